"""Langevin chains that share a wavefront (d <= 128): whole runs against the same library's windows and ``sd_advance``
call by call, bit for bit (chains change neighbours at every compaction), and one window with its diagnostics against the
oracle.  Row lengths at the edges of every lane count (8, 16, 32, 64, 128) and the first one past them; chain counts that
leave lanes, wavefronts and workgroups empty; finished chains among the others."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import langevin as L
from oracle.denoisers import GMMScore

from _gpu import as_f32_f64, dev, f32, host, make_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,M,K,T,tau", [(1, 1, 1, 1, 5, 1.0), (130, 2, 16, 8, 30, 1.0), (33, 8, 3, 6, 25, 1.0),
                                           (70, 9, 5, 24, 40, 2.0), (200, 16, 16, 4, 21, 1.0), (65, 17, 4, 8, 25, 1.0),
                                           (31, 32, 13, 16, 40, 1.0), (40, 33, 8, 5, 18, 0.5), (17, 64, 16, 64, 70, 1.0),
                                           (23, 65, 9, 8, 25, 1.0), (9, 128, 16, 40, 50, 1.0), (9, 129, 16, 8, 20, 1.0)])
def test_runs_windows_and_oracle_agree(B, d, M, K, T, tau):
    from paper_2501_05370_amd.sampler import LangevinSampler
    cfg = W.make_config("c5", B=B, d=d, M=M, K=K, T=T)
    p = cfg.params
    ids = torch.randperm(B, generator=torch.Generator().manual_seed(3)).cuda()

    def sampler():
        return LangevinSampler(make_context(cfg.schedule, d, K, seed=9, tau=tau), f32(p.means), f32(p.logw),
                               float(p.stds[0, 0]), cfg.gamma, B)

    loop = sampler()
    want, counters = loop.run(ids)
    got, run_counters = sampler().run_fused(ids)
    assert torch.equal(got, want[ids])
    assert run_counters[:3] == counters[:3] and run_counters[4] == counters[4] and counters[0] == B * T

    sc, rng = GMMScore(p), np.random.default_rng(8)
    comp = rng.integers(0, M, size=B)
    x = as_f32_f64(p.means[comp] * rng.uniform(0.3, 1.0, size=(B, 1)) + rng.standard_normal((B, d)))
    n0 = rng.integers(0, T, size=B)
    idn = host(ids)
    xo, adv, rej, lr, lu = L.ula_window(sc, x, n0, idn, K, T, cfg.gamma, seed=9, tau=tau)
    n0[-1] = T                                                       # a chain that has nothing left to do
    b, ctx = loop.buf, loop.ctx
    glr, glu = torch.full((B, K), 5.0, device="cuda"), torch.full((B, K), 5.0, device="cuda")
    ctx.sd_langevin_window(B, f32(x), dev(n0, torch.int32), ids, loop.means, loop.logw, loop.comp_std, M, cfg.gamma,
                           b.y_out, b.adv, b.rejected, glr, glu)
    live = n0 < T
    assert np.all(host(b.adv)[:B][~live] == 0) and np.all(host(b.y_out)[:B][~live] == x[~live])
    assert np.all(host(glr)[~live] == 0) and np.all(host(glu)[~live] == 0)
    same = (host(b.adv)[:B] == adv) & live
    assert same.sum() >= live.sum() - 1
    scale = np.maximum(1.0, np.abs(xo).max(axis=1, keepdims=True))
    assert np.all(np.abs(host(b.y_out)[:B] - xo)[same] / scale[same] < 1e-5)
    assert np.all(host(b.rejected)[:B][same] == rej[same])
    reached = (np.arange(K)[None, :] < adv[:, None]) & same[:, None]
    assert np.all(np.abs(host(glr) - lr)[reached] / np.maximum(1.0, np.abs(lr[reached])) < 1e-4)
    assert np.all(np.abs(host(glu) - lu)[reached] < 1e-5 * np.maximum(1.0, np.abs(lu[reached])))
    assert np.all(host(glr)[same][~reached[same]] == 0)
