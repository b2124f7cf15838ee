"""Langevin chains too long for one wavefront (d > 1024): the one-launch form of ``LangevinSampler.run`` against the same
library's windows and ``sd_advance`` call by call, bit for bit, and the windows against the oracle.  Row lengths at the
edges of the workgroup sizes (257, 512, 513, 768, 769 and 1024 groups of four) and no multiple of four."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import langevin as L
from oracle.denoisers import GMMScore

from _gpu import as_f32_f64, dev, f32, host, make_context

pytestmark = pytest.mark.gpu


def _sampler(cfg, B, tau):
    from paper_2501_05370_amd.sampler import LangevinSampler
    ctx = make_context(cfg.schedule, cfg.d, cfg.K, seed=9, tau=tau)
    p = cfg.params
    return LangevinSampler(ctx, f32(p.means), f32(p.logw), float(p.stds[0, 0]), cfg.gamma, B)


@pytest.mark.parametrize("B,d,M,K,T,tau", [(5, 1025, 1, 1, 7, 1.0), (21, 1028, 16, 8, 30, 1.0), (9, 2048, 5, 6, 17, 2.0),
                                           (9, 2051, 9, 8, 25, 1.0), (300, 2500, 9, 8, 20, 1.0), (7, 3072, 3, 16, 19, 1.0),
                                           (7, 3073, 16, 5, 12, 1.0), (11, 4096, 16, 64, 40, 0.5)])
def test_whole_chains_equal_the_window_loop(B, d, M, K, T, tau):
    from paper_2501_05370_amd.binding import SDError
    cfg = W.make_config("c5", B=B, d=d, M=M, K=K, T=T)
    ids = torch.randperm(B, generator=torch.Generator().manual_seed(3)).cuda()
    loop = _sampler(cfg, B, tau)
    n = loop.start(ids)
    while n > 0:
        loop.window(n)
        loop.advance(n)
        n = int(loop.buf.B_active.item())
    for kw in ({}, {"windows_per_sync": 4}):
        smp = _sampler(cfg, B, tau)
        out, counters = smp.run(ids, **kw)
        assert torch.equal(out, loop.buf.out)
        assert counters == loop.buf.counters.tolist() and counters[0] == B * T
        assert int(smp.buf.B_active.item()) == 0
    with pytest.raises(SDError):                                     # the back-to-back call keeps its limit
        smp.run_fused(ids)

    p, sc = cfg.params, GMMScore(cfg.params)
    rng = np.random.default_rng(8)
    comp = rng.integers(0, M, size=B)
    x = as_f32_f64(p.means[comp] * rng.uniform(0.3, 1.0, size=(B, 1)) + rng.standard_normal((B, d)))
    n0 = rng.integers(0, T, size=B)
    idn = host(ids)
    xo, adv, rej, lr, lu = L.ula_window(sc, x, n0, idn, K, T, cfg.gamma, seed=9, tau=tau)
    b, ctx = loop.buf, loop.ctx
    glr, glu = torch.full((B, K), 5.0, device="cuda"), torch.full((B, K), 5.0, device="cuda")
    ctx.sd_langevin_window(B, f32(x), dev(n0, torch.int32), ids, loop.means, loop.logw, loop.comp_std, M, cfg.gamma,
                           b.y_out, b.adv, b.rejected, glr, glu)
    same = host(b.adv)[:B] == adv
    assert same.sum() >= B - 1
    scale = np.maximum(1.0, np.abs(xo).max(axis=1, keepdims=True))
    assert np.max(np.abs(host(b.y_out)[:B] - xo)[same] / scale[same]) < 1e-5
    reached = (np.arange(K)[None, :] < adv[:, None]) & same[:, None]
    assert np.max(np.abs(host(glr) - lr)[reached] / np.maximum(1.0, np.abs(lr[reached]))) < 1e-4


@pytest.mark.parametrize("at_end", ["some", "all"])
def test_chains_handed_over_at_ragged_steps(at_end):
    """Chains at any step, step T included: such a chain's window copies its state, sd_advance leaves that in `out` and
    counts the chain-window."""
    B, d, M, K, T = 30, 1100, 4, 5, 17
    cfg = W.make_config("c5", B=B, d=d, M=M, K=K, T=T)
    n = np.random.default_rng(2).integers(0, T + 1, B) if at_end == "some" else np.full(B, T)
    if at_end == "some":
        n[[0, 1, 2, B - 1]] = [T, T - 1, 0, T]
    ids = torch.randperm(B, generator=torch.Generator().manual_seed(3)).cuda()
    smp = []
    for _ in range(2):
        s = _sampler(cfg, B, 1.0)
        s.start(ids)
        s.buf.n.copy_(torch.as_tensor(n, dtype=torch.int32))
        s.buf.out.fill_(777.0)
        smp.append(s)
    a, b = smp
    assert a._run_chains(B)
    left = B
    while left > 0:
        b.window(left)
        b.advance(left)
        left = int(b.buf.B_active.item())
    assert torch.equal(a.buf.out, b.buf.out) and not bool((b.buf.out == 777.0).any())
    assert a.buf.counters.tolist() == b.buf.counters.tolist() and int(a.buf.B_active.item()) == 0


def test_no_chains():
    """B = 0: the count says so, as sd_advance leaves it."""
    s = _sampler(W.make_config("c5", B=3, d=1100, M=4, K=5, T=17), 3, 1.0)
    b = s.buf
    b.B_active.fill_(9)
    assert s.ctx.sd_langevin_chains(0, b.y, b.n, b.chain_id, s.means, s.logw, s.comp_std, s.M, s.gamma, b.out, b.B_active, b.counters)
    assert int(b.B_active.item()) == 0 and b.counters.tolist() == [0] * 5
