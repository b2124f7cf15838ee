"""Langevin chains held by one component (d > 128): the one-launch kernels skip the logits while distances prove that the other
components cannot matter.  The window kernel with d <= 1024 and any single window always compute them, so whole runs are
compared with windows and ``sd_advance`` call by call, bit for bit, over mixtures that reach the rule and its edges: components
far apart, at log-odds around its threshold, overlapping, coincident, far from the origin, without weight; means that fit LDS
and means that do not."""
import math

import pytest
import torch

import workloads as W

from _gpu import make_context

pytestmark = pytest.mark.gpu


def _means(kind, M, d):
    g = torch.Generator().manual_seed(5)
    mu = torch.randn(M, d, generator=g)
    logw = torch.full((M,), -math.log(M))
    if kind == "apart":
        mu = 2 * mu
    elif kind == "threshold":                        # |mu_a - mu_b|^2 / 2 s^2 is about 80: gaps between 40 and 120
        mu = mu * math.sqrt(80.0 / d)
    elif kind == "overlapping":
        mu = mu * math.sqrt(2.0 / d)
    elif kind == "twins":
        mu = 2 * mu
        mu[1] = mu[0]
    elif kind == "offset":
        mu = 2 * mu + 3000.0
    else:                                            # no weight, and weights that alone decide between coincident components
        mu = 2 * mu
        mu[M - 1] = mu[0]
        logw = logw - 70.0 * torch.arange(M)
        logw[1] = -math.inf
    return mu.cuda().contiguous(), logw.cuda()


@pytest.mark.parametrize("kind", ["apart", "threshold", "overlapping", "twins", "offset", "weights"])
@pytest.mark.parametrize("B,d,M,K,T", [(9, 150, 16, 8, 140), (40, 256, 5, 16, 60), (21, 601, 7, 1, 120), (300, 1000, 16, 16, 110),
                                       (5, 1024, 3, 64, 130), (7, 1100, 16, 5, 120), (5, 2500, 16, 8, 100), (5, 4001, 4, 16, 110),
                                       (3, 4093, 10, 16, 140)])
def test_runs_equal_the_window_loop(kind, B, d, M, K, T):
    from paper_2501_05370_amd.sampler import LangevinSampler
    cfg = W.make_config("c5", B=B, d=d, M=M, K=K, T=T)
    mu, logw = _means(kind, M, d)

    def sampler():
        return LangevinSampler(make_context(cfg.schedule, d, K, seed=4), mu, logw, 1.0, cfg.gamma, B)
    ids = torch.randperm(B, generator=torch.Generator().manual_seed(3)).cuda()
    loop, smp = sampler(), sampler()
    n = loop.start(ids)
    while n > 0:
        loop.window(n)
        loop.advance(n)
        n = int(loop.buf.B_active.item())
    out, counters = smp.run(ids) if d > 1024 else smp.run_fused(ids)
    want = loop.buf.out if d > 1024 else loop.buf.out[ids]
    assert torch.equal(out, want)
    got = loop.buf.counters.tolist()
    assert [counters[i] for i in (0, 1, 2, 4)] == [got[i] for i in (0, 1, 2, 4)] and counters[0] == B * T


# Distances carry powers of the standard deviation, in other units in the two kernels, and steps far below the slack's last bit
# may follow each other for a whole run: means, steps and all at other scales, and steps of a hundredth of the usual length.
@pytest.mark.parametrize("kind", ["apart", "threshold", "offset"])
@pytest.mark.parametrize("std,length", [(0.25, 1.0), (4.0, 1.0), (1.0, 1e-2), (0.1, 1e-3)])
@pytest.mark.parametrize("d,M,K,T", [(300, 16, 8, 200), (1000, 9, 16, 200), (1100, 6, 5, 200), (3000, 16, 16, 200)])
def test_other_scales(kind, std, length, d, M, K, T):
    from paper_2501_05370_amd.sampler import LangevinSampler
    B = 5
    cfg = W.make_config("c5", B=B, d=d, M=M, K=K, T=T)
    mu, logw = _means(kind, M, d)
    gamma = cfg.gamma * (std * length) ** 2
    res = []
    for one_launch in (True, False):
        s = LangevinSampler(make_context(cfg.schedule, d, K, seed=4), (mu * std).contiguous(), logw, std, gamma, B)
        b, n = s.buf, s.start(torch.arange(B, device="cuda"))
        near = mu[torch.arange(B) % M] * torch.linspace(0.0, 1.0, B, device="cuda")[:, None]
        b.y[:B] = (std * (b.y[:B] + near)).contiguous()              # from the origin to a component's mean
        if one_launch and d <= 1024:
            s.ctx.sd_langevin_run(B, b.y, b.n, b.chain_id, s.means, s.logw, std, M, gamma, T, b.y_out, b.n, b.counters)
            res.append((b.y_out.clone(), b.counters.tolist()[:3]))
            continue
        if one_launch:
            assert s._run_chains(B)
            n = 0
        while n > 0:
            s.window(n)
            s.advance(n)
            n = int(b.B_active.item())
        res.append((b.out.clone(), b.counters.tolist()[:3]))
    assert torch.equal(res[0][0], res[1][0]) and bool(torch.isfinite(res[0][0]).all())
    assert res[0][1] == res[1][1] and res[0][1][0] == B * T


@pytest.mark.parametrize("d", [400, 1500])
def test_one_component_and_a_state_that_is_no_number(d):
    """M = 1 has no other component at all; a chain whose state holds a NaN or an infinity ends as the loop's does."""
    from paper_2501_05370_amd.sampler import LangevinSampler
    for M in (1, 6):
        B, K, T = 6, 8, 90
        cfg = W.make_config("c5", B=B, d=d, M=M, K=K, T=T)
        mu, logw = _means("apart", M, d)
        res = []
        for one_launch in (True, False):
            s = LangevinSampler(make_context(cfg.schedule, d, K, seed=4), mu, logw, 1.0, cfg.gamma, B)
            n = s.start(torch.arange(B, device="cuda"))
            s.buf.y[1, 3], s.buf.y[4, d - 1] = math.nan, math.inf
            b = s.buf
            if one_launch and d <= 1024:
                s.ctx.sd_langevin_run(B, b.y, b.n, b.chain_id, mu, logw, 1.0, M, cfg.gamma, T, b.y_out, b.n, b.counters)
                res.append(b.y_out.clone())
                continue
            if one_launch:
                assert s._run_chains(B)
                n = 0
            while n > 0:
                s.window(n)
                s.advance(n)
                n = int(b.B_active.item())
            res.append(b.out.clone())
        assert torch.equal(torch.isnan(res[0]), torch.isnan(res[1]))
        assert torch.equal(torch.nan_to_num(res[0]), torch.nan_to_num(res[1]))
        assert not bool(torch.isnan(res[0][0]).any()) and bool(torch.isnan(res[0][1]).any())
