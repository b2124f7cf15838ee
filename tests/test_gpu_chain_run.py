"""Whole chains in one launch (``sdden_run``, what ``run`` uses on mixtures) against the same library called window by
window: same counters, same states.  Predictions come from the same device function and every stored value is rounded to
fp32 at the same place; what differs is the order of the fp64 sums behind a log-ratio and a reflection (1e-15 relative),
which moves a state by at most one fp32 rounding (6e-8) per window; windows pass such a difference on with a factor of
order one, so 60 of them stay within the 1e-5 of the other parity tests.
"""
import numpy as np
import pytest
import torch

from _gpu import host

pytestmark = pytest.mark.gpu


def _mixture(rng, M, d):
    return rng.normal(0, 3.0, (M, d)), rng.uniform(0.2, 1.0, (M, d)), np.full(M, -np.log(M))


def _sampler(drafter, B, d, M, K, T, seed=3):
    import workloads as W
    from paper_2501_05370_amd.binding import Denoiser
    from paper_2501_05370_amd.sampler import DiffusionSampler, EfficientFrozenSampler, IndependentDrafterSampler
    from _gpu import make_context
    s = W.cosine_schedule(T)
    ctx = make_context(s, d, K, seed)
    mu, sd, lw = _mixture(np.random.default_rng(M * 1000 + d), M, d)
    den = Denoiser.sdden_gmm_create(mu, sd, lw, s.alpha_bar_state)
    if drafter == "independent":
        h = np.arange(0, M, 2)
        return IndependentDrafterSampler(ctx, den, Denoiser.sdden_gmm_create(mu[h], sd[h], np.full(h.size, -np.log(h.size)), s.alpha_bar_state), B)
    if drafter.startswith("reused"):
        return EfficientFrozenSampler(ctx, den, B, carry="last_accepted" if drafter.endswith("last") else "draft")
    return DiffusionSampler(ctx, den, B)


# lane layouts change at d = 64, 128, 256, 512, 1024 and with M (lanes per component); the tables leave LDS above d = 256 or
# 36 KiB; workgroups hold 1, 2 or 4 chains from 1024 and 2048 chains on; more than 64 components: window by window
@pytest.mark.parametrize("drafter,B,d,M,K,T", [
    ("frozen", 5, 1, 1, 1, 20), ("frozen", 64, 2, 8, 4, 60), ("frozen", 33, 63, 5, 64, 40), ("frozen", 2050, 64, 32, 8, 30),
    ("frozen", 9, 65, 33, 6, 40), ("frozen", 1027, 128, 3, 5, 30), ("frozen", 7, 129, 64, 7, 30), ("frozen", 3, 257, 2, 5, 40),
    ("frozen", 3, 513, 17, 4, 20), ("frozen", 2, 1030, 1, 4, 20), ("frozen", 4, 20, 65, 4, 20),
    ("reused", 40, 30, 7, 6, 50), ("reused_last", 40, 30, 7, 6, 50), ("reused", 3, 300, 4, 3, 25), ("reused", 6, 2, 3, 1, 25),
    ("independent", 50, 75, 12, 5, 40), ("independent", 3, 700, 3, 4, 20), ("independent", 4, 3, 1, 1, 30)])
def test_chain_run_equals_the_window_loop(drafter, B, d, M, K, T):
    ids = torch.randperm(B, device="cuda").to(torch.int64)
    a = _sampler(drafter, B, d, M, K, T)
    out, counters = a.run(ids)
    out = host(out).copy()
    assert host(a.buf.B_active)[0] == 0
    b = _sampler(drafter, B, d, M, K, T)
    left = b.start(ids)
    while left > 0:
        b.window(left)
        b.advance(left)
        left = int(b.buf.B_active.item())
    ref, want = host(b.buf.out), b.buf.counters.tolist()
    assert counters == want and counters[0] == B * T
    err = np.max(np.abs(out - ref) / np.maximum(1.0, np.abs(ref).max(axis=1, keepdims=True)))
    print(f"[chain run {drafter} d={d} M={M}] counters {counters}, max rel err {err:.1e}")
    assert err < 1e-5
    # a second run accumulates into the counters when asked to, and starts from zero otherwise
    assert a.run(ids, reset_counters=False)[1] == [2 * c for c in want]
    assert a.run(ids, windows_per_sync=3)[1] == want


# Chains handed over at any step, step T included: such a chain's window copies its state, sd_advance leaves that in `out`
# and counts the chain-window.
@pytest.mark.parametrize("drafter,B,d,M", [("frozen", 40, 7, 5), ("reused", 40, 30, 7), ("independent", 40, 9, 4), ("frozen", 2050, 3, 2)])
@pytest.mark.parametrize("at_end", ["some", "all"])
def test_chains_handed_over_at_ragged_steps(drafter, B, d, M, at_end):
    K, T = 5, 24
    rng = np.random.default_rng(B + d)
    n = np.full(B, T) if at_end == "all" else rng.integers(0, T + 1, B)
    if at_end == "some":
        n[[0, 1, 2, B - 1]] = [T, T - 1, 0, T]
    ids = torch.randperm(B, device="cuda").to(torch.int64)
    smp = []
    for _ in range(2):
        s = _sampler(drafter, B, d, M, K, T)
        s.start(ids)
        s.buf.n.copy_(torch.as_tensor(n, dtype=torch.int32))
        if drafter == "reused":
            s.den.sdden_eval(B, s.buf.y, s.buf.n, s.buf.Dfz)
        s.buf.out.fill_(777.0)
        smp.append(s)
    a, b = smp
    assert a._run_chains(B)
    left = B
    while left > 0:
        b.window(left)
        b.advance(left)
        left = int(b.buf.B_active.item())
    out, ref = host(a.buf.out), host(b.buf.out)
    assert not np.any(ref == 777.0)
    assert a.buf.counters.tolist() == b.buf.counters.tolist() and int(a.buf.B_active.item()) == 0
    assert np.max(np.abs(out - ref) / np.maximum(1.0, np.abs(ref).max(axis=1, keepdims=True))) < 1e-5


def test_widest_rows_of_one_component():
    """M = 1 pads a row to 2048 coordinates, 16 KiB of LDS per wavefront: four of them and the counters pass 64 KiB."""
    B, d, K, T = 2048, 1874, 2, 3
    ids = torch.arange(B, device="cuda")
    a, b = _sampler("frozen", B, d, 1, K, T), _sampler("frozen", B, d, 1, K, T)
    a.start(ids)
    assert a._run_chains(B)
    left = b.start(ids)
    while left > 0:
        b.window(left)
        b.advance(left)
        left = int(b.buf.B_active.item())
    out, ref = host(a.buf.out), host(b.buf.out)
    assert a.buf.counters.tolist() == b.buf.counters.tolist()
    assert np.max(np.abs(out - ref) / np.maximum(1.0, np.abs(ref).max(axis=1, keepdims=True))) < 1e-5


def test_denoiser_of_fewer_steps_than_the_chains():
    """Rows at a step the denoiser does not have are masked by sdden_eval; the loop over such a denoiser still runs."""
    import workloads as W
    from paper_2501_05370_amd.binding import Denoiser
    from paper_2501_05370_amd.sampler import DiffusionSampler, IndependentDrafterSampler
    from _gpu import make_context
    T, d, M, B = 12, 6, 3, 10
    s = W.cosine_schedule(T)
    mu, sd, lw = _mixture(np.random.default_rng(1), M, d)
    den = Denoiser.sdden_gmm_create(mu, sd, lw, s.alpha_bar_state[:10])
    full = Denoiser.sdden_gmm_create(mu, sd, lw, s.alpha_bar_state)
    ids = torch.arange(B, device="cuda")
    for make in (lambda: DiffusionSampler(make_context(s, d, 4, 3), den, B),
                 lambda: IndependentDrafterSampler(make_context(s, d, 4, 3), full, den, B)):
        a, b = make(), make()
        out, counters = a.run(ids)
        left = b.start(ids)
        while left > 0:
            b.window(left)
            b.advance(left)
            left = int(b.buf.B_active.item())
        assert torch.equal(out, b.buf.out) and counters == b.buf.counters.tolist()


def test_no_chains():
    """B = 0: the count says so, as sd_advance leaves it."""
    a = _sampler("frozen", 4, 6, 3, 4, 12)
    b = a.buf
    b.B_active.fill_(9)
    assert a.den.sdden_run(a.ctx, 0, b.y, b.n, b.chain_id, b.out, b.B_active, b.counters)
    assert int(b.B_active.item()) == 0 and b.counters.tolist() == [0] * 5
