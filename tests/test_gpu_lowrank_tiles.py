"""The low-rank denoiser's tiles: row counts at the edges of every tile height (16, 32, 64, 128) and of the compacting form
(512), a half slice at the end of a row (d = 16 mod 32), ranks that are padded, masked rows, a device-side chain count and
an output that is not 16-byte aligned, against the oracle.

Tolerance: the products keep 24 bits of every operand and add in fp32, so the error is that of fp32 sums over d terms in
ranges of at most 1024: below 2e-6 of the row's scale (measured 3e-7 to 7e-7).  The bits do not depend on the call's
size."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle.denoisers import LowRankDenoiser

from _gpu import as_f32_f64, dev, f32, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r", [(16, 3), (48, 33), (1104, 50), (3072, 256)])
def test_row_counts_at_tile_edges(d, r):
    from paper_2501_05370_amd.binding import Denoiser
    rng = np.random.default_rng(11)
    T, rows = 25, 18001 if d == 3072 else 4100
    p = W.lowrank_gaussian(rng, d, r)
    sched = W.cosine_schedule(T)
    g = Denoiser.sdden_lowrank_create(p.mu, p.U, p.s2, sched.alpha_bar_state)
    g.sdden_reserve(rows)
    x = as_f32_f64(rng.standard_normal((rows, d)))
    k = rng.integers(-2, T + 2, size=rows).astype(np.int32)
    k[[0, 15, 16, 31, 32, 63, 64, 127, 128, 511, 512]] = [3, -1, T, 0, T - 1, 5, -1, 2, 7, 1, 4]
    live = (k >= 0) & (k < T)
    few = np.flatnonzero(live)[:600]
    want = LowRankDenoiser(p, sched.alpha_bar_state)(x[few], k[few])
    xg, kg = f32(x), dev(k, torch.int32)
    whole = torch.full((rows, d), 777.0, dtype=torch.float32, device="cuda")
    g.sdden_eval(rows, xg, kg, whole)
    assert np.all(host(whole)[~live] == 777.0)
    err = rel_err(host(whole)[few], want)
    print(f"[lowrank d={d} r={r}] rel err {err:.2e}")
    assert err < 2e-6
    for R in (1, 15, 16, 17, 32, 33, 65, 129, 512, 513, 2049):
        out = torch.full((R, d), 777.0, dtype=torch.float32, device="cuda")
        g.sdden_eval(R, xg[:R], kg[:R], out)
        assert torch.equal(out, whole[:R]), R
        flat = torch.full((R * d + 1,), 777.0, dtype=torch.float32, device="cuda")
        g.sdden_eval(R, xg[:R], kg[:R], flat[1:].view(R, d))          # 4-byte aligned output
        assert torch.equal(flat[1:].view(R, d), whole[:R]) and flat[0] == 777.0, R
    count = torch.tensor([9], dtype=torch.int32, device="cuda")       # 9 chains of 13 rows, read on the device
    g.sdden_set_active_count(count, 13)
    for R in (500, 2000):
        out = torch.full((R, d), 777.0, dtype=torch.float32, device="cuda")
        g.sdden_eval(R, xg[:R], kg[:R], out)
        assert torch.equal(out[:117], whole[:117]) and torch.all(out[117:] == 777.0), R
    g.sdden_set_active_count(None, 1)


# Few rows add the slabs up inside the second product while a row's slabs hold 512 floats (d = 2048 at rank 64, 4096 at rank 32) and all
# tiles' 16 MB (d = 2048: 64 rows of 16 x 16 tiles, from 97 on 128 of 32 x 32).
@pytest.mark.parametrize("d,r,rows", [(2048, 50, (1, 64, 65, 96, 97, 128, 129)), (2064, 50, (1, 64)), (2048, 64, (33,)), (2048, 65, (33,)),
                                      (4096, 20, (16, 32, 33)), (4112, 20, (16, 33))])
def test_slabs_added_up_in_the_second_product(d, r, rows):
    from paper_2501_05370_amd.binding import Denoiser
    rng = np.random.default_rng(d + r)
    T, R = 25, 600
    p = W.lowrank_gaussian(rng, d, r)
    sched = W.cosine_schedule(T)
    g = Denoiser.sdden_lowrank_create(p.mu, p.U, p.s2, sched.alpha_bar_state)
    g.sdden_reserve(R)
    x = as_f32_f64(rng.standard_normal((R, d)))
    k = rng.integers(0, T, size=R).astype(np.int32)
    k[[0, 30, 63]] = [1, -1, T]
    live = (k >= 0) & (k < T)
    xg, kg = f32(x), dev(k, torch.int32)
    whole = torch.full((R, d), 777.0, dtype=torch.float32, device="cuda")
    g.sdden_eval(R, xg, kg, whole)                                   # too many rows for it
    assert rel_err(host(whole)[live], LowRankDenoiser(p, sched.alpha_bar_state)(x[live], k[live])) < 2e-6
    for n in rows:
        out = torch.full((n, d), 777.0, dtype=torch.float32, device="cuda")
        g.sdden_eval(n, xg[:n], kg[:n], out)
        assert torch.equal(out, whole[:n]), n


@pytest.mark.parametrize("r,R", [(1, 70), (2, 600), (4, 4096), (33, 4096)])
def test_axis_aligned_basis_rounds_once_per_operation(r, R):
    """Columns of U along coordinate axes: the basis holds zeros and ones, both products are exact, and what is left are the
    roundings of one multiplication (the gain) and one fused multiply-add, the same bits as in numpy.  (The fp64 image of
    that multiply-add is rounded twice: it can miss the bits once in 2^29.)"""
    from paper_2501_05370_amd.binding import Denoiser
    rng = np.random.default_rng(r)
    d, T, s2 = 80, 25, np.float32(0.01)
    axes = rng.permutation(d)[:r]
    U = np.zeros((d, r), np.float32)
    U[axes, np.arange(r)] = rng.uniform(0.5, 3.0, r)
    sched = W.cosine_schedule(T)
    g = Denoiser.sdden_lowrank_create(np.zeros(d), U, s2, sched.alpha_bar_state)
    g.sdden_reserve(R)
    k = (np.arange(R) % T).astype(np.int32)
    x = rng.standard_normal((R, d)).astype(np.float32)
    out = torch.zeros(R, d, device="cuda")
    g.sdden_eval(R, f32(x), dev(k, torch.int32), out)
    ab = np.asarray(sched.alpha_bar_state, np.float32).astype(np.float64)[k][:, None]
    sab, s2 = np.sqrt(ab), float(s2)
    ls = (U.astype(np.float64) ** 2).sum(0)[None, :] + s2
    gperp = sab * s2 / (ab * s2 + 1 - ab)
    gain = (sab * ls / (ab * ls + 1 - ab) - gperp).astype(np.float32)
    gperp = gperp.astype(np.float32)
    want = gperp * x
    p = gain * x[:, axes]
    want[:, axes] = (p.astype(np.float64) + gperp.astype(np.float64) * x[:, axes]).astype(np.float32)
    assert np.array_equal(host(out), want)
