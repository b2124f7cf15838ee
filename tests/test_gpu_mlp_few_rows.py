"""The MLP denoiser's kernels for calls of few rows: row counts at the edges of their tiles (16, 32, 64 rows) and of their
range (1024), widths at the edges of the column rule, masked rows and a device-side chain count, against the oracle.

Tolerance 2e-2 of the row's scale, as for the other MLP tests: bf16 weights and activations, fp32 sums.  Against the
kernels for many rows the results are the same bits: every kernel sums over k in one chain and in order."""
import math

import numpy as np
import pytest
import torch

import workloads as W
from oracle.denoisers import MLPDenoiser

from _gpu import as_f32_f64, dev, f32, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H", [(256, 256), (3072, 512), (768, 1280)])
def test_row_counts_at_tile_edges(d, H):
    from paper_2501_05370_amd.binding import Denoiser
    rng = np.random.default_rng(7)
    T = 25
    p = W.random_mlp(rng, d, H, 16)
    ref = MLPDenoiser(p)
    g = Denoiser.sdden_mlp_create(p, T, 1025)
    x = as_f32_f64(rng.standard_normal((1025, d)))
    k = rng.integers(-2, T + 2, size=1025).astype(np.int32)
    k[[0, 15, 16, 31, 32, 63, 64, 1023, 1024]] = [3, -1, T, 0, T - 1, 5, -1, 2, 7]
    live = (k >= 0) & (k < T)
    want = np.zeros((1025, d))
    want[live] = ref(x[live], k[live])
    xg, kg = f32(x), dev(k, torch.int32)
    whole = torch.full((1025, d), 777.0, dtype=torch.float32, device="cuda")
    g.sdden_eval(1025, xg, kg, whole)                                # the tiles for many rows
    for R in (1, 15, 16, 17, 32, 33, 64, 65, 257, 1023, 1024, 1025):
        out = torch.full((R, d), 777.0, dtype=torch.float32, device="cuda")
        g.sdden_eval(R, xg[:R], kg[:R], out)
        got = host(out)
        assert rel_err(got[live[:R]], want[:R][live[:R]]) < 2e-2, R
        assert torch.equal(out, whole[:R]), R                        # a prediction does not depend on the call's size
        img = xg[:R].to(torch.bfloat16).view(torch.int16).contiguous()
        img[~dev(live[:R], torch.bool)] = 0x7fc0                     # masked rows carry NaN in the image
        out2 = torch.full((R, d), 777.0, dtype=torch.float32, device="cuda")
        g.sdden_eval_mirror(R, xg[:R], img, kg[:R], out2)
        assert torch.equal(out2, out), R
    # 7 of 20 chains of 5 rows present; every row masked
    R = 100
    out = torch.full((R, d), 777.0, dtype=torch.float32, device="cuda")
    cnt = torch.tensor([7], dtype=torch.int32, device="cuda")
    g.sdden_set_active_count(cnt, 5)
    g.sdden_eval(R, xg[:R], kg[:R], out)
    g.sdden_set_active_count(None, 1)
    got, present = host(out), live[:R] & (np.arange(R) < 35)
    assert rel_err(got[present], want[:R][present]) < 2e-2
    assert np.all(got[~present] == 777.0)
    out.fill_(777.0)
    g.sdden_eval(R, xg[:R], torch.full((R,), -1, dtype=torch.int32, device="cuda"), out)
    assert bool((out == 777.0).all())


def test_every_tile_gives_the_same_bits():
    """The same rows in calls of every kernel: few rows (64, 1000), 64 x 128 tiles in four and two stages (1025, 4096), 128 x 128
    (8192), the 256 x 256 kernel of the batched call (10240 rows: 160 tiles of d = H = 1024 in one round of 256 CUs)."""
    from paper_2501_05370_amd.binding import Denoiser
    rng = np.random.default_rng(3)
    d = H = 1024
    T, R = 25, 10240
    g = Denoiser.sdden_mlp_create(W.random_mlp(rng, d, H, 16), T, R)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(R, d, device="cuda", generator=gen)
    k = torch.randint(0, T, (R,), device="cuda", generator=gen, dtype=torch.int32)
    whole = torch.zeros(R, d, device="cuda")
    g.sdden_eval(R, x, k, whole)
    for rows in (64, 1000, 1025, 4096, 8192):
        out = torch.zeros(rows, d, device="cuda")
        g.sdden_eval(rows, x[:rows], k[:rows], out)
        assert torch.equal(out, whole[:rows]), rows


@pytest.mark.parametrize("d", [512, 1024, 1280])
@pytest.mark.parametrize("R", [3, 16])
def test_float_rows_found_by_the_first_product(R, d):
    """The same without an image: up to 16 rows of up to 1024 coordinates the first product loads the floats, longer rows are packed."""
    from paper_2501_05370_amd.binding import Denoiser
    H, T = 256, 9
    g = Denoiser.sdden_mlp_create(W.random_mlp(np.random.default_rng(1), d, H, 16), T, 1100)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(1100, d, device="cuda", generator=gen)
    k = torch.randint(0, T, (1100,), device="cuda", generator=gen, dtype=torch.int32)
    whole = torch.zeros(1100, d, device="cuda")
    g.sdden_eval(1100, x, k, whole)                                  # the tiles for many rows
    last = torch.full_like(k[:R], T)
    last[-1:] = k[R - 1]
    for krow, there, count in ((k[:R], range(R), None), (k[:R], range(min(R, 2)), 2), (torch.full_like(last, -1), (), None),
                               (last, (R - 1,), None), (k[:R], (), 0)):
        out = torch.full((R, d), 777.0, device="cuda")
        xr = torch.full((R, d), math.nan, device="cuda")             # rows that are not there carry NaN
        rows = torch.zeros(R, dtype=torch.bool, device="cuda")
        rows[list(there)] = True
        xr[rows] = x[:R][rows]
        present = None if count is None else torch.tensor([count], dtype=torch.int32, device="cuda")
        g.sdden_set_active_count(present, 1)
        g.sdden_eval(R, xr, krow.contiguous(), out)
        g.sdden_set_active_count(None, 1)
        assert torch.equal(out[rows], whole[:R][rows]) and bool((out[~rows] == 777.0).all())


@pytest.mark.parametrize("R", [16, 30, 100, 1000])
def test_rows_found_by_the_first_product(R):
    """With a bf16 image the first product looks for the rows itself: a device-side chain count, no row at all, rows at the end of
    the buffer only; the image of masked rows is never read into a result."""
    from paper_2501_05370_amd.binding import Denoiser
    d, H, T = 512, 256, 9
    g = Denoiser.sdden_mlp_create(W.random_mlp(np.random.default_rng(1), d, H, 16), T, 1024)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(R, d, device="cuda", generator=gen)
    img = x.to(torch.bfloat16).view(torch.int16).contiguous()
    k = torch.randint(0, T, (R,), device="cuda", generator=gen, dtype=torch.int32)
    whole = torch.zeros(R, d, device="cuda")
    g.sdden_eval(R, x, k, whole)
    last = torch.full_like(k, T)
    last[-3:] = k[-3:]
    cnt = torch.tensor([3], dtype=torch.int32, device="cuda")
    for krow, present, count in ((k, 3 * 5, cnt), (torch.full_like(k, -1), 0, None), (last, None, None)):
        out = torch.full((R, d), 777.0, device="cuda")
        img2 = img.clone()
        g.sdden_set_active_count(count, 5 if count is not None else 1)
        if present is None:
            img2[:-3] = 0x7fc0
        g.sdden_eval_mirror(R, x, img2, krow, out)
        g.sdden_set_active_count(None, 1)
        rows = torch.arange(R, device="cuda")
        there = rows >= R - 3 if present is None else rows < present
        assert torch.equal(out[there], whole[there]) and bool((out[~there] == 777.0).all())
