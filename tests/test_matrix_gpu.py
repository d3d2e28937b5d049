"""GPU parity of the matrix-core kernels at the edges of their tiles.

Sizes where a tile, stage or split ends, against the fp64 oracle.  fp32 bound:
a sum of K complex products takes 12 K / 16 roundings of its accumulator, each
0.29 x 2^-24 of the partial sum (RMS); over the 2050 products of the longest
case these grow to 4.8e-7 of the result, and the transforms on either side add
about 3e-7, so 1e-6 holds for every case while a dropped part of a split value
(2^-9 to 2^-17 of it) does not.
"""
import pytest

from oracle import bl_oracle as bo
from paper_1911_09287_amd import blconv, synth
from test_parity_gpu import BF16_TOL, gpu_passes, oracle_passes, rel, say

pytestmark = pytest.mark.gpu

FP32_TOL = 1e-6


@pytest.fixture(scope="module")
def torch():
    import torch as _torch
    if not _torch.cuda.is_available():
        pytest.skip("no GPU")
    blconv.load()
    return _torch


@pytest.mark.parametrize("N,ci,co,hw,bf16", [
    (31, 17, 33, 4, 0),    # one 32-row tile, odd k (one-element loads along k), a ragged 64-wide tile
    (32, 16, 32, 2, 0),    # exactly one 32 x 32 tile and one stage of 16 k
    (65, 48, 97, 3, 0),    # one row and one column past 64-wide tiles, three stages over two wave groups
    (33, 80, 31, 5, 0),    # 64 x 32 tiles, five stages over four wave groups
    (9, 2050, 70, 1, 0),   # few tiles, long sums: k split, the last range two k long
    (64, 1024, 64, 2, 0),  # forward split along k, its partial spectra added by the inverse
    (16, 512, 512, 4, 0),  # paired backward: grad-input split along k
    (130, 24, 64, 6, 0),   # paired backward: grad-weight with the longer sums, whole
    (33, 66, 70, 4, 1),    # bfloat16 spectra: a partial stage of 32 k
    (40, 35, 37, 4, 1),    # bfloat16 spectra: odd k
])
def test_contraction_tiles(torch, N, ci, co, hw, bf16):
    layer = synth.Layer("tiles", 2, N, ci, co, hw, hw, 3, (1, 1, 1, 1), "blur")
    x, w, dy = synth.random_inputs(layer, 4100 + N)
    got = gpu_passes(torch, layer, 0.0, x, w, dy, desc_flags=blconv.BL_DESC_BF16_SPECTRA if bf16 else 0)
    plan, ws = got[3], got[4]
    xt, wt, dyt = (torch.from_numpy(a).to(ws.device) for a in (x, w, dy))
    dx, dw = torch.full_like(xt, float("nan")), torch.full_like(wt, float("nan"))
    plan.backward(dyt, wt, xt, dx, dw, ws)
    torch.cuda.synchronize()
    ref = oracle_passes(layer, 0.0, x, w, dy, rounding=bo.round_bf16 if bf16 else None)
    errs = [rel(g, r) for g, r in zip(got[:3] + (dx.cpu().numpy(), dw.cpu().numpy()), ref + ref[1:])]
    say(f"[tiles] {N} {ci}->{co} @{hw} bf16={bf16}: {errs}")
    assert max(errs) <= (BF16_TOL if bf16 else FP32_TOL), errs
