"""GPU parity of the matrix-core kernels at the edges of their tiles.

Sizes where a tile, stage or split ends, against the fp64 oracle.  fp32 bound:
a sum of K complex products takes 12 K / 16 roundings of its accumulator, each
0.29 x 2^-24 of the partial sum (RMS); over 2050 products, were they one sum,
these grow to 4.8e-7 of the result, and the transforms on either side add
about 3e-7, so 1e-6 holds for every case while a dropped part of a split value
(2^-9 to 2^-17 of it) does not.
"""
import math
import threading

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
    (9, 2050, 70, 1, 0),   # few tiles, long sums: k split in 544, 544, 544 and 418
    (64, 1024, 64, 2, 0),  # forward split along k, its partial spectra added by the inverse
    (16, 512, 512, 4, 0),  # paired backward: grad-input split along k
    (130, 24, 64, 6, 0),   # paired backward: grad-weight with the longer sums, whole
    (2, 3, 5, 4, 0),       # tiles that are mostly padding, either direction
    (8, 7, 6, 9, 0),       # eight rows; few columns with few rows
    (1, 100, 104, 13, 0),  # one row: the input gradient past its bound on vector ALUs
    (50, 20, 1, 30, 0),    # one column past its bound
    (40, 5, 40, 6, 1),     # bfloat16 spectra: few columns (backward), few products (forward)
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


def test_last_range_of_one(torch):
    """A sum split along k whose last range is one k long (less than a stage)."""
    layer = synth.Layer("last_range", 2, 40, 7681, 40, 1, 1, 3, (1, 1, 1, 1), "blur")
    x, w, _ = synth.random_inputs(layer, 4400)
    plan = blconv.plan_for_layer(layer, 0.0)
    dev = torch.device("cuda:0")
    ws = plan.workspace(dev)
    ws.fill_(0xFF)
    y = torch.full(plan.y_shape(), float("nan"), device=dev)
    with blconv.Profile() as prof:
        plan.forward(torch.from_numpy(x).to(dev), torch.from_numpy(w).to(dev), y, ws)
        torch.cuda.synchronize()
    summed = [r[2] for r in prof.records() if r[0] == "contract_reduce"]
    splits = round(summed[0] / (8 * plan.kept * layer.N * layer.C_out)) - 1
    length = -(-(-(-layer.C_in // splits)) // 32) * 32
    assert splits > 1 and layer.C_in - (splits - 1) * length == 1, splits
    err = rel(y.cpu().numpy(), bo.forward(x, w, layer.pad, 0.0))
    say(f"[last range] {splits} ranges: {err}")
    assert err <= FP32_TOL, err


@pytest.mark.parametrize("ci,co,sp,c,call", [
    (512, 64, (20, 20), 0.5, "forward"),  # one step of 32 rows and of 32 (column, part)
    (512, 64, (6, 60), 0.0, "forward"),   # one and two
    (512, 63, (4, 100), 0.0, "forward"),  # one and four
    (512, 64, (80, 6), 0.0, "forward"),   # two and one
    (64, 512, (21, 18), 0.5, "backward"),  # grad-input in four parts
])
def test_two_product_inverse_adds_partial_spectra(torch, ci, co, sp, c, call):
    """The two-product 2-D inverse adds the partial spectra of a contraction
    split along k as it loads them."""
    layer = synth.Layer("parts", 2, 15, ci, co, *sp, 3, (1, 1, 1, 1), "blur")
    x, w, dy = synth.random_inputs(layer, 4450 + sp[0])
    plan = blconv.plan_for_layer(layer, c)
    dev = torch.device("cuda:0")
    ws = plan.workspace(dev)
    ws.fill_(0xFF)
    xt, wt, dyt = (torch.from_numpy(a).to(dev) for a in (x, w, dy))
    plan.forward(xt, wt, torch.empty_like(dyt), ws)
    out = torch.full_like(dyt if call == "forward" else xt, float("nan"))
    with blconv.Profile() as prof:
        if call == "forward":
            plan.forward(None, None, out, ws, flags=blconv.BL_REUSE_X | blconv.BL_REUSE_W)
        else:
            plan.backward(dyt, None, None, out, torch.empty_like(wt), ws, flags=blconv.BL_REUSE_X | blconv.BL_REUSE_W)
        torch.cuda.synchronize()
    names = [r[0] for r in prof.records()]
    planes, points = 15 * min(ci, co), plan.fft[0] * plan.fft[1]
    (nbytes, flops), = [r[2:] for r in prof.records() if r[0] == "spec_inv_2d"]
    parts = (nbytes - 4 * planes * sp[0] * sp[1]) / (8 * planes * plan.kept)
    assert parts >= 2 and "contract_reduce" not in names, (parts, names)
    assert abs(flops - planes * 2.5 * points * math.log2(points)) > 1.0  # (what the single product reports)
    want = bo.forward(x, w, layer.pad, c) if call == "forward" else bo.backward_input(dy, w, sp, layer.pad, c)
    err = rel(out.cpu().numpy(), want)
    say(f"[parts] {ci}->{co} @{sp}: {parts:.0f} parts, {err}")
    assert err <= FP32_TOL, err


@pytest.mark.parametrize("N,ci,co,c,shared,bf16", [
    (17, 179, 181, 0.5, True, 0), (17, 179, 181, 0.5, True, 1),  # two series to a transform: 3043 and 3077
    (9, 175, 177, 0.0, False, 0), (9, 175, 177, 0.0, False, 1),  # one each: 1575 and 1593
])
def test_many_series_by_chirp_z(torch, N, ci, co, c, shared, bf16):
    """Series past the product's bound, in odd numbers: the chirp-z kernel's
    last half-wave, and its last transform with one series of two."""
    layer = synth.Layer("chirp", 1, N, ci, co, 515, 1, 3, (1, 1), "walk")
    x, w, dy = synth.random_inputs(layer, 4900 + N)
    flags = blconv.BL_DESC_BF16_SPECTRA if bf16 else 0
    got = gpu_passes(torch, layer, c, x, w, dy, desc_flags=flags)
    plan, ws = got[3], got[4]
    xt, wt = torch.from_numpy(x).to(ws.device), torch.from_numpy(w).to(ws.device)
    with blconv.Profile() as prof:
        plan.forward(xt, wt, torch.empty(plan.y_shape(), device=ws.device), ws)
        torch.cuda.synchronize()
    for name, series in (("spec_fwd_1d", N * ci), ("spec_inv_1d", N * co)):
        (flops,) = [r[3] for r in prof.records() if r[0] == name]
        assert flops == (series // 2 + 1 if shared else series) * 100.0 * 1024, (name, flops)
    ref = oracle_passes(layer, c, x, w, dy, rounding=bo.round_bf16 if bf16 else None)
    errs = [rel(g, r) for g, r in zip(got[:3], ref)]
    say(f"[chirp-z] {N} {ci}->{co} c{c} bf16={bf16}: {errs}")
    assert max(errs) <= (BF16_TOL if bf16 else FP32_TOL), errs


@pytest.mark.parametrize("N,ci,co,sp,c", [
    (3, 512, 21, (127, 3), 0.0),   # 129 x 5 grid, 387 bins: forward split in 2
    (3, 21, 512, (5, 128), 0.25),  # 7 x 130 grid, 325 bins: paired backward, grad-input split in 2
])
def test_odd_partial_spectra(torch, N, ci, co, sp, c):
    """Grids whose inverse adds no partial spectra (more than 64 rows or
    columns kept): those of an odd number of values are summed beforehand."""
    layer = synth.Layer("odd_parts", 2, N, ci, co, *sp, 3, (1, 1, 1, 1), "blur")
    x, w, dy = synth.random_inputs(layer, 4500 + ci)
    got = gpu_passes(torch, layer, c, x, w, dy)
    plan, ws = got[3], got[4]
    assert max(plan.r_h, plan.r_w) >= 64 and plan.kept > 256 and plan.kept * N * min(ci, co) % 2
    xt, wt, dyt = (torch.from_numpy(a).to(ws.device) for a in (x, w, dy))
    y, dx, dw = torch.empty_like(dyt), torch.full_like(xt, float("nan")), torch.full_like(wt, float("nan"))
    with blconv.Profile() as prof:
        plan.forward(xt, wt, y, ws)
        plan.backward(dyt, wt, xt, dx, dw, ws)
        torch.cuda.synchronize()
    assert "contract_reduce" in [r[0] for r in prof.records()]  # (or the plan splits no longer)
    ref = oracle_passes(layer, c, x, w, dy)
    errs = [rel(g, r) for g, r in zip(got[:3] + (dx.cpu().numpy(), dw.cpu().numpy()), ref + ref[1:])]
    say(f"[odd parts] {ci}->{co} @{sp}: {errs}")
    assert max(errs) <= FP32_TOL, errs


@pytest.mark.parametrize("nd,N,ci,co,sp,K,c,fft,bf16", [
    # series: one product (any length), its k-shared and its large tiles, tails of
    # samples (n % 4 and n % 32) and of rows, a Nyquist bin kept and not
    (1, 1, 1, 1, (24,), 3, 0.0, None, 0),
    (1, 2, 3, 2, (37,), 8, 0.5, None, 0),
    (1, 3, 2, 3, (3,), 3, 0.0, None, 0),
    (1, 40, 64, 60, (401,), 5, 0.0, None, 0),
    (1, 3, 5, 7, (271,), 5, 0.25, None, 0),
    (1, 2, 2, 3, (1250,), 3, 0.0, None, 0),
    (1, 20, 33, 17, (900,), 5, 0.75, None, 0),
    (1, 2, 3, 5, (333,), 7, 0.5, 700, 1),
    # planes: one product, two products with 1, 2 and 4 steps of 32 either way,
    # oblong and enlarged grids, odd and even grid sides, few and many planes
    (2, 1, 1, 2, (5, 7), 3, 0.0, None, 0),
    (2, 3, 2, 2, (1, 3), 3, 0.0, None, 0),
    (2, 2, 3, 2, (2, 2), 1, 0.0, None, 0),
    (2, 3, 5, 6, (9, 12), 5, 0.5, None, 0),
    (2, 9, 7, 10, (13, 21), 3, 0.25, None, 0),
    (2, 4, 17, 9, (33, 28), 5, 0.0, None, 0),
    (2, 2, 3, 4, (28, 33), 1, 0.5, None, 0),
    (2, 2, 2, 3, (64, 63), 3, 0.0, None, 0),
    (2, 1, 2, 1, (100, 70), 3, 0.5, None, 0),
    (2, 1, 2, 2, (31, 90), 7, 0.75, None, 0),
    (2, 2, 3, 3, (20, 24), 5, 0.5, (43, 50), 0),
    (2, 5, 40, 24, (14, 14), 7, 0.0, None, 0),
    (2, 3, 16, 12, (23, 26), 3, 0.25, None, 1),
])
def test_matrix_transforms(torch, nd, N, ci, co, sp, K, c, fft, bf16):
    """Transforms and weight-gradient inverse as matrix products on grids
    without FFT kernels, and the combined backward."""
    lo, hi = (K - 1) // 2, K - 1 - (K - 1) // 2
    layer = synth.Layer("mt", nd, N, ci, co, sp[0], sp[1] if nd == 2 else 1, K, (lo, hi) * nd, "blur")
    x, w, dy = synth.random_inputs(layer, 4300 + N)
    got = gpu_passes(torch, layer, c, x, w, dy, fft=fft, desc_flags=blconv.BL_DESC_BF16_SPECTRA if bf16 else 0)
    plan, ws = got[3], got[4]
    xt, wt, dyt = (torch.from_numpy(a).to(ws.device) for a in (x, w, dy))
    dx, dw = torch.full_like(xt, float("nan")), torch.full_like(wt, float("nan"))
    plan.backward(dyt, wt, xt, dx, dw, ws)
    torch.cuda.synchronize()
    ref = oracle_passes(layer, c, x, w, dy, fft, rounding=bo.round_bf16 if bf16 else None)
    errs = [rel(g, r) for g, r in zip(got[:3] + (dx.cpu().numpy(), dw.cpu().numpy()), ref + ref[1:])]
    say(f"[matrix] {nd}-D {N} {ci}->{co} {sp} K{K} c{c}: {errs}")
    assert max(errs) <= (BF16_TOL if bf16 else FP32_TOL), errs


def test_matrix_transforms_keep_planes_apart(torch):
    """A sample of infinities spoils only itself, and unaligned inputs and
    outputs give the same as aligned ones (the loads are 16 bytes wide)."""
    dev = torch.device("cuda:0")
    for spatial, pad, K in (((13, 11), (1, 1, 1, 1), 3), ((8, 5), (2, 2, 2, 2), 5), ((45,), (1, 1), 3)):
        plan = blconv.Plan(len(spatial), 5, 6, 4, spatial, K, pad, 0.25)
        ws = plan.workspace(dev)
        w = torch.randn(plan.w_shape(), device=dev)
        x = torch.randn(plan.x_shape(), device=dev)
        y0, y1 = torch.empty(plan.y_shape(), device=dev), torch.empty(plan.y_shape(), device=dev)
        plan.forward(x, w, y0, ws)
        bad = x.clone()
        bad[2] = float("inf")
        plan.forward(bad, w, y1, ws)
        torch.cuda.synchronize()
        keep = [0, 1, 3, 4]
        assert torch.equal(y0[keep], y1[keep]) and not torch.isfinite(y1[2]).any()
        xb, yb = torch.empty(x.numel() + 1, device=dev), torch.full((y0.numel() + 1,), float("nan"), device=dev)
        xu, yu = xb[1:].view(x.shape), yb[1:].view(y0.shape)
        xu.copy_(x)
        plan.forward(xu, w, yu, ws)
        torch.cuda.synchronize()
        assert torch.equal(yu, y0) and torch.isnan(yb[0])


def launches(torch, plan, call):
    """Names of the kernels that `call` launches, and its x, w, dy (random)."""
    dev = torch.device("cuda:0")
    ws = plan.workspace(dev)
    x, w, dy = (torch.randn(s, device=dev) for s in (plan.x_shape(), plan.w_shape(), plan.y_shape()))
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    plan.forward(x, w, y, ws)
    with blconv.Profile() as prof:
        if call == "backward":
            plan.backward(dy, None, None, dx, dw, ws, flags=blconv.BL_REUSE_X | blconv.BL_REUSE_W)
        else:
            plan.backward_weight(None, dy, dw, ws, flags=blconv.BL_REUSE_X)
        torch.cuda.synchronize()
    return [r[0] for r in prof.records()]


def test_weight_gradient_beside_the_inverse(torch):
    """On the FFT grids the combined backward call has its weight gradient's
    inverse in the launch of the input gradient's; with many planes and channel
    pairs a product of its own, before whose choice no other table is made."""
    for N, ci, co, hw, c in ((2, 3, 16, 32, 0.5), (4, 32, 32, 32, 0.5), (95, 64, 64, 32, 0.5), (96, 64, 63, 32, 0.5),
                             (2, 64, 64, 8, 0.5)):
        names = launches(torch, blconv.Plan(2, N, ci, co, (hw, hw), 3, (1, 1, 1, 1), c), "backward")
        assert "spec_inv_wgrad_2d" in names and "wgrad_idft" not in names, (N, ci, co, names)
    names = launches(torch, blconv.Plan(2, 96, 64, 64, (32, 32), 3, (1, 1, 1, 1), 0.5), "backward")
    assert "wgrad_idft" in names and "wgrad_reduce" not in names, names


@pytest.mark.parametrize("nd,N,ci,co,sp,K,c,product", [
    (2, 2, 32, 32, (26, 26), 3, 0.0, True),     # 420 bins
    (1, 2, 80, 128, (893,), 3, 0.0, True),      # 10240 channel pairs, 448 bins
    (1, 2, 80, 128, (895,), 3, 0.0, False),     # 449 bins
    (1, 2, 80, 129, (599,), 3, 0.0, False),     # one pair of channels more, 301 bins
    (1, 2, 120, 136, (509,), 3, 0.0, True),     # 16320 pairs, 256 bins
    (1, 2, 120, 136, (511,), 3, 0.0, False),    # 257 bins
    (1, 2, 2, 3, (1400,), 3, 0.0, False),       # 702 bins
])
def test_weight_gradient_by_product(torch, nd, N, ci, co, sp, K, c, product):
    """Bounds of the product that takes the place of the sliced weight-gradient
    inverse, each side against the oracle."""
    layer = synth.Layer("wgp", nd, N, ci, co, sp[0], sp[1] if nd == 2 else 1, K, (1, 1) * nd, "blur")
    plan = blconv.plan_for_layer(layer, c)
    names = launches(torch, plan, "weight")
    assert ("wgrad_reduce" not in names) == product, (plan.kept, names)
    x, w, dy = synth.random_inputs(layer, 4700 + ci)
    errs = [rel(g, r) for g, r in zip(gpu_passes(torch, layer, c, x, w, dy)[:3], oracle_passes(layer, c, x, w, dy))]
    say(f"[wgrad product] {ci}->{co} @{sp} {plan.kept} bins: {errs}")
    assert max(errs) <= FP32_TOL, errs


@pytest.mark.parametrize("N,ci,co,nd,sp,K,c,paired", [
    (18, 17, 496, 2, (8, 8), 1, 0.75, False),   # 31 stages of grad-input against 1 tile's load
    (4, 3, 340, 1, (60,), 3, 0.0, False),       # 22 stages, 6.5 apart
    (4, 3, 272, 1, (60,), 3, 0.0, True),        # 17 stages, 5.3 apart
    (18, 17, 512, 2, (8, 8), 1, 0.75, True),    # split in four: 8 stages
    (64, 64, 400, 1, (300,), 3, 0.5, True),     # two groups a tile apart: 16.5 of 25 stages
    (4, 17, 1000, 1, (700,), 3, 0.0, True),     # 63 stages within twice the load
])
def test_long_input_gradient_sums_run_apart(torch, N, ci, co, nd, sp, K, c, paired):
    """A few tiles with long sums leave the paired backward launch; either way
    against the oracle."""
    p = (K - 1) // 2
    layer = synth.Layer("long_sums", nd, N, ci, co, sp[0], sp[1] if nd == 2 else 1, K, (p, p) * nd, "blur")
    plan = blconv.plan_for_layer(layer, c)
    names = launches(torch, plan, "backward")
    assert ("contract_bwd" in names) == paired and ("contract_dgrad" in names) != paired, (plan.kept, names)
    x, w, dy = synth.random_inputs(layer, 4850 + co)
    ws = plan.workspace(torch.device("cuda:0"))
    xt, wt, dyt = (torch.from_numpy(a).to(ws.device) for a in (x, w, dy))
    dx, dw = torch.full_like(xt, float("nan")), torch.full_like(wt, float("nan"))
    plan.backward(dyt, wt, xt, dx, dw, ws)
    torch.cuda.synchronize()
    errs = [rel(g.cpu().numpy(), r) for g, r in zip((dx, dw), oracle_passes(layer, c, x, w, dy)[1:])]
    say(f"[long sums] {ci}->{co} @{sp} {plan.kept} bins: {errs}")
    assert max(errs) <= FP32_TOL, errs


@pytest.mark.parametrize("N,ci,co,nd,sp,paired", [
    (1, 16, 16, 1, (1277,), True),      # 640 bins
    (1, 16, 16, 1, (1279,), False),     # 641 bins
    (1, 128, 144, 1, (649,), False),    # 326 bins, 6008832 products
    (1, 128, 144, 1, (645,), True),     # 324 bins, 5971968 products
    (1, 256, 256, 1, (189,), True),     # 96 bins
    (1, 256, 256, 1, (191,), False),    # 97 bins
    (2, 3, 16, 1, (1399,), True),       # two images, 701 bins
])
def test_one_image_pairs_few_products(torch, N, ci, co, nd, sp, paired):
    """Bounds of the paired backward launch with one image, whose contractions
    run on the vector ALUs else; each side against the oracle."""
    layer = synth.Layer("pairs", nd, N, ci, co, sp[0], 1, 3, (1, 1) * nd, "walk")
    plan = blconv.plan_for_layer(layer, 0.0)
    names = launches(torch, plan, "backward")
    assert ("contract_bwd" in names) == paired and ("contract_dgrad" in names) != paired, (plan.kept, names)
    x, w, dy = synth.random_inputs(layer, 4800 + ci)
    ws = plan.workspace(torch.device("cuda:0"))
    xt, wt, dyt = (torch.from_numpy(a).to(ws.device) for a in (x, w, dy))
    dx, dw = torch.full_like(xt, float("nan")), torch.full_like(wt, float("nan"))
    plan.backward(dyt, wt, xt, dx, dw, ws)
    torch.cuda.synchronize()
    errs = [rel(g.cpu().numpy(), r) for g, r in zip((dx, dw), oracle_passes(layer, 0.0, x, w, dy)[1:])]
    say(f"[one image] {ci}->{co} @{sp} {plan.kept} bins: {errs}")
    assert max(errs) <= FP32_TOL, errs


@pytest.mark.parametrize("nd,N,ci,sp,K,c", [(2, 72, 64, (5, 5), 3, 0.75), (1, 32, 224, (1787,), 8, 0.0)])
def test_energies_over_many_planes(torch, nd, N, ci, sp, K, c):
    """Energies of spectra by one product: roundings of values average out over
    the planes, those of a bin's table do not.  A phase rounded to 24 bits alone
    gives 2^-25 on average; with its remainder only the operands' rounding is
    left, averaged over the sample pairs."""
    lo, hi = (K - 1) // 2, K - 1 - (K - 1) // 2
    plan = blconv.Plan(nd, N, ci, 1, sp, K, (lo, hi) * nd, c)
    dev = torch.device("cuda:0")
    x = torch.randn(plan.x_shape(), device=dev, generator=torch.Generator(device=dev).manual_seed(4970))
    got = plan.input_energy(x, plan.workspace(dev))
    u, v = (torch.from_numpy(a).to(dev).double() for a in plan.bins())
    lh, lw = plan.fft if nd == 2 else (1, plan.fft[0])
    rows = x.double().reshape(N * ci, sp[0] if nd == 2 else 1, -1)
    want = torch.zeros(plan.kept, dtype=torch.float64, device=dev)
    i, j = torch.meshgrid(*(torch.arange(n, device=dev).double() for n in rows.shape[1:]), indexing="ij")
    for at in range(0, plan.kept, 256):
        b = slice(at, at + 256)
        turns = u[b, None] * (i.reshape(1, -1) + (lo if nd == 2 else 0)) / lh + v[b, None] * (j.reshape(1, -1) + lo) / lw
        a = turns * (-2.0 * math.pi)
        flat = rows.reshape(N * ci, -1)
        want[b] = ((flat @ a.cos().T.contiguous()) ** 2 + (flat @ a.sin().T.contiguous()) ** 2).sum(0)
    want *= torch.where((v == 0) | (2 * v == lw), 1.0, 2.0)
    err = float((got - want).norm() / want.norm())
    say(f"[energies] {N * ci} planes of {sp}: {err}")
    assert err <= 1.2e-8, err


def test_tables_are_held_once(torch):
    """A series layer's transforms keep one table for the samples it takes and
    one for the samples it gives, whatever their place on the grid."""
    dev = torch.device("cuda:0")
    plan = blconv.Plan(1, 2, 2, 2, (2048,), 3, (1, 1), 0.0)
    ws = plan.workspace(dev)
    x, w, dy = (torch.randn(s, device=dev) for s in (plan.x_shape(), plan.w_shape(), plan.y_shape()))
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info(dev)[0]
    plan.forward(x, w, y, ws)
    plan.backward(dy, None, None, dx, dw, ws, flags=blconv.BL_REUSE_X | blconv.BL_REUSE_W)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info(dev)[0]
    one = 6 * plan.kept * 2048  # three bfloat16 of a cosine and a sine for a bin and two samples
    say(f"[tables] {held / 1e6:.1f} MB held, {2 * one / 1e6:.1f} MB of two tables")
    assert held <= 2 * one + (8 << 20)  # (tiles, the other tables, and memory given out in blocks of 2 MB)


@pytest.mark.parametrize("n", [240, 256, 270])
def test_small_tables_of_a_plan(torch, n):
    """Tables that share allocations: four of up to 256 KB, more than one
    allocation holds, and (270 samples) some past that size with small ones."""
    layer = synth.Layer("tables", 1, 3, 2, 5, n, 1, 8, (0, 0), "blur")
    x, w, dy = synth.random_inputs(layer, 4700 + n)
    got = gpu_passes(torch, layer, 0.0, x, w, dy, fft=300)
    errs = [rel(g, r) for g, r in zip(got[:3], oracle_passes(layer, 0.0, x, w, dy, 300))]
    say(f"[tables] {n} samples: {errs}")
    assert max(errs) <= FP32_TOL, errs


@pytest.mark.parametrize("nd,sp,K", [(2, (28, 21), 5), (2, (32, 32), 3), (1, (270,), 8)])
def test_first_calls_from_two_threads(torch, nd, sp, K):
    """A new plan's first calls, from two threads on streams and workspaces of
    their own: tables that one call makes are there for the other."""
    lo, hi = (K - 1) // 2, K - 1 - (K - 1) // 2
    layer = synth.Layer("threads", nd, 4, 24, 33, sp[0], sp[1] if nd == 2 else 1, K, (lo, hi) * nd, "blur")
    dev = torch.device("cuda:0")
    xt, wt, dyt = (torch.from_numpy(a).to(dev) for a in synth.random_inputs(layer, 4650))

    def buffers(plan):
        return plan.workspace(dev), torch.empty_like(dyt), torch.empty_like(xt), torch.empty_like(wt)

    def step(plan, b, stream=None):
        ws, y, dx, dw = b
        plan.forward(xt, wt, y, ws, stream=stream)
        plan.backward(dyt, None, None, dx, dw, ws, flags=blconv.BL_REUSE_X | blconv.BL_REUSE_W, stream=stream)

    plan = blconv.plan_for_layer(layer, 0.5)
    want = buffers(plan)
    step(plan, want)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for r in range(6):
        plan = blconv.plan_for_layer(layer, 0.5)
        got = [buffers(plan), buffers(plan)]
        torch.cuda.synchronize()
        together = threading.Barrier(2)
        failed = []

        def run(i):
            together.wait()
            try:
                step(plan, got[i], streams[i])
            except Exception as e:  # noqa: BLE001  -- reported below
                failed.append(e)

        threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not failed, failed
        for b in got:
            for a, e in zip(b[1:], want[1:]):
                assert torch.equal(a, e), r


@pytest.mark.parametrize("nd,sp,K", [(2, (28, 21), 5), (2, (9, 9), 3), (1, (270,), 8), (1, (512,), 5), (1, (900,), 3)])
def test_first_call_under_capture(torch, nd, sp, K):
    """A call captured before any table of its transforms is there (a table is
    allocated, and nothing may be during a capture) takes the paths without:
    the input gradient after an eager forward, and a plan's very first call.
    The direct sums' rounding grows as the root of their length: 2e-6 for 900
    terms, each rounding 2^-24 of partial sums up to the result."""
    lo, hi = (K - 1) // 2, K - 1 - (K - 1) // 2
    layer = synth.Layer("cold", nd, 4, 3, 5, sp[0], sp[1] if nd == 2 else 1, K, (lo, hi) * nd, "blur")
    dev = torch.device("cuda:0")
    x, w, dy = synth.random_inputs(layer, 4600)
    ref = oracle_passes(layer, 0.5, x, w, dy)
    xt, wt, dyt = (torch.from_numpy(a).to(dev) for a in (x, w, dy))
    y, dx = torch.empty_like(dyt), torch.empty_like(xt)
    for warm in (True, False):
        plan = blconv.plan_for_layer(layer, 0.5)
        ws = plan.workspace(dev)
        if warm:
            plan.forward(xt, wt, y, ws)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            if warm:
                plan.backward_input(dyt, None, dx, ws, flags=blconv.BL_REUSE_W)
            else:
                plan.forward(xt, wt, y, ws)
        for _ in range(3):
            (dx if warm else y).fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            e = rel((dx if warm else y).cpu().numpy(), ref[1 if warm else 0])
            say(f"[cold capture] {sp} K{K} warm={warm}: {e}")
            assert e <= 2e-6, (warm, e)
            plan.forward(xt, wt, y, ws)  # eager, with tables
            torch.cuda.synchronize()
            e = rel(y.cpu().numpy(), ref[0])
            assert e <= FP32_TOL, e


def test_noalloc_without_room_for_partial_spectra(torch):
    """A plan whose forward contraction splits its sums, with spectra that fill
    the allocation-free call's array: the sums stay whole and the call runs."""
    layer = synth.Layer("noalloc_full", 2, 16, 1024, 512, 4, 4, 3, (1, 1, 1, 1), "blur")
    x, w, _ = synth.random_inputs(layer, 4300)
    plan = blconv.plan_for_layer(layer, 0.25)
    spectra = plan.kept * (layer.N * layer.C_in + layer.C_in * layer.C_out + layer.N * layer.C_out) * 8
    assert spectra < 64 << 20 < spectra + 2 * plan.kept * layer.N * layer.C_out * 8
    xt, wt = (torch.from_numpy(a).to("cuda:0") for a in (x, w))
    y = torch.full(plan.y_shape(), float("nan"), device="cuda:0")
    plan.forward_noalloc(xt, wt, y)
    torch.cuda.synchronize()
    err = rel(y.cpu().numpy(), bo.forward(x, w, layer.pad, 0.25))
    say(f"[noalloc full] {err}")
    assert err <= FP32_TOL, err
