"""GPU parity of the masked SwiGLU MLP (forward and backward, both regimes) against the fp64 oracle.

Small and medium shapes: the oracle computes every output element.  Tolerances (metric in
helpers.err_report): 1e-5 for the fp32 path, 2e-2 for bf16 inputs with fp32 accumulation.
"""
import numpy as np
import pytest
import torch

import workloads
import rounding_model as rm
from helpers import assert_close, assert_close_with_model
from workloads import MlpWorkload

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def sdp():
    import paper_2507_09029_amd as m

    assert torch.cuda.is_available()
    m.lib()
    return m


def run_case(sdp, orc, w, workers, dw_layout="compact", dw_elem_tol=None):
    """dw_elem_tol: elementwise bound for the weight gradients when it differs from the tolerance (see
    test_gpu_random_shapes.py); the normwise bound is always the tolerance."""
    tol = TOL[w.dtype]
    W1, W3, W2T = workloads.mlp_weights(w)
    dW = [t.cuda() for t in (W1, W3, W2T)]
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    want_mask = orc.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    assert (mask.cpu().numpy() == want_mask).all()
    W64 = [workloads.to_f64(t) for t in (W1, W3, W2T)]
    for k in workers:
        print(f"  {w.name} worker {k} {w.mode} {w.dtype} T={w.T} d={w.d} F={w.F} p={w.p} {dw_layout}", flush=True)
        X, dY = workloads.mlp_batch(w, k)
        Y, G, U = sdp.masked_mlp_fwd(w.mode, X.cuda(), *dW, idx[k])
        if dw_layout == "scatter":
            out = (torch.empty((w.T, w.d), dtype=X.dtype, device="cuda"),) + tuple(
                torch.full((w.F, w.d), float("nan"), dtype=X.dtype, device="cuda") for _ in range(3))
        else:
            out = None
        dX, dW1, dW3, dW2T = sdp.masked_mlp_bwd(w.mode, X.cuda(), dY.cuda(), *dW, idx[k], G, U, dw_layout=dw_layout, out=out)
        torch.cuda.synchronize()
        ref = orc.worker_step(w.mode, want_mask[k], workloads.to_f64(X), workloads.to_f64(dY), *W64)
        S = np.flatnonzero(want_mask[k])
        model = None
        assert ref["nonzero_off_mask"] == 0
        assert_close(workloads.to_f64(Y), ref["Y"], tol, "Y")
        assert_close(workloads.to_f64(dX), ref["dX"], tol, "dX")
        cols = S if w.mode == "fm" else slice(None)
        assert_close(workloads.to_f64(G), ref["G"][:, cols], tol, "G")
        assert_close(workloads.to_f64(U), ref["U"][:, cols], tol, "U")
        for name, got in (("dW1", dW1), ("dW3", dW3), ("dW2T", dW2T)):
            g64 = workloads.to_f64(got)
            if dw_layout == "scatter":
                off = np.flatnonzero(want_mask[k] == 0)
                assert np.isnan(g64[off]).all(), "rows off the mask must stay untouched"
                g64 = g64[S]
            if w.dtype == "bf16":
                # no further from the oracle than the bf16 rounding points alone put the result (see helpers)
                if model is None:
                    model = rm.mlp_model(w.mode, want_mask[k], workloads.to_f64(X), workloads.to_f64(dY), *W64)
                assert_close_with_model(g64, model[name][S], ref[name][S], tol, name, elem_allow=dw_elem_tol)
            else:
                assert_close(g64, ref[name][S], tol, name, elem_tol=dw_elem_tol)


SMALL = [
    MlpWorkload("tiny_f32_fm", "f32", 8, 8, 16, 8, 2, "fm", 11),
    MlpWorkload("ragged_f32_fm", "f32", 77, 40, 130, 37, 4, "fm", 12),
    MlpWorkload("ragged_f32_bm", "f32", 77, 40, 130, 37, 4, "bm", 12),
    MlpWorkload("full_cover_f32_fm", "f32", 64, 32, 64, 64, 2, "fm", 13),       # C = 1: the dense MLP
    MlpWorkload("tiles_bf16_fm", "bf16", 264, 136, 520, 264, 4, "fm", 14),      # several tiles + ragged tails
    MlpWorkload("tiles_bf16_bm", "bf16", 264, 136, 520, 264, 4, "bm", 14),
    MlpWorkload("tails16_bf16_fm", "bf16", 272, 144, 528, 272, 4, "fm", 18),    # MFMA path, every depth ends in a partial step
    MlpWorkload("tails16_bf16_bm", "bf16", 272, 144, 528, 304, 4, "bm", 18),
    MlpWorkload("tails48_bf16_fm", "bf16", 304, 176, 560, 240, 4, "fm", 19),    # depth tails of 48, ragged rows / columns
    MlpWorkload("aligned_bf16_fm", "bf16", 512, 256, 1024, 512, 4, "fm", 15),
    MlpWorkload("aligned_bf16_bm", "bf16", 512, 256, 1024, 768, 4, "bm", 16),
    MlpWorkload("full_cover_bf16_bm", "bf16", 256, 128, 256, 256, 2, "bm", 17),
    MlpWorkload("tiny_bf16_fm", "bf16", 8, 16, 32, 16, 2, "fm", 20),            # one MFMA tile, almost all of it out of range
    MlpWorkload("tiny_bf16_bm", "bf16", 16, 16, 48, 16, 3, "bm", 21),
    MlpWorkload("full_cover_bf16_fm", "bf16", 48, 64, 128, 128, 2, "fm", 22),   # C = 1 on the MFMA path
]


# every contraction depth (d, p or F, T) an odd multiple of 8: partial last steps of 8, 24, 40 and 56
ODD_DEPTHS = [MlpWorkload(f"tails{t}_bf16_{mode}", "bf16", 128 + t, 64 + t, 256 + t, 192 + t, 2, mode, 24)
              for t in (8, 24, 40, 56) for mode in ("fm", "bm")]


@pytest.mark.parametrize("w", ODD_DEPTHS, ids=[w.name for w in ODD_DEPTHS])
def test_depths_that_are_odd_multiples_of_8(sdp, orc, w):
    run_case(sdp, orc, w, [0, 1], dw_layout="scatter" if w.mode == "bm" else "compact")


# fp32 contraction: extents around the edges of its 32- and 64-wide tiles and of its depth steps (single-element and
# 16-byte loads), and one case per operand layout that is large enough for the 128-wide tile
F32_TILES = [MlpWorkload(f"f32_{T}x{d}x{F}p{p}_{mode}", "f32", T, d, F, p, 2, mode, 25) for T, d, F, p, mode in (
    (1, 1, 3, 2, "fm"), (31, 33, 70, 65, "bm"), (32, 64, 128, 64, "fm"), (65, 31, 130, 127, "bm"), (64, 96, 192, 96, "bm"),
    (129, 63, 140, 100, "fm"), (200, 132, 516, 260, "bm"), (2040, 40, 2040, 2040, "fm"), (40, 2040, 2040, 1020, "bm"),
    (2040, 2040, 64, 33, "fm"))]


# 16 x 16 tiles (depths around the 32 steps a wave takes and the 128 its workgroup does, rows and columns that end inside a
# tile, a list longer than the kernel keeps), and dX and dW as one launch with either tile
F32_FEW = [MlpWorkload(f"few_{T}x{d}x{F}p{p}_{mode}", "f32", T, d, F, p, 2, mode, 26) for T, d, F, p, mode in (
    (4, 4, 8, 4, "fm"), (33, 36, 200, 124, "fm"), (100, 132, 300, 260, "bm"), (17, 260, 64, 36, "fm"), (260, 256, 520, 388, "fm"),
    (16, 20, 4400, 4200, "fm"), (300, 700, 400, 204, "fm"), (52, 64, 40, 40, "bm"))]


@pytest.mark.parametrize("w", F32_FEW, ids=[w.name for w in F32_FEW])
def test_f32_few_tiles(sdp, orc, w):
    run_case(sdp, orc, w, [1], dw_layout="scatter" if w.T % 2 else "compact")


def test_f32_dx_may_take_the_place_of_dy(sdp):
    """dX written over dY, which the weight gradients read."""
    w = F32_FEW[4]
    Wd = [t.cuda() for t in workloads.mlp_weights(w)]
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    X, dY = (t.cuda() for t in workloads.mlp_batch(w, 0))
    Y, G, U = sdp.masked_mlp_fwd(w.mode, X, *Wd, idx[0])
    want = sdp.masked_mlp_bwd(w.mode, X, dY, *Wd, idx[0], G, U)
    out = (dY.clone(),) + tuple(torch.empty_like(t) for t in want[1:])
    got = sdp.masked_mlp_bwd(w.mode, X, out[0], *Wd, idx[0], G, U, out=out)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert (a - b).abs().max() <= 1e-5 * b.abs().max()


# outputs in the memory of operands: (output position in the call's results, operand)
TAKEN = {"dX over dY": {0: "dY"}, "dX over X": {0: "X"}, "gradients over weights": {1: "W1", 2: "W3", 3: "W2T"},
         "dX over X, gradients over weights": {0: "X", 1: "W1", 2: "W3", 3: "W2T"}, "gradients over other weights": {1: "W3", 2: "W1"},
         "a gradient over dY and X": {1: "dY", 2: "X"}}


@pytest.mark.parametrize("taken", TAKEN.values(), ids=TAKEN.keys())
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode,layout,T,p", [("fm", "scatter", 264, 136), ("bm", "scatter", 264, 136), ("fm", "compact", 136, 136)])
def test_outputs_may_take_the_place_of_operands(sdp, mode, layout, T, p, dtype, taken):
    """The backward pass reads every operand before an output is written, in both dtypes."""
    w = MlpWorkload("in_place", dtype, T, 72, 264, p, 2, mode, 27)
    names = ("W1", "W3", "W2T")
    op = dict(zip(names, (t.cuda() for t in workloads.mlp_weights(w))))
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    op["X"], op["dY"] = (t.cuda() for t in workloads.mlp_batch(w, 0))
    Y, G, U = sdp.masked_mlp_fwd(mode, op["X"], *(op[n] for n in names), idx[0])
    dw_shape = (w.F if layout == "scatter" else p, w.d)

    def bwd(o, out):
        return sdp.masked_mlp_bwd(mode, o["X"], o["dY"], *(o[n] for n in names), idx[0], G, U, dw_layout=layout, out=out)

    fresh = [torch.zeros_like(op["X"])] + [torch.zeros(dw_shape, dtype=Y.dtype, device="cuda") for _ in range(3)]
    want = bwd(op, tuple(fresh))
    mine = {n: t.clone() for n, t in op.items()}
    out = tuple(mine[taken[i]].view(-1)[: t.numel()].view(t.shape) if i in taken and mine[taken[i]].numel() >= t.numel() else t.clone()
                for i, t in enumerate(fresh))
    got = bwd(mine, out)
    rows = idx[0].long() if layout == "scatter" else slice(None)
    for i, (a, b) in enumerate(zip(got, want)):
        if i > 0:
            a, b = a[rows], b[rows]
        # the same products; fp32 sums may come from another launch shape
        assert (a.double() - b.double()).abs().max() <= (1e-5 if dtype == "f32" else 1e-2) * b.abs().max(), f"output {i}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", ["fm", "bm"])
@pytest.mark.parametrize("taken", [0, 1, 2], ids=["Y", "G", "U"])
def test_forward_outputs_may_take_the_place_of_W2(sdp, dtype, mode, taken):
    w = MlpWorkload("in_place_fwd", dtype, 136, 264, 264, 136, 2, mode, 28)
    W1, W3, W2T = (t.cuda() for t in workloads.mlp_weights(w))
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    X = workloads.mlp_batch(w, 0)[0].cuda()
    want = sdp.masked_mlp_fwd(mode, X, W1, W3, W2T, idx[0])
    mine = W2T.clone()
    out = [torch.empty_like(t) for t in want]
    out[taken] = mine.view(-1)[: want[taken].numel()].view(want[taken].shape)
    got = sdp.masked_mlp_fwd(mode, X, W1, W3, mine, idx[0], out=tuple(out))
    for a, b in zip(got, want):
        assert (a.double() - b.double()).abs().max() <= (1e-5 if dtype == "f32" else 1e-2) * b.abs().max()


def test_f32_more_tiles_than_one_launch_holds(sdp):
    """F = 2^29 + 64 columns of one token: more 32-wide tiles than a launch of 256-thread workgroups takes."""
    F, d = (1 << 29) + 64, 4
    X = torch.tensor([[0.5, -0.25, 1.0, 0.75]], device="cuda")
    W1, W3 = (torch.ones((F, d), device="cuda") for _ in range(2))
    W2T = torch.zeros((F, d), device="cuda")
    rows = torch.tensor([0, 1, 12345, 1 << 28, F - 65, F - 2, F - 1], device="cuda")
    W2T[rows] = torch.arange(28, dtype=torch.float32, device="cuda").view(7, 4) - 11.0
    print(f"f32 bm T=1 d={d} F={F}", flush=True)
    Y, G, U = sdp.masked_mlp_fwd("bm", X, W1, W3, W2T, None)
    assert bool((G == 2.0).all()) and bool((U == 2.0).all())
    act = 4.0 / (1.0 + np.exp(-2.0))
    want = act * W2T[rows].double().sum(0)
    assert float((Y[0].double() - want).abs().max() / want.abs().max()) <= 1e-5


def test_rows_beyond_the_mfma_kernels_address_range(sdp, orc):
    """F = 2^22 + 8 under backward masking: rows of 2^22 elements and more leave the MFMA kernel's address range, so gate_up,
    down, dact (with the column-compacted copies), dX and the three weight gradients (depth-major left operands) run on the plain
    bf16 kernel, the transposes in launches of their own.  The weight gradients sum over 8 tokens only, as in the small
    random shapes (test_gpu_random_shapes.py), but have 1.7e7 elements: the rounding points alone put their elementwise maxima
    at 4.0e-2, 5.2e-2 and 5.7e-2 (rounding model, on the CPU), so the fixed bound is 8e-2 and the model-relative check (1.5 times
    those figures) is the tighter one."""
    T, d, F, p = 8, 8, (1 << 22) + 8, 1 << 21
    w = MlpWorkload("plain_bf16_bm", "bf16", T, d, F, p, 2, "bm", 29)
    Wh = workloads.mlp_weights(w)
    W, W64 = [t.cuda() for t in Wh], [workloads.to_f64(t) for t in Wh]
    mask, idx, pos, cov = sdp.make_masks(w.K, F, p, w.mask_seed, False)
    m = orc.make_masks(w.K, F, p, w.mask_seed, False)[1]
    assert (mask[1].cpu().numpy() == m).all()
    X, dY = workloads.mlp_batch(w, 1)
    sdp.profile_filter(None)
    sdp.profile_reset()
    sdp.profile_enable(True)
    try:
        Y, G, U = sdp.masked_mlp_fwd("bm", X.cuda(), *W, idx[1])
        dX, *dW = sdp.masked_mlp_bwd("bm", X.cuda(), dY.cuda(), *W, idx[1], G, U)
        torch.cuda.synchronize()
        launches = {name: calls for name, (calls, ms) in sdp.profile_read().items()}
    finally:
        sdp.profile_enable(False)
    assert launches["mlp_dw"] == 3 and launches["mlp_tr_bwd"] == 1 and launches["mlp_wt_fwd"] == 1, launches
    X, dY = workloads.to_f64(X), workloads.to_f64(dY)
    ref = orc.worker_step("bm", m, X, dY, *W64)
    for name, got in (("Y", Y), ("G", G), ("U", U), ("dX", dX)):
        assert_close(workloads.to_f64(got), ref[name], 2e-2, name)
    S = np.flatnonzero(m)
    ref = {n: ref[n][S] for n in ("dW1", "dW3", "dW2T")}
    model = rm.mlp_model("bm", m, X, dY, *W64)
    for name, got in zip(("dW1", "dW3", "dW2T"), dW):
        assert_close_with_model(workloads.to_f64(got), model[name][S], ref[name], 2e-2, name, elem_allow=8e-2)


@pytest.mark.parametrize("w", F32_TILES, ids=[w.name for w in F32_TILES])
def test_f32_tiles(sdp, orc, w):
    run_case(sdp, orc, w, [1], dw_layout="scatter" if w.T % 2 else "compact")


@pytest.mark.parametrize("w", SMALL, ids=[w.name for w in SMALL])
def test_small_shapes_all_outputs(sdp, orc, w):
    run_case(sdp, orc, w, range(min(w.K, 2)))


def test_config1_all_workers(sdp, orc):
    run_case(sdp, orc, workloads.CONFIG1, range(workloads.CONFIG1.K))


def test_scatter_layout_leaves_off_mask_rows_alone(sdp, orc):
    run_case(sdp, orc, SMALL[1], [0], dw_layout="scatter")
    run_case(sdp, orc, SMALL[5], [1], dw_layout="scatter")


def test_config1_full_step_average(sdp, orc):
    """Whole path at config 1: masks -> K workers' fwd+bwd (scatter layout) -> coverage average."""
    w = workloads.CONFIG1
    W1, W3, W2T = workloads.mlp_weights(w)
    dW = [t.cuda() for t in (W1, W3, W2T)]
    W64 = [workloads.to_f64(t) for t in (W1, W3, W2T)]
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    want_mask = orc.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    bufs = [torch.full((3 * w.F, w.d), float("nan"), dtype=torch.float32, device="cuda") for _ in range(w.K)]
    ref_bufs = []
    for k in range(w.K):
        X, dY = workloads.mlp_batch(w, k)
        Y, G, U = sdp.masked_mlp_fwd("fm", X.cuda(), *dW, idx[k])
        out = (torch.empty((w.T, w.d), dtype=torch.float32, device="cuda"),
               bufs[k][0:w.F], bufs[k][w.F:2 * w.F], bufs[k][2 * w.F:])
        sdp.masked_mlp_bwd("fm", X.cuda(), dY.cuda(), *dW, idx[k], G, U, dw_layout="scatter", out=out)
        r = orc.worker_step("fm", want_mask[k], workloads.to_f64(X), workloads.to_f64(dY), *W64)
        ref_bufs.append(np.concatenate([r["dW1"], r["dW3"], r["dW2T"]]))
    row_mask = mask.repeat(1, 3).contiguous()  # neuron j owns row j of each of the three matrices
    avg, c = sdp.coverage_grad_avg(bufs, row_mask)
    torch.cuda.synchronize()
    want, wc = orc.gated_average(ref_bufs, np.tile(want_mask, (1, 3)))
    assert (c.cpu().numpy() == wc).all() and wc.min() >= 1
    assert_close(avg.cpu().numpy(), want, 1e-5, "averaged gradient")


@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_fp32_path_and_bf16_path_agree_on_the_same_inputs(sdp, mode):
    """The same bf16-valued inputs through the fp32 kernels (fp32 matrix instructions, no intermediate rounding) and
    through the bf16 MFMA kernels: two implementations inside the library that share no contraction code must
    agree to the bf16 path's rounding (about 1e-2), without the oracle in between."""
    from helpers import err_report

    w = MlpWorkload("paths", "bf16", 512, 256, 1024, 512, 2, mode, 61)
    W = workloads.mlp_weights(w)
    X, dY = workloads.mlp_batch(w, 0)
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    outs = {}
    for name, conv in (("bf16", lambda t: t.cuda()), ("f32", lambda t: t.float().cuda())):
        Wd = [conv(t) for t in W]
        Y, G, U = sdp.masked_mlp_fwd(mode, conv(X), *Wd, idx[0])
        dX, dW1, dW3, dW2T = sdp.masked_mlp_bwd(mode, conv(X), conv(dY), *Wd, idx[0], G, U)
        torch.cuda.synchronize()
        outs[name] = [workloads.to_f64(t) for t in (Y, G, U, dX, dW1, dW3, dW2T)]
    for got, ref, what in zip(outs["bf16"], outs["f32"], ("Y", "G", "U", "dX", "dW1", "dW3", "dW2T")):
        elem, norm = err_report(got, ref)
        assert norm <= 1e-2 and elem <= 2e-2, f"{what}: elementwise {elem:.3e}, normwise {norm:.3e}"


def _filled(shape, dtype, fill):
    """A GPU tensor whose bytes are all zero, all 0xFF (NaN in bf16 and fp32) or all 0x46 (about 1.3e4 in both)."""
    t = torch.empty(shape, dtype=dtype, device="cuda")
    t.view(torch.uint8).fill_({"zero": 0, "nan": 0xFF, "big": 0x46}[fill])
    return t


POISON = [w for w in SMALL if w.name in ("ragged_f32_fm", "tiles_bf16_fm", "tiles_bf16_bm", "aligned_bf16_bm", "tiny_bf16_fm")] + [
    MlpWorkload("partial_steps_bf16_fm", "bf16", 552, 440, 1536, 1312, 4, "fm", 23),  # every depth ends in a partial step
]


@pytest.mark.parametrize("w", POISON, ids=[w.name for w in POISON])
def test_results_do_not_depend_on_what_workspace_and_outputs_held(sdp, w):
    """Nothing uninitialised is read: the same calls with the workspaces and every output buffer pre-filled with
    NaN patterns, or with large finite values, give the bits they give over zeroed buffers."""
    Wd = [t.cuda() for t in workloads.mlp_weights(w)]
    mask, idx, pos, cov = sdp.make_masks(w.K, w.F, w.p, w.mask_seed, True)
    k = w.K - 1
    X, dY = (t.cuda() for t in workloads.mlp_batch(w, k))
    n = w.p if w.mode == "fm" else w.F
    res = {}
    for fill in ("zero", "nan", "big"):
        wsf = _filled((sdp.masked_mlp_fwd_workspace_bytes(w.mode, X.dtype, w.T, w.d, w.F, w.p) + 256,), torch.uint8, fill)
        wsb = _filled((sdp.masked_mlp_bwd_workspace_bytes(w.mode, X.dtype, w.T, w.d, w.F, w.p) + 256,), torch.uint8, fill)
        fo = (_filled((w.T, w.d), X.dtype, fill), _filled((w.T, n), X.dtype, fill), _filled((w.T, n), X.dtype, fill))
        Y, G, U = sdp.masked_mlp_fwd(w.mode, X, *Wd, idx[k], out=fo, ws=wsf)
        bo = (_filled((w.T, w.d), X.dtype, fill),) + tuple(_filled((w.p, w.d), X.dtype, fill) for _ in range(3))
        back = sdp.masked_mlp_bwd(w.mode, X, dY, *Wd, idx[k], G, U, out=bo, ws=wsb)
        torch.cuda.synchronize()
        res[fill] = [t.clone().view(torch.uint8) for t in (Y, G, U) + tuple(back)]
    for fill in ("nan", "big"):
        for name, a, b in zip(("Y", "G", "U", "dX", "dW1", "dW3", "dW2T"), res["zero"], res[fill]):
            assert torch.equal(a, b), f"{w.name}: {name} depends on the previous contents of a buffer ({fill})"


def test_compiled_calls_name_the_argument_they_refuse(sdp):
    X = torch.zeros(8, 16, dtype=torch.bfloat16, device="cuda")
    W = torch.zeros(24, 16, dtype=torch.bfloat16, device="cuda")
    idx = torch.arange(8, dtype=torch.int32, device="cuda")
    for args, what in (((X, W, W.float(), W, idx), "W3: expected a contiguous torch.bfloat16"),
                       ((X, W, W.t().contiguous().t(), W, idx), "W3: expected a contiguous torch.bfloat16"),
                       ((X, W, W, W.cpu(), idx), "W2T: expected a contiguous torch.bfloat16"),
                       ((X, W, W, W, idx.long()), "idx_k: expected a contiguous torch.int32")):
        with pytest.raises(TypeError, match=what):
            sdp.masked_mlp_fwd("fm", *args)
    with pytest.raises(TypeError, match="dY: expected"):
        sdp.masked_mlp_bwd("fm", X, None, W, W, W, idx, X, X)
