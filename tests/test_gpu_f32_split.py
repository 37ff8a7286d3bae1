"""GPU: the fp32 contraction's tiles of split products (three bf16 terms an operand): one and two teams of waves, every operand
layout, partial last steps and tiles, listed rows, depths and columns, dX and the weight gradients together and apart: 1e-5 against the
fp64 oracle; each test sees to it that these tiles ran.  Which sizes take them.  Operands that are not finite, or that no bf16 holds, give
what fp32 products give."""
import pytest
import torch

import test_gpu_attn as attn
import test_gpu_mlp as mlp
from workloads import AttnWorkload, MlpWorkload

pytestmark = pytest.mark.gpu
sdp = mlp.sdp  # the fixture

# what splits of a pass: gate_up, dact, down, dX, weight gradients
CASES = [(MlpWorkload(f"{T}x{d}x{F}p{p}_{mode}", "f32", T, d, F, p, 2, mode, 91), split.split()) for T, d, F, p, mode, split in (
    # gate_up in 160 to 170 tiles (two teams), depths of one element more and less than whole steps, and of whole steps (an even and an odd
    # number); in 320
    (640, 321, 1000, 511, "fm", "gate_up"), (620, 351, 1000, 501, "fm", "gate_up"), (613, 352, 1000, 512, "fm", "gate_up"),
    (640, 320, 1000, 512, "fm", "gate_up"), (640, 320, 1000, 500, "bm", "gate_up"),
    # dact in 256 tiles, in 357, in 240 of single floats
    (1024, 256, 1100, 1024, "fm", "gate_up dact dw"), (1300, 400, 1030, 1028, "fm", "gate_up dact down dx dw"),
    (1024, 701, 1000, 901, "fm", "gate_up dact down dx dw"),
    # down and dX of single floats in 128 tiles, lists of depths of 10 and 12 steps; in 136 of four floats; in 336
    (1023, 511, 600, 301, "fm", "gate_up down dx"), (1001, 501, 400, 353, "fm", "gate_up down dx dw"), (1021, 510, 607, 321, "bm", "gate_up down dx dw"),
    (500, 1032, 1100, 1024, "fm", "gate_up down dx dw"), (1300, 1000, 600, 517, "fm", "down dx dw"),
    # weight gradients in a launch of their own: columns in order and listed, last tiles of 1 and 60 columns
    (1030, 260, 1030, 1027, "fm", "dw"), (1000, 700, 1100, 700, "fm", "gate_up dw"), (519, 769, 900, 577, "bm", "gate_up dw"),
    (600, 1100, 900, 701, "bm", "gate_up dw"),
    # and beside dX, in 32- and 16-wide tiles
    (449, 300, 1400, 701, "fm", "dw"), (480, 300, 1400, 700, "bm", "gate_up dw"), (500, 321, 1400, 705, "bm", "gate_up dact dw"),
    (450, 132, 2100, 1588, "fm", "dw"))]


def _launched(sdp, names, call, *args, **kw):
    """what the call returns, and the loop that each of the named launches took"""
    sdp.profile_filter(None)
    sdp.profile_enable(True)
    out = call(*args, **kw)
    sdp.profile_enable(False)
    return out, [sdp.profile_launch_shape(n)["loop"] for n in names]


MLP = ("gate_up", "dact", "down", "dx", "dw")


def _run(sdp, orc, w):
    return _launched(sdp, [f"mlp_{k}" for k in MLP], mlp.run_case, sdp, orc, w, [1], dw_layout="scatter" if w.p % 2 else "compact")[1]


@pytest.mark.parametrize("w,split", CASES, ids=[w.name for w, _ in CASES])
def test_f32_split_tiles(sdp, orc, w, split):
    loops = _run(sdp, orc, w)
    assert {k for k, v in zip(MLP, loops) if "split" in v} == set(split), loops


# dX in 16-wide tiles beside weight gradients in 32-wide ones of one LDS stage (513 to 768 tiles in all): none to three steps a wave, four
# floats, single ones and listed columns
ONE_STAGE = [MlpWorkload(f"one_stage_{T}x{d}x{F}p{p}_{mode}", "f32", T, d, F, p, 2, mode, 93) for T, d, F, p, mode in (
    (256, 256, 600, 512, "fm"), (256, 251, 600, 511, "fm"), (96, 960, 120, 64, "fm"), (96, 960, 100, 63, "bm"), (129, 640, 250, 128, "fm"),
    (129, 639, 250, 127, "bm"), (300, 300, 400, 204, "bm"), (300, 301, 400, 205, "fm"), (256, 256, 600, 512, "bm"), (250, 251, 600, 511, "bm"))]


@pytest.mark.parametrize("w", ONE_STAGE, ids=[w.name for w in ONE_STAGE])
def test_f32_gradients_in_one_stage(sdp, orc, w):
    assert _run(sdp, orc, w)[-1] == "waves, one stage"


# sizes at both sides of the lines between the loops
@pytest.mark.parametrize("T,d,F,p,mode,launch,loop", [
    # one round of split tiles against two and three rounds of 32-wide ones, two against four and six
    (416, 1176, 1824, 1824, "fm", "down", "staged"), (512, 1100, 1376, 1376, "fm", "down", "split, two teams"), (1518, 668, 1444, 1444, "fm", "dx", "staged"),
    (1300, 800, 816, 816, "fm", "dx", "split"), (2041, 516, 620, 620, "fm", "dw", "staged"),
    # depth against 64-wide tiles; single floats in less than 150 tiles
    (528, 280, 536, 536, "fm", "gate_up", "pipelined"), (1024, 496, 312, 312, "fm", "gate_up", "split, two teams"), (278, 367, 818, 818, "fm", "gate_up", "waves"),
    # the activation gradient's rows: no multiples of four floats; single-float loads
    (900, 576, 1407, 1407, "fm", "dact", "staged"), (599, 367, 799, 799, "fm", "dact", "waves"), (964, 807, 621, 621, "fm", "dact", "split, two teams"),
    # listed columns of the gradients
    (408, 676, 636, 372, "bm", "dw", "pipelined"), (2160, 460, 2244, 948, "bm", "dw", "split")])
def test_f32_loop_by_size(sdp, T, d, F, p, mode, launch, loop):
    assert _loop(sdp, T, d, F, p, mode, launch) == loop


# the gradients beside dX: tiles that fit the chip at once, listed columns
@pytest.mark.parametrize("T,d,F,p,mode,loop", [(948, 200, 880, 880, "fm", "waves"), (1136, 168, 1064, 1064, "fm", "split"), (468, 220, 2152, 1536, "bm", "pipelined"),
                                               (558, 388, 1144, 737, "bm", "split"), (502, 235, 2039, 1441, "bm", "pipelined"),
                                               (504, 216, 792, 776, "bm", "waves"), (609, 112, 3032, 2249, "bm", "split")])
def test_f32_loop_of_gradients_beside_dx(sdp, T, d, F, p, mode, loop):
    assert _loop(sdp, T, d, F, p, mode, "dw") == loop


# and one LDS stage or two, by dX's depth
@pytest.mark.parametrize("T,d,F,p,mode,loop", [(256, 153, 861, 861, "fm", "waves"), (256, 153, 861, 861, "bm", "waves"), (424, 121, 849, 849, "fm", "waves"),
                                               (288, 217, 677, 600, "bm", "waves, one stage"), (592, 133, 705, 705, "fm", "waves, one stage")])
def test_f32_one_stage_or_two(sdp, T, d, F, p, mode, loop):
    assert _loop(sdp, T, d, F, p, mode, "dw") == loop


def _loop(sdp, T, d, F, p, mode, launch):
    X, dY, W = _inputs(T, d, F, 96)
    idx = torch.arange(F - p, F, dtype=torch.int32, device="cuda")

    def both():
        _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
        sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U)

    return _launched(sdp, [f"mlp_{launch}"], both)[1][0]


def _inputs(T, d, F, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return _normal(T, d, scale=1.0, gen=g), _normal(T, d, scale=1.0, gen=g), [_normal(F, d, scale=0.02, gen=g) for _ in range(3)]


# the attention's gradients (three of dQKV at offset columns and one of dWo) beside its dX: heads in order and listed, 16-byte loads and
# single floats; listed heads of a multiple of 8 stay with the fp32 tiles, there and in launches of their own
@pytest.mark.parametrize("Bt,S,d,H,hd,ph,mode,layout,loop", [
    (2, 256, 512, 8, 64, 8, "fm", "compact", "split"), (1, 450, 500, 10, 50, 10, "fm", "scatter", "split"), (1, 450, 500, 10, 50, 7, "bm", "scatter", "split"),
    (2, 225, 500, 10, 50, 7, "fm", "scatter", "split"), (1, 449, 501, 10, 50, 8, "bm", "compact", "split"), (2, 242, 449, 14, 32, 12, "bm", "compact", "split"),
    (2, 256, 512, 8, 64, 5, "bm", "compact", "waves"), (1, 520, 929, 29, 32, 18, "bm", "scatter", "waves")])
def test_f32_split_gradients_of_attention(sdp, orc, Bt, S, d, H, hd, ph, mode, layout, loop):
    w = AttnWorkload(f"split_{Bt}x{S}x{d}_{H}x{hd}_{ph}", Bt, S, d, H, hd, ph, 2, 97, "f32")
    sdp.profile_reset()
    loops = _launched(sdp, ["attn_dw"], attn.run_case, sdp, orc, w, [1], dw_layout=layout, mode=mode)[1]
    assert loops == [loop] and ("attn_dx_dw" in sdp.profile_read()) == (d < 600), loops


# Error against 64 bits, normwise, of the same sums in split tiles and with the fp32 instruction.  One accumulator for all products would
# leave 3.5e-7 at 512 products (the fp32 instruction 4.4e-7); the small ones in an accumulator of their own leave 1.3e-7, which is also below
# the launch of few columns here, whose four waves add a quarter of the depth each (2.1e-7).
@pytest.mark.parametrize("T,d", [(1024, 512), (1024, 1536), (1023, 511)])
def test_f32_split_error_is_below_that_of_the_fp32_instruction(sdp, T, d):
    X, _, W = _inputs(T, d, 1024, 98)
    off = []
    for n, split in ((1024, True), (16, False)):
        idx = torch.arange(n, dtype=torch.int32, device="cuda")
        (_, G, U), loops = _launched(sdp, ["mlp_gate_up"], sdp.masked_mlp_fwd, "fm", X, *(t[:n] for t in W), idx)
        assert ("split" in loops[0]) == split, loops
        off.append(max(_off(G, X.double() @ W[0][:n].double().t()), _off(U, X.double() @ W[1][:n].double().t())))
    assert off[0] <= 0.8 * off[1], off


# Rows with one bad element: G and U are then infinite, not a number or, for the largest float, finite where fp32 products are; all
# other rows are untouched.  Reference: plain PyTorch in fp64, whose products of these do not overflow, rounded to fp32; 257 to 512
# products summed in fp32 stay below 1e-5 normwise.
@pytest.mark.parametrize("T,d,F", [(640, 257, 520), (1024, 512, 1024)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), 3.4028234e38, -3.4e38])
def test_f32_split_operands_that_are_not_finite(sdp, T, d, F, bad):
    g = torch.Generator(device="cuda")
    g.manual_seed(92)
    rnd = lambda *s, std=1.0: torch.randn(s, generator=g, device="cuda") * std
    X, W = rnd(T, d), [rnd(F, d, std=0.02) for _ in range(3)]
    W[0][5, 3] = 0.0
    X[70, 3] = X[T - 1, d - 1] = bad
    idx = torch.arange(F, dtype=torch.int32, device="cuda")
    Y, G, U = sdp.masked_mlp_fwd("fm", X, *W, idx)
    for got, w in ((G, W[0]), (U, W[1])):
        want = (X.double() @ w.double().t()).float()
        for row in (70, T - 1):
            assert torch.equal(got[row].isnan(), want[row].isnan())
            keep = ~want[row].isnan()
            inf = want[row].isinf() & keep
            assert torch.equal(got[row][inf], want[row][inf])
            assert torch.allclose(got[row][keep & ~inf], want[row][keep & ~inf], rtol=1e-5, atol=0)
        rest = torch.ones(T, dtype=torch.bool, device="cuda")
        rest[70] = rest[T - 1] = False
        assert float((got[rest].double() - want[rest].double()).norm() / want[rest].double().norm()) <= 1e-5


# One element that is not finite or too large for the split terms' scale, in each operand of the backward pass and of down, in launches that
# split: a tile that it reaches is computed again with the fp32 instruction, and its other outputs must come out as before.  Reference: plain
# PyTorch in fp64, rounded to fp32; sums of up to 1300 products are off by less than 1e-5 normwise, in the rows or columns reached and outside.
BAD = [("fm", 1300, 400, 1030, 1028, "down dact dx dw"), ("fm", 1024, 701, 1000, 901, "down dact dx dw"), ("bm", 1021, 510, 607, 321, "down dx dw"),
       ("fm", 449, 300, 1400, 701, "dw"), ("bm", 500, 321, 1400, 705, "dact dw")]


@pytest.mark.parametrize("mode,T,d,F,p,split", BAD, ids=[f"{b[0]}{b[1]}x{b[2]}p{b[4]}" for b in BAD])
@pytest.mark.parametrize("where", ["dY", "X", "W1", "W2T"])
@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 2.0**115])
def test_f32_split_backward_operands_that_are_not_finite(sdp, mode, T, d, F, p, split, where, bad):
    X, dY, W = _inputs(T, d, F, 99)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    held = idx.long()
    rows = held if mode == "fm" else torch.arange(F, device="cuda")
    _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
    j, c, t = int(held[p // 2]), d - 2, T - 3
    {"dY": dY, "X": X, "W1": W[0], "W2T": W[2]}[where][t if where in ("dY", "X") else j, c] = bad
    got, loops = _launched(sdp, [f"mlp_{k}" for k in split.split() if k != "down"], sdp.masked_mlp_bwd, mode, X, dY, *W, idx, G, U)
    assert all("split" in k for k in loops), loops
    X64, dY64, G64, U64 = (v.double() for v in (X, dY, G, U))
    W1, W3, W2T = (v[rows].double() for v in W)
    s = torch.sigmoid(G64)
    dA = (dY64 @ W2T.t()).float().double()
    dU, dG, act = dA * G64 * s, dA * U64 * (s + G64 * s * (1 - s)), G64 * s * U64
    dU, dG = dU.float().double(), dG.float().double()
    of = (lambda m: m) if mode == "fm" else (lambda m: m[:, held])
    want = (dG @ W1 + dU @ W3, of(dG).t() @ X64, of(dU).t() @ X64, of(act).t() @ dY64)
    at = int((idx == j).nonzero())
    # the row or column of each result that the element reaches, ... for all of it
    reached = {"dY": ((t, slice(None)), ..., ..., (slice(None), c)), "X": (None, (slice(None), c), (slice(None), c), None),
               "W1": ((slice(None), c), None, None, None), "W2T": (..., (at, slice(None)), (at, slice(None)), None)}[where]
    for name, a, b, r in zip(("dX", "dW1", "dW3", "dW2T"), got, want, reached):
        b = b.float()
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.isinf(), b.isinf()), name
        assert torch.equal(a[a.isinf()], b[a.isinf()]), name
        inside = torch.zeros_like(a, dtype=torch.bool)
        if r is not None:
            inside[r] = True
        assert bool(a[~inside].isfinite().all()), name
        for m in (inside & a.isfinite(), ~inside):
            if bool(m.any()):
                assert _off(a[m], b[m].double()) <= 1e-5, (name, _off(a[m], b[m].double()))
    if "down" in split and where == "W2T":
        (Y, _, _), loops = _launched(sdp, ["mlp_down"], sdp.masked_mlp_fwd, mode, X, *W, idx)
        assert "split" in loops[0], loops
        b = (act @ W2T).float()
        assert torch.equal(Y.isnan(), b.isnan()) and torch.equal(Y.isinf(), b.isinf())
        inside = torch.zeros_like(Y, dtype=torch.bool)
        inside[:, c] = True
        assert bool(Y[~inside].isfinite().all()) and _off(Y[~inside], b[~inside].double()) <= 1e-5


def _normal(*shape, scale, gen):
    return torch.randn(shape, generator=gen, device="cuda") * scale


def _off(got, want):
    return float((got.double() - want).norm() / want.norm())


# Products of operands at the ends of fp32's range, numbers below its normal ones among them, whose sums lie well inside it: G and U, and
# what dact, dX and the weight gradients make of such dY, U and weights, all in launches that split (_launched sees to it).
# Reference: plain PyTorch in fp64.  A sum is off by its own rounding (below 1e-6 normwise at these depths) and dG, dU and act by a few of theirs.
@pytest.mark.parametrize("x,w", [(-110, 100), (-114, 100), (-118, 100), (-122, 100), (-126, 110), (-130, 110), (-140, 110), (100, -122), (110, -130),
                                 (120, -140), (-55, -55), (60, 55), (100, 20)])
def test_f32_split_operands_at_the_ends_of_the_range(sdp, x, w):
    T, d, F = 1024, 544, 1024
    g = torch.Generator(device="cuda")
    g.manual_seed(94)
    idx = torch.arange(F, dtype=torch.int32, device="cuda")
    X, W = _normal(T, d, scale=2.0**x, gen=g), [_normal(F, d, scale=2.0**w, gen=g) for _ in range(3)]
    (_, G, U), loops = _launched(sdp, ("mlp_gate_up", "mlp_down"), sdp.masked_mlp_fwd, "fm", X, *W, idx)
    assert all("split" in k for k in loops), loops
    for got, m in ((G, W[0]), (U, W[1])):
        assert _off(got, X.double() @ m.double().t()) <= 1e-6, (x, w)


@pytest.mark.parametrize("dy,w2,u,w13", [(-122, 100, 0, 0), (-130, 120, 0, 0), (100, -122, 0, 0), (0, 0, -122, 100), (0, 100, -122, 0), (-122, 120, 0, 100),
                                         (-100, -10, 0, 110), (60, 40, 0, -122)])
def test_f32_split_gradients_at_the_ends_of_the_range(sdp, dy, w2, u, w13):
    T, d, F = 1024, 544, 1024
    g = torch.Generator(device="cuda")
    g.manual_seed(95)
    idx = torch.arange(F, dtype=torch.int32, device="cuda")
    X, dY, G, U = (_normal(*s, scale=2.0**e, gen=g) for s, e in (((T, d), 0), ((T, d), dy), ((T, F), 0), ((T, F), u)))
    W = [_normal(F, d, scale=2.0**e, gen=g) for e in (w13, w13, w2)]
    got, loops = _launched(sdp, ("mlp_dact", "mlp_dx", "mlp_dw"), sdp.masked_mlp_bwd, "fm", X, dY, *W, idx, G, U)
    assert all("split" in k for k in loops), loops
    X, dY, G, U, W1, W3, W2 = (t.double() for t in (X, dY, G, U, *W))
    s = torch.sigmoid(G)
    dA = dY @ W2.t()
    dU, dG, act = dA * G * s, dA * U * (s + G * s * (1 - s)), G * s * U
    for name, a, b in zip(("dX", "dW1", "dW3", "dW2T"), got, (dG @ W1 + dU @ W3, dG.t() @ X, dU.t() @ X, act.t() @ dY)):
        if not 2.0**-100 < float(b.abs().max()) < 2.0**120:
            continue  # the result itself leaves the range
        assert _off(a, b) <= 2e-6, (name, _off(a, b))
