"""GPU: small bf16 contractions that read the weights as they are stored (down, dX, the attention's out and dX), and dX beside the
weight gradients in one launch: partial tiles and depth steps, lists of depth rows at the length that still fits, and the same bits
whether or not the launches could be merged.  Tolerances: test_gpu_mlp.py, test_gpu_random_shapes.py (few tokens)."""
import pytest
import torch

import test_gpu_mlp as mlp
from test_gpu_depth_major import _Launches, _attention, _inputs
from workloads import MlpWorkload

pytestmark = pytest.mark.gpu
sdp = mlp.sdp  # the fixture

CASES = [MlpWorkload(f"stored_{T}x{d}p{p}_{mode}", "bf16", T, d, F, p, 2, mode, 71) for T, d, F, p, mode in (
    (8, 8, 16, 8, "fm"), (72, 72, 136, 120, "fm"), (56, 200, 264, 136, "bm"), (64, 64, 128, 64, "fm"), (136, 328, 72, 64, "bm"),
    (1032, 264, 520, 264, "fm"),      # 128 x 128 tiles side by side
    (1032, 264, 520, 264, "bm"),
    (64, 64, 8200, 8192, "fm"),       # the longest list behind 64 x 64 tiles
    (64, 64, 8216, 8200, "fm"),       # one chunk longer: transposed copies
    (64, 72, 2600, 2568, "fm"))]      # rows that are no whole lines, 41 steps: transposed copies


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_mlp_weights_as_stored(sdp, orc, w):
    mlp.run_case(sdp, orc, w, [1], dw_layout="scatter" if w.mode == "bm" else "compact", dw_elem_tol=4e-2)


# tiles of 64 x 64 for both; of 64 x 64 beside 128 x 128; of 128 x 128 for both (dX, weight gradients), or two launches
@pytest.mark.parametrize("mode,T,d,F,p,tiles", [
    ("fm", 136, 72, 264, 200, (64, 64)), ("fm", 1024, 768, 1288, 1024, (64, 128)), ("fm", 2048, 768, 1032, 1024, (128, 128)),
    ("bm", 136, 72, 264, 200, (64, 64)), ("bm", 168, 832, 912, 856, (64, 128)), ("bm", 1112, 936, 448, 376, (128, 128)),
    ("bm", 1024, 768, 1288, 1024, None), ("bm", 2048, 768, 1032, 1024, None)])
def test_mlp_same_bits_beside_the_weight_gradients_and_alone(sdp, mode, T, d, F, p, tiles):
    X, dY, W = _inputs(T, d, F, 9)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
    with _Launches(sdp) as n:
        want = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U)
    assert n["mlp_dx_dw"] == (tiles is not None), n
    if tiles:
        assert [sdp.profile_launch_shape(k)["tile"] for k in ("mlp_dx", "mlp_dw")] == [f"{t}x{t}" for t in tiles]
    fresh = [torch.empty_like(t) for t in want]
    dy, w3 = dY.clone(), W[1].clone()
    with _Launches(sdp) as n:  # dX over dY, which the weight gradients read
        got = sdp.masked_mlp_bwd(mode, X, dy, *W, idx, G, U, out=(dy, *fresh[1:]))
    assert n["mlp_dx_dw"] == 0 and n["mlp_dx"] == 1, n
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    got = sdp.masked_mlp_bwd(mode, X, dY, W[0], w3, W[2], idx, G, U, out=(fresh[0], fresh[1], w3[:p], fresh[3]))  # dW3 over W3
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("hd,S", [(64, 100), (50, 77), (128, 333)])
@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_attention_same_bits_beside_the_weight_gradients_and_alone(sdp, mode, hd, S):
    Bt, H, ph = 2, 4, 2
    X, dY, Wqkv, WoT, heads, (QKV, O, LSE) = _attention(sdp, mode, Bt, S, 200, H, hd, ph, 4)
    a = (mode, Bt, S, hd)
    with _Launches(sdp) as n:
        want = sdp.masked_attn_bwd(*a, X, dY, Wqkv, WoT, heads, QKV, O, LSE)
    assert n["attn_dx_dw"] == 1, n
    fresh = [torch.empty_like(t) for t in want]
    x, wq = X.clone(), Wqkv.clone()
    with _Launches(sdp) as n:
        got = sdp.masked_attn_bwd(*a, x, dY, Wqkv, WoT, heads, QKV, O, LSE, out=(x, *fresh[1:]))  # dX over X
    assert n["attn_dx_dw"] == 0 and n["attn_dx"] == 1, n
    for r, w in zip(got, want):
        assert torch.equal(r, w)
    got = sdp.masked_attn_bwd(*a, X, dY, wq, WoT, heads, QKV, O, LSE, out=(fresh[0], wq.view(-1)[: want[1].numel()].view(want[1].shape), fresh[2]))
    for r, w in zip(got, want):
        assert torch.equal(r, w)


def _workspace(nbytes):
    return torch.full((max(nbytes, 256),), 0xA5, dtype=torch.uint8, device="cuda")


def _copied(ws, base, copy):
    """whether a call wrote the `copy` bytes of a transposed copy of the weights into its workspace beside `base` bytes"""
    n = int((ws != 0xA5).sum())
    assert n <= base or n >= 0.9 * (base + copy), (n, base, copy)
    return n > base


# 20 and 21 depth steps with rows that are no whole lines (down in a launch of its own; dX's two operands count twice), the longest
# list and one chunk more; rows of whole lines and no list at any depth; copies that another launch carries, with few tokens and with
# many, and copies that would need a launch
@pytest.mark.parametrize("mode,T,d,n,down,dx,pair", [
    ("fm", 64, 72, 1280, 1, 1, 1), ("fm", 64, 72, 1288, 0, 0, 0), ("fm", 64, 72, 1000, 1, 1, 1), ("fm", 64, 64, 8192, 1, 1, 0),
    ("fm", 64, 64, 8200, 0, 0, 0), ("bm", 64, 64, 8200, 1, None, None), ("fm", 512, 1600, 1024, 1, 1, 0), ("fm", 1024, 768, 2048, 1, 0, 0),
    ("fm", 1024, 1024, 2048, 1, 0, 0), ("fm", 1024, 1600, 2048, 1, 1, 0)])
def test_mlp_limits_of_weights_as_stored(sdp, mode, T, d, n, down, dx, pair):
    F = n + 16 if mode == "fm" else n
    X, dY, W = _inputs(T, d, F, 11)
    idx = sdp.make_masks(2, F, n if mode == "fm" else (F + 15) // 16 * 8, 5, True)[1][0].contiguous()
    ws = _workspace(sdp.masked_mlp_fwd_workspace_bytes(mode, X.dtype, T, d, F, len(idx)))
    _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx, ws=ws)
    assert _copied(ws, T * n * 2, d * n * 2) == (not down)
    if dx is None:
        return
    nbytes = sdp.masked_mlp_bwd_workspace_bytes(mode, X.dtype, T, d, F, len(idx))
    ws = _workspace(nbytes)
    with _Launches(sdp) as launches:
        want = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U, ws=ws)
    assert launches["mlp_dx_dw"] == pair and _copied(ws, 3 * T * n * 2, 2 * d * n * 2) == (not (pair or dx)), launches
    dy, ws = dY.clone(), _workspace(nbytes)
    with _Launches(sdp) as launches:  # dX over dY: a launch of its own
        got = sdp.masked_mlp_bwd(mode, X, dy, *W, idx, G, U, out=(dy, *[torch.empty_like(t) for t in want[1:]]), ws=ws)
    assert launches["mlp_dx_dw"] == 0 and _copied(ws, 3 * T * n * 2, 2 * d * n * 2) == (not dx), launches
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# the same for the attention's out and dX; weights of less than 2^20 elements a matrix: copies, which the core's launch carries
@pytest.mark.parametrize("d,ph,out,dx,pair", [(840, 20, 1, 0, 0), (840, 21, 0, 0, 0), (2736, 6, 1, 1, 0), (2736, 7, 1, 0, 0), (72, 13, 0, 0, 1),
                                              (72, 14, 0, 0, 0), (1024, 16, 1, 1, 1), (1024, 15, 0, 0, 1)])
def test_attention_limits_of_weights_as_stored(sdp, d, ph, out, dx, pair):
    Bt, S, hd = 2, 32, 64
    T, E = Bt * S, ph * hd
    X, dY, Wqkv, WoT, heads, _ = _attention(sdp, "fm", Bt, S, d, ph + 1, hd, ph, 4)
    a = ("fm", Bt, S, hd)
    ws = _workspace(sdp.masked_attn_fwd_workspace_bytes("fm", X.dtype, Bt, S, d, ph + 1, hd, ph))
    _, QKV, O, LSE = sdp.masked_attn_fwd(*a, X, Wqkv, WoT, heads, ws=ws)
    assert _copied(ws, 0, E * d * 2) == (not out)
    nbytes = sdp.masked_attn_bwd_workspace_bytes("fm", X.dtype, Bt, S, d, ph + 1, hd, ph)
    base, copy = T * 4 * E * 2, 3 * E * d * 2
    ws = _workspace(nbytes)
    with _Launches(sdp) as launches:
        want = sdp.masked_attn_bwd(*a, X, dY, Wqkv, WoT, heads, QKV, O, LSE, ws=ws)
    assert launches["attn_dx_dw"] == pair and _copied(ws, base, copy) == (not (pair or dx)), launches
    x, ws = X.clone(), _workspace(nbytes)
    with _Launches(sdp) as launches:  # dX over X: a launch of its own
        got = sdp.masked_attn_bwd(*a, x, dY, Wqkv, WoT, heads, QKV, O, LSE, out=(x, *[torch.empty_like(t) for t in want[1:]]), ws=ws)
    assert launches["attn_dx_dw"] == 0 and _copied(ws, base, copy) == (not dx), launches
    for r, w in zip(got, want):
        assert torch.equal(r, w)
