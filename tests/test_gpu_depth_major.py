"""GPU: the bf16 weight gradients, which read token-major operands depth-major through transposing LDS reads, at every tile
shape and at depths of few steps, whole and partial; gradients that take the place of what that launch reads.

The reference is plain PyTorch fp32 with the saved G, U and the path's rounding of dG, dU and Act to bf16.  A result is rounded
to bf16 once (at most 2^-9 of it), and an element of dG, dU or Act may round the other way where the device's exponential
differs in its last bits (at most 2^-8 of that term): normwise at most 2^-9 + 2^-8 < 6e-3.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 6e-3
SHAPES = [(1000, 520, "128x128"), (1000, 1400, "128x192"), (2040, 1016, "128x256"), (1544, 2040, "256x192"), (2040, 2040, "256x256"),
          (40, 72, "64x64")]


@pytest.fixture(scope="module")
def sdp():
    import paper_2507_09029_amd as m

    assert torch.cuda.is_available()
    m.lib()
    return m


def _inputs(T, d, F, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).bfloat16()
    return rnd(T, d), rnd(T, d), [rnd(F, d, std=0.05) for _ in range(3)]


def _close(got, want, what):
    err = float((got.double() - want.double()).norm() / want.double().norm())
    assert err <= TOL, (what, err)


class _Launches(dict):
    """with _Launches(sdp) as n: ... afterwards n[name] = launches of that name"""

    def __init__(self, sdp):
        self.sdp = sdp

    def __missing__(self, name):
        return 0

    def __enter__(self):
        self.sdp.profile_filter(None)
        self.sdp.profile_reset()
        self.sdp.profile_enable(True)
        return self

    def __exit__(self, *exc):
        torch.cuda.synchronize()
        self.sdp.profile_enable(False)
        self.update({name: calls for name, (calls, ms) in self.sdp.profile_read().items()})


def _check_mlp_gradients(X, dY, W, G, U, rows, mode, dW1, dW3, dW2T):
    Gs, Us = (G, U) if mode == "fm" else (G[:, rows], U[:, rows])
    g, u = Gs.float(), Us.float()
    s = torch.sigmoid(g)
    dA = dY.float() @ W[2][rows].float().t()
    dG = (dA * u * (s + g * s * (1 - s))).bfloat16().float()
    dU = (dA * g * s).bfloat16().float()
    act = (g * s * u).bfloat16().float()
    _close(dW1, dG.t() @ X.float(), "dW1")
    _close(dW3, dU.t() @ X.float(), "dW3")
    _close(dW2T, act.t() @ dY.float(), "dW2T")


@pytest.mark.parametrize("T", [8, 64, 136, 200, 328])
@pytest.mark.parametrize("p,d,tile", SHAPES, ids=[s[2] for s in SHAPES])
@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_weight_gradients_every_tile_few_steps(sdp, mode, p, d, tile, T):
    F = p + 40
    X, dY, W = _inputs(T, d, F, 1000 * T + p)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    with _Launches(sdp):
        Y, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
        dX, *dW = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U, dw_layout="compact")
        assert sdp.profile_launch_shape("mlp_dw")["tile"] == tile
    _check_mlp_gradients(X, dY, W, G, U, idx.long(), mode, *dW)


# the last round's tiles cut in depth, the last range ending in a partial step (T = 64 k + 8): the one-barrier loop of a 128-row
# tile and, with 256 rows, that loop (both operands depth-major) or the phases (one)
@pytest.mark.parametrize("T,p,d,tile", [(4104, 2312, 2056, "128x192"), (6152, 2440, 2312, "256x192")])
@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_weight_gradients_cut_last_round_partial_step(sdp, mode, T, p, d, tile):
    F = p + 40
    X, dY, W = _inputs(T, d, F, T + p)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
    with _Launches(sdp) as n:
        dX, *dW = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U, dw_layout="compact")
        assert sdp.profile_launch_shape("mlp_dw")["tile"] == tile
    assert n["mlp_dw_reduce"] == 1, n
    _check_mlp_gradients(X, dY, W, G, U, idx.long(), mode, *dW)


# A gradient that overwrites what the weight-gradient launch reads: a mistake shows in the values only if one workgroup stores
# before another has read, so what is asserted first is that the launch was given copies.
@pytest.mark.parametrize("T,d,F,p", [(264, 136, 256, 200), (4104, 2056, 2352, 2312)], ids=["one_round", "cut_last_round"])
@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_mlp_gradients_over_tokens(sdp, mode, T, d, F, p):
    X, dY, W = _inputs(T, d, F, 3)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
    want = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U, dw_layout="compact")
    x, dy = X.clone(), dY.clone()
    with _Launches(sdp) as n:
        got = sdp.masked_mlp_bwd(mode, x, dy, *W, idx, G, U, dw_layout="compact",
                                 out=(torch.empty_like(X), x[:p], torch.empty_like(want[2]), dy[:p]))
    assert n["mlp_copy_bwd"] == 2, n
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_mlp_gradients_over_weights_whose_transposes_ride_on_their_launch(sdp):
    """144 tiles: the launch has room for the transposes of W1 and W3 (dact, with a full round of 256, has not), which it must not
    take while it overwrites W1: they then are a launch of their own."""
    T, d, F, p = 1024, 768, 2048, 1024
    X, dY, W = _inputs(T, d, F, 6)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    _, G, U = sdp.masked_mlp_fwd("fm", X, *W, idx)
    with _Launches(sdp) as n:
        want = sdp.masked_mlp_bwd("fm", X, dY, *W, idx, G, U, dw_layout="compact")
    assert n["mlp_tr_bwd"] == 0, n
    w1 = W[0].clone()
    with _Launches(sdp) as n:
        got = sdp.masked_mlp_bwd("fm", X, dY, w1, W[1], W[2], idx, G, U, dw_layout="compact",
                                 out=(torch.empty_like(X), w1[:p], torch.empty_like(want[2]), torch.empty_like(want[3])))
    assert n["mlp_tr_bwd"] == 1, n
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def _attention(sdp, mode, Bt, S, d, H, hd, ph, seed):
    X, dY, _ = _inputs(Bt * S, d, 8, seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 5)
    Wqkv = (torch.randn((3, H * hd, d), generator=g, device="cuda") * 0.05).bfloat16()
    WoT = (torch.randn((H * hd, d), generator=g, device="cuda") * 0.05).bfloat16()
    heads = sdp.make_masks(2, H, ph, 5, True)[1][0].contiguous()
    saved = sdp.masked_attn_fwd(mode, Bt, S, hd, X, Wqkv, WoT, heads)[1:]
    return X, dY, Wqkv, WoT, heads, saved


@pytest.mark.parametrize("mode", ["fm", "bm"])
@pytest.mark.parametrize("hd", [50, 64, 80])
@pytest.mark.parametrize("over", ["X", "dY", "X_and_dY", "O"])
def test_attention_gradients_over_tokens(sdp, mode, hd, over):
    Bt, S, H, ph = 3, 171, 4, 2  # 3 ph hd <= 480 rows of dWqkv in the place of 513 of X
    d = 4 * 88
    X, dY, Wqkv, WoT, heads, (QKV, O, LSE) = _attention(sdp, mode, Bt, S, d, H, hd, ph, 4)
    a = (mode, Bt, S, hd)
    want = sdp.masked_attn_bwd(*a, X, dY, Wqkv, WoT, heads, QKV, O, LSE)
    x, dy, o = X.clone(), dY.clone(), O.clone()
    place = lambda t, like: t.view(-1)[: like.numel()].view(like.shape)  # fails if it does not fit
    out = (torch.empty_like(X), place(x, want[1]) if "X" in over else torch.empty_like(want[1]),
           place(dy, want[2]) if "dY" in over else place(o, want[2]) if over == "O" else torch.empty_like(want[2]))
    with _Launches(sdp) as n:
        got = sdp.masked_attn_bwd(*a, x, dy, Wqkv, WoT, heads, QKV, o, LSE, out=out)
    assert n["attn_copy_bwd"] == 3, n
    for r, w in zip(got, want):
        assert torch.equal(r, w)


@pytest.mark.parametrize("over", ["X", "dY"])
def test_block_gradients_over_tokens(sdp, over):
    """dY is also what the MLP half adds to its dX, dHm what the attention half adds to dX: a gradient in the place of dY or of X
    (dHm is copied along with X) leaves both sums as they were."""
    Bt, S, d, H, hd, F = 2, 104, 72, 1, 64, 200
    X, dY, W = _inputs(Bt * S, d, F, 8)
    g = torch.Generator(device="cuda")
    g.manual_seed(21)
    Wqkv = (torch.randn((3, H * hd, d), generator=g, device="cuda") * 0.1).bfloat16()
    WoT = (torch.randn((H * hd, d), generator=g, device="cuda") * 0.1).bfloat16()
    Y, saved = sdp.block_fwd("bm", 1, Bt, S, hd, X, Wqkv, WoT, *W)
    dX, grads = sdp.block_bwd("bm", 1, Bt, S, hd, X, dY, Wqkv, WoT, *W, saved)
    want = (dX, *grads)
    x, dy = X.clone(), dY.clone()
    out = [torch.empty_like(t) for t in want]
    if over == "X":
        out[1] = x.view(-1)[: want[1].numel()].view(want[1].shape)  # dWqkv: 3 H hd = 192 rows of 208
    else:
        out[3] = dy[:F]  # dW1
    with _Launches(sdp) as n:
        dX, grads = sdp.block_bwd("bm", 1, Bt, S, hd, x, dy, Wqkv, WoT, *W, saved, out=tuple(out))
    assert (n["attn_copy_bwd"], n["mlp_copy_bwd"]) == ((3, 0) if over == "X" else (0, 2)), n
    for a, b in zip((dX, *grads), want):
        assert torch.equal(a, b)
