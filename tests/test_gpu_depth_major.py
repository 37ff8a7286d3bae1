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


@pytest.mark.parametrize("T", [8, 64, 136, 200, 328])
@pytest.mark.parametrize("p,d,tile", SHAPES, ids=[s[2] for s in SHAPES])
@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_weight_gradients_every_tile_few_steps(sdp, mode, p, d, tile, T):
    F = p + 40
    X, dY, W = _inputs(T, d, F, 1000 * T + p)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    sdp.profile_enable(True)
    try:
        Y, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
        dX, dW1, dW3, dW2T = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U, dw_layout="compact")
        torch.cuda.synchronize()
        assert sdp.profile_launch_shape("mlp_dw")["tile"] == tile
    finally:
        sdp.profile_enable(False)
    rows = idx.long()
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


@pytest.mark.parametrize("mode", ["fm", "bm"])
def test_mlp_gradients_over_tokens(sdp, mode):
    T, d, F, p = 264, 136, 256, 200
    X, dY, W = _inputs(T, d, F, 3)
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    _, G, U = sdp.masked_mlp_fwd(mode, X, *W, idx)
    want = sdp.masked_mlp_bwd(mode, X, dY, *W, idx, G, U, dw_layout="compact")
    x, dy = X.clone(), dY.clone()
    got = sdp.masked_mlp_bwd(mode, x, dy, *W, idx, G, U, dw_layout="compact",
                             out=(torch.empty_like(X), x[:p], torch.empty_like(want[2]), dy[:p]))
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("mode", ["fm", "bm"])
@pytest.mark.parametrize("hd", [50, 64, 80])
def test_attention_gradients_over_tokens(sdp, mode, hd):
    Bt, S, H, ph = 2, 171, 4, 2
    T, d = Bt * S, 4 * 88
    X, dY, _ = _inputs(T, d, 8, 4)
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    Wqkv = (torch.randn((3, H * hd, d), generator=g, device="cuda") * 0.05).bfloat16()
    WoT = (torch.randn((H * hd, d), generator=g, device="cuda") * 0.05).bfloat16()
    heads = sdp.make_masks(2, H, ph, 5, True)[1][0].contiguous()
    a = (mode, Bt, S, hd)
    _, QKV, O, LSE = sdp.masked_attn_fwd(*a, X, Wqkv, WoT, heads)
    want = sdp.masked_attn_bwd(*a, X, dY, Wqkv, WoT, heads, QKV, O, LSE)
    x, dy = X.clone(), dY.clone()
    out = (torch.empty_like(X), x.view(-1)[: want[1].numel()].view(want[1].shape) if want[1].numel() <= x.numel() else torch.empty_like(want[1]),
           dy[: want[2].shape[0]])
    got = sdp.masked_attn_bwd(*a, x, dy, Wqkv, WoT, heads, QKV, O, LSE, out=out)
    for r, w in zip(got, want):
        assert torch.equal(r, w)
