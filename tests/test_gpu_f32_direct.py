"""GPU: the fp32 contraction's direct-load tiles, pipelined (64 wide) and shared out over a tile's waves (16 and 32), with
16-byte loads and with single floats (extents that are no multiples of 4, gathered columns): partial tiles, one to several depth
steps, launches of dX and the weight gradients together and apart.  1e-5 against the fp64 oracle."""
import pytest
import torch

import test_gpu_mlp as mlp
from workloads import MlpWorkload

pytestmark = pytest.mark.gpu
sdp = mlp.sdp  # the fixture

CASES = [MlpWorkload(f"{T}x{d}x{F}p{p}_{mode}", "f32", T, d, F, p, 2, mode, 81) for T, d, F, p, mode in (
    # weight gradients of 1, 2, 3, 4 and 5 depth steps beside dX, 64-wide tiles; with single floats
    (32, 132, 1100, 1004, "fm"), (33, 132, 1100, 1001, "fm"), (64, 130, 1100, 1001, "fm"), (96, 132, 1100, 1004, "bm"),
    (97, 132, 1100, 1004, "fm"), (129, 264, 1100, 1003, "bm"), (130, 254, 1102, 1003, "bm"),
    # gate_up and dact in 64-wide tiles of 1, 2 and 4 steps; of 128
    (1000, 32, 1032, 1004, "fm"), (1000, 36, 1030, 1001, "fm"), (1001, 100, 1031, 1002, "bm"), (2044, 36, 2040, 2036, "fm"),
    # dX alone (more than 256 tiles of 32) and down in 32-wide tiles; gathered columns with 16-byte loads on the other side
    (520, 516, 300, 200, "fm"), (521, 515, 300, 201, "bm"), (100, 64, 300, 151, "bm"),
    # register-staged tiles with 16-byte loads: down in tiles of 64 and of 128; weight gradients beyond a round in a launch of their own
    (1000, 1000, 64, 36, "fm"), (2044, 2044, 64, 36, "fm"), (520, 516, 2044, 2036, "fm"),
    # a list of depth rows that LDS does not take
    (8, 16, 4200, 4100, "fm"), (8, 17, 4200, 4097, "fm"))]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_f32_direct_load_tiles(sdp, orc, w):
    mlp.run_case(sdp, orc, w, [1], dw_layout="scatter" if w.p % 2 else "compact")


# weight gradients in 128-wide register-staged tiles: too few tokens for the split ones, too many tiles of dX for one launch
def test_f32_gradients_in_128_wide_tiles(sdp, orc):
    w = MlpWorkload("wide_gradients", "f32", 250, 1060, 1100, 1000, 2, "fm", 83)
    sdp.profile_filter(None)
    sdp.profile_enable(True)
    mlp.run_case(sdp, orc, w, [1])
    sdp.profile_enable(False)
    assert sdp.profile_launch_shape("mlp_dw") == {"tile": "128x128", "loop": "staged"}


# lists that LDS does not take, beyond the 16- and 32-wide tiles: split products (256 and 1024 tiles of 64), with 16-byte loads and with
# single floats, and 64-wide register-staged tiles where an output of less than 64 columns keeps the split ones away.  Reference:
# plain PyTorch in fp64; 4100 products summed in fp32 stay below 1e-5 normwise.
@pytest.mark.parametrize("T,d,F,p,loop", [(1024, 1024, 4200, 4100, "split, two teams"), (1023, 1021, 4201, 4097, "split, two teams"),
                                          (2048, 2048, 4200, 4100, "split"), (2047, 2045, 4201, 4097, "split"), (16384, 40, 4200, 4100, "staged"),
                                          (16384, 41, 4201, 4097, "staged")])
def test_f32_long_lists_on_large_tiles(sdp, T, d, F, p, loop):
    g = torch.Generator(device="cuda")
    g.manual_seed(82)
    rnd = lambda *s, std=1.0: torch.randn(s, generator=g, device="cuda") * std
    X, dY, W = rnd(T, d), rnd(T, d), [rnd(F, d, std=0.02) for _ in range(3)]
    idx = sdp.make_masks(2, F, p, 5, True)[1][0].contiguous()
    sdp.profile_filter(None)
    sdp.profile_enable(True)
    Y, G, U = sdp.masked_mlp_fwd("fm", X, *W, idx)
    dX = sdp.masked_mlp_bwd("fm", X, dY, *W, idx, G, U)[0]
    sdp.profile_enable(False)
    for name in ("mlp_down", "mlp_dx"):
        assert sdp.profile_launch_shape(name) == {"tile": "64x64", "loop": loop}
    W1, W3, W2T = (t[idx.long()].double() for t in W)
    G64, U64 = X.double() @ W1.t(), X.double() @ W3.t()
    s = torch.sigmoid(G64)
    dA = dY.double() @ W2T.t()
    for got, want in ((Y, (G64 * s * U64) @ W2T), (dX, (dA * U64 * (s + G64 * s * (1 - s))) @ W1 + (dA * G64 * s) @ W3)):
        assert float((got.double() - want).norm() / want.norm()) <= 1e-5
