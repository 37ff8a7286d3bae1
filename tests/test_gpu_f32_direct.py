"""GPU: the fp32 contraction's direct-load tiles, pipelined (64 and 128 wide) and shared out over a tile's waves (16 and 32), with
16-byte loads and with single floats (extents that are no multiples of 4, gathered columns): partial tiles, one to several depth
steps, launches of dX and the weight gradients together and apart.  1e-5 against the fp64 oracle."""
import pytest

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
    # a list of depth rows that LDS does not take
    (8, 16, 4200, 4100, "fm"), (8, 17, 4200, 4097, "fm"))]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_f32_direct_load_tiles(sdp, orc, w):
    mlp.run_case(sdp, orc, w, [1], dw_layout="scatter" if w.p % 2 else "compact")
