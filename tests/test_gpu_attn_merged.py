"""GPU: the bf16 attention backward as one launch (heads up to 64, few blocks): one row to several tiles, every kind of width, the
last number of blocks that qualifies and one head more.  Tolerances and their reasons: test_gpu_attn.py."""
import pytest

import test_gpu_attn as t
from test_gpu_depth_major import _Launches
from workloads import AttnWorkload

pytestmark = pytest.mark.gpu
sdp = t.sdp  # the fixture

CASES = [(AttnWorkload(f"merged{hd}_S{S}_{Bt}x{H}", Bt, S, 72, H, hd, H, 2, 91), one) for hd, Bt, S, H, one in
         ((64, 1, 1, 2, 1), (50, 3, 31, 2, 1), (64, 2, 33, 3, 1), (32, 1, 129, 2, 1), (64, 1, 300, 2, 1),
          (64, 8, 130, 16, 1), (50, 8, 130, 17, 0))]


@pytest.mark.parametrize("mode", ["fm", "bm"])
@pytest.mark.parametrize("w,one", CASES, ids=[w.name for w, _ in CASES])
def test_backward_in_one_launch(sdp, orc, w, one, mode):
    with _Launches(sdp) as n:
        t.run_case(sdp, orc, w, [0], mode=mode)
    assert (n["attn_core_bwd"], n["attn_core_bwd_dq"]) == (one, 1 - one), n
