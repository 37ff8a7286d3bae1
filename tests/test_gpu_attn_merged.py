"""GPU: the attention backward as one launch (few blocks): one row to several tiles, every kind of width, the last number of blocks
that qualifies and one head or a tile more.  Tolerances and their reasons: test_gpu_attn.py."""
import pytest

import test_gpu_attn as t
from test_gpu_depth_major import _Launches
from workloads import AttnWorkload

pytestmark = pytest.mark.gpu
sdp = t.sdp  # the fixture

CASES = [(AttnWorkload(f"merged_{dt}_{hd}_S{S}_{Bt}x{H}", Bt, S, 72, H, hd, H, 2, 91, dt), one) for dt, hd, Bt, S, H, one in
         (("bf16", 64, 1, 1, 2, 1), ("bf16", 50, 3, 31, 2, 1), ("bf16", 64, 2, 33, 3, 1), ("bf16", 32, 1, 129, 2, 1), ("bf16", 64, 1, 300, 2, 1),
          ("bf16", 64, 8, 130, 16, 1), ("bf16", 50, 8, 130, 17, 0),
          ("bf16", 64, 4, 1040, 7, 1), ("bf16", 64, 1, 2112, 8, 0),  # four waves on a block, in two launches
          # wider heads: four waves on a block, then eight
          ("bf16", 72, 1, 1, 2, 1), ("bf16", 96, 2, 33, 3, 1), ("bf16", 104, 1, 300, 2, 1), ("bf16", 128, 4, 200, 8, 1), ("bf16", 80, 4, 200, 9, 0),
          ("bf16", 88, 1, 545, 2, 1), ("bf16", 120, 1, 1024, 8, 1), ("bf16", 80, 1, 1056, 8, 0),
          # short sequences: as many blocks of 32 rows as of 128
          ("bf16", 128, 48, 32, 4, 1), ("bf16", 128, 50, 32, 4, 0), ("bf16", 80, 56, 17, 4, 0),
          ("f32", 7, 1, 1, 2, 1), ("f32", 64, 2, 33, 3, 1), ("f32", 75, 1, 130, 2, 1), ("f32", 128, 8, 49, 12, 1), ("f32", 36, 8, 49, 13, 0))]


@pytest.mark.parametrize("mode", ["fm", "bm"])
@pytest.mark.parametrize("w,one", CASES, ids=[w.name for w, _ in CASES])
def test_backward_in_one_launch(sdp, orc, w, one, mode):
    with _Launches(sdp) as n:
        t.run_case(sdp, orc, w, [0], mode=mode)
    assert (n["attn_core_bwd"], n["attn_core_bwd_dq"]) == (one, 1 - one), n


# the smaller cases of test_gpu_attn.py run as one launch
@pytest.mark.parametrize("w", [AttnWorkload("bad_two_f32", 8, 75, 24, 10, 32, 10, 2, 92, "f32"), AttnWorkload("bad_two_bf16", 4, 200, 72, 9, 72, 9, 2, 92)],
                         ids=lambda w: w.name)
def test_bad_token_with_two_launches(sdp, w):
    with _Launches(sdp) as n:
        t._check_bad_token(sdp, w, "fm", 33)
    assert n["attn_core_bwd"] == 0 and n["attn_core_bwd_dq"] > 0, n
