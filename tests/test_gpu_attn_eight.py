"""GPU: bf16 heads wider than 64 where eight waves share a block's walk (from 512 tokens on, up to 8 pairs of sequence and head; the
rule itself: test_attn_rule.py), at the edges of its 32-row tiles and of the widths.  Tolerances and their reasons: test_gpu_attn.py."""
import pytest

import test_gpu_attn as t
from workloads import AttnWorkload

pytestmark = pytest.mark.gpu
sdp = t.sdp  # the fixture

CASES = [AttnWorkload(f"eight{hd}_S{S}_{Bt}x{ph}", Bt, S, 72, H, hd, ph, 2, 61) for hd, Bt, S, H, ph in
         ((72, 1, 512, 3, 2), (96, 2, 545, 3, 2), (104, 1, 575, 3, 2), (128, 1, 513, 3, 2), (120, 1, 800, 2, 1),
          (80, 1, 512, 9, 8),    # the most pairs that qualify (forward masking)
          (80, 1, 512, 10, 9),   # one head more
          (88, 2, 515, 5, 4), (128, 1, 515, 9, 8),  # as many pairs, tokens that are no multiple of 32
          (128, 1, 511, 3, 2))]  # one token short


@pytest.mark.parametrize("mode", ["fm", "bm"])
@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_eight_waves_on_a_block(sdp, orc, w, mode):
    t.run_case(sdp, orc, w, [0], dw_layout="scatter" if w.hd % 16 else "compact", mode=mode)


@pytest.mark.parametrize("tok", [0, 33, 255, -1])
@pytest.mark.parametrize("w", [AttnWorkload(f"bad{hd}_S{S}", 2, S, 72, 2, hd, 2, 2, 62) for hd, S in ((72, 520), (96, 512), (128, 545))],
                         ids=lambda w: w.name)
def test_bad_token_reaches_only_what_depends_on_it(sdp, w, tok):
    t._check_bad_token(sdp, w, "fm", tok % w.S)
