"""GPU: the average, its norm and the fused update where a row is no whole number of 512-parameter segments: rows in whole groups of 8
parameters, groups that straddle two rows (one of them trained by nobody, or by another worker), a buffer that ends inside a group, more
workers than one batch, and buffers just below the size from which they are taken.  Rows outside a worker's mask hold NaN."""
import pytest

import test_gpu_adamw as adamw
import test_gpu_avg as avg

pytestmark = pytest.mark.gpu
sdp = avg.sdp  # the fixture

CASES = [(3, 40961, 8, 20000, "bf16"), (3, 87382, 9, 29000, "f32"), (9, 90001, 9, 30000, "bf16"), (4, 52431, 15, 20000, "f32"),
         (12, 8000, 100, 2500, "f32"), (4, 1541, 511, 700, "bf16"), (4, 1535, 513, 700, "f32"), (4, 1533, 513, 700, "bf16"),
         (20, 12485, 63, 900, "bf16"), (2, 787, 1001, 400, "bf16"), (8, 5000, 72, 2500, "bf16"), (8, 1240, 264, 700, "bf16"),
         (1, 700, 520, 300, "f32")]
IDS = [f"K{K}_R{R}_D{D}_{dt}" for K, R, D, p, dt in CASES]


@pytest.mark.parametrize("c", CASES, ids=IDS)
def test_average(sdp, orc, c):
    avg.test_avg_matches_oracle_with_poisoned_off_mask_rows(sdp, orc, *c)


@pytest.mark.parametrize("c", CASES, ids=IDS)
def test_norm(sdp, orc, c):
    avg.test_squared_norm_of_the_average_matches_oracle(sdp, orc, *c)


@pytest.mark.parametrize("c", CASES, ids=IDS)
def test_update(sdp, orc, c):
    adamw.test_adamw_matches_oracle(sdp, orc, *c, 3)
