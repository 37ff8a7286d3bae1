"""GPU, bit-exact against numpy: the compaction of rows of at most 32768 neurons at the edges of its 2048-byte chunks, from rows at any
address, mask bytes of any value but zero, and gather rows longer and shorter than the count."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 7, 8, 9, 2047, 2048, 2049, 4095, 4101, 6144, 32760, 32767, 32768])
@pytest.mark.parametrize("K,density", [(3, 0.5), (2, 1.0), (1, 0.0)])
def test_index_of_short_rows(F, K, density):
    import paper_2507_09029_amd as sdp

    rng = np.random.default_rng(F * 7 + K)
    mask = np.where(rng.random((K, F)) < density, rng.integers(1, 256, (K, F)), 0).astype(np.uint8)
    held = torch.full((K * F + 3,), 9, dtype=torch.uint8, device="cuda")
    on = held[3:].view(K, F)  # off any word's boundary
    on.copy_(torch.from_numpy(mask))
    counts = (mask != 0).sum(1)
    for idx_ld in sorted({F, max(1, int(counts.min()) - 1)}):
        idx, pos, count, cov = (t.cpu().numpy() for t in sdp.index_masks_static(on, idx_ld=idx_ld))
        for k in range(K):
            rows = np.flatnonzero(mask[k])
            want = np.full(F, -1)
            want[rows] = np.arange(len(rows))
            assert (pos[k] == want).all() and count[k] == len(rows)
            assert (idx[k] == np.append(rows, np.full(F, -1))[:idx_ld]).all()
        assert (cov == (mask != 0).sum(0)).all()
