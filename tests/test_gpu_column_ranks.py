"""GPU: backward masking hands dact's columns to their compact places for lists that leave long gaps, fill or skip a block of 256
neurons, begin or end at its edges, or hold all of them.  The gradients of the listed rows are those of the list of all neurons, to the
rounding of one bf16 result: the terms are the same and only their order over the tokens may differ."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LISTS = {
    "first": lambda F: np.arange(8),
    "last": lambda F: np.arange(F - 8, F),
    "ends": lambda F: np.r_[0:4, F - 4:F],
    "a block": lambda F: np.arange(256, 512),
    "around a block": lambda F: np.r_[248:256, 512:520],
    "every second": lambda F: np.arange(0, F, 2),
    "all but one in 67": lambda F: np.flatnonzero(np.arange(F) % 67)[: (F - F // 67 - 1) // 8 * 8],
    "all": lambda F: np.arange(F),
}


@pytest.mark.parametrize("F", [528, 768, 4352, 20000])
@pytest.mark.parametrize("which", LISTS)
def test_listed_rows_of_the_full_gradients(F, which):
    import paper_2507_09029_amd as sdp

    T, d = 128, 64
    rows = LISTS[which](F).astype(np.int32)
    assert len(rows) % 8 == 0 and (np.diff(rows) > 0).all()
    g = torch.Generator().manual_seed(F)
    t = lambda *s: torch.randn(*s, generator=g).bfloat16().cuda()
    X, dY, W = t(T, d), t(T, d), [t(F, d) * 0.125 for _ in range(3)]
    every = torch.arange(F, dtype=torch.int32, device="cuda")
    idx = torch.from_numpy(rows).cuda()
    _, G, U = sdp.masked_mlp_fwd("bm", X, *W, every)
    full = sdp.masked_mlp_bwd("bm", X, dY, *W, every, G, U)
    got = sdp.masked_mlp_bwd("bm", X, dY, *W, idx, G, U)
    for name, a, b in zip(("dW1", "dW3", "dW2T"), got[1:], full[1:]):
        a, b = a.double(), b[idx.long()].double()
        # sums of T terms in fp32 that differ by their order round to the same bf16 value or to its neighbour, which with 8 significant
        # bits lies at most 2^-7 of the value away
        assert ((a - b).abs() <= 2.0**-7 * b.abs() + T * 2.0**-23 * b.abs().max()).all(), name
