"""The Brent check of a batch against the host's at the edges of the GPU
check: factor lengths around the 32-bit words, term counts around its 64-term
sets, and sums up to the largest capacity."""
import numpy as np
import pytest

from paper_2511_20317_amd import tsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [tsf.TSF_TERNARY, tsf.TSF_Z2])
@pytest.mark.parametrize("fmt,cap", [((1, 1, 1), 1), ((4, 1, 8), 64), ((3, 1, 11), 65),
                                     ((8, 1, 8), 128), ((4, 4, 4), 129), ((2, 2, 3), 512),
                                     ((8, 8, 8), 512)])
def test_violations_equal_the_hosts(mode, fmt, cap):
    import torch
    rng = np.random.default_rng(cap)
    base = tsf.init_scheme(*fmt, mode=mode)
    schemes = [base]
    for k in range(11):
        U, V, W = (x.astype(np.int64) for x in base.live())
        r = U.shape[0]
        if k % 3 == 0 and cap > r:       # copies of one term: large sums
            extra = int(rng.integers(1, cap - r + 1)) if k else cap - r
            U, V, W = (np.concatenate([x, np.repeat(x[:1], extra, 0)]) for x in (U, V, W))
        else:                            # changed coefficients, also to rank 0 and 1
            keep = int(rng.integers(0, r + 1)) if k % 3 == 1 else r
            U, V, W = U[:keep], V[:keep], W[:keep]
            for x in (U, V, W):
                if x.size:
                    at = rng.integers(0, x.size, 1 + x.size // 7)
                    x.reshape(-1)[at] = rng.integers(0 if mode else -1, 2, at.size)
        schemes.append(tsf.Scheme(*fmt, U, V, W, mode, cap))
    b = tsf.WalkBatch([(base, len(schemes), cap, 0)], capacity=cap, rec_cap=1)
    hdr = b.headers()
    start = np.zeros((len(schemes), cap, 6), np.uint64)
    for w, s in enumerate(schemes):
        hdr["start_rank"][w] = s.rank
        start[w] = tsf.pack(s, cap)
    b.hdr.copy_(torch.from_numpy(hdr.view(np.uint8).reshape(-1).copy()))
    b.start.copy_(torch.from_numpy(start.view(np.int64)))
    got = b.verify_device(2).cpu().numpy()
    assert got.tolist() == [tsf.verify(s) for s in schemes]
    assert got[0] == 0 and (got[1:] > 0).any()
