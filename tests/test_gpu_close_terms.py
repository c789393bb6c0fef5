"""The search for mergeable terms is left out for terms known to be alone: long
walks with many expands, merges and restarts, in which a missed merge shows as a
walk that differs from the oracle's; with the state checks, which compare what
is known of every term with its factors, after every iteration."""
import numpy as np
import pytest

from paper_2511_20317_amd import tsf
from tests.gpu_parity import compare, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [tsf.TSF_TERNARY, tsf.TSF_Z2])
@pytest.mark.parametrize("fmt,cap,reduce_p", [((2, 2, 2), 12, 1 << 32), ((2, 2, 2), 12, 1 << 31),
                                              ((3, 3, 3), 40, 1 << 32), ((3, 3, 3), 100, 1 << 31),
                                              ((2, 5, 7), 200, 1 << 32)])
def test_long_walks_equal_the_oracles(mode, fmt, cap, reduce_p):
    import torch
    s = tsf.init_scheme(*fmt, mode=mode)
    groups = [(s, 10, cap, 0)]
    prm = tsf.walk_params(base_seed=5, max_iters=3000, plateau=700, t_expand=1 << 28,
                          t_reduce=reduce_p)
    ctx = tsf.Context()
    a = tsf.WalkBatch(groups, capacity=cap, rec_cap=16)
    b = tsf.WalkBatch(groups, capacity=cap, rec_cap=16)
    for x in (a, b):
        x.init(ctx)
    a.walk(ctx, prm, 3000, 64, 1, 2)
    b.walk(ctx, prm, 3000, 64, 1, 2, checked=True)
    torch.cuda.synchronize()
    compare(a, run_oracle(groups, prm, range(10), 3000, [3000]), "%s cap %d" % (fmt, cap))
    ha, hb = a.headers(), b.headers()
    assert (hb["done"] != tsf.DONE_CHECK_FAILED).all()
    assert np.array_equal(ha, hb)
