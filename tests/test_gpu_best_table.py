"""The best-scheme table where its sort can go wrong: tables that are full,
fill one workgroup's 64 slots exactly, one fewer or one more, or stay nearly
empty; against the oracle's order of the same population."""
import itertools

import numpy as np
import pytest

from oracle import pyoracle as O
from paper_2511_20317_amd import tsf
from tests.test_gpu_explore import _gpu_table, _oracle_table

pytestmark = pytest.mark.gpu

FORMATS = [f for f in itertools.product(range(1, 9), repeat=3) if f[0] * f[1] * f[2] <= 48]


def _standard(m, n, p):
    d = O.from_c(O.standard(m, n, p))
    return tsf.Scheme(m, n, p, d["U"], d["V"], d["W"])


@pytest.mark.parametrize("slots,formats", [(1, 1), (3, 3), (63, 63), (64, 64), (65, 65), (130, 127),
                                           (1000, 5), (1025, 200), (4096, 1), (4096, 217)])
def test_table_is_the_sorted_population(slots, formats):
    import torch
    rng = np.random.default_rng(slots * 1000 + formats)
    picked = [FORMATS[k] for k in rng.permutation(len(FORMATS))[:formats]]
    assert len(picked) == formats
    schemes = [_standard(*f) for f in picked + picked[: formats // 2 + 1]]
    schemes = [schemes[k] for k in rng.permutation(len(schemes))]
    b = tsf.WalkBatch([(s, 1, s.rank, 0) for s in schemes], capacity=48)
    b.max_len = 64
    b.init(tsf.Context())
    want = _oracle_table(schemes)
    assert _gpu_table(*b.population_best(slots)) == want
    table = torch.zeros(slots * tsf.BEST_ENTRY_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    count, dropped = (torch.full((1,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    b.population_best_noalloc(table, count, slots, dropped)
    assert _gpu_table(table, count) == want and int(dropped.item()) == 0
