"""The lifting search's node budget against the oracle's count of nodes, in
one tree (no prefix): with as many nodes as the oracle needed the GPU ends as
it does, with one fewer it runs out."""
import numpy as np
import pytest

from oracle import pyoracle as O
from paper_2511_20317_amd import tsf
from tests.test_gpu_lift import _cases, _to_tsf

pytestmark = pytest.mark.gpu


def test_budget_counts_the_oracles_nodes():
    checked = 0
    for name, z in _cases():
        st, t, nodes = O.lift(z, 20000)
        if st < 0 or nodes < 2:
            continue
        info, got = tsf.lift(_to_tsf(z), max_nodes=nodes, max_subtrees=1)
        assert (info["status"], info["subtrees"], info["exhausted"]) == (st, 1, 1), (name, nodes)
        if st == 1:
            want = O.from_c(t)
            for g, k in zip(got.live(), "UVW"):
                assert np.array_equal(g, want[k]), name
        info, got = tsf.lift(_to_tsf(z), max_nodes=nodes - 1, max_subtrees=1)
        assert (info["status"], info["exhausted"], got) == (-1, 0, None), (name, nodes)
        checked += 1
    assert checked >= 3
