"""The subtrees that a lifting search counts as searched to the end, where many end at once:
schemes that have no lifting, because they are no schemes (an entry of Strassen's is
missing), at every number of subtrees up to the default."""
import numpy as np
import pytest

from paper_2511_20317_amd import tsf
from tests.golden_io import load_formula_scheme

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", [0, 3, 7])
@pytest.mark.parametrize("limit", [1, 64, 65, 1000, 1 << 14, 1 << 16])
def test_every_subtree_is_counted(entry, limit):
    U, V, W = (np.abs(x) for x in load_formula_scheme("strassen_formulas.txt")[3:])
    W = W.copy()
    # an entry of a term that keeps others
    row, col = [at for at in np.argwhere(W) if W[at[0]].sum() > 1][entry]
    W[row, col] = 0
    z = tsf.Scheme(2, 2, 2, U, V, W, tsf.TSF_Z2)
    info, got = tsf.lift(z, max_nodes=1 << 40, max_subtrees=limit)
    assert got is None and info["status"] == 0 and info["subtree"] == -1
    assert info["exhausted"] == info["subtrees"] <= limit
    # with one node a subtree most run out of budget, and none is counted twice
    info, got = tsf.lift(z, max_nodes=1, max_subtrees=limit)
    assert got is None and info["status"] in (0, -1)
    assert (info["exhausted"] == info["subtrees"]) == (info["status"] == 0)
    assert info["exhausted"] <= info["subtrees"]
