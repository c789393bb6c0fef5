"""Checked walks in every shape that the library chooses by itself, and in the shapes that a
launch may name: no check fails, every walk ends as without checks, and a damaged state is
found."""
import numpy as np
import pytest

from paper_2511_20317_amd import tsf

pytestmark = pytest.mark.gpu

OPEN = (0, 0, 0)
# format, capacity, walks, launch: packed factors, 32-bit and 64-bit pairs with 32, 16 and 8
# lanes; beyond 64 terms 16 and 8 lanes; one walk per wavefront
CASES = [((2, 2, 3), 20, 65, OPEN), ((2, 2, 3), 20, 4097, OPEN), ((2, 2, 3), 20, 8193, OPEN),
         ((1, 4, 5), 28, 65, OPEN), ((1, 4, 5), 28, 4097, OPEN), ((1, 4, 5), 28, 8193, OPEN),
         ((3, 4, 4), 56, 8193, OPEN), ((1, 6, 6), 44, 65, OPEN), ((1, 6, 6), 44, 4097, OPEN),
         ((3, 4, 5), 68, 12289, OPEN), ((3, 4, 5), 68, 17000, OPEN), ((3, 4, 5), 68, 33, OPEN),
         ((3, 3, 3), 35, 65, OPEN), ((3, 3, 3), 35, 65, (8, 1, 3)), ((3, 3, 3), 35, 65, (8, 4, 1)),
         ((3, 4, 5), 68, 33, (0, 2, 1)), ((3, 3, 3), 35, 65, (64, 0, 2))]


@pytest.mark.parametrize("mode", [tsf.TSF_TERNARY, tsf.TSF_Z2])
@pytest.mark.parametrize("fmt,cap,walks,launch", CASES)
def test_checked_equals_unchecked(fmt, cap, walks, launch, mode):
    import torch
    ctx = tsf.Context()
    groups = [(tsf.init_scheme(*fmt, mode=mode), walks, cap, -10 ** 6)]
    prm = tsf.walk_params(base_seed=cap + walks, max_iters=10 ** 6, plateau=30, t_expand=1 << 30)
    done = []
    for checked in (False, True):
        b = tsf.WalkBatch(groups, capacity=cap, rec_cap=4)
        b.init(ctx)
        for part in (37, 23):
            b.walk(ctx, prm, part, *launch, checked=checked)
        done.append(b)
    torch.cuda.synchronize()
    a, c = done
    assert (c.headers()["done"] == 0).all() and (c.headers()["t"] == 60).all()
    assert torch.equal(a.hdr, c.hdr) and torch.equal(a.rec, c.rec)
    assert torch.equal(a.cur, c.cur) and torch.equal(a.best, c.best)


@pytest.mark.parametrize("fmt,cap,walks", [c[:3] for c in CASES if c[3] == OPEN])
def test_damage_is_found(fmt, cap, walks):
    import torch
    ctx = tsf.Context()
    b = tsf.WalkBatch([(tsf.init_scheme(*fmt), walks, cap, -10 ** 6)], capacity=cap, rec_cap=4)
    prm = tsf.walk_params(base_seed=9, max_iters=10 ** 6, plateau=30)
    b.init(ctx)
    b.walk(ctx, prm, 20)
    b.cur[walks - 1, 1, 2:4] = 0          # a zero factor
    b.walk(ctx, prm, 20, checked=True)
    torch.cuda.synchronize()
    hdr = b.headers()
    assert hdr["done"][walks - 1] == tsf.DONE_CHECK_FAILED
    assert int(hdr["reserved"][walks - 1]) & tsf.CHECK_ZERO_FACTOR
    assert (hdr["done"][:walks - 1] == 0).all() and np.all(hdr["t"][:walks - 1] == 40)
