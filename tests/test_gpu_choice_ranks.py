"""The library's choice of strategy and lanes near its bounds, with as many terms as the
bounds speak of: walks that start from a standard scheme just below the capacity, against
an explicit launch in every walk and against the oracle in some."""
import pytest

from paper_2511_20317_amd import tsf
from tests.gpu_parity import compare, run_oracle

pytestmark = pytest.mark.gpu

# format, capacity, walks on both sides of a bound, and the terms that some walk must have
CASES = [((3, 3, 4), 40, (1024, 1025), 33), ((3, 3, 4), 41, (3072, 3073), 33),
         ((3, 4, 4), 49, (8192, 16384, 18432), 33), ((4, 4, 4), 64, (4096, 4097, 8193), 64),
         ((3, 4, 6), 76, (11264, 11265, 20480), 65), ((5, 5, 3), 80, (12288, 12289, 16385), 65),
         ((4, 4, 5), 96, (12288, 12289), 80), ((4, 4, 6), 97, (12289,), 96),
         ((5, 5, 5), 128, (17,), 125)]


@pytest.mark.parametrize("fmt,cap,walks,terms", [(f, c, n, t) for f, c, ns, t in CASES for n in ns])
@pytest.mark.parametrize("mode,wide,objective", [(tsf.TSF_TERNARY, False, tsf.OBJ_RANK),
                                                 (tsf.TSF_Z2, False, tsf.OBJ_RANK),
                                                 (tsf.TSF_TERNARY, True, tsf.OBJ_RANK),
                                                 (tsf.TSF_TERNARY, False, tsf.OBJ_ADDITIONS)])
def test_choice_near_its_bounds(fmt, cap, walks, terms, mode, wide, objective):
    import torch
    ctx = tsf.Context()
    groups = [(tsf.init_scheme(*fmt, mode=mode), walks, cap, -10 ** 6)]
    prm = tsf.walk_params(base_seed=cap * 65536 + walks, max_iters=40, plateau=25,
                          t_expand=1 << 31, objective=objective)
    explicit = (16, 1, 2) if cap > 64 else (8, 1, 1)
    states = []
    for launch in ((0, 0, 0), explicit):
        b = tsf.WalkBatch(groups, capacity=cap, rec_cap=4)
        if wide:
            b.max_len = 64
        b.init(ctx)
        for part in (29, 11):
            b.walk(ctx, prm, part, *launch)
        states.append(b)
    torch.cuda.synchronize()
    a, e = states
    ranks = [torch.from_numpy(a.headers()[k].copy()).cuda() for k in ("rank", "best_rank")]
    assert int(ranks[0].max()) >= terms
    assert torch.equal(a.hdr, e.hdr) and torch.equal(a.rec, e.rec)
    slot = torch.arange(cap, device="cuda")
    for rank, x, y in zip(ranks, (a.cur, a.best), (e.cur, e.best)):
        live = (slot[None, :] < rank[:, None])[:, :, None]
        assert torch.equal(x * live, y * live)
    some = {0, walks // 2, walks - 1, int(ranks[0].argmax())}
    compare(a, run_oracle(groups, prm, sorted(some), 40, splits=[29, 11]), "choice")


def test_tuning_a_batch_whose_default_has_32_lanes():
    """the tuned launch is one of the autotuner's, 32 lanes among them, the batch is left as
    it was, and both objectives walk on from it as the oracle does"""
    import torch
    ctx = tsf.Context()
    groups = [(tsf.init_scheme(2, 2, 2), 200, 16, -10 ** 6)]
    for objective in (tsf.OBJ_RANK, tsf.OBJ_ADDITIONS):
        prm = tsf.walk_params(base_seed=77, max_iters=500, plateau=200, objective=objective)
        b = tsf.WalkBatch(groups, rec_cap=8)
        b.init(ctx)
        b.walk(ctx, prm, 100)
        torch.cuda.synchronize()
        before = (b.hdr.clone(), b.cur.clone(), b.best.clone())
        lanes, waves, strategy = b.autotune(ctx, prm, trial_iters=100)
        assert waves in (1, 2, 4) and (lanes in (4, 8, 16, 32) if strategy != 2 else
                                       lanes in (16, 32, 64))
        assert all(torch.equal(x, y) for x, y in zip(before, (b.hdr, b.cur, b.best)))
        b.walk(ctx, prm, 400)
        torch.cuda.synchronize()
        compare(b, run_oracle(groups, prm, range(0, 200, 13), 500), "tuned")
