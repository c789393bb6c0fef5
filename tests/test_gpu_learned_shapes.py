"""Walks with the learned proposal end in the same state whatever the lanes
per walk, the wavefronts per workgroup and the split into calls (calls that
end before, at and after a captured chunk of 16 iterations)."""
import pytest

from oracle import mlp as ref
from paper_2511_20317_amd import tsf

pytestmark = pytest.mark.gpu


def _run(groups, prm, calls, n_calls, capacity, max_len, lanes, wpb):
    import torch
    ctx = tsf.Context()
    p = ref.init_params(3)
    net = tsf.Mlp()
    net.set_params(p["W1"], p["b1"], p["W2"], p["b2"], p["w3"], p["b3"])
    b = tsf.WalkBatch(groups, capacity=capacity, rec_cap=8)
    b.max_len = max(b.max_len, max_len)
    ws = tsf.LearnWorkspace(b.n_walks, choice_cap=n_calls)
    b.init(ctx)
    for n in calls:
        b.walk_learned(ctx, prm, net, ws, n, lanes_per_walk=lanes, waves_per_block=wpb)
    torch.cuda.synchronize()
    return [x.clone() for x in (b.hdr, b.cur, b.best, b.rec, ws.choice, ws.cand, ws.feat, ws.logit)]


@pytest.mark.parametrize("capacity,max_len,wpb", [(35, 1, 1), (64, 64, 4), (128, 64, 3)])
def test_shapes_and_splits_agree(capacity, max_len, wpb):
    import torch
    # the second walk group is at its target from the start, the third reaches it
    groups = [(tsf.init_scheme(3, 3, 3), 37, 35, 0), (tsf.init_scheme(2, 2, 2), 5, 16, 8),
              (tsf.init_scheme(2, 2, 2), 9, 16, 7)]
    prm = tsf.walk_params(base_seed=41, max_iters=45, plateau=30, t_expand=1 << 28)
    want = _run(groups, prm, [1] * 50, 50, capacity, max_len, 8, 1)
    for calls in ([50], [15, 35], [16, 17, 17], [33, 1, 16]):
        got = _run(groups, prm, calls, 50, capacity, max_len, 0 if calls[0] != 15 else 16, wpb)
        for x, y in zip(want, got):
            assert torch.equal(x, y), calls
