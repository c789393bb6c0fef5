"""What tsf_walk_learned leaves in its workspace: calls that end before, at and after a
captured chunk of 16 iterations."""
import pytest

from oracle import mlp as ref
from paper_2511_20317_amd import tsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("calls", [[1], [7], [16], [17, 40]])
def test_workspace_holds_the_last_iteration(calls):
    """after a call the hidden layers and scores are those of the rows in the workspace"""
    import torch
    ctx = tsf.Context()
    p = ref.init_params(5)
    net = tsf.Mlp()
    net.set_params(p["W1"], p["b1"], p["W2"], p["b2"], p["w3"], p["b3"])
    b = tsf.WalkBatch([(tsf.init_scheme(3, 3, 3), 41, 35, 0)], rec_cap=8)
    ws = tsf.LearnWorkspace(b.n_walks)
    prm = tsf.walk_params(base_seed=4, max_iters=100, plateau=30)
    b.init(ctx)
    for n in calls:
        ws.h1.fill_(-1)
        ws.h2.fill_(-1)
        b.walk_learned(ctx, prm, net, ws, n)
        h1, h2, logit = net.forward(ws.feat)
        assert torch.equal(ws.h1, h1) and torch.equal(ws.h2, h2) and torch.equal(ws.logit, logit)
