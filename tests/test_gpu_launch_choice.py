"""The library's choice of strategy and lanes against an explicit launch, on
both sides of every bound of the choice: identical states, bit for bit."""
import pytest

from paper_2511_20317_amd import tsf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,walks", [
    (32, 1024), (33, 1024), (33, 1025), (41, 3072), (41, 3073), (65, 12288), (65, 12289),
    (40, 1024), (41, 1024), (41, 1025), (48, 4096), (48, 4097), (48, 8193), (49, 8193),
    (64, 33), (65, 33), (65, 8192), (65, 8193), (72, 16385), (73, 16385), (96, 8193),
    (97, 8193), (128, 17)])
@pytest.mark.parametrize("mode,wide,objective", [(tsf.TSF_TERNARY, False, tsf.OBJ_RANK),
                                                 (tsf.TSF_Z2, False, tsf.OBJ_RANK),
                                                 (tsf.TSF_TERNARY, True, tsf.OBJ_RANK),
                                                 (tsf.TSF_TERNARY, False, tsf.OBJ_ADDITIONS)])
def test_choice_equals_explicit_launch(cap, walks, mode, wide, objective):
    import torch
    ctx = tsf.Context()
    # grown by expands towards the capacity, restarted from the best scheme
    groups = [(tsf.init_scheme(2, 3, 3, mode=mode), walks, cap, -10 ** 6)]
    prm = tsf.walk_params(base_seed=cap * 65536 + walks, max_iters=60, plateau=25,
                          t_expand=1 << 31, restart_from_best=1, objective=objective)
    explicit = (16, 1, 2) if cap > 64 else (8, 1, 1)
    states = []
    for launch in ((0, 0, 0), explicit):
        b = tsf.WalkBatch(groups, capacity=cap, rec_cap=4)
        if wide:
            b.max_len = 64
        b.init(ctx)
        for part in (41, 19):
            b.walk(ctx, prm, part, *launch)
        states.append((b.hdr, b.rec, b.cur, b.best))
    torch.cuda.synchronize()
    hdr = states[0][0].cpu().numpy().view(tsf.HEADER_DTYPE)
    assert (hdr["t"] == 60).all()
    ranks = torch.from_numpy(hdr["rank"].copy()).cuda(), torch.from_numpy(
        hdr["best_rank"].copy()).cuda()
    assert torch.equal(states[0][0], states[1][0])
    assert torch.equal(states[0][1], states[1][1])
    slot = torch.arange(cap, device="cuda")
    for k, rank in enumerate(ranks):       # the live terms
        live = (slot[None, :] < rank[:, None])[:, :, None]
        assert torch.equal(states[0][2 + k] * live, states[1][2 + k] * live)
