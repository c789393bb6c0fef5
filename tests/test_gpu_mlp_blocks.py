"""The proposal network at the sizes where its row blocks change (32, 64 and
128 rows a workgroup; a partly filled last block) and with buffers that are
not 16-byte aligned, against the fp64 oracle.  The bounds are those that
test_gpu_mlp derives from the bf16 roundings an output passes through."""
import ctypes as C

import numpy as np
import pytest

from oracle import mlp as ref
from paper_2511_20317_amd import tsf
from tests.test_gpu_mlp import _net, _problem

pytestmark = pytest.mark.gpu


def _shifted(torch, shape, dtype, by):
    """a tensor whose data starts `by` elements into its allocation"""
    n = int(np.prod(shape))
    return torch.zeros(n + by, dtype=dtype, device="cuda")[by:by + n].view(shape)


@pytest.mark.parametrize("M,shift", [(31, 0), (33, 1), (8193, 0), (16385, 0)])
def test_row_blocks_match_oracle(M, shift):
    import torch
    p, X, y = _problem(500 + M, M)
    net = _net(torch, p)
    Xd = _shifted(torch, (M, 512), torch.int16, shift)
    Xd.copy_(torch.from_numpy(tsf.bf16_bits(X)))
    h1, h2, d1, d2 = (_shifted(torch, (M, 256), torch.int16, shift) for _ in range(4))
    logit, d3 = (torch.zeros(M, dtype=torch.float32, device="cuda") for _ in range(2))
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    yd = torch.from_numpy(y.astype(np.float32)).cuda()
    net.forward(Xd, h1, h2, logit)
    tsf.check(tsf.lib().tsf_mlp_bwd(
        C.byref(net.c()), *[C.c_void_p(t.data_ptr()) for t in (Xd, yd)], M,
        *[C.c_void_p(t.data_ptr()) for t in (h1, h2, logit, d2, d1, d3, loss)], net._stream()))
    torch.cuda.synchronize()
    f = ref.forward(p, X)
    assert (np.abs(tsf.bf16_to_float(h1.cpu().numpy()) - f["h1"]) <= 2 ** -6 * f["m1"] + 1e-6).all()
    m2 = np.abs(f["h1"]) @ np.abs(ref.bf16_round(p["W2"])) + np.abs(p["b2"])
    assert (np.abs(tsf.bf16_to_float(h2.cpu().numpy()) - f["h2"])
            <= 2 ** -5 * (m2 + f["m1"].max()) + 1e-6).all()
    assert (np.abs(logit.cpu().numpy() - f["logit"]) <= 2 ** -5 * (f["m3"] + 1) + 1e-6).all()
    g, _ = ref.backward(p, X, y)
    gg = net.unpack(net.grad.cpu().numpy())
    e3 = (1.0 / (1.0 + np.exp(-f["logit"])) - y) / M
    e2 = np.abs(np.outer(e3, ref.bf16_round(p["w3"])))
    e1 = e2 @ np.abs(ref.bf16_round(p["W2"])).T
    mass = {"w3": np.abs(f["h2"]).T @ np.abs(e3), "b3": np.array([np.abs(e3).sum()]),
            "W2": np.abs(f["h1"]).T @ e2, "b2": e2.sum(axis=0),
            "W1": np.abs(X).T @ e1, "b1": e1.sum(axis=0)}
    for k, S in mass.items():
        assert (np.abs(gg[k] - g[k]) <= 2 ** -5 * S + 2 ** -5 * np.abs(g[k]) + 1e-6).all(), k
    assert abs(float(loss.item()) - ref.loss(p, X, y)) <= 1e-3 * (1 + ref.loss(p, X, y))
