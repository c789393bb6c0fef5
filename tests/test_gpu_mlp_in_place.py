"""Network passes whose outputs or workspaces lie over inputs that the pass has used by
then: the same results, bit for bit, as with buffers of their own."""
import ctypes as C
import functools

import numpy as np
import pytest

from paper_2511_20317_amd import tsf
from tests.test_gpu_mlp import _net, _problem

pytestmark = pytest.mark.gpu


def _ptr(t):
    return C.c_void_p(t.data_ptr())


_made = functools.lru_cache(None)(_problem)


def _inputs(M, shift):
    import torch
    p, X, y = _made(900 + M, M)
    Xd = torch.zeros(M * 512 + shift, dtype=torch.int16, device="cuda")[shift:].view(M, 512)
    Xd.copy_(torch.from_numpy(tsf.bf16_bits(X)))
    return _net(torch, p), Xd, torch.from_numpy(y.astype(np.float32)).cuda()


SIZES = [(1, 0), (33, 0), (33, 1), (5000, 0), (20000, 0)]


@pytest.mark.parametrize("M,shift", SIZES)
@pytest.mark.parametrize("over", ["h2 in X", "h2 in the end of X", "logit in X", "logit in h1"])
def test_forward(M, shift, over):
    import torch
    net, X, _ = _inputs(M, shift)
    h1, h2, logit = net.forward(X)
    want = [t.clone() for t in (h1, h2, logit)]
    g1, g2, gl = torch.zeros_like(h1), torch.zeros_like(h2), torch.zeros_like(logit)
    if over == "h2 in X":
        g2 = X.view(-1)[:M * 256].view(M, 256)
    elif over == "h2 in the end of X":
        g2 = X.view(-1)[M * 256:].view(M, 256)
    elif over == "logit in X":
        gl = X.view(-1)[shift:][:2 * M].view(torch.float32)
    else:
        gl = g1.view(-1)[:2 * M].view(torch.float32)
    net.forward(X, g1, g2, gl)
    assert torch.equal(g2, want[1]) and torch.equal(gl, want[2])
    if over != "logit in h1":
        assert torch.equal(g1, want[0])


@pytest.mark.parametrize("M,shift", SIZES)
@pytest.mark.parametrize("over", ["d1 is h1", "d1 is h2", "d3 is logit", "d1 is h1, d3 is logit",
                                  "d1 over logit", "d1 over y"])
def test_backward(M, shift, over):
    import torch
    net, X, y = _inputs(M, shift)
    h1, h2, logit = net.forward(X)

    def backward(h1, h2, logit, y, d1, d3):
        d2, loss = torch.zeros_like(h2), torch.zeros(1, device="cuda")
        net.grad.fill_(7)
        tsf.check(tsf.lib().tsf_mlp_bwd(C.byref(net.c()), _ptr(X), _ptr(y), M, _ptr(h1), _ptr(h2),
                                        _ptr(logit), _ptr(d2), _ptr(d1), _ptr(d3), _ptr(loss),
                                        net._stream()))
        return [t.clone() for t in (net.grad, loss, d2, d1, d3)]

    want = backward(h1, h2, logit, y, torch.zeros_like(h1), torch.zeros_like(logit))
    d1, d3 = torch.zeros_like(h1), torch.zeros_like(logit)
    if "d1 is h1" in over:
        d1 = h1
    if "d1 is h2" in over:
        d1 = h2
    if "d3 is logit" in over:
        d3 = logit
    if "d1 over" in over:                 # the last rows of d1 hold the logits or the labels
        tail = d1.view(-1)[-2 * M:].view(torch.float32)
        tail.copy_(logit if over == "d1 over logit" else y)
        logit, y = (tail, y) if over == "d1 over logit" else (logit, tail)
    got = backward(h1, h2, logit, y, d1, d3)
    for w, g in zip(want, got):
        assert torch.equal(w, g), over
