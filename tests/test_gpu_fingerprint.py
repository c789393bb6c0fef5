"""The term-parallel kernels with one walk per wavefront against the oracle
where their parts change: numbers of attempts at the edges of the shared draws
(2^k lanes an iteration, one draw for 64 lanes), calls that end within a draw,
term slots per lane, factor widths, and both sets of coefficients."""
import pytest

from paper_2511_20317_amd import tsf
from tests.gpu_parity import compare, run_oracle

pytestmark = pytest.mark.gpu


def _check(fmt, cap, mode, tries, max_len, splits, walks=12, **kw):
    s = tsf.init_scheme(*fmt, mode=mode)
    groups = [(s, walks, cap, 0)]
    iters = sum(splits)
    prm = tsf.walk_params(base_seed=77, max_iters=iters, plateau=90, flip_tries=tries, **kw)
    ctx = tsf.Context()
    b = tsf.WalkBatch(groups, capacity=cap, rec_cap=16)
    b.max_len = max(b.max_len, max_len)
    b.init(ctx)
    for n in splits:
        b.walk(ctx, prm, n, 64, 1 if tries % 2 else 4, 2)
    import torch
    torch.cuda.synchronize()
    compare(b, run_oracle(groups, prm, range(walks), iters, splits),
            "%s cap %d tries %d" % (fmt, cap, tries))


@pytest.mark.parametrize("tries", [1, 2, 3, 4, 7, 8, 15, 16, 31, 32, 62, 63, 64])
def test_draws_shared_by_iterations(tries):
    _check((2, 3, 3), 30, tsf.TSF_TERNARY, tries, 1, [1, 5, 64, 130], t_expand=1 << 30)


@pytest.mark.parametrize("mode", [tsf.TSF_TERNARY, tsf.TSF_Z2])
@pytest.mark.parametrize("fmt,cap,max_len", [
    ((3, 3, 3), 64, 1), ((3, 3, 3), 65, 1), ((4, 4, 5), 128, 1), ((3, 3, 3), 64, 64),
    ((3, 3, 3), 129, 64), ((2, 2, 17), 76, 1), ((4, 4, 5), 257, 64), ((5, 5, 5), 321, 64)])
def test_slots_and_widths(mode, fmt, cap, max_len):
    _check(fmt, cap, mode, 7, max_len, [150, 51], t_expand=1 << 29, t_reduce=3 << 30)
