"""Feature rows of more log records than a launch has wavefronts, and of more than 2^26."""
import pytest

from paper_2511_20317_amd import tsf

pytestmark = pytest.mark.gpu


def _records(n):
    """records whose masks, slot and rank differ from row to row"""
    import torch
    q = torch.arange(n, device="cuda")
    rec = torch.zeros((n, 16), dtype=torch.int64, device="cuda")
    rec[:, 0] = q
    rec[:, 1] = 20 + q % 70
    rec[:, 2] = q % 16
    for k in range(6):
        rec[:, 3 + 2 * k] = (q * 2654435761 + k * 40503) % (1 << 62)
        rec[:, 4 + 2 * k] = rec[:, 3 + 2 * k] & (q * 7919 + k)
    return rec


@pytest.mark.parametrize("n", [1, 3, 4, 5, 262143, 262144, 262145, 3 * 262144 + 2])
def test_rows_in_turn_equal_rows_of_small_calls(n):
    import torch
    rec = _records(n)
    X = tsf.features_from_log(rec)
    step = 100003
    for at in range(0, n, step):
        assert torch.equal(X[at:at + step], tsf.features_from_log(rec[at:at + step].contiguous()))


def test_more_than_2_to_26_rows():
    import torch
    n = (1 << 26) + 3                      # 64 GiB of rows, 8 GiB of records
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GiB of free GPU memory")
    rec = torch.zeros((n, 16), dtype=torch.int64, device="cuda")
    few = _records(1000)
    places = [0, 262144, (1 << 25) + 7, n - 1000]
    for at in places:
        rec[at:at + 1000] = few
    X = tsf.features_from_log(rec)
    want = tsf.features_from_log(few)
    for at in places:
        assert torch.equal(X[at:at + 1000], want)
    del X, rec
    torch.cuda.empty_cache()
