"""GPU kernels at the edges of their words, tiles and row layouts, against the
CPU oracle.  Every result is a whole number: equality."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2504_00987_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lb():
    from paper_2504_00987_amd.labs import Labs
    h = Labs(0)
    yield h
    h.close()


def _packed_rows(ns, stride, shift, seed):
    """Rows of ns[b] spins, `stride` bytes apart, the first `shift` bytes into
    an allocation; the bytes between rows hold -1, which no result may see.
    The allocation ends with the last row's last spin padded to the stride."""
    rows = I.random_pm1_ragged(np.asarray(ns, dtype=np.int32), stride, seed)
    rows[np.arange(stride)[None, :] >= np.asarray(ns)[:, None]] = -1
    flat = torch.full((shift + rows.size,), -1, dtype=torch.int8, device="cuda")
    flat[shift:] = torch.from_numpy(rows.reshape(-1)).cuda()
    return rows, flat[shift:].view(len(ns), stride)


@pytest.mark.parametrize("n", [3, 4, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160,
                               192, 193, 224, 225, 255, 256])
@pytest.mark.parametrize("pad,shift,count", [(0, 0, 64), (1, 1, 65), (5, 3, 1), (16, 16, 130)])
def test_energy_rows_of_any_alignment(lb, n, pad, shift, count):
    rows, dev = _packed_rows([n] * count, n + pad, shift, seed=7 * n + pad)
    got = lb.energy_batch(dev, n_uniform=n).cpu().numpy()
    assert np.array_equal(got, O.energy_batch(rows, n_uniform=n))


@pytest.mark.parametrize("lo,hi,count", [(3, 20, 200), (3, 256, 129), (100, 256, 63)])
def test_energy_mixed_lengths_in_one_group(lb, lo, hi, count):
    ns = I.uneven_lengths(count, lo, hi, seed=lo + hi)
    rows, dev = _packed_rows(ns, hi + 3, 5, seed=hi)
    got = lb.energy_batch(dev, ns=torch.from_numpy(ns).cuda()).cpu().numpy()
    assert np.array_equal(got, O.energy_batch(rows, ns=ns))


@pytest.mark.parametrize("n", [3, 4, 31, 32, 62, 63, 64, 65, 66, 67, 68, 127, 128, 129, 130, 131,
                               132, 191, 192, 193, 194, 195, 255, 256])
def test_skew_deviation_word_edges(lb, n):
    # around the lengths where a candidate's pairs fill whole 32-bit words,
    # all-equal and alternating rows (the most and fewest broken pairs) included
    rows, dev = _packed_rows([n] * 7, n + 1, 1, seed=n)
    rows[0, :n] = 1
    rows[1, :n] = 1 - 2 * (np.arange(n) % 2)
    dev[:2, :n] = torch.from_numpy(rows[:2, :n]).cuda()
    got = lb.skew_deviation(dev, n_uniform=n).cpu().numpy()
    assert np.array_equal(got, [O.skew_deviation(r[:n]) for r in rows])
