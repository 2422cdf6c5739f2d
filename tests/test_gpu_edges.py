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


def _enumerated_min(n):
    """(E_min, count over all 2^n, smallest code with s_0 = +1) by Eq. 1-2 on
    every code, as plain tensor arithmetic on 64-bit integers."""
    best, count, first = 1 << 30, 0, None
    step = 1 << 22
    for c0 in range(0, 1 << (n - 1), step):
        code = torch.arange(c0, min(c0 + step, 1 << (n - 1)), device="cuda") * 2
        bit = [1 - 2 * ((code >> i) & 1) for i in range(n)]
        e = torch.zeros_like(code)
        for k in range(1, n):
            c = torch.zeros_like(code)
            for i in range(n - k):
                c += bit[i] * bit[i + k]
            e += c * c
        m = int(e.min())
        if m <= best:
            at = code[e == m]
            if m < best:
                best, count, first = m, 0, int(at[0])
            count += 2 * at.numel()
    return best, count, first


# both sides of the line between enumeration and branch and bound
@pytest.mark.parametrize("n", [23, 24, 25, 26])
def test_exhaustive_minimum_both_methods(lb, n):
    e, count, seq = lb.bruteforce_min(n)
    code = sum(1 << i for i, s in enumerate(seq) if s < 0)
    assert (e, count, code) == _enumerated_min(n)


# odd and even lengths, 32- and 64-bit masks; values of the plain enumeration of all 2^(n-1) codes
@pytest.mark.parametrize("n,e,count,code", [
    (28, 50, 8, 0x4b7770e), (29, 62, 8, 0x31fd5b2), (30, 59, 16, 0x1f6d5ce),
    (31, 67, 8, 0x52b26380), (32, 64, 8, 0x14ae326), (33, 64, 8, 0x13355a780),
    (34, 65, 8, 0xcc01e5aa), (35, 73, 8, 0x9b2b51c)])
def test_exhaustive_minimum_search(lb, n, e, count, code):
    got_e, got_count, seq = lb.bruteforce_min(n)
    assert (got_e, got_count) == (e, count)
    assert sum(1 << i for i, s in enumerate(seq) if s < 0) == code
