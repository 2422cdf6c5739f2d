"""GPU kernels at the edges of their words, tiles and row layouts, against the
CPU oracle.  Every result is a whole number: equality."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2504_00987_amd import inputs as I
from tests.test_gpu_parity import _oracle_memetic, _oracle_walks

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


# neighbours per lane and their masks change at 64, 128 and 192, several walks share a wavefront at
# N <= 32 (16 lanes with one or two neighbours each), the last group of such a batch is partly idle
@pytest.mark.parametrize("n", [15, 16, 17, 32, 33, 64, 65, 128, 129, 191, 192, 193, 256])
@pytest.mark.parametrize("launch,walks", [((64, 1), 3), ((128, 2), 5), ((256, 4), 7),
                                          ((64, 2), 5), ((64, 4), 1), ((64, 4), 9)])
def test_walk_class_edges(lb, n, launch, walks):
    rules = I.Rules(I.STEPS_MULT_N, 1, I.TENURE_LINEAR, 1, 10, 0, 1, 5, 0, 1)
    lb.set_launch(*launch)
    try:
        res = lb.tabu_batch(rules, walks, 99 + n, n_uniform=n, out_stride=256, trace_stride=n)
    finally:
        lb.set_launch(None)
    best, be, fe, trs = _oracle_walks(walks, n, rules, 99 + n)
    assert np.array_equal(res.best_e.cpu().numpy(), be)
    assert np.array_equal(res.final_e.cpu().numpy(), fe)
    assert np.array_equal(res.best_seq.cpu().numpy()[:, :best.shape[1]], best)
    assert np.array_equal(res.trace.cpu().numpy()[:, :n], np.stack(trs))


# the default layout changes between 2048 and 2049 walks (N <= 16) and 4096 and 4097 (N <= 32)
@pytest.mark.parametrize("lo,hi,walks", [(9, 16, 2048), (9, 16, 2049), (12, 32, 4096),
                                         (12, 32, 4097), (12, 40, 4097)])
def test_default_layout_lines(lb, lo, hi, walks):
    rules = I.rules_tabu(2)
    ns = I.uneven_lengths(walks, lo, hi, seed=walks)
    res = lb.tabu_batch(rules, walks, 5, ns=ns)
    lb.set_launch(64, 1)
    try:
        one = lb.tabu_batch(rules, walks, 5, ns=ns)
    finally:
        lb.set_launch(None)
    for a, b in ((res.best_e, one.best_e), (res.final_e, one.final_e), (res.best_seq, one.best_seq)):
        assert torch.equal(a, b)
    head = _oracle_walks(20, ns, rules, 5, with_trace=False)[1]
    assert np.array_equal(res.best_e.cpu().numpy()[:20], head)


# children in flight: with K = 2 and 3 nearly every child waits for the one before it, with 128
# few do; more and fewer generations than wavefronts; generations of one, three, seven and eight
@pytest.mark.parametrize("K,gens,chunk", [(2, 21, 21), (3, 40, 7), (17, 5, 3), (128, 33, 33)])
@pytest.mark.parametrize("children", [1, 3, 7, 8])
def test_memetic_children_in_flight(lb, K, gens, chunk, children):
    ns = np.array([24, 33, 64, 65, 96, 129, 193], dtype=np.int32)
    rules = I.RULES_MEMETIC
    batch = 0 if children == 1 else children
    ref = _oracle_memetic(ns, K, rules, gens, 31 + K, children=batch)
    res = lb.memetic_run(K, rules, gens, len(ns), 31 + K, ns=ns, chunk=chunk, children=children,
                         out_stride=256)
    for p, st in enumerate(ref):
        assert (int(res.best_e[p]), int(res.gens_done[p])) == (st.bestE, gens)
        assert np.array_equal(res.best_seq[p, :int(ns[p])].cpu().numpy(), st.best)
    # a target that some replicas reach on the way, with later children in flight
    target = sorted(st.bestE for st in ref)[len(ns) // 2]
    ref = _oracle_memetic(ns, K, rules, gens, 31 + K, target=target, children=batch)
    res = lb.memetic_run(K, rules, gens, len(ns), 31 + K, ns=ns, chunk=chunk, children=children,
                         out_stride=256, target=target)
    for p, st in enumerate(ref):
        assert (int(res.best_e[p]), int(res.hit_gen[p])) == (st.bestE, st.hit)
        assert int(res.gens_done[p]) == st.gen


# both sides of the lines where a replica gets fewer wavefronts
@pytest.mark.parametrize("n,pops", [(70, 256), (70, 257), (24, 2048), (24, 2049), (70, 2049),
                                    (130, 512), (130, 513)])
def test_memetic_wavefront_lines(lb, n, pops):
    rules = I.RULES_MEMETIC
    kw = dict(n_uniform=n, out_stride=256)
    many = lb.memetic_run(20, rules, 11, pops, 6, **kw)
    few = lb.memetic_run(20, rules, 11, 24, 6, **kw)
    assert torch.equal(many.best_e[:24], few.best_e)
    assert torch.equal(many.best_seq[:24], few.best_seq)
    ref = _oracle_memetic([n] * 4, 20, rules, 11, 6)
    assert [int(e) for e in many.best_e[:4]] == [st.bestE for st in ref]


# batches of one length run with raised issue priority from 2048 walks (two wavefronts per SIMD) on;
# a batch of two lengths runs without
@pytest.mark.parametrize("n", [40, 64, 65, 130, 200])
@pytest.mark.parametrize("walks", [2047, 2048])
def test_one_length_priority_line(lb, n, walks):
    rules = I.Rules(I.STEPS_FIXED, 70, I.TENURE_LINEAR, 1, 10, 0, 1, 5, 0, 1)
    kw = dict(out_stride=256)
    one = lb.tabu_batch(rules, walks, 17, n_uniform=n, **kw)
    ns = np.full(walks + 1, n, dtype=np.int32)
    ns[walks] = n - 1
    two = lb.tabu_batch(rules, walks + 1, 17, ns=ns, **kw)
    for a, b in ((one.best_e, two.best_e), (one.final_e, two.final_e), (one.best_seq, two.best_seq)):
        assert torch.equal(a, b[:walks])
    assert np.array_equal(one.best_e.cpu().numpy()[:8],
                          _oracle_walks(8, n, rules, 17, with_trace=False)[1])
