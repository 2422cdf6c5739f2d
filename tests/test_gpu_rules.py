"""GPU kernels on both sides of the lines where the library picks another form
of a launch, against the CPU oracle.  Every result is a whole number:
equality."""
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


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


# walks of N <= 32: two per wavefront up to 16 (as a persistent grid 8) walks per compute unit, four
# beyond, the last wavefront partly idle; lengths at the edges of the lanes and mixed ones
@pytest.mark.parametrize("lengths", [(17, 17), (31, 31), (32, 32), (3, 32)])
@pytest.mark.parametrize("launch,line", [((64, 2), 16), ((128, 4), 16), ((64, 2, 1), 8),
                                         ((64, 4), 16)])
@pytest.mark.parametrize("aspiration", [0, 1])
def test_short_walk_forms(lb, launch, line, lengths, aspiration):
    rules = I.Rules(I.STEPS_MULT_N, 2, I.TENURE_LINEAR, 1, 10, 0, 1, 5, 0, aspiration)
    lo, hi = lengths
    for walks in (1, 3, line * _cus(), line * _cus() + 1, line * _cus() + 3):
        ns = None if lo == hi else I.uneven_lengths(walks, lo, hi, seed=walks)
        kw = dict(ns=ns, n_uniform=hi if lo == hi else 0, out_stride=128, trace_stride=2 * hi)
        res = {}
        for form in (launch, (64, 1)):
            lb.set_launch(*form)
            try:
                res[form] = lb.tabu_batch(rules, walks, 23, **kw)
            finally:
                lb.set_launch(None)
        a, b = res.values()
        for x, y in ((a.best_e, b.best_e), (a.final_e, b.final_e), (a.best_seq, b.best_seq),
                     (a.trace, b.trace)):
            assert torch.equal(x, y), walks
        head = min(walks, 12)
        best, be, fe, _ = _oracle_walks(head, hi if ns is None else ns, rules, 23, with_trace=False)
        assert np.array_equal(a.best_e[:head].cpu().numpy(), be[:head])
        assert np.array_equal(a.best_seq[:head, :best.shape[1]].cpu().numpy(), best[:head])


# both sides of the lines where a replica gets fewer wavefronts: replicas per compute unit, and
# populations too small to keep more of them busy
@pytest.mark.parametrize("n,per_cu", [(24, 1), (24, 8), (70, 1), (70, 8), (130, 1), (130, 2)])
@pytest.mark.parametrize("K,children", [(2, 1), (7, 1), (8, 1), (24, 1), (2, 3), (40, 2)])
def test_memetic_wavefronts(lb, n, per_cu, K, children):
    rules = I.RULES_MEMETIC
    gens = 13 if children == 1 else 5
    kw = dict(n_uniform=n, out_stride=256, children=children)
    line = per_cu * _cus()
    runs = [lb.memetic_run(K, rules, gens, pops, 6, **kw) for pops in (line, line + 1, 3)]
    for r in runs[:2]:
        assert torch.equal(r.best_e[:3], runs[2].best_e)
        assert torch.equal(r.best_seq[:3], runs[2].best_seq)
    assert torch.equal(runs[0].best_seq, runs[1].best_seq[:line])
    ref = _oracle_memetic([n] * 3, K, rules, gens, 6, children=0 if children == 1 else children)
    assert [int(e) for e in runs[2].best_e] == [st.bestE for st in ref]


# both sides of the lines where one wavefront draws a population, and populations at the edges of a
# wavefront's lanes
@pytest.mark.parametrize("n,per_cu", [(3, 4), (33, 4), (128, 4), (129, 16), (256, 16)])
@pytest.mark.parametrize("K", [2, 63, 64, 65, 128])
def test_memetic_populations(lb, n, per_cu, K):
    line = per_cu * _cus()
    runs = []
    for pops in (line, line + 1):
        r = lb.memetic_run(K, I.RULES_MEMETIC, 0, pops, 11, n_uniform=n, out_stride=256)
        runs.append((r, np.frombuffer(lb.memetic_save(), dtype=np.uint8)))
    (a, blob_a), (b, blob_b) = runs
    assert torch.equal(a.best_e, b.best_e[:line]) and torch.equal(a.best_seq, b.best_seq[:line])
    # every member of the common replicas: 32 bytes each, after the header and the lengths
    at = [256 + (4 * p + 255) // 256 * 256 for p in (line, line + 1)]
    size = line * K * 32
    assert np.array_equal(blob_a[at[0]:at[0] + size], blob_b[at[1]:at[1] + size])
    ref = _oracle_memetic([n] * 2, K, I.RULES_MEMETIC, 0, 11)
    assert [int(e) for e in a.best_e[:2]] == [st.bestE for st in ref]


# launches of one generation, and of many on one wavefront per replica: more children than
# wavefronts, targets reached on the way, generations past a replica's limit
@pytest.mark.parametrize("mode,chunk", [(0, 5), (1, 5), (2, 1)])
@pytest.mark.parametrize("K,children", [(2, 1), (3, 2), (100, 1), (100, 3), (128, 8)])
def test_memetic_generations_one_at_a_time(lb, mode, chunk, K, children):
    ns = np.array([3, 24, 64, 65, 128, 129, 193, 256], dtype=np.int32)
    rules, gens = I.RULES_MEMETIC, 7
    batch = 0 if children == 1 else children
    ref = _oracle_memetic(ns, K, rules, gens, 91, children=batch)
    kw = dict(ns=ns, out_stride=256, children=children, mode=mode, chunk=chunk)
    res = lb.memetic_run(K, rules, gens, len(ns), 91, **kw)
    for p, st in enumerate(ref):
        assert (int(res.best_e[p]), int(res.gens_done[p])) == (st.bestE, gens)
        assert np.array_equal(res.best_seq[p, :int(ns[p])].cpu().numpy(), st.best)
    target = sorted(st.bestE for st in ref)[len(ns) // 2]
    ref = _oracle_memetic(ns, K, rules, gens, 91, target=target, children=batch)
    res = lb.memetic_run(K, rules, gens, len(ns), 91, target=target, **kw)
    for p, st in enumerate(ref):
        assert (int(res.best_e[p]), int(res.hit_gen[p]), int(res.gens_done[p])) == (
            st.bestE, st.hit, st.gen)
    # many replicas of a small population: one wavefront each, also in longer launches
    pops = 16 * _cus() + 1
    many = lb.memetic_run(2, rules, gens, pops, 91, n_uniform=65, out_stride=256, children=children,
                          chunk=4)
    one = lb.memetic_run(2, rules, gens, 8, 91, n_uniform=65, out_stride=256, children=children,
                         mode=mode, chunk=chunk)
    assert torch.equal(many.best_seq[:8], one.best_seq) and torch.equal(many.best_e[:8], one.best_e)


# the longest lengths of the exhaustive search: the roots' depth stops at 13 pairs, a node's halves
# are full at n = 40; values of the plain enumeration of all 2^(n-1) codes
@pytest.mark.parametrize("n,e,count,code", [
    (36, 82, 8, 0x1f8c51252), (37, 86, 8, 0x13354b0f00), (38, 87, 8, 0x3c34aa66),
    (39, 99, 8, 0x49a150179c), (40, 108, 8, 0x2223dc3a5a)])
def test_exhaustive_minimum_longest(lb, n, e, count, code):
    got_e, got_count, seq = lb.bruteforce_min(n)
    assert (got_e, got_count) == (e, count) and O.energy(seq) == e
    assert sum(1 << i for i, s in enumerate(seq) if s < 0) == code
    # the smallest of its images with s_0 = +1
    alternating = 1 - 2 * (np.arange(n) % 2)
    for image in (seq, seq * alternating, seq[::-1], seq[::-1] * alternating):
        image = image * image[0]
        assert code <= sum(1 << i for i, s in enumerate(image) if s < 0)


# both sides of the line from which walks of one length issue ahead, on any number of compute units
@pytest.mark.parametrize("n", [40, 200])
def test_issue_priority_line(lb, n):
    rules = I.Rules(I.STEPS_FIXED, 70, I.TENURE_LINEAR, 1, 10, 0, 1, 5, 0, 1)
    line = 8 * _cus()
    few, many = (lb.tabu_batch(rules, w, 17, n_uniform=n, out_stride=256) for w in (line - 1, line))
    for a, b in ((few.best_e, many.best_e), (few.final_e, many.final_e),
                 (few.best_seq, many.best_seq)):
        assert torch.equal(a, b[:line - 1])
    assert np.array_equal(many.best_e.cpu().numpy()[:8],
                          _oracle_walks(8, n, rules, 17, with_trace=False)[1])


def test_server_forgets_a_cancelled_request_that_was_waiting(lb):
    # cancelled and polled while another request holds the slots: nothing is admitted in its place
    import time
    from paper_2504_00987_amd import _lib
    from paper_2504_00987_amd.labs import Server
    srv = Server(lb, 16, I.RULES_MEMETIC, max_slots=4, chunk=8)
    try:
        first = srv.submit(120, 11, 4, 4000)
        drop = srv.submit(41, 12, 4, 5)
        srv.cancel(drop)
        with pytest.raises(_lib.LabsError) as err:
            srv.poll(drop, 41)
        assert err.value.code == _lib.LABS_E_CANCELLED
        last = srv.submit(40, 13, 3, 5)
        got, t0 = {}, time.time()
        while len(got) < 2 and time.time() - t0 < 60:
            for rid, n in ((first, 120), (last, 40)):
                if rid not in got and (r := srv.poll(rid, n)) is not None:
                    got[rid] = r
            assert sum(srv.stats()[:2]) <= 2
            time.sleep(0.002)
        assert len(got) == 2
        assert srv.stats() == (0, 0, 2, 0)
    finally:
        srv.close()
    ref = _oracle_memetic([40] * 3, 16, I.RULES_MEMETIC, 5, 13)
    assert got[last][1] == min(st.bestE for st in ref)


@pytest.mark.parametrize("n_min,n_max,most", [(32, 32, 25), (3, 32, 30), (64, 64, 15)])
def test_autotune_of_short_walks_is_short(n_min, n_max, most):
    # a persistent grid of each size that fits, no larger ones
    from paper_2504_00987_amd.labs import Labs
    h = Labs(0)
    try:
        assert h.autotune(I.rules_tabu(2), n_min, n_max, 256) <= most
    finally:
        h.close()


# up to N = 32 a row's rotations come from registers, beyond from LDS
@pytest.mark.parametrize("n", [5, 6, 16, 17, 21, 22, 30, 31, 32, 33, 34])
def test_skew_deviation_short_rows(lb, n):
    rows = I.random_pm1(70, n, n + 3, seed=n)
    rows[:, n:] = -1  # past the rows: not looked at
    rows[0, :n] = 1
    rows[1, :n] = 1 - 2 * (np.arange(n) % 2)
    got = lb.skew_deviation(torch.from_numpy(rows).cuda(), n_uniform=n).cpu().numpy()
    assert np.array_equal(got, [O.skew_deviation(r[:n]) for r in rows])
