"""GPU parity of ps_route (the router's scoring over a micro-batch, paper Sec. 3.4.3) against the
oracle, through the C ABI: decisions, scores and the updated state are integers and must match."""
import numpy as np
import pytest
import torch

from oracle import router as orr
from paper_2504_03702_amd import binding as ps

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_route(P, D, win, cap, qp, cd, **kw):
    K, l = win.shape
    t32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(DEV)
    t64 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int64)).to(DEV)
    n = len(P)
    w_t, qp_t, cd_t = t32(win).reshape(-1), t64(qp), t64(cd)
    a_t = torch.full((n,), -7, dtype=torch.int32, device=DEV)
    s_t = torch.full((n,), -7, dtype=torch.int64, device=DEV)
    st = ps.new_status(DEV)
    ps.ps_route(t32(P), t32(D), K, l, w_t if l > 0 else None, t32(cap), qp_t, cd_t, a_t, s_t, status=st, **kw)
    flags, bad = ps.ps_status_read(st)
    return (a_t.cpu().numpy(), s_t.cpu().numpy(), w_t.cpu().numpy().reshape(K, l), qp_t.cpu().numpy(),
            cd_t.cpu().numpy(), flags, bad)


def random_case(rng, K, l, n, hot):
    cap = rng.integers(2000, 6000, K) if hot else rng.integers(100_000, 400_000, K)
    win = rng.integers(0, cap.max() // 2, (K, l))
    qp, cd = rng.integers(0, 3000, K), rng.integers(0, 20000, K)
    P = np.clip(np.rint(np.exp(rng.normal(np.log(52.0), 1.2, n))), 7, 2048).astype(np.int64)
    D = np.clip(np.rint(np.exp(rng.normal(np.log(87.0), 1.3, n))), 0, 4096).astype(np.int64)
    return P, D, win, cap, qp, cd


@pytest.mark.parametrize("K,l,n,hot", [(1, 1, 5, False), (3, 8, 40, True), (4, 100, 300, True), (64, 100, 1000, False),
                                       (256, 100, 4096, True), (256, 100, 512, False), (1000, 30, 200, True),
                                       (17, 333, 100, True), (5, 0, 20, False)])
def test_decisions_scores_and_state_match(K, l, n, hot):
    print(f"route K={K} l={l} n={n} hot={hot}", flush=True)
    P, D, win, cap, qp, cd = random_case(np.random.default_rng(K * 1000 + l), K, l, n, hot)
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd)
    assert flags == 0
    assert np.array_equal(a, ra) and np.array_equal(s, rs)
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)
    if K > 1 and n >= 40:
        assert len(np.unique(ra)) > 1                       # the batch really is spread over instances


def test_hand_cases_ties_penalty_and_other_parameters():
    win = np.array([[900] * 4, [0] * 4])
    a, s, *_ = run_route([50], [4], win, [1000, 1000], [0, 200], [0, 0])
    assert a.tolist() == [0] and s.tolist() == [20700]
    a, s, *_ = run_route([50], [4], win, [1000, 1000], [0, 200], [0, 0], beta=2)        # twice the penalty
    assert a.tolist() == [1] and s.tolist() == [100 * 254]
    a, s, *_ = run_route([50], [4], win, [1000, 1000], [0, 200], [0, 0], t_mem_pct=96)   # no penalty yet
    assert a.tolist() == [0] and s.tolist() == [5400]
    a, s, w, qp, cd, *_ = run_route([10] * 4, [5] * 4, np.zeros((3, 8), np.int64), [10**6] * 3, [0] * 3, [0] * 3)
    assert a.tolist() == [0, 1, 2, 0] and qp.tolist() == [20, 10, 10] and w[0].tolist() == [20, 22, 24, 26, 28, 0, 0, 0]


def test_missing_predictions_and_limits():
    win = np.zeros((2, 4), np.int64)
    a, s, w, qp, cd, flags, bad = run_route([10, 10, -3], [5, -1, 5], win, [1000, 1000], [0, 0], [0, 0])
    assert a.tolist() == [0, -1, -1] and s.tolist() == [1500, 0, 0] and qp.tolist() == [10, 0]
    assert flags == ps.PS_ST_BAD_RECORD and bad == 1
    z32 = torch.zeros(2048, dtype=torch.int32, device=DEV)
    z64 = torch.zeros(2048, dtype=torch.int64, device=DEV)
    with pytest.raises(ps.PsError) as e:                    # more instances than one workgroup has threads
        ps.ps_route(z32[:1], z32[:1], 1025, 0, None, z32[:1025], z64[:1025], z64[:1025], z32[:1], z64[:1])
    assert e.value.code == -6
    big = torch.zeros(256 * 200, dtype=torch.int32, device=DEV)
    with pytest.raises(ps.PsError) as e:                    # windows that do not fit the LDS
        ps.ps_route(z32[:1], z32[:1], 256, 200, big, z32[:256], z64[:256], z64[:256], z32[:1], z64[:1])
    assert e.value.code == -6


@pytest.mark.parametrize("K,l,n", [(64, 128, 150), (65, 129, 150), (2, 4, 200), (3, 5, 200), (63, 1, 130), (128, 127, 64),
                                   (1024, 29, 70),        # fills the LDS: one block per window
                                   (256, 134, 66),        # larger blocks than the smallest, to fit
                                   (7, 1000, 40), (1, 8000, 12), (2, 17000, 5),
                                   # requests and blocks at which the scan of whole windows takes over
                                   (64, 100, 1), (64, 100, 2), (64, 100, 3), (64, 500, 31), (64, 500, 32), (16, 1500, 127),
                                   (16, 1500, 128), (2, 1536, 130), (2, 1537, 130), (1024, 29, 2), (33, 600, 33), (9, 0, 1)])
def test_block_edges_and_full_lds(K, l, n):
    """The kernel keeps maxima per block of a window: predictions on, beside and beyond the block boundaries, maps of one
    wavefront and of several, and the largest maps the call accepts.  Integers: everything must match."""
    print(f"route blocks K={K} l={l} n={n}", flush=True)
    rng = np.random.default_rng(K * 7919 + l)
    P, D, win, cap, qp, cd = random_case(rng, K, l, n, True)
    edges = np.array([0, 1, 3, 4, 5, 8, l // 2, max(l - 4, 0), max(l - 1, 0), l, l + 1, 4096])
    D = np.where(rng.random(n) < 0.7, edges[rng.integers(0, len(edges), n)], D)
    win[0, :] = -5                                              # (values below zero keep their place in the maxima)
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd)
    assert flags == 0
    assert np.array_equal(a, ra) and np.array_equal(s, rs)
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)


@pytest.mark.parametrize("K,l,n", [(65, 100, 200), (129, 12, 257), (256, 128, 300), (257, 60, 150), (600, 40, 190),
                                   (130, 140, 140), (90, 0, 70), (1024, 29, 130), (256, 120, 40),
                                   (250, 125, 3), (256, 128, 200)])
@pytest.mark.parametrize("near", ["spread", "one instance", "last instance", "two wavefronts"])
def test_choices_that_follow_each_other(K, l, n, near):
    """Choices that stay with one instance, alternate between wavefronts, or fall on one that is alone in its wavefront;
    requests without a prediction between them, a whole group of 64 of them, and at both ends.  Integers: everything must
    match."""
    print(f"route choices K={K} l={l} n={n} {near}", flush=True)
    rng = np.random.default_rng(K * 31 + l)
    P, D, win, cap, qp, cd = random_case(rng, K, l, n, True)
    few = {"spread": [], "one instance": [min(K - 1, 70)], "last instance": [K - 1], "two wavefronts": [5, K - 1]}[near]
    if few:
        qp = qp + 10_000_000                                    # far more than the calls below add to the others
        qp[few] = 0
    D[rng.random(n) < 0.2] = 0
    bad = rng.random(n) < 0.1
    bad[[0, -1]] = True
    if n >= 192:
        bad[64:128] = True
    D[bad & (rng.random(n) < 0.5)] = -1
    P[bad & (D >= 0)] = -2
    a, s, w, q2, c2, flags, first = run_route(P, D, win, cap, qp, cd)
    ok = ~bad
    ra, rs, rw, rq, rc = orr.route(P[ok], D[ok], win, cap, qp, cd)
    assert flags == ps.PS_ST_BAD_RECORD and first == 0
    assert np.array_equal(a[ok], ra) and np.array_equal(s[ok], rs)
    assert (a[bad] == -1).all() and (s[bad] == 0).all()
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)


@pytest.mark.parametrize("K,l", [(5, 50), (64, 50), (130, 50), (260, 50), (70, 140), (100, 260), (6, 500), (256, 128)])
@pytest.mark.parametrize("beta,peak,queued", [(1, (1 << 29) // 100, 0), (1, (1 << 24), 0), (3, (1 << 29) // 300, 0),
                                              (1, 1000, (1 << 29) // 100), (0, 1 << 24, 5000), (700, 4000, 100),
                                              (1, 1000, -5), (1, -70000, 10)])
def test_values_that_pass_the_bounds_of_the_short_form(K, l, beta, peak, queued):
    """Scores and peaks of a call that start below the bounds for one-register scores and pass them on the way (each
    bound, with the penalty's factor), or lie outside from the start; limits of 0 and queues below 0 among them."""
    print(f"route bounds K={K} l={l} beta={beta} peak={peak} queued={queued}", flush=True)
    rng = np.random.default_rng(K + beta)
    P, D, win, cap, qp, cd = random_case(rng, K, l, 300, True)
    win = peak - rng.integers(0, 60_000, (K, l)) - np.arange(K)[:, None] % 7 * 3000
    cap[::3] = 0
    if queued > 1 << 20:
        qp = queued - rng.integers(0, 90_000, K)
    elif queued < 0:
        qp[K // 2] = queued
        cd[K // 2] = 0
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd, beta=beta)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd, beta=beta)
    assert flags == 0
    assert np.array_equal(a, ra) and np.array_equal(s, rs)
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)


@pytest.mark.parametrize("K,l,n", [(1, 16, 70), (5, 100, 300), (64, 128, 200), (65, 33, 130), (130, 100, 400),
                                   (256, 100, 1000), (256, 128, 150), (300, 60, 200), (700, 40, 300), (1000, 30, 300),
                                   # one wavefront's walk: beside larger blocks, without room for it, and at its most instances
                                   (250, 125, 300), (260, 100, 300), (512, 56, 200), (500, 60, 300), (513, 56, 200), (70, 50, 31),
                                   (70, 50, 32)])
@pytest.mark.parametrize("load", ["free", "mixed", "filling", "ties", "all over", "one by one", "uneven", "rising"])
def test_walks_over_free_and_full_windows(K, l, n, load):
    """Windows below their limits, over and near them, limits reached on the way, equal scores, requests that add nothing,
    faulty ones and lists that end inside a group of 64: what one wavefront walks to the end, does not begin or leaves on the
    way to the tables.  Integers: everything must match."""
    print(f"route walks K={K} l={l} n={n} {load}", flush=True)
    rng = np.random.default_rng(K * 131 + l + n)
    P, D, win, cap, qp, cd = random_case(rng, K, l, n, False)
    level = {"free": 0.1, "mixed": 1.0, "filling": 0.0, "ties": 0.0, "all over": 1.0, "one by one": 0.0}.get(load, 0.0)
    win = np.rint(rng.random((K, 1)) * level * cap[:, None] * (1.0 - 0.5 * np.arange(l) / l)).astype(np.int64)
    if load == "all over":
        win += cap[:, None]
    if load == "uneven":                                        # most requests' windows have to be read, after a while
        win = rng.integers(0, 200_000, (K, l))
    if load == "rising":
        win = np.rint(rng.random((K, 1)) * cap[:, None] * (0.5 + 0.5 * np.arange(l) / l)).astype(np.int64)
    if load == "filling":                                       # some requests each before the limit
        cap = 600 + 40 * np.arange(K) % 3000
    if load == "ties":
        qp[:], cd[:] = 7, 11
        P[rng.random(n) < 0.3] = 40
        D[P == 40] = 60
    if load == "one by one":                                    # one instance takes all, until it is at its limit
        qp = qp + 30_000
        qp[K // 2] = 0
        cap[K // 2] = 4000
    P[rng.random(n) < 0.1] = 0
    D[rng.random(n) < 0.1] = 0
    bad = rng.random(n) < 0.03
    P[bad] = -1
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ok = ~bad
    ra, rs, rw, rq, rc = orr.route(P[ok], D[ok], win, cap, qp, cd)
    assert flags == (ps.PS_ST_BAD_RECORD if bad.any() else 0)
    assert np.array_equal(a[ok], ra) and np.array_equal(s[ok], rs) and (a[bad] == -1).all() and (s[bad] == 0).all()
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)


@pytest.mark.parametrize("what", ["prompt", "prediction"])
@pytest.mark.parametrize("at", [0, 63, 64, 150, 259])
def test_a_huge_request_between_ordinary_ones(what, at):
    """A request of 2^20 tokens ends one wavefront's walk at the group it is in; those after it go on from its state."""
    print(f"route huge {what} at {at}", flush=True)
    rng = np.random.default_rng(at)
    P, D, win, cap, qp, cd = random_case(rng, 130, 40, 260, False)
    win = np.rint(rng.random((130, 1)) * 0.5 * cap[:, None] * (1.0 - 0.5 * np.arange(40) / 40)).astype(np.int64)
    (P if what == "prompt" else D)[at] = 1 << 20
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd)
    assert flags == 0
    assert np.array_equal(a, ra) and np.array_equal(s, rs)
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)


def test_windows_at_their_limits_go_by_the_tables():
    """4096 requests over full windows of 256 instances take no longer than the tables do (1.4 times as long as over 64
    instances, where there is no other walk; 1.9 when one wavefront read every window over and over)."""
    def fastest(K):
        rng = np.random.default_rng(K)
        P, D, _, cap, qp, cd = random_case(rng, K, 100, 4096, False)
        win = np.rint(cap[:, None] * (0.78 + 0.06 * rng.random((K, 100)))).astype(np.int64)
        t32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(DEV)
        t64 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int64)).to(DEV)
        P, D, win, cap, qp, cd = t32(P), t32(D), t32(win).reshape(-1), t32(cap), t64(qp), t64(cd)
        a, s, took = t32(np.zeros(4096)), t64(np.zeros(4096)), []
        for _ in range(8):
            state = win.clone(), qp.clone(), cd.clone()
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            ps.ps_route(P, D, K, 100, state[0], cap, state[1], state[2], a, s)
            e[1].record()
            torch.cuda.synchronize()
            took.append(e[0].elapsed_time(e[1]))
        return min(took)
    one, several = fastest(64), fastest(256)
    assert several < 1.6 * one, (one, several)


def test_state_of_an_instance_with_huge_queues():
    """The state is carried exactly in int64 also where a hundredfold no longer fits (10^17 tokens as a mark of an
    instance that is out of use)."""
    mark = 10**17
    a, s, w, qp, cd, flags, _ = run_route([10, 20, 30], [3, 1, 2], np.zeros((1, 4), np.int64), [1000], [mark], [mark + 7])
    assert flags == 0 and a.tolist() == [0, 0, 0]
    assert qp.tolist() == [mark + 60] and cd.tolist() == [mark + 7 + 6] and w[0].tolist() == [60, 42, 12, 0]


# one wavefront and several, blocks of one 16-byte piece and longer ones, more slots than a thread's registers
SHAPES = [(3, 8, 12), (70, 20, 40), (64, 129, 40), (256, 134, 12), (8, 3000, 6), (5, 2000, 6), (1, 100, 5)]


@pytest.mark.parametrize("K,l,n", SHAPES)
def test_peaks_beyond_int32(K, l, n):
    """Instances whose windows lie so high that a request's tokens would take them past 2^31: nothing is stored out of
    range as long as they are not chosen (their peak is the largest of all), so nothing is flagged and all results
    are exact.  Values just below, at and above the line at which 32 bits would still do."""
    print(f"route near 2^31 K={K} l={l} n={n}", flush=True)
    rng = np.random.default_rng(K + l)
    P, D, win, cap, qp, cd = random_case(rng, K, l, n, False)
    hot = rng.permutation(K)[: (K + 1) // 2] if K > 1 else np.array([], int)
    for k in hot:
        win[k, rng.integers(0, l, 3)] = 2**31 - 1 - rng.integers(0, 4000, 3)
    if K == 1:
        win[0, :] = 2**31 - 1 - 5000 - rng.integers(0, 100, l)
        P = np.array([200, 300, 150, 400, 7][:n])
        D = np.minimum(D, l)
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd)
    assert rw.max() < 2**31 and flags == 0
    assert np.array_equal(a, ra) and np.array_equal(s, rs)
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)


@pytest.mark.parametrize("K,l", [(k, l) for k, l, _ in SHAPES])
def test_stored_values_beyond_int32_are_flagged(K, l):
    """Every instance is full to the brim, so the request that is dispatched takes slots out of the int32 range: flagged,
    low 32 bits kept, score and queues exact."""
    print(f"route past 2^31 K={K} l={l}", flush=True)
    rng = np.random.default_rng(K * l)
    _, _, win, cap, qp, cd = random_case(rng, K, l, 1, False)
    win[:, :] = 2**31 - 1 - rng.integers(0, 50, (K, l))
    P, D = np.array([100]), np.array([l - l // 3])
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd)
    assert flags == ps.PS_ST_RANGE and rw.max() >= 2**31
    assert np.array_equal(a, ra) and np.array_equal(s, rs) and np.array_equal(q2, rq) and np.array_equal(c2, rc)
    assert np.array_equal(w.astype(np.int64) & 0xffffffff, rw & 0xffffffff)


@pytest.mark.parametrize("where", ["everywhere", "one wavefront", "ties"])
@pytest.mark.parametrize("K,l,n", [(64, 12, 50), (200, 16, 60), (130, 140, 40), (6, 3000, 5)])
def test_scores_beyond_32_bits(K, l, n, where):
    """Queues so long that scores need 64 bits: on all instances, on those of one wavefront only (the exchange then mixes
    minima found either way), and equal ones, which go to the lowest instance."""
    print(f"route 64-bit scores K={K} l={l} n={n} {where}", flush=True)
    rng = np.random.default_rng(K + n)
    P, D, win, cap, qp, cd = random_case(rng, K, l, n, True)
    big = rng.integers(2**25, 2**40, K)
    if where == "everywhere":
        qp, cd = big, rng.integers(2**25, 2**40, K)
    elif where == "one wavefront":
        qp = np.where(np.arange(K) // 64 == (K - 1) // 64, big, qp)
    else:
        win[:, :], cap[:], cd[:] = 0, 10**6, 0
        qp = np.full(K, 2**33)
    a, s, w, q2, c2, flags, _ = run_route(P, D, win, cap, qp, cd)
    ra, rs, rw, rq, rc = orr.route(P, D, win, cap, qp, cd)
    assert flags == 0
    assert np.array_equal(a, ra) and np.array_equal(s, rs)
    assert np.array_equal(w, rw) and np.array_equal(q2, rq) and np.array_equal(c2, rc)
