"""A prepared set against few query points, against the general kernel: pairs, squared distances bit for bit, counts and status."""
import pytest
import torch

import paper_2508_21230_amd as pkg
from tests import parity
from tests.test_gpu_strip import epsilon, rows, same_pairs, sorted_pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def both():
    g, e = parity.general_context(), pkg.EJoin(0)
    yield g, e
    g.close()
    e.close()


def rules_say(n, nq, d):
    """Whether lists and counts go to the kernel of few query points (see the rules' own test)."""
    groups, blocks = (2 if nq <= 32 else 4 if nq <= 64 else 8 if nq <= 128 else 16), max(2, -(-d // 32))
    kb = groups * blocks
    if nq > 256 or groups * 16 * (blocks * 64 + 24) + 128 + 8 * 128 * 12 > 159 * 1024:
        return [False, False]
    if groups == 16:
        return [n >= 14000 + 300 * kb, n >= 9 * kb * kb // 5]
    return [-(-n // 64) * -(-nq // 64) > 300 or n >= (300 if groups == 4 else 600) * (kb - 32)] * 2


def compare(both, P, Q, eps, d):
    (n, nq), few = (P.shape[0], Q.shape[0]), rules_say(P.shape[0], Q.shape[0], d)
    assert [both[1].join_kernel(n, d, nq, count=c, prepared=True) == "few" for c in (False, True)] == few
    sets = [e.prepare(P, d=d) for e in both]
    want = sets[0].join_count(Q, eps)
    cap = int(want[2])
    for _ in range(2):  # (the first call leaves the context as it found it)
        for u, v in zip(want, sets[1].join_count(Q, eps)):
            assert torch.equal(u, v)
        same_pairs(sets[0].join_pairs(Q, eps, cap), sets[1].join_pairs(Q, eps, cap))
    cp, none, total = sets[1].join_count(Q, eps, want_counts_q=False)
    assert none is None and torch.equal(cp, want[0]) and torch.equal(total, want[2]) and both[1].status() == 0
    for s in sets:
        s.close()


# every number of groups of query points and its edges, one more than any takes, sets of which some wavefronts have no point
@pytest.mark.parametrize("d", [20, 64, 100, 130, 300, 960])
@pytest.mark.parametrize("nq", [1, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257])
def test_number_of_query_points(both, nq, d):
    print(f"few n=20011 nq={nq} d={d}", flush=True)
    P, Q = rows(20011, d, seed=d), rows(nq, d, seed=d + nq)
    Q[:(nq + 1) // 2] = P[:(nq + 1) // 2]
    compare(both, P, Q, epsilon(P, d, 0.002), d)


@pytest.mark.parametrize("share", [0.03, 0.3])
@pytest.mark.parametrize("nq, d", [(60, 416), (60, 448), (60, 512), (60, 544), (60, 1056), (60, 1152), (120, 512), (120, 544)])
def test_staged_results(both, nq, d, share):
    """The dimensions where a wavefront stages fewer results, or the LDS is full."""
    print(f"few staged nq={nq} d={d} share={share}", flush=True)
    P, Q = rows(20011, d, seed=d), rows(nq, d, seed=d + nq)
    compare(both, P, Q, epsilon(P, d, share), d)


@pytest.mark.parametrize("share", [0.02, 1.0])
@pytest.mark.parametrize("n", [1, 31, 33, 255, 257, 513, 70000, 140001])
def test_number_of_points(both, n, share):
    """One to several panels a workgroup; sparse results, and all pairs, which no wavefront can stage."""
    print(f"few n={n} share={share}", flush=True)
    d, nq = 70, 50 if share < 1 else 20
    P, Q = rows(n, d, seed=n), rows(nq, d, seed=n + 1)
    compare(both, P, Q, epsilon(torch.cat([P[:500], Q]), d, share) * (1.0 if share < 1 else 3.0), d)


@pytest.mark.parametrize("share", [0.04, 0.14, 0.76])
@pytest.mark.parametrize("n, nq, d", [(140001, 20, 40), (140001, 60, 40), (140001, 120, 40), (70001, 250, 64), (20011, 250, 64), (70001, 120, 530)])
def test_lists_of_more_than_is_staged(both, n, nq, d, share):
    """Two and three panels a wavefront: results that wait for an atomic of their own, and, in its last panel, for the workgroup's; whole, cut off and not wanted."""
    print(f"few dense n={n} nq={nq} d={d} share={share}", flush=True)
    P, Q = rows(n, d, seed=d + 1), rows(nq, d, seed=nq)
    eps = epsilon(torch.cat([P[:2000], Q]), d, share)
    compare(both, P, Q, eps, d)
    s = both[1].prepare(P, d=d)
    total = int(s.join_count(Q, eps)[2])
    whole, d2 = sorted_pairs(s.join_pairs(Q, eps, total))
    pairs, dist2, found = s.join_pairs(Q, eps, total // 2)
    keys, order = torch.sort(pairs.reshape(-1).view(torch.int64))
    at = torch.searchsorted(whole, keys)
    assert int(found) == total and torch.equal(whole[at], keys) and torch.equal(d2[at], dist2[order]) and bool((keys[1:] != keys[:-1]).all())
    assert int(s.join_pairs(Q, eps, 0)[2]) == total
    s.close()


def test_query_norms_far_above_the_sets_and_out_of_range(both):
    P, Q = rows(9000, 96, seed=1), rows(40, 96, seed=2)
    P[:3000] *= 0.01
    Q[7] *= 300
    for eps in (0.02, 1.0, 3.0):
        compare(both, P, Q, eps, 96)
    s = both[1].prepare(P, d=96)
    for value, status in ((float("nan"), 2), (60000.0, 1)):
        bad = Q.clone()
        bad[39, :90] = value
        cp, cq, total = s.join_count(bad, 3.0)
        assert both[1].status() == status and int(total) == 0 and not cp.any() and not cq.any()
        assert int(s.join_pairs(bad, 3.0, 100)[2]) == 0 and both[1].status() == status
    s.close()
    compare(both, P, Q, 1.0, 96)


def test_a_list_that_is_cut_off(both):
    P, Q = rows(3000, 64, seed=3), rows(30, 64, seed=4)
    s = both[1].prepare(P, d=64)
    whole, d2 = sorted_pairs(s.join_pairs(Q, 100.0, 90000))
    pairs, dist2, found = s.join_pairs(Q, 100.0, 1000)
    keys, order = torch.sort(pairs.reshape(-1).view(torch.int64))
    at = torch.searchsorted(whole, keys)
    assert int(found) == whole.numel() == 90000 and torch.equal(whole[at], keys) and torch.equal(d2[at], dist2[order])
    s.close()


def test_captured_and_replayed_on_new_queries(both):
    e = both[1]
    P = rows(30000, 96, seed=5)
    s, Q = e.prepare(P, d=96), rows(60, 96, seed=6)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s.join_count(Q, 2.8)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = s.join_count(Q, 2.8)
    for seed in (7, 8, 9, 7):
        Q.copy_(rows(60, 96, seed=seed))
        g.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in out]
        for u, v in zip(got, s.join_count(Q, 2.8)):
            assert torch.equal(u, v)
    s.close()
