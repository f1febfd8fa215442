"""The join of the smallest problems, in one launch, against the general kernel: pairs, squared distances bit for bit, counts and status;
each by workgroups that wait for the others' norms, by ones that do not and work (nearly) all of them out, and by ones that miss every third."""
import pytest
import torch

import paper_2508_21230_amd as pkg
from paper_2508_21230_amd import build
from tests import parity
from tests.test_gpu_strip import epsilon, rows, same_pairs, sorted_pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def general():
    e = parity.general_context()
    yield e
    e.close()


@pytest.fixture(scope="module", params=["waits", "late", "blind"])
def once(request):
    e = pkg.EJoin(0) if request.param == "waits" else parity.variant_context({"late": build.LATE_LIB, "blind": build.BLIND_LIB}[request.param])
    yield e
    e.close()


LAST_IN_64 = {1: 1216, 64: 1216, 96: 1344, 130: 1472, 960: 1984}  # (lists)


# one tile; edges of tiles; the last list in tiles of 64 and the first of 128; the last counts in tiles of 64
# (2,432) and the first of 128; the last problem of all (4,864; lists of many coordinates 3,968, two tiles a CU), and one of the kernel after it
@pytest.mark.parametrize("d", [1, 64, 96, 130, 960])
@pytest.mark.parametrize("n,share", [(1, 0.5), (63, 0.3), (65, 0.3), (129, 1.0), (1216, 0.01), (1217, 0.01), (1344, 0.01), (1345, 0.01), (1472, 0.01), (1473, 0.01), (1984, 0.01), (1985, 0.01), (2432, 0.003), (2433, 0.003), (3968, 0.0005), (3969, 0.0005), (4864, 0.0005), (4865, 0.0005)])
def test_self_join(general, once, n, d, share):
    print(f"once self n={n} d={d} share={share}", flush=True)
    assert (once.join_kernel(n, d) == "once") == (n <= (3968 if d == 960 else 4864)) and (once.join_kernel(n, d, count=True) == "once") == (n <= 4864)
    assert n > 3968 or once.join_work(n, d)[0] == (64 if n <= LAST_IN_64[d] else 128)
    X = rows(n, d, seed=n + d)
    eps = epsilon(X, d, share)
    cap = n + int(general.selfjoin_count(X, eps, d=d)[1])
    for _ in range(2):  # (the first call leaves the context as it found it)
        same_pairs(general.selfjoin_pairs(X, eps, cap, d=d), once.selfjoin_pairs(X, eps, cap, d=d))
        for u, v in zip(general.selfjoin_count(X, eps, d=d), once.selfjoin_count(X, eps, d=d)):
            assert torch.equal(u, v)
        assert once.status() == 0


@pytest.mark.parametrize("d", [40, 200])
@pytest.mark.parametrize("n,nq", [(1, 1), (64, 1), (65, 63), (1000, 10), (10, 1000), (4000, 500), (20000, 60), (700, 7000), (3000, 1900), (300, 20000), (300, 90000)])
def test_two_sets(general, once, n, nq, d):
    print(f"once two sets n={n} nq={nq} d={d}", flush=True)
    assert (once.join_kernel(n, d, nq) == "once") == (once.join_kernel(n, d, nq, count=True) == "once") == (nq < 90000)  # (2,112 tiles of 128: another kernel)
    P, Q = rows(n, d, seed=d), rows(nq, d, seed=d + 1)
    Q[:min(n, nq) // 3] = P[:min(n, nq) // 3]
    eps = epsilon(Q, d, 0.01)
    cap = int(general.join_count(P, Q, eps, d=d)[2])
    same_pairs(general.join_pairs(P, Q, eps, cap, d=d), once.join_pairs(P, Q, eps, cap, d=d))
    for wanted in (True, False):
        for u, v in zip(general.join_count(P, Q, eps, d=d, want_counts_q=wanted), once.join_count(P, Q, eps, d=d, want_counts_q=wanted)):
            assert u is v is None or torch.equal(u, v)


@pytest.mark.parametrize("n", [1500, 3000])
@pytest.mark.parametrize("value,row", [(float("nan"), 0), (float("inf"), 1499), (60000.0, 700)])
def test_data_out_of_range_reports_nothing(once, n, value, row):
    X = rows(n, 96, seed=1)
    X[row, :90] = value
    pairs, _, found = once.selfjoin_pairs(X, 100.0, 1000, d=96)
    assert once.status() == (1 if value == 60000.0 else 2) and int(found) == 0
    counts, total = once.selfjoin_count(X, 100.0, d=96)
    assert once.status() != 0 and int(total) == 0 and not counts.any()
    X[row] = 0
    assert int(once.selfjoin_count(X, 100.0, d=96)[1]) == n * (n - 1) // 2 and once.status() == 0  # (zero, and all within epsilon)


def test_norms_of_very_different_sizes(general, once):
    """The scale of the norm terms is that of all points, not of a tile's."""
    X = rows(1400, 96, seed=2)
    X[:600] *= 0.004
    X[9] *= 250
    for eps in (0.01, 0.05, 4.0):
        cap = 1400 + int(general.selfjoin_count(X, eps, d=96)[1])
        same_pairs(general.selfjoin_pairs(X, eps, cap, d=96), once.selfjoin_pairs(X, eps, cap, d=96))


def test_joins_of_two_sets_in_a_few_tiles_leave_nothing_for_the_next(general, once):
    """Two to seven tiles fill slots in copies that no workgroup of theirs reads; the next join has more workgroups and far smaller norms."""
    X = rows(1500, 96, seed=8) * 0.004
    eps = 0.01
    cap = 1500 + int(general.selfjoin_count(X, eps, d=96)[1])
    want = general.selfjoin_pairs(X, eps, cap, d=96), general.selfjoin_count(X, eps, d=96)
    for n, nq in ((60, 100), (60, 200), (100, 200), (30, 300), (300, 30), (180, 100), (1, 440)) * 5:
        P, Q = rows(n, 96, seed=n), rows(nq, 96, seed=nq) * 50
        for u, v in zip(general.join_count(P, Q, 200.0, d=96), once.join_count(P, Q, 200.0, d=96)):
            assert torch.equal(u, v)
        same_pairs(want[0], once.selfjoin_pairs(X, eps, cap, d=96))
        once.join_pairs(P, Q, 200.0, n * nq, d=96)
        for u, v in zip(want[1], once.selfjoin_count(X, eps, d=96)):
            assert torch.equal(u, v)


@pytest.mark.parametrize("n", [300, 3000])
def test_a_list_that_is_cut_off(once, n):
    X = rows(n, 64, seed=3)
    whole, d2 = sorted_pairs(once.selfjoin_pairs(X, 100.0, n * (n + 1) // 2, d=64))
    assert whole.numel() == n * (n + 1) // 2  # (more than a wavefront stages in the LDS)
    pairs, dist2, found = once.selfjoin_pairs(X, 100.0, 1000, d=64)
    keys, order = torch.sort(pairs.reshape(-1).view(torch.int64))
    at = torch.searchsorted(whole, keys)
    assert int(found) == whole.numel() and torch.equal(whole[at], keys) and torch.equal(d2[at], dist2[order]) and bool((keys[1:] != keys[:-1]).all())


def test_captured_and_replayed_on_new_data(once):
    X = rows(2000, 96, seed=4)
    other = [rows(2000, 96, seed=s) * f for s, f in ((5, 1.0), (6, 3.0), (7, 0.2))]
    side = torch.cuda.Stream()
    counts, total = torch.empty(2000, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int64, device="cuda")
    call = lambda: once.selfjoin_count(X, 2.5, d=96, counts=counts, total=total)
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for Y in other * 2:
        X.copy_(Y)
        g.replay()
        torch.cuda.synchronize()
        got = counts.clone(), total.clone()
        call()
        torch.cuda.synchronize()
        assert torch.equal(got[0], counts) and torch.equal(got[1], total)


def test_several_contexts_on_streams_of_their_own():
    """Their workgroups share the CUs: some may be started only when others' have ended."""
    X = [rows(4800, 64, seed=20 + k) for k in range(4)]
    want = [general_count(x) for x in X]
    each = [(pkg.EJoin(0), torch.cuda.Stream()) for _ in X]
    torch.cuda.synchronize()
    got = [[] for _ in X]
    for _ in range(20):
        for k, (e, stream) in enumerate(each):
            with torch.cuda.stream(stream):
                got[k].append(e.selfjoin_count(X[k], 1.2, d=64))
    torch.cuda.synchronize()
    for k in range(4):
        assert all(torch.equal(c, want[k][0]) and torch.equal(t, want[k][1]) for c, t in got[k])


def general_count(X):
    e = parity.general_context()
    counts = e.selfjoin_count(X, 1.2, d=64)
    torch.cuda.synchronize()
    return counts


# the norms by workgroups of the launch: one tile; tiles of 64, ragged; of 128; the last block and set in one launch (320 workgroups, 312 of them
# for the norms, more than a workgroup has threads) and the first in two
@pytest.mark.parametrize("n,d,i0,j0,rows_,cols", [(1, 20, 0, 0, 1, 1), (300, 70, 7, 100, 3, 200), (2000, 384, 1, 700, 501, 499), (8000, 100, 1000, 3000, 1800, 1750),
                                                  (19968, 64, 0, 19600, 20, 300), (19969, 64, 0, 19600, 20, 300)])
def test_dense_block(general, once, n, d, i0, j0, rows_, cols):
    """The distances of the joins, zero on the diagonal; and data out of range is reported."""
    print(f"once dense n={n} d={d} rows={rows_} cols={cols}", flush=True)
    X = rows(n, d, seed=n)
    X[:n // 3] *= 0.01
    for _ in range(2):
        D = once.dist2_tile(X, i0, j0, rows_, cols, d=d)
        assert once.status() == 0
    pairs, d2, _ = sorted_triples(general.join_pairs(X[i0:i0 + rows_].clone(), X[j0:j0 + cols].clone(), 1e3, rows_ * cols, d=d))
    i, j = pairs[:, 0].long(), pairs[:, 1].long()
    off = i0 + i != j0 + j
    scale = torch.sqrt((X.float() ** 2).sum(1).max())  # (the scale of the norm terms of a part of the points may be another)
    assert i.numel() == rows_ * cols and bool(((D[i, j] - d2)[off].abs() <= 2e-6 * scale ** 2).all()) and not D[i, j][~off].any()
    if 1 < n < 9000:  # (bit for bit, of the same set)
        keys, dist2 = sorted_pairs(general.selfjoin_pairs(X, epsilon(X, d, 0.01), n * (n + 1) // 2, d=d))
        p = keys.view(torch.int32).view(-1, 2).long()
        inside = (p[:, 0] >= i0) & (p[:, 0] < i0 + rows_) & (p[:, 1] >= j0) & (p[:, 1] < j0 + cols)
        assert torch.equal(D[p[inside, 0] - i0, p[inside, 1] - j0], dist2[inside])
    X[n - 1, 0] = float("nan")
    once.dist2_tile(X, 0, 0, 1, 1, d=d)
    assert once.status() == 2


def sorted_triples(call):
    pairs, d2, found = call
    return pairs[:int(found)], d2[:int(found)], int(found)
