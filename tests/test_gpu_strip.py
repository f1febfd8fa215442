"""The join kernel that keeps its rows in registers, against the general kernel: pairs, squared distances bit for bit and counts, on a
build that takes problems of every size there."""
import pytest
import torch

import paper_2508_21230_amd as pkg
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def both():
    g, s = parity.general_context(), parity.strip_context()
    yield g, s
    g.close()
    s.close()


def rows(n, d, seed):
    """FP16 rows in [0, 1), some duplicates, on the device with a stride that is a multiple of 64."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    out = torch.zeros((n, (d + 63) // 64 * 64), dtype=torch.float16, device="cuda")
    out[:, :d] = torch.rand((n, d), generator=gen, device="cuda")
    out[n // 2:n // 2 + n // 20] = out[n // 3]
    return out


def sorted_pairs(call):
    pairs, d2, found = call
    m = int(found.cpu()[0])
    assert m <= pairs.shape[0]
    keys, order = torch.sort(pairs[:m].reshape(-1).view(torch.int64))
    return keys, d2[:m][order]


def same_pairs(a, b):
    (ka, da), (kb, db) = sorted_pairs(a), sorted_pairs(b)
    assert torch.equal(ka, kb) and torch.equal(da, db)
    assert ka.numel() < 2 or bool((ka[1:] != ka[:-1]).all())


def epsilon(X, d, share):
    D = torch.cdist(X[:400, :d].float(), X[-400:, :d].float())
    return float(torch.quantile(D.flatten()[:100000], share))


D_OF_BLOCKS = [20, 70, 128, 133, 190, 220, 256, 270, 300, 350, 384]  # two to ten blocks of 32 coordinates, and two widths that go to the general kernel in either build


@pytest.mark.parametrize("d", D_OF_BLOCKS)
@pytest.mark.parametrize("n,share", [(1, 0.5), (64, 0.2), (65, 0.02), (511, 0.004), (769, 0.3), (1700, 0.03), (5200, 0.002), (5200, 0.00002)])
def test_self_join(both, n, d, share):
    print(f"strip self n={n} d={d} share={share}", flush=True)
    X = rows(n, d, seed=n + d)
    eps = epsilon(X, d, share)
    cap = n * (n + 1) // 2
    same_pairs(both[0].selfjoin_pairs(X, eps, cap, d=d), both[1].selfjoin_pairs(X, eps, cap, d=d))
    (cg, tg), (cs, ts) = both[0].selfjoin_count(X, eps, d=d), both[1].selfjoin_count(X, eps, d=d)
    assert torch.equal(cg, cs) and torch.equal(tg, ts) and both[1].status() == 0


@pytest.mark.parametrize("d", D_OF_BLOCKS)
@pytest.mark.parametrize("n,nq,share", [(1, 900, 0.3), (900, 1, 0.3), (3000, 520, 0.01), (520, 3000, 0.01), (1300, 1290, 0.2), (9000, 70, 0.0005)])
def test_two_sets(both, n, nq, d, share):
    """Both ways round: the points in the rows, and the query points."""
    print(f"strip two sets n={n} nq={nq} d={d} share={share}", flush=True)
    P, Q = rows(n, d, seed=d), rows(nq, d, seed=d + 1)
    Q[:min(n, nq) // 3] = P[:min(n, nq) // 3]
    eps = epsilon(Q, d, share)
    same_pairs(both[0].join_pairs(P, Q, eps, n * nq, d=d), both[1].join_pairs(P, Q, eps, n * nq, d=d))
    sets = [e.prepare(P, d=d) for e in both]
    for call in (lambda e, s: e.join_count(P, Q, eps, d=d), lambda e, s: s.join_count(Q, eps)):
        for u, v in zip(call(both[0], sets[0]), call(both[1], sets[1])):
            assert torch.equal(u, v)
    for s in sets:
        s.close()


@pytest.mark.parametrize("d", [64, 128, 224, 320])
def test_dense_results_huge_epsilon_and_overflow(both, d):
    n, nq = 1300, 700
    print(f"strip dense d={d}", flush=True)
    X, Q = rows(n, d, seed=3), rows(nq, d, seed=4)
    for eps in (0.0, 1e3, 2e19):  # (the last: its square is beyond FP32)
        same_pairs(both[0].selfjoin_pairs(X, eps, n * n, d=d), both[1].selfjoin_pairs(X, eps, n * n, d=d))
        for u, v in zip(both[0].join_count(X, Q, eps, d=d), both[1].join_count(X, Q, eps, d=d)):
            assert torch.equal(u, v)
        for u, v in zip(both[0].selfjoin_count(X, eps, d=d), both[1].selfjoin_count(X, eps, d=d)):
            assert torch.equal(u, v)
    eps = epsilon(X, d, 0.1)
    keys, _ = sorted_pairs(both[0].selfjoin_pairs(X, eps, n * n, d=d))
    pairs, d2, found = both[1].selfjoin_pairs(X, eps, keys.numel() // 3, d=d)
    some = pairs.reshape(-1).view(torch.int64)
    assert int(found.cpu()[0]) == keys.numel() and torch.unique(some).numel() == some.numel() and bool(torch.isin(some, keys).all())


@pytest.mark.parametrize("n,d,batches", [(12345, 100, 3), (20000, 224, 32)])
def test_batched_return(both, n, d, batches):
    print(f"strip to host n={n} d={d} batches={batches}", flush=True)
    X = rows(n, d, seed=n)
    eps = epsilon(X, d, 0.0002)
    keys, d2 = sorted_pairs(both[0].selfjoin_pairs(X, eps, 4000000, d=d))
    m = keys.numel() + 100
    pairs, dist2 = torch.empty((m, 2), dtype=torch.int32, device="cuda"), torch.empty(m, device="cuda")
    host, host2 = torch.empty((m, 2), dtype=torch.int32, pin_memory=True), torch.empty(m, pin_memory=True)
    assert both[1].selfjoin_pairs_to_host(X, eps, batches, pairs, dist2, host, host2, d=d) == keys.numel()
    k, order = torch.sort(host[:keys.numel()].reshape(-1).view(torch.int64))
    assert torch.equal(k, keys.cpu()) and torch.equal(host2[:keys.numel()][order], d2.cpu())


def test_sets_of_many_norms_and_captured_replays(both):
    """Norms over many powers of two (the pieces of the norm terms at their limits), and replays of a captured call."""
    n, nq, d = 2600, 900, 200
    X, Q = rows(n, d, seed=11), rows(nq, d, seed=12)
    X *= torch.logspace(-3, 2, n, device="cuda")[:, None].half()
    Q *= torch.logspace(2, -3, nq, device="cuda")[:, None].half()
    for eps in (0.05, 3.0, 300.0):
        same_pairs(both[0].join_pairs(X, Q, eps, n * nq, d=d), both[1].join_pairs(X, Q, eps, n * nq, d=d))
        same_pairs(both[0].join_pairs(Q, X, eps, n * nq, d=d), both[1].join_pairs(Q, X, eps, n * nq, d=d))
    want = both[0].selfjoin_count(X, 3.0, d=d)
    counts, total = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int64, device="cuda")
    both[1].selfjoin_count(X, 3.0, d=d, counts=counts, total=total)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        both[1].selfjoin_count(X, 3.0, d=d, counts=counts, total=total)
    for _ in range(3):
        counts.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(counts, want[0]) and torch.equal(total, want[1])
        both[1].selfjoin_count(Q, 1.0, d=d)
        torch.cuda.synchronize()


@pytest.mark.parametrize("n,nq,d", [(52000, 0, 256), (52000, 0, 270), (52000, 0, 320), (70000, 0, 150), (40000, 33000, 240), (33000, 40000, 300), (60000, 41000, 100),
                                    (3500, 300000, 320)])
def test_realignment(both, n, nq, d):
    """Launches long enough that the workgroups of an XCD are re-aligned: stages of 64 and of 32 columns, two sets either way round."""
    print(f"strip re-alignment n={n} nq={nq} d={d}", flush=True)
    stages = (n + 511) // 512 * ((nq or n) // 64) // (1 if nq else 2)  # (either way round)
    assert stages > 1.1 * 256 * (1024 // ((d + 31) // 32)) and both[1].join_kernel(n, d, nq) == "strip"
    X = rows(n, d, seed=d)
    eps = epsilon(X, d, 0.00002)
    if nq:
        Q = rows(nq, d, seed=d + 1)
        calls = (lambda e: e.join_pairs(X, Q, eps, 4000000, d=d)), (lambda e: e.join_count(X, Q, eps, d=d))
    else:
        calls = (lambda e: e.selfjoin_pairs(X, eps, 8000000, d=d)), (lambda e: e.selfjoin_count(X, eps, d=d))
    same_pairs(calls[0](both[0]), calls[0](both[1]))
    for u, v in zip(calls[1](both[0]), calls[1](both[1])):
        assert torch.equal(u, v)


@pytest.fixture(scope="module")
def product():
    e = pkg.EJoin(0)
    yield e
    e.close()


@pytest.mark.parametrize("n,d", [(14501, 128), (20011, 40), (33001, 60), (40000, 200), (65001, 96), (70000, 256), (52000, 310)])
@pytest.mark.parametrize("share", [0.00001, 0.002])
def test_self_joins_that_go_there(both, product, n, d, share):
    """The product's own build at sizes that it sends there: few neighbours, and a hundred and more of them."""
    print(f"strip product self n={n} d={d} share={share}", flush=True)
    assert product.join_kernel(n, d) == "strip"
    X = rows(n, d, seed=n)
    X[n // 2:n // 2 + n // 20] = rows(n, d, seed=n + 1)[:n // 20]  # (other points in place of the duplicates)
    eps = epsilon(X, d, share)
    cap = int(4 * share * n * n) + 100000
    same_pairs(both[0].selfjoin_pairs(X, eps, cap, d=d), product.selfjoin_pairs(X, eps, cap, d=d))
    for u, v in zip(both[0].selfjoin_count(X, eps, d=d), product.selfjoin_count(X, eps, d=d)):
        assert torch.equal(u, v)


@pytest.mark.parametrize("n,nq,d,count", [(300000, 300, 128, True), (200000, 500, 300, True), (200000, 1000, 64, False), (1000, 200000, 60, True), (30011, 7001, 200, False),
                                          (7001, 30011, 200, True), (500000, 700, 100, True), (2500, 100000, 256, False)])
def test_two_sets_that_go_there(both, product, n, nq, d, count):
    print(f"strip product two sets n={n} nq={nq} d={d} count={count}", flush=True)
    assert product.join_kernel(n, d, nq, count=count) == "strip"
    P, Q = rows(n, d, seed=d), rows(nq, d, seed=d + 1)
    eps = epsilon(Q, d, 0.0002)
    if count:
        for u, v in zip(both[0].join_count(P, Q, eps, d=d), product.join_count(P, Q, eps, d=d)):
            assert torch.equal(u, v)
    else:
        same_pairs(both[0].join_pairs(P, Q, eps, n * nq // 500, d=d), product.join_pairs(P, Q, eps, n * nq // 500, d=d))
