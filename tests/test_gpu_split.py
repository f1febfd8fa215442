"""GPU parity of the split-FP16 self-join of FP32 rows against the CPU oracle evaluated on the FP32 data in FP64."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ej(request):
    e = parity.open_context(request)
    yield e
    e.close()


def run_f32(ej, X32, eps, capacity):
    pairs, d2, npairs = ej.selfjoin_pairs_f32(torch.from_numpy(X32).cuda(), float(eps), capacity)
    torch.cuda.synchronize()
    assert ej.status() == 0
    return parity.to_host_pairs(pairs, d2, npairs)


def data(kind, n, d, seed):
    rng = np.random.default_rng(seed)
    if kind == "uniform":
        return rng.random((n, d), dtype=np.float32)
    if kind == "offset":      # far from the origin: FP16 spacing near 10 is 2^-7
        return (np.float32(10.0) + rng.random((n, d), dtype=np.float32)).astype(np.float32)
    if kind == "clustered":
        c = rng.random((12, d), dtype=np.float32)
        return (c[rng.integers(0, 12, size=n)] + np.float32(0.03) * rng.standard_normal((n, d)).astype(np.float32)).astype(np.float32)
    raise ValueError(kind)


@parity.BOTH_KERNELS
@pytest.mark.parametrize("kind,n,d,ld_extra", [("uniform", 1500, 100, 0), ("offset", 1300, 64, 5), ("clustered", 2100, 257, 0),
                                               ("uniform", 1, 8, 0), ("uniform", 700, 1, 3), ("clustered", 6300, 48, 0)])
def test_split_join_matches_fp64_on_the_fp32_data(ej, kind, n, d, ld_extra):
    print(f"split {kind} n={n} d={d}", flush=True)
    X = data(kind, n, d, seed=n + d)
    if ld_extra:
        buf = np.full((n, d + ld_extra), np.float32(123.0))  # columns beyond d must be ignored
        buf[:, :d] = X
        Xarg = buf[:, :d]
    else:
        Xarg = X
    P = X.astype(np.float64)
    eps = orc.select_eps_all_pairs(P, 8) if n >= 3 else np.float32(0.5)
    ora_pairs, ora_d2 = orc.selfjoin_pairs(P, eps)
    Xd = torch.from_numpy(np.ascontiguousarray(buf) if ld_extra else X).cuda()
    if ld_extra:
        Xd = Xd[:, :d]
    pairs, d2, npairs = ej.selfjoin_pairs_f32(Xd, float(eps), ora_pairs.shape[0] * 2 + 1024)
    torch.cuda.synchronize()
    assert ej.status() == 0
    gp, gd2, found = parity.to_host_pairs(pairs, d2, npairs)
    assert found == gp.shape[0]
    st = parity.check_pair_sets(P, eps, gp, gd2, ora_pairs, ora_d2)
    print("  ", st, flush=True)
    counts, total = ej.selfjoin_count_f32(Xd, float(eps))
    torch.cuda.synchronize()
    assert int(total.cpu()[0]) == found - n
    off = gp[gp[:, 0] != gp[:, 1]]
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), np.bincount(off[:, 0], minlength=n) + np.bincount(off[:, 1], minlength=n))


def test_split_join_is_more_accurate_than_the_fp16_join_where_conversion_hurts(ej):
    """Points in [10, 11]^64: converted to FP16 their coordinates move by up to 2^-8, a quarter of the typical
    neighbour distance; the split join sees 22 bits of every coordinate."""
    n, d = 2000, 64
    X = data("offset", n, d, seed=5)
    P = X.astype(np.float64)
    eps = orc.select_eps_all_pairs(P, 16)
    truth = orc.selfjoin_pairs(P, eps)[0]
    gp, gd2, found = run_f32(ej, X, eps, 400000)
    acc_split = orc.overlap_accuracy(n, truth, gp)
    X16 = ej.convert_f32(torch.from_numpy(X).cuda())
    p16, d16, n16 = ej.selfjoin_pairs(X16, float(eps), 400000, d=d)
    torch.cuda.synchronize()
    g16, _, _ = parity.to_host_pairs(p16, d16, n16)
    acc_fp16 = orc.overlap_accuracy(n, truth, g16)
    print(f"  overlap accuracy: split {acc_split:.5f}, fp16 {acc_fp16:.5f}", flush=True)
    assert acc_split > 0.995 and acc_split > acc_fp16 + 0.01  # what is left is the FP32 accumulation at s ~ 7000
    # squared distances: the split join's error is that of the FP32 accumulation, not of the conversion
    common = np.isin(orc.pair_keys(gp), orc.pair_keys(truth))
    o = {int(k): v for k, v in zip(orc.pair_keys(truth), orc.selfjoin_pairs(P, eps)[1])}
    err = np.array([abs(float(v) - o[int(k)]) for k, v in zip(orc.pair_keys(gp)[common], gd2[common])])
    s_max = (P ** 2).sum(axis=1).max()
    assert err.max() <= 2e-6 * s_max


@parity.BOTH_KERNELS
def test_split_join_duplicates_and_self_pairs(ej):
    rng = np.random.default_rng(9)
    X = rng.standard_normal((900, 70)).astype(np.float32)
    X[100] = X[5]
    X[899] = X[5]
    gp, gd2, found = run_f32(ej, X, 0.0, 4000)
    keys = set(map(tuple, gp.tolist()))
    assert found == 900 + 3 and {(5, 100), (5, 899), (100, 899)} <= keys
    assert np.all(gd2 == 0.0)


def test_split_join_rejects_bad_arguments_and_reports_out_of_range_data(ej):
    import paper_2508_21230_amd as pkg
    X = torch.zeros((10, 8), dtype=torch.float32, device="cuda")
    with pytest.raises(pkg.EJoinError):
        ej.selfjoin_pairs_f32(X, -1.0, 100)
    with pytest.raises(pkg.EJoinError):
        ej.selfjoin_pairs_f32(X.to(torch.float64), 1.0, 100)
    big = torch.full((10, 8), 1.0e5, dtype=torch.float32, device="cuda")  # beyond FP16's largest number
    pairs, d2, npairs = ej.selfjoin_pairs_f32(big, 1.0, 100)
    torch.cuda.synchronize()
    assert ej.status() == 2 and int(npairs.cpu()[0]) == 0


@pytest.mark.parametrize("d", [20, 33, 130, 400])
def test_split_results_do_not_depend_on_the_kernel(ej, d):
    """A set large enough for the general kernel, and its first 1,000 and 2,600 points, which the kernel of small problems takes
    in tiles of 64 and of 128: the same pairs and counts among them, the same squared distances bit for bit."""
    n = 14500
    assert [ej.join_work(m, d, split=True)[0] for m in (n, 2600, 1000)] == [256, 128, 64]
    print(f"split kernels d={d}", flush=True)
    X = data("uniform", n, d, seed=d)
    X[700] = X[3]
    eps = orc.select_eps_sample(X[:900].astype(np.float64), 12, 900)
    Xd = torch.from_numpy(X).cuda()
    pairs, d2, found = run_f32(ej, X, eps, 12 * n * 20)
    assert found == pairs.shape[0]
    for m in (1000, 2600):
        want = (pairs < m).all(axis=1)
        sub, sub_d2, sub_found = run_f32(ej, X[:m], eps, m * m)
        assert sub_found == sub.shape[0]
        kw, kg = orc.pair_keys(pairs[want]), orc.pair_keys(sub)
        ow, og = np.argsort(kw), np.argsort(kg)
        assert np.array_equal(kw[ow], kg[og]) and np.array_equal(d2[want][ow], sub_d2[og])
        counts, total = ej.selfjoin_count_f32(Xd[:m], float(eps))
        ns = sub[sub[:, 0] != sub[:, 1]]
        hist = np.bincount(ns[:, 0], minlength=m) + np.bincount(ns[:, 1], minlength=m)
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), hist) and int(total.cpu()[0]) == ns.shape[0]
    counts, total = ej.selfjoin_count_f32(Xd, float(eps))
    ns = pairs[pairs[:, 0] != pairs[:, 1]]
    hist = np.bincount(ns[:, 0], minlength=n) + np.bincount(ns[:, 1], minlength=n)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), hist) and int(total.cpu()[0]) == ns.shape[0]


@pytest.mark.parametrize("d,S", [(20, 1500), (33, 40), (160, 900)])
def test_split_counts_of_large_sets(ej, d, S):
    """More than 32,768 points, one, two and five k-blocks a part, wave tiles whose candidates fit the queue and ones that overflow it
    (the points are stored cluster by cluster): counts = histogram of the pairs."""
    n = 33100
    assert ej.join_work(n, d, split=True)[0] == 256 and n > 32768
    print(f"split counts of a large set d={d} S={S}", flush=True)
    rng = np.random.default_rng(d)
    ids = np.sort(rng.integers(0, 33, size=n))
    X = (rng.random((33, d), dtype=np.float32)[ids] + np.float32(0.03) * rng.standard_normal((n, d)).astype(np.float32)).astype(np.float32)
    take = np.sort(rng.choice(n, size=1500, replace=False))
    eps = orc.select_eps_sample(X[take].astype(np.float64), S, n)
    Xd = torch.from_numpy(X).cuda()
    pairs, d2, npairs = ej.selfjoin_pairs_f32(Xd, float(eps), 2 * n * S)
    found = int(npairs.cpu()[0])
    assert ej.status() == 0 and n < found <= 2 * n * S
    ns = pairs[:found].long()
    ns = ns[ns[:, 0] != ns[:, 1]]
    hist = torch.bincount(ns[:, 0], minlength=n) + torch.bincount(ns[:, 1], minlength=n)
    counts, total = ej.selfjoin_count_f32(Xd, float(eps))
    assert torch.equal(counts.long(), hist) and int(total.cpu()[0]) == ns.shape[0]


@parity.BOTH_KERNELS
@pytest.mark.parametrize("d,share", [(20, 0.05), (130, 0.05), (64, 0.6)])
def test_split_pairs_of_dense_tiles(ej, d, share):
    """Wave tiles whose candidates overflow the queue: pairs against the oracle, counts against the pairs."""
    n = 900
    print(f"split dense pairs d={d} share={share}", flush=True)
    X = data("uniform", n, d, seed=n + d)
    P = X.astype(np.float64)
    eps = orc.select_eps_all_pairs(P, share * n)
    ora_pairs, ora_d2 = orc.selfjoin_pairs(P, eps)
    pairs, d2, found = run_f32(ej, X, eps, n * n)
    assert found == pairs.shape[0]
    parity.check_pair_sets(P, eps, pairs, d2, ora_pairs, ora_d2)
    counts, total = ej.selfjoin_count_f32(torch.from_numpy(X).cuda(), float(eps))
    ns = pairs[pairs[:, 0] != pairs[:, 1]]
    hist = np.bincount(ns[:, 0], minlength=n) + np.bincount(ns[:, 1], minlength=n)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), hist) and int(total.cpu()[0]) == ns.shape[0]
