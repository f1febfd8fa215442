"""Shared helpers of the GPU parity tests: the parity rule between the HIP path and the CPU oracle.

Rule: the GPU pair set must equal the oracle's except for pairs whose
FP64 distance lies within a relative 1e-3 of epsilon; squared distances of common pairs must agree
within a relative 1e-3.

Two floors complete the rule where a relative bound cannot hold for the method itself:
  * As D2 -> 0 an FP32 expansion s_i + s_j - 2a cancels two numbers of size s, so the value tolerance is
    max(1e-3 * D2, 5e-7 * (s_i + s_j), ...): about four FP32 ulps of the operands; it only matters for
    near-duplicates.
  * The method is meant for data commensurate with the dynamic range of FP16 (Section 4.5).  The kernel
    carries the norm term -s/2 as FP16 pieces scaled to the largest norm s_max of the data, which is
    exact for every point with s >= max(2^-16 s_max, 2^-14) and resolves smaller norms to 2^-40 s_max
    (2^-39 at least).  RES(s_max) = max(2^-38 s_max, 2^-36) bounds what that costs a squared distance:
    it matters only for pairs of points whose norms are 2^16 below the largest one, or for squared
    distances below FP16's smallest normal number squared (2^-28).
A pair whose D2 is closer to eps^2 than these two floors may fall on either side, like the pairs in
the relative band.  For the workloads of the task both floors are orders of magnitude inside the
1e-3 band (w3: 3e-4 and 1.5e-9 against 1.4e-3).
"""
from __future__ import annotations

import os

import numpy as np
import pytest

from oracle import oracle as orc

#: for tests of the general join kernel at sizes that the library's rule gives to the small kernel: once as the rule has it, once by
#: the build in which every size goes to the general one (their fixture `ej` is open_context)
BOTH_KERNELS = pytest.mark.parametrize("ej", ["by_size", "general"], indirect=True)


def open_context(request):
    import paper_2508_21230_amd as pkg
    return pkg.EJoin(0) if getattr(request, "param", "by_size") == "by_size" else general_context()


def variant_context(path):
    """A context of one of the tests' builds, which must be of the sources as they are."""
    import paper_2508_21230_amd as pkg
    from paper_2508_21230_amd import build
    sources = [os.path.join(os.path.dirname(build.SRC), f) for f in os.listdir(os.path.dirname(build.SRC)) if f.endswith((".hip", ".h"))]
    built = os.path.exists(path) and os.path.getmtime(path) >= max(map(os.path.getmtime, sources))
    assert built, "build the variants first: python -m paper_2508_21230_amd.build --ablations"
    return pkg.EJoin(0, lib_path=path)


def general_context():
    from paper_2508_21230_amd import build
    e = variant_context(build.GENERAL_KERNEL_LIB)
    assert e.join_kernel(100, 64) == e.join_kernel(100000, 64) == "tiles"
    return e


def strip_context():
    from paper_2508_21230_amd import build
    e = variant_context(build.STRIP_KERNEL_LIB)
    assert e.join_kernel(100, 64) == e.join_kernel(100, 320, 50, count=True) == "strip"
    return e


REL = 1e-3
FLOOR = 5e-7


def resolution(s_max):
    return max(2.0 ** -38 * float(s_max), 2.0 ** -36)


def value_tolerance(d2, s_sum, s_max):
    """Allowed |dist2_gpu - D2| for oracle squared distances d2 of pairs whose norms sum to s_sum."""
    return np.maximum(np.maximum(REL * np.asarray(d2), FLOOR * np.asarray(s_sum)), resolution(s_max))


def in_band(d2, eps, s_sum, s_max):
    """True where a pair may fall on either side of epsilon."""
    d2 = np.asarray(d2, dtype=np.float64)
    e2 = float(eps) * float(eps)
    return orc.boundary_band(d2, eps, REL) | (np.abs(d2 - e2) <= np.maximum(FLOOR * np.asarray(s_sum), resolution(s_max)))


def to_host_pairs(pairs_t, d2_t, n_pairs_t):
    found = int(n_pairs_t.cpu()[0])
    cap = pairs_t.shape[0]
    m = min(found, cap)
    pairs = pairs_t[:m].cpu().numpy().view(np.uint32).reshape(m, 2)
    d2 = None if d2_t is None else d2_t[:m].cpu().numpy()
    return pairs, d2, found


def check_pair_sets(P, eps, gpu_pairs, gpu_d2, ora_pairs, ora_d2, strict=False):
    """Asserts the parity rule; returns a dict of statistics (mismatch rate among boundary pairs etc.).

    strict: the rule without its two floors (relative band and relative value tolerance only), which is what
    the five workloads of the task are held to."""
    def may_differ(d2, s_sum, s_max):
        return orc.boundary_band(d2, eps, REL) if strict else in_band(d2, eps, s_sum, s_max)
    n = P.shape[0]
    gp = np.asarray(gpu_pairs, dtype=np.uint32)
    assert gp.ndim == 2 and gp.shape[1] == 2
    assert (gp[:, 0] <= gp[:, 1]).all(), "pairs must have i <= j"
    assert gp.size == 0 or gp.max() < n, "index out of range"
    kg = orc.pair_keys(gp)
    order = np.argsort(kg, kind="stable")
    kg_sorted = kg[order]
    assert np.all(kg_sorted[1:] != kg_sorted[:-1]), "duplicate pairs in the GPU result"
    ko = orc.pair_keys(ora_pairs)  # sorted by construction
    assert np.all(ko[1:] > ko[:-1])
    # self pairs: all present on both sides
    assert (gp[:, 0] == gp[:, 1]).sum() == n and (ora_pairs[:, 0] == ora_pairs[:, 1]).sum() == n
    common_g = np.isin(kg_sorted, ko, assume_unique=True)
    common_o = np.isin(ko, kg_sorted, assume_unique=True)
    only_g = kg_sorted[~common_g]
    only_o_d2 = ora_d2[~common_o]
    s = orc.norms(P)
    s_max = s.max() if s.size else 0.0
    # pairs only the oracle has must be boundary pairs
    oo = ora_pairs[~common_o]
    assert may_differ(only_o_d2, s[oo[:, 0]] + s[oo[:, 1]], s_max).all(), "GPU missed a pair outside the boundary band"
    # pairs only the GPU has: evaluate them with the oracle, must be boundary pairs
    if only_g.size:
        gi = (only_g >> np.uint64(32)).astype(np.int64)
        gj = (only_g & np.uint64(0xFFFFFFFF)).astype(np.int64)
        d2x = np.array([orc.dist2(P, i, j) for i, j in zip(gi, gj)])
        assert may_differ(d2x, s[gi] + s[gj], s_max).all(), "GPU reported a pair outside the boundary band"
    stats = dict(pairs_gpu=int(gp.shape[0]), pairs_oracle=int(ora_pairs.shape[0]), only_gpu=int(only_g.size),
                 only_oracle=int(only_o_d2.size))
    band_total = int(orc.boundary_band(ora_d2, eps, REL).sum()) + int(only_g.size)
    stats["boundary_pairs"] = band_total
    stats["mismatches"] = int(only_g.size + only_o_d2.size)
    stats["boundary_mismatch_rate"] = (only_g.size + only_o_d2.size) / band_total if band_total else 0.0
    if gpu_d2 is not None:
        g_d2 = np.asarray(gpu_d2)[order][common_g].astype(np.float64)
        o_d2 = ora_d2[common_o]
        op = ora_pairs[common_o]
        tol = REL * o_d2 if strict else value_tolerance(o_d2, s[op[:, 0]] + s[op[:, 1]], s_max)
        err = np.abs(g_d2 - o_d2)
        worst = int(np.argmax(err - tol))
        assert (err <= tol).all(), f"dist2 off: pair {op[worst]} gpu {g_d2[worst]} oracle {o_d2[worst]} tol {tol[worst]}"
        stats["floor_used"] = int((err > REL * o_d2).sum())  # common pairs that needed a floor
        nz = o_d2 > 0
        stats["max_rel_err_d2"] = float((err[nz] / o_d2[nz]).max()) if nz.any() else 0.0
        m, sd = orc.distance_error_stats(g_d2, o_d2)
        stats["dist_err_mean"], stats["dist_err_std"] = m, sd
    stats["overlap_accuracy"] = orc.overlap_accuracy(n, gp, ora_pairs)
    return stats


def check_rows(P, eps, rows, row_start, nbr, nd2, gpu_pairs, gpu_d2, strict=False):
    """Neighbour lists of sampled query rows (oracle) against the GPU pairs that touch those rows.

    rows: sorted distinct row indices; row_start / nbr / nd2: the oracle's lists (oracle.rows_join);
    gpu_pairs: the pairs of the GPU list with an end among `rows` (others are ignored), gpu_d2 their squared
    distances (or None).  strict: the rule without its two floors -- a mismatched pair must lie in the relative
    band |dist - eps| <= 1e-3 eps, a common pair's squared distance within 1e-3 relative -- which is the rule
    the five workloads of the task are held to.  Returns statistics (counts, mismatch rate among the boundary
    pairs, overlap accuracy of Eq. 3 over the sampled rows, distance error of Section 4.5).
    """
    n = P.shape[0]
    rows = np.asarray(rows, dtype=np.int64)
    R = rows.size
    assert np.all(rows[1:] > rows[:-1])
    ridx = np.full(n, -1, dtype=np.int64)
    ridx[rows] = np.arange(R)
    gp = np.asarray(gpu_pairs, dtype=np.uint32).astype(np.int64)
    gd = None if gpu_d2 is None else np.asarray(gpu_d2, dtype=np.float64)
    nonself = gp[:, 0] != gp[:, 1]
    gp = gp[nonself]
    if gd is not None:
        gd = gd[nonself]
    # every (query row, neighbour) the GPU list holds: a pair counts for each of its ends that is a query row
    ra, rb = ridx[gp[:, 0]], ridx[gp[:, 1]]
    ma, mb = ra >= 0, rb >= 0
    gkey = np.concatenate([(ra[ma] << 32) | gp[ma, 1], (rb[mb] << 32) | gp[mb, 0]])
    gval = None if gd is None else np.concatenate([gd[ma], gd[mb]])
    order = np.argsort(gkey, kind="stable")
    gkey = gkey[order]
    if gval is not None:
        gval = gval[order]
    assert np.all(gkey[1:] != gkey[:-1]), "duplicate neighbour in the GPU result"
    per_row_o = np.diff(row_start)
    okey = (np.repeat(np.arange(R, dtype=np.int64), per_row_o) << 32) | nbr.astype(np.int64)
    assert np.all(okey[1:] > okey[:-1])
    in_g = np.isin(okey, gkey, assume_unique=True)   # oracle neighbours the GPU has too
    in_o = np.isin(gkey, okey, assume_unique=True)   # GPU neighbours the oracle has too
    only_o_d2 = nd2[~in_g]
    only_g_key = gkey[~in_o]
    only_g_q = rows[only_g_key >> 32]
    only_g_j = only_g_key & 0xFFFFFFFF
    only_g_d2 = np.array([orc.dist2(P, q, j) for q, j in zip(only_g_q, only_g_j)], dtype=np.float64)
    s_all = None
    if strict:
        ok_o = orc.boundary_band(only_o_d2, eps, REL)
        ok_g = orc.boundary_band(only_g_d2, eps, REL)
    else:
        s_all = orc.norms(P)
        s_max = s_all.max()
        oq = rows[okey[~in_g] >> 32]
        oj = okey[~in_g] & 0xFFFFFFFF
        ok_o = in_band(only_o_d2, eps, s_all[oq] + s_all[oj], s_max)
        ok_g = in_band(only_g_d2, eps, s_all[only_g_q] + s_all[only_g_j], s_max)
    assert ok_o.all(), f"GPU missed {int((~ok_o).sum())} neighbours outside the boundary band"
    assert ok_g.all(), f"GPU reported {int((~ok_g).sum())} neighbours outside the boundary band"
    band = int(orc.boundary_band(nd2, eps, REL).sum() + orc.boundary_band(only_g_d2, eps, REL).sum())
    mism = int(only_o_d2.size + only_g_d2.size)
    st = dict(rows=int(R), neighbours_oracle=int(okey.size), neighbours_gpu=int(gkey.size), boundary_pairs=band, mismatches=mism,
              boundary_mismatch_rate=(mism / band if band else 0.0), d2_checked=0)
    # Eq. 3 over the sampled rows
    inter = np.bincount(okey[in_g] >> 32, minlength=R).astype(np.float64)
    union = per_row_o + np.bincount(gkey >> 32, minlength=R) - inter
    score = np.ones(R)
    score[union > 0] = inter[union > 0] / union[union > 0]
    st["overlap_accuracy"] = float(score.mean())
    if gval is not None and in_g.any():
        o_d2 = nd2[in_g]
        g_d2 = gval[in_o]  # same order: both key arrays are sorted
        err = np.abs(g_d2 - o_d2)
        rel_tol = REL * o_d2
        if strict:
            tol = rel_tol
        else:
            ck = okey[in_g]
            tol = value_tolerance(o_d2, s_all[rows[ck >> 32]] + s_all[ck & 0xFFFFFFFF], s_max)
        worst = int(np.argmax(err - tol))
        assert (err <= tol).all(), f"dist2 off: gpu {g_d2[worst]} oracle {o_d2[worst]} tol {tol[worst]}"
        st["d2_checked"] = int(err.size)
        st["floor_used"] = int((err > rel_tol).sum())  # common pairs that needed a floor (0 in strict mode by the assertion)
        nz = o_d2 > 0
        st["max_rel_err_d2"] = float((err[nz] / o_d2[nz]).max()) if nz.any() else 0.0
        st["dist_err_mean"], st["dist_err_std"] = orc.distance_error_stats(g_d2, o_d2)
    return st
