"""The rules that choose a call's kernel (csrc/rules.h compiled with g++), at the edges where one changes to the other."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = tmp_path_factory.mktemp("rules") / "librules.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2508_21230_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "rules_dump.cpp"), "-o", str(out)], check=True)
    lib = ctypes.CDLL(str(out))
    lib.ejoin_test_norms_from_the_end.argtypes = [ctypes.c_int64] * 2
    lib.ejoin_test_ingest_wide.argtypes, lib.ejoin_test_ingest_wide.restype = [ctypes.c_int64], ctypes.c_uint32
    lib.ejoin_test_ingest_past_the_caches.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_int64, ctypes.c_uint64]
    lib.ejoin_test_few_pays.argtypes = [ctypes.c_int64] * 2 + [ctypes.c_int32] * 2
    lib.ejoin_test_once_edge.argtypes = [ctypes.c_int64] * 2 + [ctypes.c_int32] * 2
    lib.ejoin_test_dense_norm_groups.argtypes, lib.ejoin_test_dense_norm_groups.restype = [ctypes.c_int64] * 3, ctypes.c_int64
    lib.ejoin_test_few_groups_of.argtypes = [ctypes.c_int64]
    return lib


def test_norms_start_at_the_end_only_of_rows_that_the_memory_side_cache_does_not_hold(rules):
    for n, ld in ((1, 64), (20000, 384), (10**6, 64), (500000, 192), (1_900_000, 64), (6_300_000, 64), (6 * 10**6, 1024)):  # up to 243 MB, from 806 MB on
        assert not rules.ejoin_test_norms_from_the_end(n, ld)
    for n, ld in ((2_000_000, 64), (500000, 256), (10**6, 256), (6_290_000, 64)):  # from 256 MB on
        assert rules.ejoin_test_norms_from_the_end(n, ld)


def test_ingestion_past_the_caches_only_where_lines_are_rarely_read_twice(rules):
    assert [rules.ejoin_test_ingest_wide(c) for c in (8, 16, 24, 32, 40, 48, 64, 80, 96, 128, 176, 192, 8192)] == [8, 16, 8, 32, 8, 16, 64, 16, 32, 64, 16, 64, 64]
    # (d, stride, address, MB of input): one piece a row; whole lines; pieces of 1 KB, 512 and 256 bytes that share lines; rows that are not 16-byte aligned
    for d, ld, address, mb, past in ((100, 100, 0, 250, 0), (100, 100, 0, 260, 1), (200, 200, 16, 2000, 1), (200, 200, 8, 2000, 0), (32, 32, 0, 2000, 0), (101, 101, 0, 400, 0),
                                     (192, 192, 0, 760, 1), (192, 192, 0, 780, 0), (192, 192, 64, 300, 0), (180, 192, 128, 400, 1), (512, 512, 0, 2000, 1), (768, 768, 0, 700, 1), (768, 768, 0, 1700, 0),
                                     (1000, 1000, 0, 570, 1), (1000, 1000, 0, 580, 0), (324, 324, 0, 470, 1), (324, 324, 0, 490, 0), (300, 300, 0, 260, 0), (668, 668, 0, 653, 0)):
        assert rules.ejoin_test_ingest_past_the_caches((mb << 20) // (4 * d), d, ld, address) == past, (d, ld, address, mb)


def test_few_query_points_against_sets_where_that_is_the_better_kernel(rules):
    assert [rules.ejoin_test_few_groups_of(nq) for nq in (1, 32, 33, 64, 65, 128, 129, 256, 257)] == [2, 2, 4, 4, 8, 8, 16, 16, 0]
    # (n, nq, d): measured as slower by a tenth or more, counts and lists; and as faster
    for n, nq, d in ((16000, 60, 960), (18500, 60, 768), (6000, 120, 384), (9000, 120, 480), (13000, 30, 1024), (3000, 60, 512), (20000, 140, 250), (28000, 250, 250), (16000, 250, 200)):
        assert not rules.ejoin_test_few_pays(n, nq, d, 0) and not rules.ejoin_test_few_pays(n, nq, d, 1)
    for n, nq, d in ((100000, 120, 530), (20000, 60, 960), (20000, 30, 1500), (12000, 120, 480), (1500, 30, 512), (1500, 60, 256), (6000, 120, 128), (24000, 250, 64), (60000, 250, 250)):
        assert rules.ejoin_test_few_pays(n, nq, d, 0) and rules.ejoin_test_few_pays(n, nq, d, 1)
    # lists of more than 128 query points take more points than counts
    for n, nq, d, count, there in ((13000, 250, 64, 1, 1), (13000, 250, 64, 0, 0), (23599, 250, 64, 0, 0), (23600, 250, 64, 0, 1), (24000, 250, 220, 0, 0), (7371, 250, 128, 1, 0), (7372, 250, 128, 1, 1)):
        assert rules.ejoin_test_few_pays(n, nq, d, count) == there
    # the other kernel's tiles of 64: up to 300 of them
    for n, nq, d, there in ((19200, 64, 960, 0), (19201, 64, 960, 1), (9600, 128, 480, 0), (9601, 128, 480, 1), (9599, 64, 512, 0), (9600, 64, 512, 1)):
        assert rules.ejoin_test_few_pays(n, nq, d, 1) == there


def test_tiles_of_the_one_launch_join(rules):
    """(n, nq or 0, d, counts): the last problem in tiles of 64 and the first of 128, the last of all and the first of another kernel."""
    for n, nq, d, count, edge in ((1216, 0, 64, 0, 64), (1217, 0, 64, 0, 128), (1344, 0, 96, 0, 64), (1345, 0, 96, 0, 128), (1472, 0, 130, 0, 64), (1473, 0, 130, 0, 128),
                                  (2432, 0, 96, 1, 64), (2433, 0, 96, 1, 128), (4864, 0, 96, 0, 128), (4865, 0, 96, 0, 0), (4864, 0, 96, 1, 128), (4865, 0, 96, 1, 0),
                                  (3968, 0, 960, 0, 128), (3969, 0, 960, 0, 0), (4864, 0, 512, 0, 128), (4864, 0, 513, 0, 0), (4864, 0, 1152, 1, 128), (4864, 0, 1153, 1, 0),
                                  (3968, 0, 1153, 1, 128), (3968, 0, 4096, 0, 128), (3968, 0, 4097, 0, 0), (4000, 3000, 768, 1, 128), (4000, 3000, 769, 1, 0), (4000, 3000, 512, 0, 128),
                                  (4000, 3000, 513, 0, 0), (300, 90000, 40, 0, 0), (300, 20000, 40, 0, 128), (100, 60000, 40, 1, 128), (10, 131062, 40, 1, 0)):
        assert rules.ejoin_test_once_edge(n, nq, d, count) == edge, (n, nq, d, count)


def test_dense_blocks_whose_norms_are_worked_out_in_their_launch(rules):
    """(n, rows, columns): the workgroups for the norms; the last set of a block of five tiles, blocks of tiles of 64 and of 128, and what takes two launches."""
    for n, rows, cols, groups in ((1, 1, 1, 8), (19968, 20, 300, 312), (19969, 20, 300, 0), (8000, 300, 300, 128), (8000, 1800, 1750, 64), (8000, 600, 600, 128), (20000, 4000, 5000, 0), (120000, 300, 300, 0)):
        assert rules.ejoin_test_dense_norm_groups(n, rows, cols) == groups, (n, rows, cols)
