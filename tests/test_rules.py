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
    return lib


def test_norms_start_at_the_end_only_of_rows_that_the_memory_side_cache_does_not_hold(rules):
    for n, ld in ((1, 64), (20000, 384), (10**6, 64), (500000, 192), (1_900_000, 64), (6_300_000, 64), (6 * 10**6, 1024)):  # up to 243 MB, from 806 MB on
        assert not rules.ejoin_test_norms_from_the_end(n, ld)
    for n, ld in ((2_000_000, 64), (500000, 256), (10**6, 256), (6_290_000, 64)):  # from 256 MB on
        assert rules.ejoin_test_norms_from_the_end(n, ld)
