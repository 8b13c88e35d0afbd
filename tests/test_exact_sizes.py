"""Index arithmetic of the exact minimum (csrc/oob_exact_sizes.h), compiled for the host and checked
over everything the entry points accept."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_08125_amd", "csrc")
WRAPPERS = r"""
#include "oob_exact_sizes.h"
using namespace oob_exact;
extern "C" {
// first index at which the quotient is wrong, -1: none
int wrong_quotient(int M) {
    for (int i = 0; i < 256 * M; ++i) if (quot(i, recip(M)) != i / M) return i;
    return -1;
}
// LDS of k_exact_eval for each accepted n_max of (L, M) against the tables of its largest slowest stage, the bands as wide
// as the sides: the smallest surplus in doubles over all that take the LDS path (1 << 30: none does).
int smallest_surplus(int L, int M) {
    size_t tables = 0; // covers next to the stage, both W, one one-node table, by the layers before it
    for (int P = 0; P <= L - 1; ++P) {
        const int S = L - 1 - P, most = P > S ? P : S;
        const size_t n = (size_t)(L - 1) * M + band_size(P, P) + band_size(S, S) + (size_t)(most + 1) * (M + 1);
        tables = n > tables ? n : tables;
    }
    int least = 1 << 30;
    for (int n = 1; n * M <= 4096; ++n) {
        const size_t lds = eval_lds(L, M, n, 1, false);
        if (lds == 0) continue;
        if (lds > kLdsLimit - kLdsStatic) return -1;
        const long long pool = (long long)(lds / 8) - (long long)(eval_fixed(L, M, n, 1) + n), surplus = pool - (long long)tables;
        if (surplus < least) least = (int)surplus;
    }
    return least;
}
}
"""


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    d = tmp_path_factory.mktemp("exact_sizes")
    (d / "wrappers.cpp").write_text(WRAPPERS)
    lib = str(d / "wrappers.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, "-o", lib, str(d / "wrappers.cpp")], check=True)
    return C.CDLL(lib)


def test_quotient_by_the_number_of_gpus(sizes):
    """Every index below 256 layers x M, every M: a reciprocal of 16 bits fails from M = 31 on."""
    assert [sizes.wrong_quotient(M) for M in range(1, 65)] == [-1] * 64


def test_tables_of_any_slowest_stage_fit_the_lds_of_a_workgroup(sizes):
    """All shapes the entry point accepts, n_max far beyond the layers included (a workgroup's share of a
    compute unit's LDS, two to four of them, must not fall below its tables)."""
    short = [(L, M) for M in range(1, 65) for L in range(1, 256) if sizes.smallest_surplus(L, M) < 0]
    assert short == []
