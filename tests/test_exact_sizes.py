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
