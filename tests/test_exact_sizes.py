"""Index arithmetic of the exact minimum (csrc/oob_exact_sizes.h), compiled for the host and checked
over everything the entry points accept."""
import pytest

import exact_sizes


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    return exact_sizes.build(tmp_path_factory.mktemp("exact_sizes"))


def test_quotient_by_the_number_of_gpus(sizes):
    """Every index below 256 layers x M, every M: a reciprocal of 16 bits fails from M = 31 on."""
    assert [sizes.wrong_quotient(M) for M in range(1, 65)] == [-1] * 64


def test_tables_of_any_slowest_stage_fit_the_lds_of_a_workgroup(sizes):
    """All shapes the entry point accepts, n_max far beyond the layers included (a workgroup's share of a
    compute unit's LDS, two to four of them, must not fall below its tables)."""
    short = [(L, M) for M in range(1, 65) for L in range(1, 256) if sizes.smallest_surplus(L, M) < 0]
    assert short == []
