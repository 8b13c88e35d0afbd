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


def test_launches_beyond_the_default_limit_of_lds_are_announced(sizes):
    """64 KB a workgroup, static arrays (as they are in the library) included, over all shapes that the entry points accept; none beyond 160 KB."""
    import ctypes as C

    static = exact_sizes.static_lds()
    assert len(static) == 3 and all(static.values())
    sizes.launch.restype = C.c_size_t
    announced, wrong = C.c_int(), []
    for kernel, own in enumerate(static[k] for k in ("k_exact_prep", "k_exact_bounds", "k_exact_eval")):
        for counts in range(2):
            for M in range(1, 65):
                for L in range(1, 256):
                    n = sizes.launch(kernel, L, M, counts, C.byref(announced))
                    if n + own > 160 * 1024 or (n + own > 64 * 1024 and not announced.value):
                        wrong.append((kernel, counts, L, M, n))
    assert not wrong, (len(wrong), wrong[:12])
