"""Instantiation enumeration (Section 4.2.1, Eq. 5) through the C ABI against the CPU oracle:
every vector, in list order, bit for bit (integer work: no tolerance)."""
import random

import numpy as np
import pytest

from oracle import instantiation as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_2309_08125_amd as pkg

    assert torch.cuda.is_available()
    pkg.load()
    return pkg


def compare(P, sizes, N_lo, N_hi, f, consecutive=None):
    if consecutive is None:
        inst = P.Instantiator(sizes, N_lo, N_hi, f)
    else:
        n0, p = consecutive
        sizes = list(range(n0, n0 + p))
        inst = P.Instantiator(None, N_lo, N_hi, f, n0=n0, p=p)
    off, x, st = inst.enumerate()
    want_off, want = I.instantiations_range(sizes, N_lo, N_hi, f)
    assert st == P.OOB_OK
    assert np.array_equal(off, want_off), (sizes, N_lo, N_hi, f)
    assert x.shape == want.shape and np.array_equal(x, want), (sizes, N_lo, N_hi, f)
    return len(want)


def test_paper_example_and_degenerate_cases(P):
    print("sizes (2,3,4)", flush=True)
    assert compare(P, [2, 3, 4], 0, 13, 0) > 0
    assert compare(P, [2, 3, 4], 13, 13, 0) == 5
    assert compare(P, [2, 3, 4], 7, 7, 0) == 2
    assert compare(P, [5], 15, 15, 3) == 0        # empty list: nothing to write
    assert compare(P, [5], 0, 0, 0) == 0          # no node, no pipeline
    assert compare(P, [1], 0, 9, 4) == 5          # one size: one vector per N' >= 5
    assert compare(P, [7, 9], 1, 6, 0) == 0       # nothing representable


def test_random_size_lists(P):
    rng = random.Random(11)
    for case in range(40):
        p = rng.randint(1, 9)
        sizes = sorted(rng.sample(range(1, 16), p))
        N_lo = rng.randint(0, 30)
        N_hi = N_lo + rng.randint(0, 25)
        f = rng.randint(0, 7)
        print(f"case {case}: sizes {sizes} N' {N_lo}..{N_hi} f {f}", flush=True)
        compare(P, sizes, N_lo, N_hi, f)


@pytest.mark.parametrize("n0,n_hi,f", [(1, 4, 1), (2, 16, 3), (4, 32, 4), (1, 32, 8), (8, 64, 8)])
def test_node_specifications_of_the_planning_workloads(P, n0, n_hi, f):
    """Consecutive sizes n0..n_hi, every N' from (f+1) n0 to N = n_hi + f n0 (Section 4.1.1):
    the five planning configurations; the last is the headline one (57 sizes, 1 343 380 vectors
    over several thousand wave-sized pieces with a ragged tail)."""
    N = n_hi + f * n0
    print(f"n0 {n0} n_hi {n_hi} f {f} N {N}", flush=True)
    total = compare(P, None, (f + 1) * n0, N, f, consecutive=(n0, n_hi - n0 + 1))
    if (n0, n_hi, f) == (8, 64, 8):
        assert total == 1343380


@pytest.mark.parametrize("p,N_lo,N_hi,f,spare", [(1, 0, 130, 0, 1), (3, 0, 40, 0, 3), (7, 10, 40, 1, 1), (8, 0, 36, 2, 2), (9, 0, 36, 1, 5),
                                                 (16, 0, 40, 1, 1), (17, 3, 40, 1, 0), (4, 0, 63, 3, 1), (4, 0, 64, 3, 2), (4, 100, 229, 30, 3)])
def test_rows_written_by_whole_waves(P, p, N_lo, N_hi, f, spare):
    """Full waves store four rows at a time, the last one row by row; rows that start at any multiple of two bytes, templates around a
    group's and a store's number, more lists than a wave has lanes, empty lists in front; entries past the total are left alone."""
    import torch

    inst = P.Instantiator(None, N_lo, N_hi, f, n0=1, p=p)
    off, st = inst.count()
    want_off, want = I.instantiations_range(list(range(1, p + 1)), N_lo, N_hi, f)
    assert st == P.OOB_OK and np.array_equal(off, want_off) and (len(want) > 64 or p == 1)
    x = torch.full((p, len(want) + spare), 9, dtype=torch.int16, device="cuda:0")
    inst.enqueue(x, len(want) + spare)
    got = x.cpu().numpy()
    assert np.array_equal(got[:, : len(want)].T, want) and (got[:, len(want):] == 9).all()


@pytest.mark.parametrize("sizes,N_lo,N_hi,f", [([64], 0, 4095, 0), ([64, 128], 0, 4095, 0), ([64, 128, 192], 1, 4095, 1), ([500, 700, 900], 0, 4095, 0),
                                               ([31, 57], 0, 2047, 1), ([5, 9], 7, 70, 0), ([5, 9], 7, 71, 0), ([1, 2], 100, 100, 0),
                                               ([1], 0, 4094, 0), ([1, 90], 4031, 4095, 0)])
def test_many_cluster_sizes_and_gaps_between_their_lists(P, sizes, N_lo, N_hi, f):
    """Lists of one vector, of none for tens of cluster sizes between two and of more than a wave, from one to 4 096 of them: where a
    vector's list is found by two reads, and by halving for the lanes behind the wave's first list."""
    print(sizes, N_lo, N_hi, f, flush=True)
    assert compare(P, sizes, N_lo, N_hi, f) >= 40


def test_gaps_between_the_lists_take_no_walk(P):
    """63 vectors of up to 63 pipelines, in 4 096 lists of which 63 are not empty, against 64 such vectors in 65 lists: the search for a
    vector's list grows with the logarithm of their number (1.2 times the time; past one empty list after the other it was 19 times)."""
    import torch

    def us(sizes, N_hi):
        inst = P.Instantiator(sizes, 1, N_hi, 0)
        off, st = inst.count()
        assert st == P.OOB_OK and off[-1] in (63, 64)
        x = torch.empty((1, int(off[-1])), dtype=torch.int16, device="cuda:0")
        best = float("inf")
        for _ in range(5):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            inst.enqueue(x, int(off[-1]))
            ev[0].record()
            for _ in range(20):
                inst.enqueue(x, int(off[-1]))
            ev[1].record()
            torch.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) / 20 * 1e3)
        return best

    sparse, dense = us([64], 4095), us([1], 64)
    print(f"{sparse:.1f} and {dense:.1f} us", flush=True)
    assert sparse < 4 * dense


def test_large_cluster_sizes_take_the_table_from_global_memory(P):
    """Two planes of the count table exceed the LDS here: the counting kernel's other path."""
    print("sizes 500,700,900", flush=True)
    assert compare(P, [500, 700, 900], 1900, 2000, 3) > 0
    sizes = list(range(90, 130, 3))
    print("sizes", sizes, flush=True)
    assert compare(P, sizes, 1000, 1100, 2) > 1000


def test_largest_dimensions_the_entry_points_take(P):
    """OOB_INST_MAX_P template sizes and cluster sizes up to OOB_INST_MAX_N: 1023 sizes
    3073..4095, N' = 3990..4095: one pipeline of exactly N' nodes is the only way each time."""
    sizes = list(range(3073, 4096))
    print("1023 sizes, N' 3990..4095", flush=True)
    assert compare(P, sizes, 3990, 4095, 0) == 106
    assert compare(P, sizes, 4000, 4095, 1) == 0          # two pipelines never fit


def test_integer_table_path(P):
    """Counts of 2^53 and more keep the table in int64 (no case the oracle could enumerate gets
    there): the test hook forces that path on ordinary cases."""
    lib = P.load()
    assert lib.oob_inst_keep_wide_table(1) == 0
    try:
        assert compare(P, [2, 3, 4], 0, 13, 0) > 0
        assert compare(P, None, 20, 48, 4, consecutive=(4, 29)) == 10251
        assert compare(P, list(range(90, 130, 3)), 1000, 1100, 2) > 1000
    finally:
        assert lib.oob_inst_keep_wide_table(0) == 1


def test_status_codes_and_capacity(P):
    import torch

    inst = P.Instantiator([3, 3, 4], 0, 12, 0)          # not strictly increasing
    off, st = inst.count()
    assert st == P.OOB_EINVAL and not off.any()
    inst = P.Instantiator([0, 2], 0, 12, 0)             # not positive
    assert inst.count()[1] == P.OOB_EINVAL
    inst = P.Instantiator(list(range(1, 31)), 30, 30, 0)
    off, st = inst.count()
    assert st == P.OOB_OK and int(off[-1]) == 5604       # partitions of 30
    x = torch.full((30, 100), 7777, dtype=torch.int16, device="cuda")
    inst.enqueue(x, 100)                                 # too small: nothing may be written
    torch.cuda.synchronize()
    assert int(inst.status.item()) == P.OOB_ECAPACITY
    assert bool((x.cpu() == 7777).all())
    assert int(inst.offsets[-1].item()) == 5604
    # lists longer than 2^62 are reported, not enumerated
    inst = P.Instantiator(None, 1000, 1000, 0, n0=1, p=200)   # partitions of 1000 into parts <= 200
    assert inst.count()[1] == P.OOB_EOVERFLOW


def test_capacity_larger_than_total_leaves_the_tail_untouched(P):
    import torch

    inst = P.Instantiator([2, 3, 4], 13, 13, 0)
    assert inst.count()[1] == P.OOB_OK
    x = torch.full((3, 64), 7777, dtype=torch.int16, device="cuda")
    inst.enqueue(x, 64)
    torch.cuda.synchronize()
    h = x.cpu().numpy()
    assert int(inst.status.item()) == P.OOB_OK
    assert h[:, :5].T.tolist() == [[5, 1, 0], [2, 3, 0], [3, 1, 1], [0, 3, 1], [1, 1, 2]]
    assert (h[:, 5:] == 7777).all()


@pytest.mark.parametrize("p,N_hi,f", [(1, 0, 0), (1, 1215, 0), (7, 1215, 0), (8, 1215, 0), (9, 1216, 0), (16, 242, 8), (15, 243, 8),
                                      (23, 127, 17), (24, 128, 17)])
def test_count_table_at_the_edges_of_its_lds(P, p, N_hi, f):
    """8 planes of (N_hi + 1) (f + 2) counts fit 152 KB up to 2 432 of them; planes are written in groups of 8."""
    step = max(1, N_hi // 40)
    sizes = [3 + step * (j + 1) for j in range(p)]
    print(f"p {p} N_hi {N_hi} f {f}", flush=True)
    compare(P, sizes, max(0, N_hi - 70), N_hi, f)


@pytest.mark.parametrize("N_hi,p,f", [(200, 200, 8), (300, 61, 3), (600, 600, 2), (1000, 40, 0)])
def test_list_lengths_beyond_32_bits(P, N_hi, p, f):
    """Lengths (no list is enumerated) against the recurrence of the count in Python integers."""
    C = [[0] * (f + 2) for _ in range(N_hi + 1)]
    C[0][0] = 1
    for n in range(1, p + 1):
        for x in range(n, N_hi + 1):
            C[x] = [C[x][q] + C[x - n][max(q - 1, 0)] for q in range(f + 2)]
    N_lo = max(0, N_hi - 150)
    want = [0]
    for x in range(N_lo, N_hi + 1):
        want.append(want[-1] + C[x][f + 1])
    assert want[-1] > 1 << 32
    off, st = P.Instantiator(None, N_lo, N_hi, f, n0=1, p=p).count()
    assert off.tolist() == [min(w, 1 << 62) for w in want]
    assert st == (P.OOB_OK if want[-1] < 1 << 62 else P.OOB_EOVERFLOW)


@pytest.mark.parametrize("N_hi,p,f,first", [(1200, 9, 0, 6), (600, 8, 0, 7), (365, 20, 3, 8), (340, 9, 3, 9), (250, 12, 3, 10),
                                            (135, 24, 3, 24), (140, 60, 3, 21), (128, 128, 3, 53)])
def test_table_that_outgrows_32_bits_on_the_way(P, N_hi, p, f, first):
    """Counts that fit 32 bits up to a plane, at any place in its group of eight planes: from there on 64 bits, and the
    planes before are widened.  The same table as counted in 64 bits from the start."""
    import torch

    C = [[0] * (f + 2) for _ in range(N_hi + 1)]
    C[0][0] = 1
    planes = [[row[:] for row in C]]
    for n in range(1, p + 1):
        for x in range(n, N_hi + 1):
            C[x] = [C[x][q] + C[x - n][max(q - 1, 0)] for q in range(f + 2)]
        planes.append([row[:] for row in C])
    assert [max(map(max, c)) >= (1 << 32) - 1 for c in planes].index(True) == first
    R = (p + 8) // 8 * 8
    want = np.array(planes).transpose(1, 2, 0)                              # [N'][q][j]
    lib = P.load()
    for wide in (1, 0):
        lib.oob_inst_keep_wide_table(wide)
        try:
            inst = P.Instantiator(None, N_hi, N_hi, f, n0=1, p=p)
            off, st = inst.count()
        finally:
            lib.oob_inst_keep_wide_table(0)
        assert st == P.OOB_OK and int(off[-1]) == planes[p][N_hi][f + 1]
        n = (N_hi + 1) * (f + 2) * R
        table = inst.workspace[256: 256 + 8 * n].view(torch.int64).reshape(N_hi + 1, f + 2, R)[:, :, : p + 1]
        assert np.array_equal(table.cpu().numpy(), want), wide


@pytest.mark.parametrize("f", [0, 1, 2, 3, 4, 5, 9, 16, 30])
def test_count_table_by_node_counts(P, f):
    """Every number of q's of a wave and of waves for a node count; one to sixteen node counts a step; the last lane; sizes
    beyond N_hi; gaps; counts around 2^32, where the table is counted in 64 bits after all.  Whole tables against the recurrence."""
    import torch

    for sizes, N_hi in [(range(8, 65), 128 if f < 10 else 70), (range(2, 65), 40), (range(3, 60, 2), 50), (range(20, 83), 75), (range(40, 60), 30),
                        (range(5, 40), 97), (range(7, 70), 230), (range(7, 70), 290)]:
        sizes = list(sizes)
        p, R = len(sizes), (len(sizes) + 8) // 8 * 8
        C = np.zeros((N_hi + 1, f + 2, p + 1), dtype=np.int64)
        C[0, 0] = 1
        for j, n in enumerate(sizes):
            C[:, :, j + 1] = C[:, :, j]
            for x in range(n, N_hi + 1):
                C[x, 1:, j + 1] += C[x - n, :-1, j + 1]
                C[x, 0, j + 1] += C[x - n, 0, j + 1]
        print(f"sizes {sizes[0]}..{sizes[-1]} N_hi {N_hi} f {f}: up to {C.max()}", flush=True)
        inst = P.Instantiator(sizes, 0, N_hi, f)
        off, st = inst.count()
        assert st == P.OOB_OK and np.array_equal(off, np.concatenate([[0], np.cumsum(C[:, f + 1, p])]))
        ws, n = inst.workspace.cpu(), (N_hi + 1) * (f + 2) * R
        narrow = int(ws[:4].view(torch.int32))
        assert narrow == int(C.max() < (1 << 32) - 1)
        if narrow:
            at = 256 + (8 * n + 255) // 256 * 256
            table = ws[at: at + 4 * n].view(torch.int32).numpy().view("uint32").reshape(N_hi + 1, f + 2, R)
            assert (table[:, :, p + 1:] == 0xFFFFFFFF).all()
        else:
            table = ws[256: 256 + 8 * n].view(torch.int64).numpy().reshape(N_hi + 1, f + 2, R)
        assert np.array_equal(table[:, :, : p + 1], C)


@pytest.mark.parametrize("listed", [False, True])
@pytest.mark.parametrize("N_hi,f,least", [(40, 2, 24), (126, 2, 41), (127, 2, 35), (63, 6, 22), (100, 0, 36)])
def test_count_table_at_the_line_between_planes_and_scans(P, N_hi, f, least, listed):
    """`least` sizes from 5 on are counted by node counts (steps of five), fewer by sizes: 10 and N_hi / 5 sizes, 16 where a plane has
    fewer than 512 counts; lists may be counted by sizes beyond that.  The lengths and the whole table against the recurrence, on both sides of the line."""
    assert least == (16 if (N_hi + 1) * (f + 2) < 512 else 10) + N_hi // 5
    for p in (least - 1, least, least + 1):
        R = (p + 8) // 8 * 8
        C = np.zeros((N_hi + 1, f + 2, p + 1), dtype=np.int64)
        C[0, 0] = 1
        for j in range(p):
            n = 5 + j
            C[:, :, j + 1] = C[:, :, j]
            for x in range(n, N_hi + 1):
                C[x, 1:, j + 1] += C[x - n, :-1, j + 1]
                C[x, 0, j + 1] += C[x - n, 0, j + 1]
        assert C.max() < 1 << 32
        inst = P.Instantiator(list(range(5, 5 + p)), 0, N_hi, f) if listed else P.Instantiator(None, 0, N_hi, f, n0=5, p=p)
        off, st = inst.count()
        assert st == P.OOB_OK and np.array_equal(off, np.concatenate([[0], np.cumsum(C[:, f + 1, p])])), p
        ws, n = inst.workspace.cpu().numpy(), (N_hi + 1) * (f + 2) * R
        at = 256 + (8 * n + 255) // 256 * 256
        table = ws[at: at + 4 * n].view("uint32").reshape(N_hi + 1, f + 2, R)
        assert np.array_equal(table[:, :, : p + 1], C), p
