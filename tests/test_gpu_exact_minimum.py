"""Exact minimum of the pipeline cost (all explicit pipelines; Section 4.1.2's closed form) through
the C ABI against the CPU oracle: integers, compared exactly."""
import json
import os

import pytest

import exact_sizes
import inputs
from oracle import exact_minimum as E

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_2309_08125_amd as pkg

    assert torch.cuda.is_available()
    pkg.load()
    return pkg


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    return exact_sizes.build(tmp_path_factory.mktemp("exact_sizes"))


SHAPES = [(1, 1, 1, 1, 4), (5, 1, 1, 3, 6), (6, 2, 1, 3, 8), (7, 2, 1, 2, 9), (6, 4, 1, 2, 12), (8, 4, 2, 2, 12),
          (9, 2, 2, 3, 9), (12, 3, 1, 4, 12), (15, 2, 1, 5, 15), (23, 8, 1, 3, 30), (37, 3, 1, 5, 40), (20, 16, 1, 2, 33),
          # more GPU positions than one tile of the kernel holds: several blocks of whole nodes
          (12, 8, 1, 10, 12), (10, 4, 2, 20, 10), (14, 3, 1, 30, 14), (9, 16, 1, 6, 9), (30, 5, 1, 27, 30)]


@pytest.mark.parametrize("shape", SHAPES)
def test_small_random_against_the_oracle(P, shape):
    L, M, n_min, n_max, nb = shape
    for seed in range(3):
        for var in ("plain", "tight", "forbid"):
            inp = inputs.random_small(seed, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"),
                                      forbid_some_d=(var == "forbid"))
            print("case", inp.name, shape, var, flush=True)
            st, got = P.ExactMinimum(inp).run()
            assert st == P.OOB_OK and got == E.exact_minimum(inp), (shape, seed, var)


def test_stage_times_that_are_not_monotone_in_the_last_layer(P):
    """A stage that ends at the model's last layer pays no boundary term, so it can be faster than
    the stage ending one layer earlier: the hand case of the oracle's pins (32, 20, 20), and small
    times against boundary terms up to 5 on two hundred seeds."""
    from test_oracle_exact_minimum import boundary_heavy_case

    inp = boundary_heavy_case()
    st, got = P.ExactMinimum(inp).run()
    assert st == P.OOB_OK and got == [32, 20, 20] == E.exact_minimum(inp)
    for seed in range(1000, 1200):
        inp = inputs.random_small(seed, 6, 2, 1, 3, 8, t_lo=1, t_hi=4)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp), seed
    for seed in range(40):  # longer models, more GPUs per node
        inp = inputs.random_small(2000 + seed, 14, 4, 1, 4, 16, t_lo=1, t_hi=3)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp), seed


MODE_SHAPES = [(7, 3, 1, 2, 0), (6, 2, 1, 3, 0), (8, 1, 1, 4, 0), (12, 4, 1, 3, 0), (25, 8, 1, 4, 0), (40, 2, 1, 9, 0),
               (7, 1, 1, 4, 3), (7, 2, 1, 3, 4), (8, 2, 1, 3, 3), (6, 4, 1, 2, 3), (14, 4, 1, 4, 6), (20, 2, 2, 6, 7),
               (9, 3, 1, 2, 2), (16, 8, 1, 2, 5)]


@pytest.mark.parametrize("shape", MODE_SHAPES)
def test_4S_mode_and_stage_limit_against_the_oracle(P, shape):
    """N_b = 4 S per pipeline (microbatches = 0) and N_b below min(L, n M), where the limit S <= N_b
    binds: the entry point with the stage count in its tables against the oracle that carries it too;
    the one without it against the oracle without it on the templates it answers for, -2 on the others."""
    L, M, n_min, n_max, nb = shape
    for seed in range(3):
        for var in ("plain", "tight", "forbid"):
            inp = inputs.random_small(seed, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"),
                                      forbid_some_d=(var == "forbid"))
            print("case", inp.name, shape, var, flush=True)
            st, got = P.ExactMinimum(inp, staged=True).run()
            assert st == P.OOB_OK and got == E.exact_minimum_staged(inp), (shape, seed, var)
            st, got = P.ExactMinimum(inp).run()
            want = E.exact_minimum(inp, allow_bound=True)  # marks the other templates as the boundary does
            assert E.LIMIT_CAN_BIND == P.OOB_EXACT_LIMIT_CAN_BIND
            assert st == P.OOB_OK and got == want, (shape, seed, var)


def test_stage_limit_at_middle_sizes(P):
    """Tables of 49 x 65 x 21 and 65 x 65 x 33 entries per workgroup, many workgroups in flight."""
    for shape in [(24, 4, 1, 6, 10), (36, 2, 2, 12, 14), (48, 8, 1, 8, 20), (64, 4, 1, 16, 32)]:
        L, M, n_min, n_max, nb = shape
        inp = inputs.random_small(1, L, M, n_min, n_max, nb, f=1)
        print("case", shape, flush=True)
        st, got = P.ExactMinimum(inp, staged=True).run()
        assert st == P.OOB_OK and got == E.exact_minimum_staged(inp), shape


def test_shapes_beyond_lds_take_the_general_path(P):
    """More layers or GPUs per node than the LDS tables hold: the recurrence over tables in the
    workspace, same results."""
    for shape in [(200, 2, 1, 2, 200), (120, 48, 1, 1, 0), (140, 1, 1, 3, 140), (150, 2, 1, 2, 0)]:
        L, M, n_min, n_max, nb = shape
        inp = inputs.random_small(7, L, M, n_min, n_max, nb, f=1, tight_mem=True)
        print("case", shape, flush=True)
        if shape[0] >= 200 or shape[1] >= 48:
            assert P.oob_exact_workspace_size(L, n_max, M) > (16 << 20)   # tables of the workgroups in flight
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp), shape


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_configurations_1_to_3(P, cfg):
    inp = inputs.config(cfg)
    st, got = P.ExactMinimum(inp).run()
    assert st == P.OOB_OK and got == E.exact_minimum(inp)
    # never above what the recursion finds
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    res = planner.plan(inp)
    planner.close()
    for i, e in enumerate(got):
        assert (e is None) == (not res["feasible"][i])
        assert e is None or e <= int(res["T"][i])


@pytest.mark.timeout(600)
def test_headline_configuration_against_stored_oracle_results(P):
    """Configuration 4 as bench.py runs it; the oracle's minima are stored by
    tests/golden/make_golden.py cfg4_exact (which calls only the oracle)."""
    inp = inputs.config(4)
    want = json.load(open(os.path.join(GOLD, "cfg4_exact_minimum.json")))["exact_minimum"]
    st, got = P.ExactMinimum(inp).run()
    assert st == P.OOB_OK and got == want
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    res = planner.plan(inp)
    planner.close()
    gaps = [int(res["T"][i]) / e - 1 for i, e in enumerate(got)]
    assert min(gaps) >= 0
    print(f"configuration 4: recursion above the exact minimum by at most {max(gaps):.4%}, "
          f"equal for {sum(g == 0 for g in gaps)} of {len(gaps)} templates", flush=True)


def test_status_for_negative_profile_entries(P):
    import dataclasses

    inp = inputs.random_small(3, 8, 2, 1, 3, 8)
    fwd = inp.fwd_ns.copy()
    fwd[2, 0] = -5
    st, _ = P.ExactMinimum(dataclasses.replace(inp, fwd_ns=fwd)).run()
    assert st == P.OOB_EINVAL
    # several workgroups' worth of (layer, GPU count) pairs, the bad entry in the last one
    inp = inputs.random_small(3, 40, 4, 1, 3, 40)
    fwd = inp.fwd_ns.copy()
    fwd[39, 3] = -1
    st, _ = P.ExactMinimum(dataclasses.replace(inp, fwd_ns=fwd)).run()
    assert st == P.OOB_EINVAL


def test_status_for_times_too_large_to_be_exact(P):
    import dataclasses

    inp = inputs.random_small(4, 8, 2, 1, 3, 8)
    # tables in LDS hold doubles: (N_b + 2) * sum of the layers' slowest times must stay below 2^52
    big = dataclasses.replace(inp, fwd_ns=inp.fwd_ns + (1 << 50))
    st, _ = P.ExactMinimum(big).run()
    assert st == P.OOB_EOVERFLOW
    ok = dataclasses.replace(inp, fwd_ns=inp.fwd_ns + (1 << 44))
    st, got = P.ExactMinimum(ok).run()
    assert st == P.OOB_OK and got == E.exact_minimum(ok)
    # tables in the workspace hold int64: below 2^61
    st, got = P.ExactMinimum(big, staged=True).run()
    assert st == P.OOB_OK and got == E.exact_minimum_staged(big)
    huge = dataclasses.replace(inp, fwd_ns=inp.fwd_ns + (1 << 57))
    st, _ = P.ExactMinimum(huge, staged=True).run()
    assert st == P.OOB_EOVERFLOW


def test_many_random_shapes(P):
    """400 seeded random shapes (1..16 GPUs per node, all three N_b regimes, tight memory, forbidden GPU
    counts, small times against boundary terms) against the oracle; templates whose stage limit can bind
    carry the marker on both sides."""
    import random

    rng = random.Random(2309)
    for n in range(400):
        M = rng.choice([1, 2, 3, 4, 5, 7, 8, 8, 9, 12, 16])
        L = rng.randint(1, 44 if M <= 8 else 30)
        n_max = rng.randint(1, max(1, min(10, L)))
        n_min = rng.randint(1, n_max)
        nb = rng.choice([0, 0, rng.randint(1, 2 * L + 2), L * M + 5, rng.randint(1, 12)])
        var = rng.choice(["plain", "tight", "forbid"])
        kw = {}
        if rng.random() < 0.3:
            kw = dict(t_lo=1, t_hi=rng.choice([3, 4, 8]))
        if rng.random() < 0.2:
            kw["uniform_layers"] = True
        inp = inputs.random_small(rng.randint(0, 10 ** 6), L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"),
                                  forbid_some_d=(var == "forbid"), **kw)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (n, L, M, n_min, n_max, nb, var, kw)


@pytest.mark.parametrize("shape", [(64, 3, 1, 5, 64), (92, 1, 1, 20, 92), (98, 8, 1, 2, 98), (75, 2, 3, 20, 75),
                                   (72, 5, 2, 6, 0), (90, 2, 1, 30, 90), (64, 3, 1, 4, 12), (92, 1, 1, 9, 8), (70, 2, 1, 5, 9)])
def test_jobs_large_enough_for_bounds(P, shape):
    """More (layer pair, GPU count) triples than are evaluated without lower bounds: one GPU per node, GPU
    counts that are no power of two, few nodes (long stages: wide bands, tables over layers and GPUs), many
    nodes, a stage limit that binds; random times, equal layers (every stage time occurs many times, bounds
    and minima tie) and one layer that dwarfs the others."""
    import dataclasses

    L, M, n_min, n_max, nb = shape
    assert L * (L + 1) // 2 * M > 4096
    for var in ("plain", "tight", "forbid", "equal", "dwarf"):
        inp = inputs.random_small(11, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"),
                                  forbid_some_d=(var == "forbid"))
        if var == "equal":
            inp = dataclasses.replace(inp, fwd_ns=inp.fwd_ns[:1].repeat(L, 0).copy(), bwd_ns=inp.bwd_ns[:1].repeat(L, 0).copy())
        if var == "dwarf":
            fwd = inp.fwd_ns.copy()
            fwd[L // 3] = fwd.sum(0)
            inp = dataclasses.replace(inp, fwd_ns=fwd)
        print("case", shape, var, flush=True)
        staged = 0 < nb < min(L, n_max * M)
        st, got = P.ExactMinimum(inp, staged=staged).run()
        want = E.exact_minimum_staged(inp) if staged else E.exact_minimum(inp)
        assert st == P.OOB_OK and got == want, (shape, var)


@pytest.mark.parametrize("shape", [(100, 1, 20, 92, 0), (66, 2, 1, 66, 132), (66, 2, 3, 68, 132)])
def test_more_templates_than_bounds_are_kept_for(P, shape):
    """More than 64 templates: every stage is evaluated but those too dear by their time alone."""
    L, M, n_min, n_max, nb = shape
    assert n_max - n_min + 1 > 64 and L * (L + 1) // 2 * M > 4096
    for var in ("plain", "tight", "forbid"):
        inp = inputs.random_small(23, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"), forbid_some_d=(var == "forbid"))
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp), (shape, var)


def test_buckets_of_more_entries_than_are_bounded_at_once(P, sizes):
    """More possible slowest stages than 512 buckets of 64 hold."""
    inp = inputs.random_small(29, 98, 8, 1, 2, 98, f=1)
    e = P.ExactMinimum(inp)
    st, got = e.run()
    h = exact_sizes.head(e.workspace)
    assert h["bucket"] > 64 and h["nbuckets"] <= 512
    assert st == P.OOB_OK and got == E.exact_minimum(inp)


@pytest.mark.parametrize("shape", [(74, 31, 1, 2, 0), (66, 32, 1, 2, 66), (46, 48, 1, 2, 0), (30, 60, 1, 2, 30), (20, 64, 1, 2, 0),
                                   (26, 64, 1, 1, 0)])
def test_many_gpus_per_node_with_tables_in_lds(P, shape):
    """Indices (layer, GPU count) beyond 2^16 / M, tables in LDS (a small workspace)."""
    L, M, n_min, n_max, nb = shape
    assert P.oob_exact_workspace_size(L, n_max, M) < (16 << 20)
    for var in ("plain", "tight", "forbid"):
        inp = inputs.random_small(13, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"),
                                  forbid_some_d=(var == "forbid"))
        print("case", shape, var, flush=True)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (shape, var)


@pytest.mark.parametrize("shape", [(35, 1, 1, 1389, 0), (31, 2, 1, 840, 62), (1, 1, 1, 1681, 0), (90, 1, 4, 69, 90), (10, 1, 1, 1641, 10),
                                   (130, 2, 1, 3, 0), (105, 1, 1, 104, 105), (100, 3, 2, 2, 0), (88, 2, 4, 4, 88)])
def test_shares_of_the_lds_that_just_hold_the_tables(P, shape):
    """Far more nodes than layers (tables as for as many nodes as layers), and two, three or four workgroups per compute
    unit whose tables take the whole of their share."""
    L, M, n_min, n_max, nb = shape
    for var in ("plain", "tight"):
        inp = inputs.random_small(5, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"))
        print("case", shape, var, flush=True)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (shape, var)


@pytest.mark.parametrize("shape,padded", [((32, 8, 1, 4, 0), 1), ((31, 8, 1, 4, 0), 1), ((59, 8, 1, 60, 0), 0), ((61, 8, 1, 60, 0), 1),
                                          ((58, 8, 2, 18, 60), 1), ((36, 8, 1, 25, 49), 1), ((40, 4, 1, 9, 0), 0)])
def test_padded_and_plain_rows_of_the_profile(P, sizes, shape, padded):
    """Eight GPUs per node: rows of nine doubles, or of eight where nine would cost a workgroup of a compute unit (and in jobs
    without bounds, up to 31 layers); one-node tables shared out evenly to the waves where they do not all fit."""
    L, M, n_min, n_max, nb = shape
    assert sizes.padded(L, M, n_max) == padded
    for var in ("plain", "tight", "forbid"):
        inp = inputs.random_small(23, L, M, n_min, n_max, nb, f=1, tight_mem=(var == "tight"), forbid_some_d=(var == "forbid"))
        print("case", shape, var, flush=True)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (shape, var)


@pytest.mark.parametrize("shape", [(72, 64, 1, 1, 0), (105, 32, 1, 2, 105), (142, 16, 1, 2, 0), (167, 8, 1, 3, 167), (178, 5, 1, 2, 0)])
def test_tables_in_lds_without_the_ends_of_the_stages(P, sizes, shape):
    """The largest shapes whose times are held as doubles: their tables leave no room for the ends of the
    stages, which are added up where they are read; a small workspace."""
    L, M, n_min, n_max, nb = shape
    assert sizes.sums(L, M, n_max) == 1 and P.oob_exact_workspace_size(L, n_max, M) < (16 << 20)
    for var in ("plain", "forbid"):
        inp = inputs.random_small(17, L, M, n_min, n_max, nb, f=1, forbid_some_d=(var == "forbid"))
        print("case", shape, var, flush=True)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (shape, var)


@pytest.mark.parametrize("shape", [(192, 1, 1, 8, 192), (189, 2, 1, 2, 0), (171, 8, 1, 1, 0)])
def test_shapes_beyond_doubles_take_times_beyond_them(P, sizes, shape):
    """Shapes whose tables would fit the LDS but whose times may exceed 2^52: answered in 64-bit integers."""
    import dataclasses

    L, M, n_min, n_max, nb = shape
    assert sizes.sums(L, M, n_max) >= 0
    inp = inputs.random_small(19, L, M, n_min, n_max, nb, f=1)
    for add in (0, 1 << 42):
        big = dataclasses.replace(inp, fwd_ns=inp.fwd_ns + add)
        want = E.exact_minimum(big)
        for staged in (False, True):
            print("case", shape, add, staged, flush=True)
            st, got = P.ExactMinimum(big, staged=staged).run()
            assert st == P.OOB_OK and got == want, (shape, add, staged)


# (layers, GPUs per node, templates, N_b): a node covers up to 64 layers, one more, few; starts that fill a wave and do not
@pytest.mark.parametrize("ends", ["ascending", "mixed"])
@pytest.mark.parametrize("shape", [(64, 1, 1, 4, 64), (65, 1, 1, 3, 0), (64, 2, 1, 2, 0), (66, 2, 1, 3, 70), (67, 4, 1, 2, 70), (65, 8, 1, 1, 70),
                                   (66, 8, 1, 3, 0), (33, 4, 1, 5, 33), (17, 8, 2, 4, 20), (31, 8, 4, 12, 0)])
def test_tables_of_a_node_in_registers_and_in_lds(P, shape, ends):
    """Ends of stages that ascend with the layer (tables in registers where a node covers at most 64) and boundary terms
    that outweigh layers."""
    import dataclasses

    import numpy as np

    L, M, n_min, n_max, nb = shape
    for var in ("plain", "tight", "forbid"):
        inp = inputs.random_small(41, L, M, n_min, n_max, nb, f=1, t_lo=60, t_hi=99, tight_mem=(var == "tight"), forbid_some_d=(var == "forbid"))
        if ends == "mixed":
            inp = dataclasses.replace(inp, boundary_ns=np.random.default_rng(L).integers(0, 400, L))
        print("case", shape, ends, var, flush=True)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (shape, ends, var)


# (layers, GPUs per node, templates, N_b) whose bands are a layer or two off the lines between the tables of a node and those over all GPUs
@pytest.mark.parametrize("shape", [(26, 8, 1, 2, 40), (28, 8, 1, 3, 0), (35, 4, 1, 2, 50), (36, 4, 2, 4, 0), (43, 4, 1, 5, 45), (34, 8, 1, 4, 34)])
def test_few_nodes_of_many_layers(P, shape):
    L, M, n_min, n_max, nb = shape
    for var in ("plain", "tight", "uniform"):
        inp = inputs.random_small(47, L, M, n_min, n_max, nb, f=1, t_lo=60, t_hi=99, tight_mem=(var == "tight"), uniform_layers=(var == "uniform"))
        print("case", shape, var, flush=True)
        st, got = P.ExactMinimum(inp).run()
        assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True), (shape, var)


def call_us(exact):
    """Time of a call, the best of five."""
    import torch

    best = float("inf")
    for _ in range(5):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        exact.enqueue()
        ev[0].record()
        for _ in range(10):
            exact.enqueue()
        ev[1].record()
        torch.cuda.synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]) / 10 * 1e3)
    return best


@pytest.mark.parametrize("job", [226, 171])
def test_two_nodes_of_many_layers_take_little_longer_than_one(P, job):
    """61 and 66 ragged layers, 8 GPUs per node: where a node may cover most of the model a table per start layer is the longer way for
    two nodes (1.8 and 1.6 times the time of one node, 1.3 with the tables over all GPUs)."""
    import dataclasses

    inp = inputs.config(5)[job]
    one, two = (call_us(P.ExactMinimum(dataclasses.replace(inp, n_min=1, n_max=n, microbatches=0))) for n in (1, 2))
    print(f"{one:.0f} and {two:.0f} us", flush=True)
    assert two < 1.7 * one


@pytest.mark.parametrize("ends", ["ascending", "mixed"])
@pytest.mark.parametrize("shape", [(20, 8, 1, 4, 9), (33, 4, 1, 4, 12), (40, 2, 1, 6, 11), (30, 1, 1, 24, 10), (66, 2, 1, 2, 3)])
def test_tables_of_a_node_with_stage_counts(P, shape, ends):
    import dataclasses

    import numpy as np

    L, M, n_min, n_max, nb = shape
    for var in ("plain", "tight"):
        inp = inputs.random_small(43, L, M, n_min, n_max, nb, f=1, t_lo=60, t_hi=99, tight_mem=(var == "tight"))
        if ends == "mixed":
            inp = dataclasses.replace(inp, boundary_ns=np.random.default_rng(L).integers(0, 400, L))
        print("case", shape, ends, var, flush=True)
        st, got = P.ExactMinimum(inp, staged=True).run()
        assert st == P.OOB_OK and got == E.exact_minimum_staged(inp), (shape, ends, var)


@pytest.mark.parametrize("shape", [(2, 8, 1, 2, 1), (17, 8, 1, 4, 9), (18, 8, 1, 4, 9), (20, 8, 1, 3, 12), (23, 8, 2, 3, 11), (20, 8, 1, 4, 8),
                                   (20, 8, 1, 3, 9), (20, 8, 1, 3, 10), (23, 8, 2, 3, 9)])
def test_stage_counts_with_tables_in_lds_and_in_registers(P, shape):
    """As many start layers as waves and one more, and few nodes up to the layers whose tables still fit LDS."""
    L, M, n_min, n_max, nb = shape
    for var in ("plain", "tight"):
        inp = inputs.random_small(53, L, M, n_min, n_max, nb, f=1, t_lo=60, t_hi=99, tight_mem=(var == "tight"))
        print("case", shape, var, flush=True)
        st, got = P.ExactMinimum(inp, staged=True).run()
        assert st == P.OOB_OK and got == E.exact_minimum_staged(inp), (shape, var)


def test_stage_counts_of_a_short_model_take_little_longer(P):
    """Ten layers, 8 GPUs per node: where every start layer has a wave and a table in LDS, the tables in registers are the longer way (1.9 times
    the time of the call without stage counts, 1.4 with those in LDS)."""
    with_counts = call_us(P.ExactMinimum(inputs.random_small(5, 10, 8, 1, 2, 3, f=1, t_lo=60, t_hi=99), staged=True))
    without = call_us(P.ExactMinimum(inputs.random_small(5, 10, 8, 1, 2, 10, f=1, t_lo=60, t_hi=99)))
    print(f"{with_counts:.0f} and {without:.0f} us", flush=True)
    assert with_counts < 1.6 * without


@pytest.mark.parametrize("L,M", [(92, 1), (60, 8), (150, 8), (66, 33)])
def test_list_of_the_possible_slowest_stages(P, sizes, L, M):
    """Every stage that fits once, with its time, ascending by the leading bits -- lists put in order in LDS and longer ones."""
    import numpy as np
    import torch

    inp = inputs.random_small(17, L, M, 1, 1, L, f=1, t_lo=200, t_hi=3000, tight_mem=True)
    e = P.ExactMinimum(inp)
    st, _ = e.run()
    assert st == P.OOB_OK
    h, at = exact_sizes.head(e.workspace), exact_sizes.offsets(sizes, L, M, inp.n_max)
    n = h["ncand"]
    tau = e.workspace[at["ctau"]: at["ctau"] + 8 * n].view(torch.float64).cpu().numpy()
    uvd = e.workspace[at["cuvd"]: at["cuvd"] + 4 * n].view(torch.int32).cpu().numpy()
    PT = np.concatenate([np.zeros((1, M), dtype=np.int64), np.cumsum(inp.fwd_ns + inp.bwd_ns, axis=0)])
    X = np.concatenate([[0], inp.boundary_ns[:-1], [0]])
    mem = np.concatenate([[0], np.cumsum(inp.mem_bytes)])
    want = {(u, v, d): int(PT[v, d - 1] - PT[u, d - 1] + X[v]) for v in range(1, L + 1) for u in range(v) for d in range(1, M + 1)
            if -(-int(mem[v] - mem[u]) // d) <= inp.mem_cap}
    got = list(zip((uvd & 255).tolist(), (uvd >> 8 & 255).tolist(), (uvd >> 16).tolist()))
    assert len(set(got)) == n == len(want) and all(want[k] == t for k, t in zip(got, tau.tolist()))
    lead = tau.view(np.int64) >> 44
    assert (np.diff(lead - lead.min()).clip(max=1)[: int((lead - lead.min() < 4095).sum()) - 1] >= 0).all()


@pytest.mark.parametrize("L,M", [(87, 3), (107, 2), (23, 37)])
def test_list_that_ends_at_the_default_limit_of_lds(P, sizes, L, M):
    """The list fits beside its tables in 48 KB, but not in 64 KB with the static arrays of the kernel."""
    test_list_of_the_possible_slowest_stages(P, sizes, L, M)


@pytest.mark.parametrize("M", [1, 3, 4, 8])
@pytest.mark.parametrize("nb", [2, 7, 8, 9, 10])
def test_stage_counts_around_whole_groups(P, M, nb):
    """Counts 0 .. N_b in groups of four: one short group, and every remainder; one side without layers and two."""
    for L, n_max in ((18, 3), (26, 6)):
        inp = inputs.random_small(nb, L, M, 1, n_max, nb, f=1, t_lo=60, t_hi=99)
        st, got = P.ExactMinimum(inp, staged=True).run()
        assert st == P.OOB_OK and got == E.exact_minimum_staged(inp), (L, M, nb)


def test_leftovers_with_stage_counts_are_listed_once(P, sizes):
    """Slowest stages whose tables exceed LDS are left to the general path: each at most once, whatever the
    number of templates that pick it first."""
    import torch

    L, M, n_min, n_max, nb = 65, 8, 1, 8, 40
    inp = inputs.random_small(7, L, M, n_min, n_max, nb, f=1)
    e = P.ExactMinimum(inp, staged=True)
    st, got = e.run()
    assert st == P.OOB_OK and got == E.exact_minimum_staged(inp)
    h = exact_sizes.head(e.workspace)
    o = exact_sizes.offsets(sizes, L, M, n_max, counts=True, staged=True)["over"]
    left = e.workspace[o: o + 4 * h["over"]].view(torch.int32).tolist()
    assert 0 < len(left) == len(set(left)) <= h["alive"] <= h["ncand"]


LAMBDA_GIVEN = (0, 0.04, 0.1, 0.2, 0.4, 0.8, 1.6, 3.5)  # prices per GPU of the bounds, N_b given


def bounds_of_a_job(P, sizes, inp):
    """(bounds on the device [entries, prices], the same sums in 80-bit floats, their rounding): least sums over the
    stages before and after each possible slowest stage, GPUs priced, N_b given, no stage limit."""
    import numpy as np
    import torch

    L, M = inp.L, inp.gpus_per_node
    e = P.ExactMinimum(inp)
    st, got = e.run()
    assert st == P.OOB_OK and got == E.exact_minimum(inp, allow_bound=True)
    h, at = exact_sizes.head(e.workspace), exact_sizes.offsets(sizes, L, M, inp.n_max)
    n = h["ncand"]
    part = lambda k, size, dt: e.workspace[at[k]: at[k] + size * n].view(dt).cpu().numpy()
    tau, uvd = part("ctau", 8, torch.float64), part("cuvd", 4, torch.int32)
    lb = part("lb", 4 * len(LAMBDA_GIVEN), torch.float32).reshape(n, len(LAMBDA_GIVEN))
    big = np.longdouble
    forbidden = (inp.fwd_ns >= 1 << 62) | (inp.bwd_ns >= 1 << 62)
    assert not forbidden.any() and int(inp.mem_bytes.sum()) <= inp.mem_cap
    PT = np.concatenate([np.zeros((1, M), dtype=np.int64), np.cumsum(inp.fwd_ns + inp.bwd_ns, axis=0)]).astype(big)
    X = np.concatenate([[0], inp.boundary_ns[:-1], [0]]).astype(big)
    d1 = np.arange(1, M + 1)
    want, err = np.empty((n, len(LAMBDA_GIVEN)), dtype=big), np.empty((n, 1))
    for c0 in range(0, n, h["bucket"]):
        c = slice(c0, min(n, c0 + h["bucket"]))
        lo, hi = tau[c].min(), tau[c].max()
        err[c] = 6 * L * 2.0 ** -63 * (L * hi + 2 * float(PT.max()) + L * M * LAMBDA_GIVEN[-1] * lo)
        for k, price in enumerate(LAMBDA_GIVEN):
            lam = big(price * lo)
            before, after = np.full(L + 1, big(np.inf)), np.full(L + 1, big(np.inf))
            before[0] = after[L] = 0
            for p in range(1, L + 1):
                t = PT[p] + X[p] - PT[:p]  # stages [x, p)
                before[p] = np.where(t <= hi, before[:p, None] + t + lam * d1, big(np.inf)).min()
            for p in range(L - 1, -1, -1):
                t = PT[p + 1:] + X[p + 1:, None] - PT[p]
                after[p] = np.where(t <= hi, after[p + 1:, None] + 2 * t - big(hi) + lam * d1, big(np.inf)).min()
            u, v, d = uvd[c] & 255, uvd[c] >> 8 & 255, uvd[c] >> 16
            want[c, k] = inp.microbatches * tau[c].astype(big) + before[u] + after[v] + lam * d
    return lb, want, err


@pytest.mark.parametrize("never", [(), (0,), (3, 40)])
def test_lower_bounds_are_below_what_they_bound(P, sizes, never):
    """The bounds of every possible slowest stage against the sums they stand for, in more precision.  `never`: layers
    whose time on two GPUs no pipeline of a minimum takes, near the largest that is accepted -- doubles of that size
    round by a quarter of a nanosecond and more."""
    import dataclasses

    import numpy as np

    inp = inputs.random_small(3, 66, 2, 1, 2, 4, f=1, t_lo=20, t_hi=50)
    if never:
        fwd = inp.fwd_ns.copy()
        fwd[list(never), 1] = ((1 << 52) // (inp.microbatches + 2) - 10 ** 7) // len(never)
        inp = dataclasses.replace(inp, fwd_ns=fwd)
    lb, want, err = bounds_of_a_job(P, sizes, inp)
    finite = np.isfinite(want)
    assert finite.sum() > 4096 and (lb <= want + err)[finite].all(), float((lb - want)[finite].max())
    # stages that no pipeline has as its slowest: the layers before or after them need a slower one
    assert (~finite).any() and np.isposinf(lb[~finite]).all()


@pytest.mark.parametrize("L,M,n_max", [(92, 1, 60), (92, 1, 4), (65, 2, 20), (66, 2, 2), (48, 4, 10), (47, 4, 1), (34, 8, 6), (34, 8, 1)])
def test_lower_bounds_whatever_the_longest_stage(P, sizes, L, M, n_max):
    """The same for every number of GPUs that has kernels of its own: buckets whose longest stage has a few layers (eight, sixteen and more of
    them are different paths), up to the whole model."""
    import numpy as np

    inp = inputs.random_small(5, L, M, 1, n_max, L, f=1, t_lo=60, t_hi=99)
    lb, want, err = bounds_of_a_job(P, sizes, inp)
    finite = np.isfinite(want)
    assert finite.any() and (lb <= want + err)[finite].all(), float((lb - want)[finite].max())
    # and not below by more than what is taken off for the rounding, where no end of a stage is let through that is too slow
    assert (lb[finite] >= want[finite] * (1 - 1e-5) - 1).mean() > 0.9


def test_stages_that_leave_a_layer_uncovered_are_ruled_out(P):
    """One layer that dwarfs the others, more GPUs per node than the count of the fewest nodes takes: what is
    faster than that layer on all its GPUs is the slowest stage of no pipeline and is not evaluated."""
    import dataclasses

    L, M = 40, 9
    inp = inputs.random_small(2, L, M, 1, 6, 0, f=1, t_lo=20, t_hi=50)
    fwd = inp.fwd_ns.copy()
    fwd[13] += 5000
    inp = dataclasses.replace(inp, fwd_ns=fwd)
    e = P.ExactMinimum(inp)
    st, got = e.run()
    assert st == P.OOB_OK and got == E.exact_minimum(inp)
    least = (inp.fwd_ns + inp.bwd_ns)[13].min()  # (boundary terms only add to it)
    cum = inp.fwd_ns + inp.bwd_ns
    slow = 0
    for d in range(M):
        for u in range(L):
            t = cum[u:, d].cumsum() + [b if v < L - 1 else 0 for v, b in enumerate(inp.boundary_ns[u:].tolist(), u)]
            slow += int((t >= least).sum())
    h = exact_sizes.head(e.workspace)
    assert slow < h["ncand"] // 2 and h["alive"] <= slow + h["bucket"]


@pytest.mark.parametrize("templates", [1, 3, 4, 5, 32, 33, 63, 64])
@pytest.mark.parametrize("job", [(40, 6, 0), (66, 2, 0), (66, 2, 20)])
def test_filter_with_one_to_sixty_four_templates(P, templates, job):
    """The filter gives an entry as many lanes as its templates round up to (those of at most a node per layer): from one
    template to all of a wave, with stage counts (the limit binds: 64 multipliers) and without."""
    L, M, nb = job
    staged = nb > 0
    n_max = max(templates, 12) if staged else templates
    inp = inputs.random_small(31, L, M, n_max - templates + 1, n_max, nb, f=1, t_lo=20)
    e = P.ExactMinimum(inp, staged=staged)
    st, got = e.run()
    h = exact_sizes.head(e.workspace)
    want = E.exact_minimum_staged(inp) if staged else E.exact_minimum(inp)
    assert st == P.OOB_OK and got == want
    assert 0 < h["alive"] <= h["ncand"] and h["bucket"] >= (64 if staged else 32)


@pytest.mark.parametrize("shape", [(70, 2, 1, 30, 40), (50, 8, 1, 20, 33)])
def test_templates_without_an_answer_cost_no_evaluations(P, shape):
    """Templates whose stage limit can bind beside others: what the filter keeps is what it keeps for the
    others alone, up to the order of equal times in the list."""
    L, M, n_min, n_max, nb = shape
    inp = inputs.random_small(4, L, M, n_min, n_max, nb, f=1, t_lo=20)
    e = P.ExactMinimum(inp)
    st, got = e.run()
    want = E.exact_minimum(inp, allow_bound=True)
    assert st == P.OOB_OK and got == want and got[-1] == P.OOB_EXACT_LIMIT_CAN_BIND
    few = inputs.random_small(4, L, M, n_min, n_min + want.index(P.OOB_EXACT_LIMIT_CAN_BIND) - 1, nb, f=1, t_lo=20)
    alone = P.ExactMinimum(few)
    assert alone.run()[1] == want[: few.n_max - few.n_min + 1]
    a, b = exact_sizes.head(e.workspace)["alive"], exact_sizes.head(alone.workspace)["alive"]
    assert a <= 2 * b, (a, b)
