"""Parity of the HIP path with the CPU oracle, through the C ABI, on a real MI355X.

Integer work: everything must match bit for bit -- every field of every state record of
every level, the templates, the stage lists, the coverage and the work counters.
"""
import hashlib
import json
import os
import sys

import numpy as np
import pytest

import inputs
from oracle import capi
import parity_util as PU

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_2309_08125_amd as pkg

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.load()
    return pkg


def oracle_expected(inp):
    o = capi.Oracle(inp)
    want = o.templates(inp.n_min, inp.n_max)
    c = capi.coverage(want["feasible"], inp.n_min, inp.f)
    want["cover_hdr"], want["cover_maxpipes"] = c["hdr"], c["maxpipes"]
    want["states"], want["candidates"] = o.states, o.candidates
    return o, want


def full_check(P, planner, inp):
    """Templates and every block of every level against the oracle."""
    say(f"case {inp.name} L={inp.L} M={inp.gpus_per_node} n={inp.n_min}-{inp.n_max} "
        f"nb={inp.microbatches} f={inp.f} cap={inp.mem_cap}")
    got = planner.plan(inp)
    o, want = oracle_expected(inp)
    try:
        PU.compare_templates(got, want, inp.n_max - inp.n_min + 1)
        nstates = 0
        for S in range(1, o.Smax + 1):
            for delta in range(o.D):
                gb = planner.block(S, delta)
                assert (gb is not None) == o.valid(S, delta), (S, delta)
                if gb is not None:
                    nstates += PU.compare_block(gb, o.block(S, delta), S, inp.L)
        return got, nstates
    finally:
        o.close()


SHAPES = [(5, 1, 1, 3, 6), (6, 2, 1, 3, 8), (7, 2, 1, 2, 5), (6, 4, 1, 2, 12), (8, 4, 2, 3, 12),
          (6, 3, 1, 2, 0), (7, 1, 1, 4, 0), (9, 3, 1, 4, 4), (12, 2, 2, 5, 0), (10, 8, 1, 2, 16),
          (1, 1, 1, 1, 4), (1, 4, 1, 2, 4), (3, 2, 1, 5, 2), (37, 3, 1, 5, 9), (70, 2, 1, 6, 11),
          # more than 64 target device sets (two workgroup groups), 16 GPUs per node, many nodes
          (72, 1, 1, 70, 0), (20, 16, 1, 2, 8), (40, 2, 1, 40, 64), (30, 3, 2, 30, 0),
          # the largest node the library takes: 64 GPUs (OOB_MAX_GPUS), 63 device sets inside it
          (40, 64, 1, 1, 0), (20, 64, 1, 2, 24)]


# Levels of few candidates are done by one launch, which leaves little of a small job to the split and select kernels:
# the sweeps below run as a caller gets them and with every level through those kernels.
every_kernel = pytest.mark.parametrize("small_state", [640, 0])


@every_kernel
@pytest.mark.parametrize("shape", SHAPES)
def test_small_random_every_state(P, shape, small_state):
    """Small and ragged shapes (L not a multiple of any tile, L = 1, more nodes than layers,
    N_b below the stage limit, the paper's N_b = 4 S' mode), three variants of the memory cap /
    forbidden GPU counts, every state compared."""
    L, M, n_min, n_max, nb = shape
    planner = P.Planner(L, n_max, M)
    planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
    for seed in range(3):
        for var in ("plain", "tight", "forbid"):
            inp = inputs.random_small(seed, L, M, n_min, n_max, nb, f=seed,
                                      tight_mem=(var == "tight"), forbid_some_d=(var == "forbid"))
            full_check(P, planner, inp)
            assert small_state or planner.flags()[2] == 0
    planner.close()


def test_longest_model_the_library_takes(P):
    """OOB_MAX_L layers (1023): 129 x 129 blocks of the plane, up to 128 segments per block."""
    planner = P.Planner(1023, 2, 1)
    full_check(P, planner, inputs.random_small(5, 1023, 1, 1, 2, 0, f=1))
    planner.close()
    planner = P.Planner(300, 2, 2)
    full_check(P, planner, inputs.random_small(5, 300, 2, 1, 2, 5, f=1))
    planner.close()


@every_kernel
def test_many_random_shapes_on_one_handle(P, small_state):
    """Four hundred random shapes (L, GPUs per node, template range, N_b, f, memory and
    forbidden-GPU-count variants, large times, uniform layers) back to back on one handle, every
    state of every case against the oracle."""
    import random

    rng = random.Random(2309)
    planner = P.Planner(60, 24, 16)
    planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
    states = 0
    for case in range(400):
        M = rng.choice([1, 1, 2, 3, 4, 5, 8, 8, 12, 16])
        L = rng.randint(1, 60 if M <= 4 else 34)
        n_max = rng.randint(1, max(1, min(24, L)))
        n_min = rng.randint(1, n_max)
        nb = rng.choice([0, 0, rng.randint(1, 2 * L + 2), rng.randint(1, 12)])
        kw = {}
        if rng.random() < 0.15:
            kw["t_lo"] = 1 << rng.randint(20, 30)
            kw["t_hi"] = 2 * kw["t_lo"]
        if rng.random() < 0.2:
            kw["uniform_layers"] = True
        if rng.random() < 0.3:
            kw["boundary"] = rng.random() < 0.5
        var = rng.choice(["plain", "tight", "forbid"])
        inp = inputs.random_small(rng.randint(0, 10**6), L, M, n_min, n_max, nb, f=rng.randint(0, 4),
                                  tight_mem=(var == "tight"), forbid_some_d=(var == "forbid"), **kw)
        states += full_check(P, planner, inp)[1]
    planner.close()
    assert states > 1_000_000


@every_kernel
def test_handle_reuse_across_shapes(P, small_state):
    """One handle sized for the maxima serves smaller jobs back to back."""
    planner = P.Planner(40, 6, 4)
    planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
    for i, (L, M, n_max, nb) in enumerate([(40, 4, 6, 16), (9, 2, 3, 5), (25, 3, 6, 0), (40, 1, 6, 40)]):
        full_check(P, planner, inputs.random_small(50 + i, L, M, 1, n_max, nb, f=1, tight_mem=(i % 2 == 0)))
    planner.close()


@pytest.mark.parametrize("cfg", [1, 2, 3])
def test_configs_1_to_3_every_state(P, cfg):
    inp = inputs.config(cfg)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    got, nstates = full_check(P, planner, inp)
    assert got["feasible"].all()
    say(f"config {cfg}: {got['states']} states ({nstates} exist), {got['candidates']} candidates: bit-exact")
    planner.close()


def check_against_golden(P, inp, path):
    g = json.load(open(path))
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    got = planner.plan(inp)
    want = {k: np.array(v) for k, v in g.items() if isinstance(v, list)}
    want["states"], want["candidates"] = g["states"], g["candidates"]
    PU.compare_templates(got, want, inp.n_max - inp.n_min + 1)
    Smax = P.oob_plan_max_stages(inp.L, inp.n_max, inp.gpus_per_node, inp.microbatches)
    D = inp.gpus_per_node - 1 + inp.n_max
    bad = []
    for S in range(1, Smax + 1):
        h = hashlib.sha256()
        for delta in range(D):
            gb = planner.block(S, delta)
            if gb is not None:
                h.update(PU.canonical_gpu_block(gb, S, inp.L))
        if h.hexdigest() != g["level_sha256"][str(S)]:
            bad.append(S)
    planner.close()
    assert not bad, f"levels whose state records differ from the oracle's: {bad[:10]}"
    return got


@pytest.mark.timeout(900)
def test_config4_full_size_against_stored_oracle_results(P):
    """The headline workload in the configuration bench.py times.  The oracle needs minutes
    for it, so its templates and a SHA-256 per level over all state records are stored by
    tests/golden/make_golden.py (which calls only the oracle)."""
    inp = inputs.config(4)
    say("config 4 (L=98, n=8..64 x 8 GPUs)")
    got = check_against_golden(P, inp, os.path.join(GOLD, "cfg4_expected.json"))
    assert (got["states"], got["candidates"]) == (3724666, 16232508904)


@pytest.mark.timeout(900)
def test_config4_with_the_papers_microbatch_choice_against_stored_oracle_results(P):
    """Configuration 4 with N_b = 4 S' per state (the paper's planning-time choice, Section
    4.1.2): the cost coefficients then differ per level (cl = 3 r, cr = 4 s).  Stored results
    written by tests/golden/make_golden.py cfg4_paper_nb (oracle only)."""
    import dataclasses

    inp = dataclasses.replace(inputs.config(4), microbatches=0, name="cfg4_gpt175b_paper_nb")
    say("config 4, N_b = 4 S'")
    got = check_against_golden(P, inp, os.path.join(GOLD, "cfg4_paper_nb_expected.json"))
    assert (got["states"], got["candidates"]) == (3724666, 16232508904)


@pytest.mark.timeout(900)
def test_config4_repeated_calls_on_one_handle_stay_identical(P):
    """Levels run on two streams with events between them: five calls back to back on one handle
    (no host synchronisation in between) must leave exactly the stored oracle results, every
    time -- a missing dependency between the streams would show up here as a changed record."""
    import torch

    inp = inputs.config(4)
    g = json.load(open(os.path.join(GOLD, "cfg4_expected.json")))
    want = {k: np.array(v) for k, v in g.items() if isinstance(v, list)}
    want["states"], want["candidates"] = g["states"], g["candidates"]
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    prof = P.DeviceProfile(inp)
    outs = [planner.new_outputs(inp) for _ in range(5)]
    for o in outs:
        planner.enqueue(prof, o)
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        say(f"call {i}")
        PU.compare_templates(o.to_host(), want, inp.n_max - inp.n_min + 1)
    D = inp.gpus_per_node - 1 + inp.n_max
    for S in (2, 3, 17, 50, 51, 97, 98):  # the records the last call left behind
        h = hashlib.sha256()
        for delta in range(D):
            gb = planner.block(S, delta)
            if gb is not None:
                h.update(PU.canonical_gpu_block(gb, S, inp.L))
        assert h.hexdigest() == g["level_sha256"][str(S)], S
    planner.close()


@pytest.mark.parametrize("fork", [False, True])
def test_call_can_be_captured_into_a_graph_and_replayed(P, fork):
    """The call stays on the caller's stream, or forks to the streams of the handle and joins them again with
    events, so a caller may capture it.  The graph is replayed three times with eager work in between; every replay
    must give the oracle's templates again (the output buffers are cleared before each)."""
    import torch

    inp = inputs.config(2)
    o, want = oracle_expected(inp)
    o.close()
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    if fork:
        planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
        planner.set_option(P.OOB_OPT_OVERLAP_FROM, 0)
    prof = P.DeviceProfile(inp)
    out = planner.new_outputs(inp)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        planner.enqueue(prof, out)  # first call: the handle creates its streams and events
    torch.cuda.synchronize()
    assert planner.flags()[2:] == ([0, 23] if fork else [25, 0])
    PU.compare_templates(out.to_host(), want, inp.n_max - inp.n_min + 1)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        planner.enqueue(prof, out)
    for i in range(3):
        say(f"replay {i}")
        for v in out.t.values():
            v.zero_()
        torch.randn(1 << 20, device="cuda").sum().item()  # eager work and a synchronisation between replays
        graph.replay()
        torch.cuda.synchronize()
        PU.compare_templates(out.to_host(), want, inp.n_max - inp.n_min + 1)
    full = {(S, d): planner.block(S, d) for S in (2, 9, 17) for d in range(2, 8)}
    assert any(b is not None for b in full.values())
    planner.close()


def test_capture_with_launches_beyond_64_kb_of_lds(P):
    """Sixty nodes: launches of up to 67 KB of LDS, which the library announces to the runtime in the captured call itself.
    Replays with eager work in between give what the plain split kernel gives."""
    import torch

    inp = inputs.random_small(67, 60, 8, 1, 60, 0, f=2)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 1)
    want = planner.plan(inp)
    planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 0)
    planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
    planner.set_option(P.OOB_OPT_OVERLAP_FROM, 1000)
    prof = P.DeviceProfile(inp)
    out = planner.new_outputs(inp)
    planner.plan(inp)
    flags = planner.flags()
    assert flags[:3] == [1, 0, 0] and flags[3] > 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        planner.enqueue(prof, out)
    for i in range(3):
        say(f"replay {i}")
        out.base.zero_()
        torch.randn(1 << 20, device="cuda").sum().item()
        graph.replay()
        torch.cuda.synchronize()
        got = out.to_host()
        for k in want:
            assert np.array_equal(got[k], want[k]), (i, k)
    planner.close()


def test_device_status_reports_bad_profile_values(P):
    import torch

    inp = inputs.random_small(3, 8, 2, 1, 2, 6)
    planner = P.Planner(8, 2, 2)
    bad = inputs.PlanInput("neg", inp.fwd_ns.copy(), inp.bwd_ns, inp.mem_bytes, inp.boundary_ns, 1, 2, 2, 6,
                           inp.mem_cap, 1)
    bad.fwd_ns[3, 0] = -5
    assert int(planner.plan(bad)["status"][0]) == P.OOB_EINVAL
    big = inputs.PlanInput("big", inp.fwd_ns * (1 << 45), inp.bwd_ns, inp.mem_bytes, inp.boundary_ns, 1, 2, 2,
                           6, inp.mem_cap, 1)
    assert int(planner.plan(big)["status"][0]) == P.OOB_EOVERFLOW
    assert int(planner.plan(inp)["status"][0]) == P.OOB_OK
    planner.close()


@every_kernel
def test_large_times_stay_exact_on_both_paths(P, small_state):
    """Times near the top of the exactly representable range.  Up to a bound the set-up
    kernel checks, (total, split point) pairs fit one double and the keyed split kernel runs;
    above it the select kernel evaluates every candidate itself.  Both must match the oracle
    bit for bit; so must the launch of the small levels, which has no keys."""
    planner = P.Planner(12, 4, 3)
    planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
    seen = set()
    for seed in range(4):
        for inp in (inputs.random_small(20 + seed, 9, 2, 1, 3, 7, t_lo=(1 << 38), t_hi=(1 << 39)),
                    inputs.random_small(30 + seed, 12, 3, 1, 4, 0, t_lo=(1 << 36), t_hi=(1 << 37),
                                        tight_mem=True),
                    inputs.random_small(40 + seed, 9, 2, 1, 3, 7, t_lo=(1 << 30), t_hi=(1 << 31)),
                    inputs.random_small(50 + seed, 12, 3, 1, 4, 9)):
            full_check(P, planner, inp)
            seen.add(tuple(planner.flags()[:2]))
            assert small_state or planner.flags()[2] == 0
    assert seen == {(0, 0), (1, 0)}, "keyed kernel and in-select evaluation must both have run"
    planner.close()


@pytest.mark.parametrize("shape", [(40, 1, 1, 5, 4000), (63, 1, 1, 4, 3000), (64, 1, 2, 3, 2500), (20, 2, 1, 4, 2000), (12, 3, 1, 4, 0)])
def test_totals_just_below_and_above_what_a_key_holds(P, shape):
    """The largest profile whose totals fit keys and the smallest whose do not, one unit of the bound apart.  A key of a
    level is total, split and split point: with a microbatch count far above the stage count the totals come within a
    few per cent of the field they have (one GPU per node, most of the time in one layer)."""
    import dataclasses

    L, M, n_min, n_max, nb = shape
    base = inputs.random_small(17, L, M, n_min, n_max, nb, t_lo=1 << 10, t_hi=1 << 11)
    base.fwd_ns[L // 3] = 1 << 24
    Smax = P.oob_plan_max_stages(L, n_max, M, nb)
    mult = (nb or 4 * Smax) + 4 * Smax + 4
    line = ((1 << 52) >> L.bit_length()) // mult  # keys fit iff the sum below stays under this
    w = int((base.fwd_ns + base.bwd_ns).sum() + base.boundary_ns.sum())
    scale = (line - 1) // w
    for above in (False, True):
        inp = dataclasses.replace(base, fwd_ns=base.fwd_ns * scale, bwd_ns=base.bwd_ns * scale, boundary_ns=base.boundary_ns * scale)
        inp.fwd_ns[L // 3, 0] += line - 1 + above - w * scale  # the sum is now line - 1 or line
        planner = P.Planner(L, n_max, M)
        planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
        got, _ = full_check(P, planner, inp)
        assert planner.flags()[:3] == [0 if above else 1, 0, 0], above
        top = int(got["T"][got["S"] > 1].max()) << L.bit_length()  # (one stage: no key)
        assert top < 1 << 52 and (M > 1 or top > 0.95 * (1 << 52)), top / (1 << 52)
        planner.close()


def test_plain_split_kernel(P):
    """The tiled split kernel without keys serves shapes that stage more tables than the keyed
    kernel holds (hundreds of nodes); the handle option routes ordinary shapes through it."""
    for inp in (inputs.config(1), inputs.config(2),
                inputs.random_small(3, 37, 3, 1, 5, 9, f=1, tight_mem=True),
                inputs.random_small(4, 30, 3, 2, 30, 0, f=2),
                inputs.random_small(21, 9, 2, 1, 3, 7, t_lo=(1 << 38), t_hi=(1 << 39))):
        print("plain", inp.name, inp.L, flush=True)
        planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
        planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 1)
        full_check(P, planner, inp)
        assert planner.flags()[:2] == [0, 1]
        planner.close()


@pytest.mark.parametrize("nb", [0, 300])
def test_split_kernel_with_more_than_half_of_the_lds(P, nb):
    """128 layers on up to 128 nodes: full groups of 64 targets and second groups, launches of 64-88 KB of LDS (four waves'
    staged tables), against the plain split kernel, which the tests above compare with the oracle."""
    inp = inputs.random_small(61, 128, 8, 1, 128, nb, f=2)
    say(f"keyed and plain, N_b {nb}")
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    got = planner.plan(inp)
    assert planner.flags()[:2] == [1, 0]
    planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 1)
    want = planner.plan(inp)
    assert planner.flags()[:2] == [0, 1]
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert int(got["status"][0]) == P.OOB_OK
    planner.close()


@pytest.mark.parametrize("shape", [(150, 1, 150, 8, 0), (140, 1, 140, 64, 290), (176, 1, 176, 8, 0), (200, 1, 200, 8, 410)])
def test_split_kernel_of_the_most_nodes_it_serves(P, shape):
    """One hundred and forty to two hundred nodes: 76 to 120 tables staged per split point, launches of 81 to 125 KB of LDS,
    against the plain split kernel."""
    L, n_min, n_max, M, nb = shape
    inp = inputs.random_small(61, L, M, n_min, n_max, nb, f=2)
    planner = P.Planner(L, n_max, M)
    got, flags = planner.plan(inp), planner.flags()
    assert flags[:2] == [1, 0]
    planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 1)
    want = planner.plan(inp)
    assert planner.flags()[:2] == [0, 1]
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert int(got["status"][0]) == P.OOB_OK
    planner.close()


@pytest.mark.parametrize("shape", [(44, 1, 36, 8, 0), (47, 4, 44, 8, 50), (62, 6, 60, 8, 0), (76, 5, 37, 2, 100)])
def test_splits_of_a_short_and_a_long_side(P, shape):
    """Levels whose launch has the shorter side of such splits stream (36 to 61 targets across nodes), every state."""
    L, n_min, n_max, M, nb = shape
    inp = inputs.random_small(67, L, M, n_min, n_max, nb, f=2, t_lo=20)
    planner = P.Planner(L, n_max, M)
    full_check(P, planner, inp)
    planner.close()


def test_xcd_chunked_task_order(P):
    """The other order of the workgroup tasks (block row by block row, each XCD walking one
    contiguous stretch of the list) computes the same tables."""
    for inp in (inputs.config(2), inputs.config(3),
                inputs.random_small(3, 37, 3, 1, 5, 9, f=1, tight_mem=True),
                inputs.random_small(5, 60, 2, 1, 6, 11, f=2),
                inputs.random_small(4, 30, 3, 2, 30, 0, f=2)):
        print("xcd", inp.name, inp.L, flush=True)
        planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
        planner.set_option(P.OOB_OPT_XCD_ORDER, 1)
        planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
        full_check(P, planner, inp)
        planner.close()


def test_select_with_eight_lanes_per_state(P):
    """The select kernel of the top levels (eight lanes per state), forced onto every level of
    shapes the oracle finishes in seconds: once reading the keys of all splits, once evaluating
    the two outer splits of every level itself (both device-set families, both N_b modes, a
    profile whose totals are too large for keys, so that its one-lane fallback runs too), the
    latter also with every launch on one stream."""
    seen = set()
    for fuse_from, one_stream in ((1 << 20, 0), (2, 0), (2, 1)):
        for inp in (inputs.config(1), inputs.config(2),
                    inputs.random_small(3, 37, 3, 1, 5, 9, f=1, tight_mem=True),
                    inputs.random_small(5, 60, 2, 1, 6, 11, f=2),
                    inputs.random_small(4, 30, 3, 2, 30, 0, f=2),
                    inputs.random_small(7, 12, 8, 1, 3, 5),
                    inputs.random_small(21, 9, 2, 1, 3, 7, t_lo=(1 << 38), t_hi=(1 << 39))):
            print("select8", fuse_from, inp.name, inp.L, flush=True)
            planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
            planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
            planner.set_option(P.OOB_OPT_SELECT8_FROM, 2)
            planner.set_option(P.OOB_OPT_FUSE_FROM, fuse_from)
            planner.set_option(P.OOB_OPT_ONE_STREAM, one_stream)
            full_check(P, planner, inp)
            seen.add(tuple(planner.flags()[:2]))
            planner.close()
    assert seen == {(0, 0), (1, 0)}, "keys and the evaluation without keys must both have run"


@pytest.mark.parametrize("overlap_from", [0, 20, 200])
def test_levels_on_several_streams(P, overlap_from):
    """The inner splits of the levels of at least `overlap_from` thousand candidates on streams of the library: all
    levels, or a stretch of them with levels before and behind it on the caller's stream; called directly and replayed
    from a captured graph."""
    import torch

    for inp in (inputs.config(2), inputs.random_small(5, 60, 2, 1, 6, 11, f=2), inputs.random_small(4, 30, 3, 2, 30, 0, f=2)):
        say(f"overlap from {overlap_from} {inp.name} {inp.L}")
        planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
        planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
        planner.set_option(P.OOB_OPT_OVERLAP_FROM, overlap_from)
        full_check(P, planner, inp)
        prof, out = P.DeviceProfile(inp), planner.new_outputs(inp)
        planner.enqueue(prof, out)
        want = out.to_host()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            planner.enqueue(prof, out)
        for i in range(3):
            out.base.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = out.to_host()
            assert all(np.array_equal(got[k], want[k]) for k in out.t), (inp.name, i)
        planner.close()


def test_overlapped_jobs_of_several_handles_stay_behind_their_callers_streams(P):
    """Three handles with overlapped levels on two caller streams, profile written before and overwritten after each call on the
    same stream without a wait in between: the job runs between the two."""
    import torch

    inp = inputs.config(2)
    planners = [P.Planner(inp.L, inp.n_max, inp.gpus_per_node) for _ in range(3)]
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    jobs, good = [], P.DeviceProfile(inp)
    for i, planner in enumerate(planners):
        planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
        planner.set_option(P.OOB_OPT_OVERLAP_FROM, 0)
        jobs.append((planner, P.DeviceProfile(inp), planner.new_outputs(inp), streams[i % 2]))
    planners[0].enqueue(good, jobs[0][2])
    want = jobs[0][2].to_host()
    torch.cuda.synchronize()
    for rep in range(4):
        for planner, prof, out, stream in jobs:
            with torch.cuda.stream(stream):
                prof.base.copy_(good.base)
                out.base.zero_()
                planner.enqueue(prof, out)
                prof.base.fill_(rep)
    torch.cuda.synchronize()
    for planner, prof, out, _ in jobs:
        got = out.to_host()
        assert all(np.array_equal(got[k], want[k]) for k in out.t)
        planner.close()


def level_counts(inp):
    """Per level S' >= 2: candidates, and those of the widest state of the device set with most (s, m) pairs."""
    L, M = inp.L, inp.gpus_per_node
    out = {}
    for S in range(2, min(L, inp.n_max * M, inp.microbatches or L) + 1):
        pairs = {}
        for s in range(1, S):
            r = S - s
            for a in range(s, M):  # GPUs inside a node
                for b in range(r, M - a + 1):
                    if b < M:
                        pairs[0, a + b] = pairs.get((0, a + b), 0) + 1
            for a in range(-(-s // M), min(s, inp.n_max) + 1):  # whole nodes
                for b in range(-(-r // M), min(r, inp.n_max - a) + 1):
                    pairs[1, a + b] = pairs.get((1, a + b), 0) + 1
        n = L - S + 1
        out[S] = sum(pairs.values()) * (n * (n + 1) * (n + 2) // 6), max(pairs.values(), default=0) * n
    return out


@pytest.mark.parametrize("job", [1, 2, 3, (60, 2, 1, 6, 11), (30, 3, 2, 30, 0), (40, 16, 1, 3, 0)])
def test_flags_say_which_launches_did_the_levels(P, job):
    """How many levels one launch did, and how many put their inner splits on other streams."""
    inp = inputs.config(job) if isinstance(job, int) else inputs.random_small(5, *job, f=2)
    levels = level_counts(inp)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    got = planner.plan(inp)
    assert got["candidates"] == sum(c for c, _ in levels.values())
    small = {S for S, (c, widest) in levels.items() if widest <= 640 and c <= 500000}
    assert planner.flags() == [1, 0, len(small), 0]
    planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 1)
    planner.plan(inp)
    assert planner.flags() == [0, 1, 0, 0]
    planner.set_option(P.OOB_OPT_PLAIN_SPLIT, 0)
    planner.set_option(P.OOB_OPT_OVERLAP_FROM, 20)
    planner.set_option(P.OOB_OPT_SMALL_STATE, 0)
    planner.plan(inp)
    large = [S for S, (c, _) in levels.items() if S >= 4 and c >= 20000]
    assert planner.flags() == [1, 0, 0, max(large) - min(large) + 1 if large else 0]
    planner.set_option(P.OOB_OPT_ONE_STREAM, 1)
    planner.plan(inp)
    assert planner.flags() == [1, 0, 0, 0]
    planner.close()


def test_options_do_not_change_each_other(P):
    """An option at its default value changes nothing, and the order of the calls does not matter."""
    inp = inputs.config(3)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    planner.plan(inp)
    flags = planner.flags()
    assert flags[2] > 0 and flags[3] == 0
    for option, value in ((P.OOB_OPT_PLAIN_SPLIT, 0), (P.OOB_OPT_XCD_ORDER, 0), (P.OOB_OPT_ONE_STREAM, 0),
                          (P.OOB_OPT_SELECT8_FROM, 82), (P.OOB_OPT_FUSE_FROM, 82), (P.OOB_OPT_OVERLAP_FROM, 24000),
                          (P.OOB_OPT_SMALL_STATE, 640)):
        planner.set_option(option, value)
        planner.plan(inp)
        assert planner.flags() == flags, option
    planner.close()
    seen = []
    options = [(P.OOB_OPT_SMALL_STATE, 1000), (P.OOB_OPT_OVERLAP_FROM, 200), (P.OOB_OPT_XCD_ORDER, 1)]
    for order in (options, options[::-1]):
        planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
        for option, value in order:
            planner.set_option(option, value)
        planner.plan(inp)
        seen.append(planner.flags())
        planner.close()
    assert seen[0] == seen[1] and seen[0][2] > 0 and seen[0][3] > 0, seen


@pytest.mark.parametrize("small_state", [0, 100, 1 << 30])
def test_levels_by_one_launch(P, small_state):
    """Levels of at most `small_state` candidates a state candidate by candidate: none, some, all of them; one to
    sixteen GPUs per node, both N_b modes, tight memory, totals too large for keys, more than 64 pairs of a device
    set, blocks whose first column lacks layers."""
    for inp in (inputs.config(1), inputs.config(2), inputs.random_small(3, 37, 3, 1, 5, 9, f=1, tight_mem=True),
                inputs.random_small(5, 60, 2, 1, 6, 11, f=2), inputs.random_small(4, 30, 3, 2, 30, 0, f=2),
                inputs.random_small(7, 12, 8, 1, 3, 5), inputs.random_small(8, 40, 16, 1, 3, 0), inputs.random_small(9, 7, 1, 1, 7, 0),
                inputs.random_small(21, 9, 2, 1, 3, 7, t_lo=(1 << 38), t_hi=(1 << 39))):
        say(f"small state {small_state} {inp.name} {inp.L}")
        planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
        planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
        full_check(P, planner, inp)
        planner.close()


@pytest.mark.parametrize("job", [(26, 4, 2, 16, 32), (9, 1, 1, 9, 0), (17, 8, 1, 3, 0), (66, 2, 1, 3, 5), (7, 2, 1, 2, 0), (120, 1, 1, 2, 2)])
def test_small_levels_with_one_to_eight_columns_a_workgroup(P, job):
    """Levels by one launch in workgroups of one, two, four and eight states: many and few candidates a state, blocks of one state and whole
    ones, launches at and above the most workgroups that are split further."""
    inp = inputs.random_small(12, *job, f=1)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    for small_state in (1 << 30, 640):
        planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
        full_check(P, planner, inp)
        assert planner.flags()[2] > 0
    planner.close()


@every_kernel
def test_two_calls_same_answer(P, small_state):
    """Determinism: the same job twice on one handle gives identical tables."""
    inp = inputs.config(2)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    planner.set_option(P.OOB_OPT_SMALL_STATE, small_state)
    a = planner.plan(inp)
    blocks_a = {(S, d): planner.block(S, d) for S in (2, 5, 9) for d in range(3, 12)}
    b = planner.plan(inp)
    for k in a:
        assert np.array_equal(np.asarray(a[k]), np.asarray(b[k])), k
    for (S, d), ba in blocks_a.items():
        bb = planner.block(S, d)
        assert (ba is None) == (bb is None)
        if ba is not None:
            for k in ba:
                assert np.array_equal(ba[k], bb[k])
    planner.close()
