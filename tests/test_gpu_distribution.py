"""Batch distribution (Section 4.2.2, Eq. 6) and plan choice through the C ABI against the CPU oracle.
The minimum of Eq. 6 is unique and compared exactly (128-bit integers); the distribution that
reaches it is not, so it is checked for validity: it uses Q microbatches, at least one per pipeline,
and has exactly the minimal variance and the reported slowest time."""
import random

import numpy as np
import pytest

import inputs
from oracle import batch_distribution as BD

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_2309_08125_amd as pkg

    assert torch.cuda.is_available()
    pkg.load()
    return pkg


def distribution_of(X, base, extra):
    N = []
    for c, b, e in zip(X, base, extra):
        assert (c > 0) or (b == 0 and e == 0)
        assert e <= c
        N += [int(b) + 1] * int(e) + [int(b)] * (int(c) - int(e))
    return N


def compare(P, vectors, template_T, Q, exhaustive):
    st, vx, slow, base, extra = P.Distributor(vectors, len(vectors), template_T, Q).solve()
    for i, X in enumerate(vectors):
        T = BD.pipelines_of(X, template_T)
        if not T:
            assert st[i] == P.OOB_DIST_NO_PIPELINE
            continue
        if len(T) > Q:
            assert st[i] == P.OOB_DIST_TOO_FEW_MICROBATCHES and vx[i] == 0 and slow[i] == 0 and not base[i].any()
            continue
        assert st[i] == P.OOB_DIST_OK, (X, st[i])
        N = distribution_of(X, base[i], extra[i])
        assert sum(N) == Q and min(N) >= 1, (X, N)
        want = BD.exhaustive(T, Q)[0] if exhaustive else BD.sweep(T, Q)[0]
        assert vx[i] == want == BD.vx(T, N), (X, template_T, Q, N)
        assert slow[i] == max(n * t for n, t in zip(N, T))
    return st, vx, slow


def test_hand_cases(P):
    # templates with T = 10 and 6, five microbatches (worked in the oracle's pins): (10,10) -> 2+3, slowest 30;
    # (10,6) -> N = (2,3), x sum of squares 4, slowest 20; (6,6) -> slowest 18
    d = P.Distributor([[2, 0], [1, 1], [0, 2]], 3, [10, 6], 5)
    st, vx, slow, base, extra = d.solve()
    assert st.tolist() == [0, 0, 0] and vx == [100, 4, 36] and slow.tolist() == [30, 20, 18]
    assert base.tolist() == [[2, 0], [2, 3], [0, 2]] and extra.tolist() == [[1, 0], [0, 0], [0, 1]]
    assert d.choose([0, 3]).tolist() == [2]
    assert d.choose([0, 1, 2, 3, 3]).tolist() == [0, 1, 2, -1]
    # T = (2, 3), five microbatches: N = (3, 2), all pipelines take 6
    st, vx, slow, base, extra = P.Distributor([[1, 1]], 1, [2, 3], 5).solve()
    assert (vx, slow.tolist(), base.tolist(), extra.tolist()) == ([0], [6], [[3, 2]], [[0, 0]])


def test_small_plans_against_the_definition(P):
    """Every plan against exhaustive search: few pipelines, few microbatches, equal and very
    different times, plans that cannot be distributed, several workgroups and a ragged last one."""
    rng = random.Random(4)
    plans = 0
    for case in range(120):
        p = rng.randint(1, 5)
        tT = [rng.choice([rng.randint(1, 60), rng.randint(10**8, 10**9), 7]) for _ in range(p)]
        Q = rng.randint(1, 13)
        vecs = [[rng.choice([0, 0, 1, 1, 2, 3]) for _ in range(p)] for _ in range(rng.randint(1, 150))]
        vecs = [v for v in vecs if sum(v) <= 6]
        if vecs:
            compare(P, vecs, tT, Q, exhaustive=True)
            plans += len(vecs)
    assert plans > 3000


def test_realistic_plans_against_the_parametric_oracle(P):
    """Up to 16 pipelines, up to 512 microbatches, times of seconds in ns (up to the library's limit)."""
    rng = random.Random(5)
    for case in range(25):
        p = rng.randint(2, 24)
        tT = sorted(rng.randint(2 * 10**9, (1 << 35)) for _ in range(p))
        Q = rng.choice([32, 100, 256, 512])
        vecs = []
        for _ in range(24):
            v = [0] * p
            for _ in range(rng.randint(1, 16)):
                v[rng.randrange(p)] += 1
            vecs.append(v)
        print("case", case, p, Q, flush=True)
        compare(P, vecs, tT, Q, exhaustive=False)


def test_templates_of_nearly_equal_time(P):
    """Times that differ by a few ns in 10^10: the levels of the exchanges then cancel to a small
    part of their terms: only exact integer comparisons order them correctly."""
    rng = random.Random(9)
    for case in range(30):
        base = rng.randint(10**9, 3 * 10**10)
        tT = sorted(set(base + rng.randint(0, 6) for _ in range(rng.randint(2, 8))))
        Q = rng.choice([20, 64, 200])
        vecs = [[rng.choice([0, 1, 1, 2]) for _ in range(len(tT))] for _ in range(40)]
        vecs = [v for v in vecs if 0 < sum(v) <= Q]
        compare(P, vecs, tT, Q, exhaustive=False)


def test_status_codes_and_limits(P):
    tT = list(range(100, 120))
    x17 = [1] * 17 + [0] * 3          # seventeen templates in one plan
    x16 = [1] * 16 + [0] * 4
    st, vx, slow, base, extra = P.Distributor([x17, x16, [0] * 20], 3, tT, 40).solve()
    assert st.tolist() == [P.OOB_DIST_TOO_MANY_TEMPLATES, P.OOB_DIST_OK, P.OOB_DIST_NO_PIPELINE]
    assert vx[0] == 0 and not base[0].any() and vx[1] == BD.sweep(BD.pipelines_of(x16, tT), 40)[0]
    st = P.Distributor([[1, 1, 0], [1, 0, 1], [1, 0, 0]], 3, [5, 0, (1 << 35) + 1], 9).solve()[0]
    assert st.tolist() == [P.OOB_DIST_BAD_TIME, P.OOB_DIST_BAD_TIME, P.OOB_DIST_OK]
    # the largest time and the largest Q the library takes, two pipelines
    big = 1 << 35
    st, vx, slow, base, extra = P.Distributor([[1, 1]], 1, [big, big - 1], 65535).solve()
    assert st.tolist() == [0] and vx[0] == BD.sweep([big, big - 1], 65535)[0]
    fake = 0x10000
    assert P.oob_dist_solve(0, 1, 1, 1, fake, 1, fake, fake, 0, 0, fake, 0) == P.OOB_EINVAL
    assert P.oob_dist_solve(fake, 2, 1, 1, fake, 1, fake, fake, 0, 0, fake, 0) == P.OOB_EINVAL   # capacity < count
    assert P.oob_dist_solve(fake, 1, 1, 1, fake, 0, fake, fake, 0, 0, fake, 0) == P.OOB_EINVAL   # Q
    assert P.oob_dist_solve(fake, 1, 1, 1, fake, 1, fake, fake, fake, 0, fake, 0) == P.OOB_EINVAL  # base without extra
    assert P.oob_dist_solve(fake, 0, 0, 1, fake, 1, fake, fake, 0, 0, fake, 0) == P.OOB_OK        # nothing to do


@pytest.mark.parametrize("Q,distribution", [(17, True), (40, True), (40, False), (300, True)])
def test_many_plans_in_two_launches(P, Q, distribution):
    """More plans than one launch takes (196 608): plans of 1 to 16 templates (registers hold ten), many of them with exchanges on
    their path, twins, plans that cannot be solved, a ragged end and an odd capacity; the same plans in one launch are compared
    with the oracle."""
    rng = random.Random(Q)
    tT = [rng.randint(10**9, 4 * 10**9) for _ in range(19)]
    tT[7] = tT[3]
    vecs = []
    for i in range(160):
        v = [0] * 19
        for j in rng.sample(range(19), 1 + i % 16):
            v[j] = rng.choice([1, 1, 1, 2, 3])
        vecs.append(v)
    vecs += [[0] * 19, [1] * 19]
    assert sum(sum(v) > Q for v in vecs) > (10 if Q == 17 else -1)
    few = vecs[:160]
    compare(P, few, tT, Q, exhaustive=False)
    want = P.Distributor(vecs, len(vecs), tT, Q).solve()
    pick = np.random.Generator(np.random.PCG64(Q)).integers(0, len(vecs), size=196608 + 1024 + 65)
    got = P.Distributor(np.asarray(vecs)[pick], len(pick), tT, Q, distribution=distribution).solve()
    assert np.array_equal(got[0], want[0][pick]) and np.array_equal(got[2], want[2][pick])
    assert got[1] == [want[1][i] for i in pick]
    if distribution:
        assert np.array_equal(got[3], want[3][pick]) and np.array_equal(got[4], want[4][pick])
    else:
        assert got[3] is None and got[4] is None


@pytest.mark.parametrize("p,count,spare", [(1, 64, 0), (3, 128, 1), (7, 65, 2), (8, 64, 3), (9, 191, 0), (63, 64, 1), (64, 130, 5), (65, 64, 2), (130, 257, 7),
                                           (65, 131072 + 192, 1), (9, 196608 + 320, 3)])
def test_plans_read_and_written_by_whole_waves(P, p, count, spare):
    """A full wave moves its counts and its distribution four rows at a time, the plans of a last one that is not full a row at a time: the
    same 63 plans (none of them in a full wave) give the same; entries past the plans are left alone.  Row counts around the tile's and rows
    that start at any multiple of two bytes."""
    import torch

    rng = np.random.Generator(np.random.PCG64(p * 1000 + count))
    T = rng.integers(10**6, 3 * 10**6, size=p).tolist()
    vecs = np.zeros((63, p), dtype=np.int64)
    for i, v in enumerate(vecs):
        used = rng.choice(p, size=min(p, [1, 2, 5, 10, 11, 16, 17][i % 7]), replace=False)
        v[used] = rng.integers(1, 4, size=len(used))
    vecs[17] = 0
    want = P.Distributor(vecs, 63, T, 60).solve()
    pick = rng.integers(0, 63, size=count)
    x = torch.full((p, count + spare), 9, dtype=torch.int16)
    x[:, :count] = torch.from_numpy(vecs[pick].T.astype(np.int16))
    d = P.Distributor(x.to("cuda:0"), count, T, 60)
    d.base.fill_(77), d.extra.fill_(78)
    got = d.solve()
    assert got[1] == [want[1][i] for i in pick]
    for k in (0, 2, 3, 4):
        assert np.array_equal(got[k], want[k][pick])
    assert (d.base[:, count:] == 77).all() and (d.extra[:, count:] == 78).all()


def times_of(kind, p, rng):
    if kind == "equal":
        return [2 * 10**9 + 7] * p
    if kind == "falling":
        return [16 * 10**9 // (8 + j) for j in range(p)]
    if kind == "plateau":
        return [max(16 * 10**9 // (8 + j), 10**9) for j in range(p)]
    if kind == "coarse":
        return [rng.randint(5, 20) * 10**8 for _ in range(p)]
    if kind == "tiny":
        return [rng.randint(1, 12) for _ in range(p)]
    return [rng.choice([2046, 2047, 2048, 2049, 1024, 4096, 3]) for _ in range(p)]  # around what doubles hold exactly


@pytest.mark.parametrize("kind", ["equal", "falling", "plateau", "coarse", "tiny", "edge"])
def test_ties_and_long_paths_in_every_launch(P, kind):
    """Times that make exact ties of costs and of levels, twins and plans of which most have a path: up to ten templates, more, and more
    than there may be; all plans in one launch, with paths in the first launch, in the second one, and in the place of their counts."""
    rng = random.Random(kind)
    p, Q = 30, 45
    tT = times_of(kind, p, rng)
    vecs = []
    for i in range(96):
        v = [0] * p
        for j in rng.sample(range(p), 1 + i % 16):
            v[j] = rng.choice([1, 1, 1, 2, 3])
        vecs.append(v)
    compare(P, vecs, tT, Q, exhaustive=False)
    vecs += [[0] * p, [1] * 17 + [0] * 13, [2] * p, [0] * 29 + [Q + 1]]
    want = P.Distributor(vecs, len(vecs), tT, Q).solve()
    assert want[0][96:].tolist() == [P.OOB_DIST_NO_PIPELINE, P.OOB_DIST_TOO_MANY_TEMPLATES, P.OOB_DIST_TOO_MANY_TEMPLATES,
                                     P.OOB_DIST_TOO_FEW_MICROBATCHES]
    for count in (131072, 131073, 196608, 196609, 1024 * 200 + 1):
        pick = np.random.Generator(np.random.PCG64(count)).integers(0, len(vecs), size=count)
        for inplace in (False, True):
            d = P.Distributor(np.asarray(vecs)[pick], count, tT, Q)
            if inplace:
                d.extra = d.x
            got = d.solve()
            assert np.array_equal(got[0], want[0][pick]) and np.array_equal(got[2], want[2][pick]), (count, inplace)
            assert got[1] == [want[1][i] for i in pick]
            assert np.array_equal(got[3], want[3][pick]) and np.array_equal(got[4], want[4][pick])


@pytest.mark.parametrize("share", [0, 1, 15, 16, 17, 63, 64, 65, 255, 256])
def test_numbers_of_plans_left_to_the_second_launch(P, share):
    """Of every 256 plans `share` have an exchange on their path, of few templates or of many, the others do not: around the shares of a wave.
    The plans left over are the first, the last and scattered ones."""
    tT = [10**9 + j for j in range(12)] + [3 * 10**9]
    few = [1] * 4 + [0] * 8 + [1]
    many = [1] * 12 + [0]
    plain = [0] * 12 + [5]
    compare(P, [plain, few, many], tT, 45, exhaustive=False)
    want = P.Distributor([plain, few, many], 3, tT, 45).solve()
    for count in (131072 + 300, 196608 + 1024 * 3 + 300):
        at = np.arange(count) % 256
        left = [at < share, at >= 256 - share, np.random.Generator(np.random.PCG64(share)).permutation(256)[at] < share]
        for where in left:
            pick = np.where(where, 1 + (np.arange(count) // 256 % 3 == 0), 0)
            got = P.Distributor(np.asarray([plain, few, many])[pick], count, tT, 45).solve()
            assert np.array_equal(got[0], want[0][pick]) and np.array_equal(got[2], want[2][pick])
            assert got[1] == [want[1][i] for i in pick]
            assert np.array_equal(got[3], want[3][pick]) and np.array_equal(got[4], want[4][pick])


def test_time_does_not_hang_on_the_template_times(P):
    """200 000 plans of one to ten templates, or of eleven to sixteen: times that are all equal, fall as 1 / nodes or lie on a coarse grid make
    ties and paths for most plans.  What a call takes may differ by a small factor (two and five here), not by forty."""
    import torch

    rng = random.Random(1)
    p, count = 57, 200000

    def us(lo, hi, kind):
        tT = times_of(kind, p, rng) if kind else [2 * 10**9 + j * (3 * 10**7 + 12345) for j in range(p)]
        vecs = np.zeros((512, p), dtype=np.uint16)
        for v in vecs:
            v[rng.sample(range(p), rng.randint(lo, hi))] = 1
        d = P.Distributor(vecs[np.arange(count) % 512], count, tT, 512)
        took = []
        for _ in range(5):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            d.enqueue()
            ev[1].record()
            torch.cuda.synchronize()
            took.append(ev[0].elapsed_time(ev[1]) * 1e3)
        return sorted(took)[2]

    spread = us(1, 10, None)
    for kind, factor in (("equal", 6), ("falling", 6), ("coarse", 20)):
        took = us(1, 10, kind)
        print(kind, round(spread), round(took), flush=True)
        assert took < factor * spread, kind
    assert us(11, 16, None) < 12 * spread


@pytest.mark.parametrize("out", ["base", "extra"])
def test_a_distribution_may_overwrite_the_counts(P, out):
    """base or extra in the place of x, with more plans than one launch takes, a part of them beyond what the first launch does:
    the counts of a plan are read before its distribution is written."""
    rng = random.Random(7)
    tT = [10**9, 10**9 + 1, 10**9 + 2] + [rng.randint(10**9, 4 * 10**9) for _ in range(13)]
    vecs = []
    for i in range(200):
        v = [0] * len(tT)
        for j in rng.sample(range(3 if i % 4 == 0 else 16), 1 + i % (3 if i % 4 == 0 else 13)):
            v[j] = rng.choice([1, 1, 2, 3])
        vecs.append(v)
    pick = np.random.Generator(np.random.PCG64(7)).integers(0, len(vecs), size=196608 + 65)
    want = P.Distributor(vecs, len(vecs), tT, 60).solve()
    d = P.Distributor(np.asarray(vecs)[pick], len(pick), tT, 60)
    setattr(d, out, d.x)
    got = d.solve()
    assert np.array_equal(got[0], want[0][pick]) and np.array_equal(got[2], want[2][pick])
    assert got[1] == [want[1][i] for i in pick]
    assert np.array_equal(got[3], want[3][pick]) and np.array_equal(got[4], want[4][pick])


@pytest.mark.parametrize("count", [500, 150001, 196608 + 65])
@pytest.mark.parametrize("rows", [-3, -1, 0, 2])
def test_a_distribution_whole_rows_from_the_counts(P, count, rows):
    """base a number of rows before or behind x in the same buffer, in one launch and in several; plans with ties and with exchanges
    on their path, which are read once more after the first launch."""
    import torch

    rng = random.Random(11)
    tT = [10**9, 10**9, 2 * 10**9, 3 * 10**9, 4 * 10**9] + [rng.randint(10**9, 4 * 10**9) for _ in range(9)]
    p = len(tT)
    vecs = []
    for i in range(200):
        v = [0] * p
        for j in rng.sample(range(5 if i % 2 else p), 1 + i % (5 if i % 2 else 12)):
            v[j] = rng.choice([1, 1, 2, 3])
        vecs.append(v)
    pick = np.random.Generator(np.random.PCG64(count)).integers(0, len(vecs), size=count)
    want = P.Distributor(vecs, len(vecs), tT, 50).solve()
    buf = torch.full((p + abs(rows), count), -7, dtype=torch.int16, device="cuda")
    at, out = (0, rows) if rows > 0 else (-rows, 0)
    buf[at: at + p] = torch.from_numpy(np.ascontiguousarray(np.asarray(vecs, dtype=np.int16)[pick].T)).cuda()
    d = P.Distributor(buf[at: at + p], count, tT, 50)
    d.base = buf[out: out + p]
    got = d.solve()
    assert np.array_equal(got[0], want[0][pick]) and np.array_equal(got[2], want[2][pick])
    assert got[1] == [want[1][i] for i in pick]
    assert np.array_equal(got[3], want[3][pick]) and np.array_equal(got[4], want[4][pick])


@pytest.mark.parametrize("count", [500, 196608 + 65])
def test_one_array_for_both_parts_of_a_distribution(P, count):
    """base and extra the same array: it holds what is written last, extra."""
    rng = random.Random(12)
    tT = [rng.randint(10**9, 4 * 10**9) for _ in range(14)]
    vecs = [[rng.choice([0, 0, 1, 3]) for _ in tT] for _ in range(200)]
    pick = np.random.Generator(np.random.PCG64(count)).integers(0, len(vecs), size=count)
    want = P.Distributor(vecs, len(vecs), tT, 60).solve()
    d = P.Distributor(np.asarray(vecs)[pick], count, tT, 60)
    d.base = d.extra
    got = d.solve()
    assert np.array_equal(got[0], want[0][pick]) and np.array_equal(got[2], want[2][pick])
    assert got[1] == [want[1][i] for i in pick]
    assert np.array_equal(got[3], want[4][pick]) and np.array_equal(got[4], want[4][pick])


def test_choice_of_the_plan_against_the_oracle(P):
    """Groups of plans as the enumeration produces them (one group per cluster size); cases in which
    every minimiser of a plan has the same slowest time, so that the choice is unique."""
    rng = random.Random(7)
    checked = 0
    for case in range(40):
        sizes = sorted(rng.sample(range(2, 9), rng.randint(2, 4)))
        tT = [rng.randint(20, 60) * 100 // n for n in sizes]
        Q = rng.randint(6, 12)
        from oracle import instantiation

        off, vecs = instantiation.instantiations_range(sizes, 6, 16, 1)
        vecs = [list(map(int, v)) for v in vecs]
        unique = all(len({max(n * t for n, t in zip(N, BD.pipelines_of(X, tT))) for N in BD.exhaustive(BD.pipelines_of(X, tT), Q)[1]}) <= 1
                     for X in vecs)
        if not unique or not vecs:
            continue
        d = P.Distributor(vecs, len(vecs), tT, Q)
        d.solve()
        best = d.choose(off)
        for g in range(len(off) - 1):
            want = BD.best_plan(vecs[off[g]:off[g + 1]], tT, Q, solver=BD.exhaustive)
            assert best[g] == (-1 if want is None else off[g] + want), (sizes, tT, Q, g)
        checked += 1
    assert checked >= 15


@pytest.mark.parametrize("groups", [[1], [0, 255, 256, 257, 0], [70000, 3, 65537], [5] * 300, [2047, 2048, 2049, 4097], [140000],
                                    [1, 0, 2] * 6000, [1] * 300 + [9000]])
def test_choice_in_groups_of_any_size(P, groups):
    """Groups below, at and above the shares of a workgroup, empty ones, more groups than lanes; few distinct times, so
    that the first of equals decides, and plans that cannot be distributed."""
    rng = np.random.Generator(np.random.PCG64(len(groups)))
    total = sum(groups)
    vecs = rng.integers(0, 3, size=(total, 3))
    tT = [40, 50, 50]
    d = P.Distributor(vecs, total, tT, 5)
    st, vx, slow, base, extra = d.solve()
    off = np.concatenate([[0], np.cumsum(groups)])
    best = d.choose(off)
    for g in range(len(groups)):
        ok = np.flatnonzero(st[off[g]:off[g + 1]] == P.OOB_DIST_OK) + off[g]
        assert best[g] == (ok[np.argmin(slow[ok])] if len(ok) else -1), g


def test_headline_node_specification_at_full_size(P):
    """All 1 343 380 plans of the headline workload's node specification (templates for 8..64 nodes,
    f = 8, 72..128 nodes), the planner's own T1 per template as the time per microbatch, 512
    microbatches, as bench.py runs it: sampled plans against the oracle, all of them against what
    holds for any correct output."""
    import torch

    inp = inputs.config(4)
    planner = P.Planner(inp.L, inp.n_max, inp.gpus_per_node)
    res = planner.plan(inp)
    planner.close()
    n0, n_hi, p, N = (int(v) for v in res["cover_hdr"][:4])
    tT = [int(v) for v in res["T1"][n0 - inp.n_min: n0 - inp.n_min + p]]
    inst = P.Instantiator(None, (inp.f + 1) * n0, N, inp.f, n0=n0, p=p)
    off, st = inst.count()
    total = int(off[-1])
    x = torch.empty((p, total), dtype=torch.int16, device="cuda")
    inst.enqueue(x, total)
    Q = 512
    d = P.Distributor(x, total, tT, Q)
    st, vx, slow, base, extra = d.solve()
    assert total == 1343380 and (st == P.OOB_DIST_OK).all()
    X = x.cpu().numpy().view("uint16").T
    pipes = X.sum(axis=1)
    assert (((base.astype(np.int64) * X) + extra).sum(axis=1) == Q).all()      # every microbatch is handed out
    assert (base[X > 0] >= 1).all() and (extra <= X).all()
    times = (base.astype(np.int64) + (extra > 0)) * np.asarray(tT, dtype=np.int64)[None, :]
    assert (times.max(axis=1) == slow).all()
    assert (slow * pipes >= Q * min(tT)).all()
    rng = np.random.Generator(np.random.PCG64(2))
    for i in rng.integers(0, total, size=120).tolist() + [0, total - 1]:
        T = BD.pipelines_of(X[i].tolist(), tT)
        Nd = distribution_of(X[i].tolist(), base[i], extra[i])
        assert vx[i] == BD.sweep(T, Q)[0] == BD.vx(T, Nd), i
    best = d.choose(off)
    for g in range(len(off) - 1):
        seg = slow[off[g]:off[g + 1]]
        assert best[g] == off[g] + int(np.argmin(seg))


def test_times_and_groups_handed_over_on_a_stream_of_the_callers(P):
    """The times and the groups travel on the current stream: everything on one that is not the default, behind work
    of its own, and the arrays that come back are the caller's."""
    import torch

    n0, p, N, f = 2, 5, 20, 2
    inst = P.Instantiator(None, (f + 1) * n0, N, f, n0=n0, p=p)
    off, x, st = inst.enumerate()
    assert st == P.OOB_OK
    times = [7, 11, 13, 17, 19]
    want = P.Distributor(x, len(x), times, 40)
    want.solve()
    best = want.choose(off)
    s = torch.cuda.Stream()
    busy = torch.empty(1 << 26, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for _ in range(20):
            busy.zero_()
        again, st = inst.count()
        xd = torch.empty((p, int(again[-1])), dtype=torch.int16, device="cuda")
        inst.enqueue(xd, int(again[-1]))
        d = P.Distributor(xd, int(again[-1]), times, 40)
        d.enqueue()
        got = d.choose(again)
    assert st == P.OOB_OK and (again == off).all() and again is not off and (got == best).all()
    inst.offsets.zero_()
    torch.cuda.synchronize()
    assert (again == off).all() and torch.equal(d.slowest, want.slowest) and torch.equal(d.vx, want.vx)


def test_solved_on_another_stream_than_it_was_made_on(P):
    """Counts, times and cleared results are still on their way on a busy stream when another one is asked to solve; then the same from a graph."""
    import torch

    n0, p, N, f = 2, 5, 20, 2
    inst = P.Instantiator(None, (f + 1) * n0, N, f, n0=n0, p=p)
    off, x, st = inst.enumerate()
    assert st == P.OOB_OK
    times = [7, 11, 13, 17, 19]
    want = P.Distributor(x, len(x), times, 40)
    want.solve()
    same = lambda: all(torch.equal(getattr(d, k), getattr(want, k)) for k in ("status", "vx", "slowest", "base", "extra"))
    s = torch.cuda.Stream()
    busy = torch.empty(1 << 26, dtype=torch.int32, device="cuda")
    xd = torch.zeros((p, len(x)), dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for _ in range(20):
            busy.zero_()
        inst.enqueue(xd, len(x))
        d = P.Distributor(xd, len(x), times, 40)
    d.enqueue()
    assert same()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        d.enqueue()
    for _ in range(3):
        for t in (d.status, d.vx, d.slowest, d.base, d.extra):
            t.fill_(9)
        g.replay()
        torch.cuda.synchronize()
        assert same()
