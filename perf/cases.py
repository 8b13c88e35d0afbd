"""Performance cases of the planner: what a job scheduler asks of it, through its public entry points.

A case is a dict of plain values; "op" says which part of the framework it exercises:
  plan        templates for every node count of a range (Section 4.1), one job
  batch       many independent planning jobs in one call
  exact       exact minimum of the template cost, per template
  enumerate   every instantiation of a node specification (Section 4.2.1, Eq. 5)
  distribute  batch distribution of every instantiation (Section 4.2.2, Eq. 6) and the plan choice
  choose      the whole of Section 4.2: enumerate, distribute, choose, starting from a node specification
  reconf      failure sequences (Section 5.1)
Shapes are those of the planning configurations (tiny, GPT-1.3B-, 6.7B-, 175B-shaped, the ragged batch) and
sizes between them.  All results are integers: every output is compared exactly.
"""
import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2309_08125_amd as P

MiB, GiB, LINK = 1 << 20, 1 << 30, 25 * 10**9


def listed():
    return [
        # The smallest job (12 layers, up to 4 nodes of one GPU), from host memory to host memory: what a
        # scheduler pays to re-plan a small job on the spot.  Launches and copies count, arithmetic does not.
        dict(name="plan-tiny-host", op="plan", L=12, M=1, n_min=1, n_max=4, nb=8, f=1, kind="gpt", f_ns=1000000, emb=1,
             state_mib=250, act_mib=40, bnd_mib=8, cap_gib=80, host=True),
        # GPT-1.3B-shaped: 24 layers and two embeddings, 2..16 nodes of 4 GPUs, profile resident on the GPU.
        dict(name="plan-26-layers", op="plan", L=26, M=4, n_min=2, n_max=16, nb=32, f=3, kind="gpt", f_ns=2200000, emb=3,
             state_mib=300, act_mib=96, bnd_mib=16, cap_gib=192, host=False),
        # An odd depth with uneven layers and the paper's own planning-time choice N_b = 4 S' (nb = 0),
        # host to host.
        dict(name="plan-61-layers-4S-host", op="plan", L=61, M=8, n_min=3, n_max=27, nb=0, f=4, kind="ragged", f_ns=5000000,
             emb=1, state_mib=1024, act_mib=0, bnd_mib=32, cap_gib=192, host=True),
        # The headline workload: GPT-175B-shaped, 8..64 nodes of 8 GPUs, profile resident.
        dict(name="plan-98-layers", op="plan", L=98, M=8, n_min=8, n_max=64, nb=128, f=8, kind="gpt", f_ns=47500000, emb=6,
             state_mib=30720, act_mib=1536, bnd_mib=96, cap_gib=192, host=False),
        # A ragged batch of independent jobs of 24..128 uneven layers, four side by side, profiles resident.
        dict(name="batch-32-jobs", op="batch", jobs=32, L_lo=24, L_hi=128, M=8, n_min=1, n_max=32, nb=64, lanes=4),
        # Exact minimum of the cost for all templates of the headline workload.
        dict(name="exact-98-layers", op="exact", staged=False, L=98, M=8, n_min=8, n_max=64, nb=128, f=8, kind="gpt",
             f_ns=47500000, emb=6, state_mib=30720, act_mib=1536, bnd_mib=96, cap_gib=192),
        # The same for the GPT-1.3B shape under N_b = 4 S.
        dict(name="exact-26-layers-4S", op="exact", staged=False, L=26, M=4, n_min=2, n_max=16, nb=0, f=3, kind="gpt",
             f_ns=2200000, emb=3, state_mib=300, act_mib=96, bnd_mib=16, cap_gib=192),
        # Exact minimum where the stage limit S <= N_b binds (tables with the stage count).
        dict(name="exact-staged-48-layers", op="exact", staged=True, L=48, M=8, n_min=1, n_max=8, nb=20, f=2, kind="ragged",
             f_ns=5000000, emb=1, state_mib=1024, act_mib=0, bnd_mib=32, cap_gib=192),
        # All instantiations (about 1.3 million) of the headline node specification: templates for 8..64 nodes
        # but one (a node count that has none), f = 8, into a buffer that the program keeps.
        dict(name="enumerate-8-64", op="enumerate", n0=8, n_hi=64, f=8),
        # The batch distribution of the 1 343 380 instantiations of all sizes 8..64 for 512 microbatches, and
        # the best plan per cluster size; the instantiations are in hand.
        dict(name="distribute-8-64", op="distribute", n0=8, n_hi=64, f=8, Q=512),
        # Section 4.2 as a whole for the GPT-6.7B-shaped node specification (10 251 instantiations).
        dict(name="choose-4-32", op="choose", n0=4, n_hi=32, f=4, Q=256),
        # A million failure sequences of the headline cluster (128 nodes), one node at a time down to the end.
        dict(name="reconf-128-nodes", op="reconf", n0=8, n_hi=64, f=8, pipelines=13, burst=1, trajectories=1 << 20),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_job(rng, L_hi, n_hi):
    L = _log_int(rng, 12, L_hi)
    M = rng.choice([1, 2, 4, 8, 8])
    n_max = min(_log_int(rng, 4, n_hi), L)
    kind = rng.choice(["gpt", "ragged"])
    return dict(L=L, M=M, n_min=max(1, n_max // 8), n_max=n_max, nb=rng.choice([0, 2 * n_max, 2 * n_max]), f=rng.randint(1, 8),
                kind=kind, f_ns=_log_int(rng, 1000000, 50000000), emb=rng.randint(1, 6) if kind == "gpt" else 1,
                state_mib=_log_int(rng, 250, 30720 if M == 8 and n_max >= 32 else 2048), act_mib=rng.choice([0, 96, 256]),
                bnd_mib=rng.choice([8, 16, 32, 96]), cap_gib=192)


def _draw_spec(rng):
    """A node specification with at least a few hundred and at most as many instantiations as the headline's."""
    while True:
        n0 = rng.randint(2, 8)
        spec = dict(n0=n0, n_hi=_log_int(rng, 5 * n0, 64), f=rng.randint(1, 8))
        if spec["n_hi"] >= 3 * n0 and 300 <= plan_count(**spec)[1] <= 1343380:
            return spec


def draw(rng):
    op = rng.choice(["plan", "plan", "plan", "batch", "exact", "exact", "staged", "enumerate", "distribute", "choose", "reconf"])
    if op == "plan":
        return dict(op="plan", **_draw_job(rng, 98, 64), host=rng.random() < 0.5)
    if op == "batch":
        return dict(op="batch", jobs=_log_int(rng, 3, 32), L_lo=24, L_hi=rng.randint(40, 120), M=8, n_min=1,
                    n_max=rng.randint(8, 32), nb=64, lanes=rng.choice([1, 4]))
    if op == "exact":
        job = _draw_job(rng, 98, 64)
        return dict(job, op="exact", staged=False, nb=rng.choice([0, job["L"] + rng.randint(0, 30)]))
    if op == "staged":
        job = _draw_job(rng, 44, 9)
        return dict(job, op="exact", staged=True, nb=rng.randint(max(2, job["L"] // 3), max(3, job["L"] // 2)))
    if op == "reconf":
        n0, f = rng.randint(2, 8), rng.randint(1, 8)
        c = f + 1 + rng.randint(0, 6)
        return dict(op="reconf", n0=n0, n_hi=rng.randint(6 * n0, 64), f=f, pipelines=c, burst=rng.choice([1, 1, 2, 3]),
                    trajectories=_log_int(rng, 1 << 12, 1 << 20))
    spec = _draw_spec(rng)
    return dict(op=op, **spec) if op == "enumerate" else dict(op=op, **spec, Q=rng.choice([128, 256, 512]))


# ---- inputs ---------------------------------------------------------------------------------------
def make_job(c, rng):
    """Layer profile of one planning job.  kind "gpt": equal layers up to a few per cent, the first and
    the last one (embedding, head) `emb` times a layer; "ragged": log-normal layers.  F on d GPUs = F / d plus a
    ring all-reduce of the boundary tensor; a stage that is not last pays a boundary transfer each way."""
    L, M = c["L"], c["M"]
    if c["kind"] == "gpt":
        mult = np.ones(L, dtype=np.int64)
        mult[0] = mult[-1] = c["emb"]
        F = rng.integers(int(0.95 * c["f_ns"]), int(1.05 * c["f_ns"]), size=L) * mult
        B = 2 * F
        state = mult * (c["state_mib"] * MiB)
    else:
        F = np.maximum(1, np.rint(c["f_ns"] * np.exp(0.5 * rng.standard_normal(L)))).astype(np.int64)
        B = np.rint(F * rng.uniform(1.8, 2.2, size=L)).astype(np.int64)
        state = np.rint(c["state_mib"] * MiB * np.exp(0.7 * rng.standard_normal(L))).astype(np.int64)
        mult = 1
    d = np.arange(1, M + 1, dtype=np.int64)
    bnd = c["bnd_mib"] * MiB
    sync = np.where(d > 1, -(-(2 * (d - 1) * bnd * 10**9) // (d * 8 * LINK)), 0)
    return SimpleNamespace(
        name="job", L=L, n_min=c["n_min"], n_max=c["n_max"], gpus_per_node=M, microbatches=c["nb"], mem_cap=c["cap_gib"] * GiB,
        f=c["f"], fwd_ns=-(-F[:, None] // d) + sync, bwd_ns=-(-B[:, None] // d) + sync,
        mem_bytes=state + c["act_mib"] * MiB * mult, boundary_ns=np.full(L, 2 * -(-(bnd * 10**9) // LINK), dtype=np.int64))


def batch_jobs(c, rng):
    jobs = []
    for i in range(c["jobs"]):
        # depths evenly spread over the range, so that the batch's work does not hang on the seed
        L = c["L_lo"] + (c["L_hi"] - c["L_lo"]) * i // max(1, c["jobs"] - 1)
        jobs.append(make_job(dict(L=L, M=c["M"], n_min=c["n_min"], n_max=c["n_max"], nb=c["nb"], f=int(rng.integers(1, 9)),
                                  kind="ragged", f_ns=5000000, state_mib=1024, act_mib=0, bnd_mib=32, cap_gib=192), rng))
    return [jobs[i] for i in np.random.Generator(np.random.PCG64(5)).permutation(len(jobs))]


def template_times(p, rng):
    """Time per microbatch of a pipeline of each template, in ns: seconds, growing slowly with the nodes."""
    return np.rint(2.1e9 * (1 + 0.9 * np.arange(p) / max(1, p - 1)) * rng.uniform(0.9, 1.1, size=p)).astype(np.int64)


@functools.lru_cache(maxsize=None)
def plan_count(n0, n_hi, f, without=0):
    """(N, number of instantiations for (f+1) n0 .. N nodes) of the node specification, one size left out or none."""
    N, Q = n_hi + f * n0, f + 1
    C = np.zeros((N + 1, Q + 1), dtype=np.int64)  # [nodes, pipelines still required]
    C[0, 0] = 1
    for n in range(n0, n_hi + 1):
        for x in range(n, N + 1 if n != without else 0):
            C[x, 1:] += C[x - n, :-1]
            C[x, 0] += C[x - n, 0]
    return N, int(C[(f + 1) * n0:, Q].sum())


def prepare(case, seed):
    c, rng = case, np.random.Generator(np.random.PCG64(seed))
    s = SimpleNamespace(case=c)
    if c["op"] == "plan":
        s.job = make_job(c, rng)
        s.planner = P.Planner(c["L"], c["n_max"], c["M"])
        if not c["host"]:
            s.prof = P.DeviceProfile(s.job)
            s.out = s.planner.new_outputs(s.job)
    elif c["op"] == "batch":
        jobs = batch_jobs(c, rng)
        s.planner = P.Planner(max(j.L for j in jobs), c["n_max"], c["M"], lanes=c["lanes"])
        profs = [P.DeviceProfile(j) for j in jobs]
        s.outs = [s.planner.new_outputs(j) for j in jobs]
        s.keep = profs
        s.args = ([p.c for p in profs], [j.L for j in jobs], [j.n_min for j in jobs], [j.n_max for j in jobs],
                  [j.gpus_per_node for j in jobs], [j.microbatches for j in jobs], [j.mem_cap for j in jobs],
                  [j.f for j in jobs], [o.c for o in s.outs])
    elif c["op"] == "exact":
        s.exact = P.ExactMinimum(make_job(c, rng), staged=c["staged"])
    elif c["op"] == "reconf":
        n0, n_hi, k = c["n0"], c["n_hi"], c["pipelines"]
        N = n_hi + c["f"] * n0
        sizes = np.full(k, n0)
        if k * n0 > N:
            sizes = sizes[: N // n0]
        for _ in range(N - int(sizes.sum())):
            sizes[rng.choice(np.flatnonzero(sizes < n_hi))] += 1
        steps = -(-(N - (c["f"] + 1) * n0 + 1) // c["burst"])
        draws = rng.integers(0, 1 << 32, size=(steps, c["burst"], c["trajectories"]), dtype=np.uint32)
        s.sim = P.FailureSimulator(sizes.tolist(), n0, n_hi, c["f"], draws)
    elif c["op"] == "enumerate":
        n0, n_hi = c["n0"], c["n_hi"]
        N, most = plan_count(n0, n_hi, c["f"])
        missing = n_hi - 1 - int(rng.integers(0, max(1, (n_hi - n0) // 4)))
        s.inst = P.Instantiator([n for n in range(n0, n_hi + 1) if n != missing], (c["f"] + 1) * n0, N, c["f"])
        s.x = torch.zeros((n_hi - n0, most), dtype=torch.int16, device="cuda")
    else:
        n0, p = c["n0"], c["n_hi"] - c["n0"] + 1
        N, _ = plan_count(n0, c["n_hi"], c["f"])
        s.inst = P.Instantiator(None, (c["f"] + 1) * n0, N, c["f"], n0=n0, p=p)
        s.times = template_times(p, rng).tolist()
        if c["op"] == "distribute":
            s.off, x = _enumerate(s.inst)
            s.dist = P.Distributor(x, int(s.off[-1]), s.times, c["Q"])
    return s


def _enumerate(inst, x=None):
    off, st = inst.count()
    P.binding.check(st, "oob_inst_count")
    if x is None:
        x = torch.empty((inst.p, int(off[-1])), dtype=torch.int16, device=inst.device)
    inst.enqueue(x, int(x.shape[1]))
    return off, x


def _distributed(d, best):
    return {"best": best, "vx": d.vx, "slowest": d.slowest, "base": d.base, "extra": d.extra, "status": d.status}


def run(s):
    op = s.case["op"]
    if op == "plan":
        if s.case["host"]:
            return s.planner.plan(s.job)
        s.planner.enqueue(s.prof, s.out)
        return s.out.t
    if op == "batch":
        rc = P.oob_plan_templates_batch(s.planner.h, *s.args, torch.cuda.current_stream().cuda_stream)
        P.binding.check(rc, "oob_plan_templates_batch")
        return [o.base for o in s.outs]
    if op == "exact":
        P.binding.check(s.exact.enqueue(), "oob_exact_minimum")
        return s.exact.best, s.exact.status
    if op == "enumerate":
        return _enumerate(s.inst, s.x)
    if op == "distribute":
        s.dist.enqueue()
        return _distributed(s.dist, s.dist.choose(s.off))
    if op == "choose":
        off, x = _enumerate(s.inst)
        d = P.Distributor(x, int(off[-1]), s.times, s.case["Q"])
        d.enqueue()
        return dict(_distributed(d, d.choose(off)), x=x)
    s.sim.enqueue()
    return {"trace": s.sim.trace, "final": s.sim.final_sizes, "summary": s.sim.summary, "status": s.sim.status}


# ---- what a pass cannot do without ------------------------------------------------------------------
def plan_work(L, M, n_max, nb):
    """(states, candidate splits) of the recursion, closed form over the (level, device set) pairs."""
    top = min(L, n_max * M, nb or L)
    states = cands = 0
    for S in range(1, top + 1):
        n = L - S + 1
        for units, across in [(g, False) for g in range(S, M + 1)] + [(a, True) for a in range(max(2, -(-S // M)), min(S, n_max) + 1)]:
            states += n * (n + 1) // 2
            for k in range(1, S):
                if across:
                    lo, hi = max(-(-k // M), units - min(S - k, n_max)), min(k, n_max, units - -(-(S - k) // M))
                else:
                    lo, hi = max(k, units - (M - 1)), min(M - 1, units - (S - k))
                if hi >= lo:
                    cands += (hi - lo + 1) * (n * (n + 1) * (n + 2) // 6)
    return states, cands


def _plan_work(c):
    _, cands = plan_work(c["L"], c["M"], c["n_max"], c["nb"])
    stages = min(c["L"], c["n_max"] * c["M"], c["nb"] or c["L"])
    n_out = c["n_max"] - c["n_min"] + 1
    return 8 * c["L"] * (2 * c["M"] + 2) + n_out * (8 * stages + 60), 6 * cands  # two adds, a compare, two selects and a min per split


def work(case):
    c = case
    if c["op"] == "plan":
        b, f = _plan_work(c)
        return {"bytes": b, "flops": f}
    if c["op"] == "batch":
        got = [_plan_work(dict(c, L=c["L_lo"] + (c["L_hi"] - c["L_lo"]) * i // max(1, c["jobs"] - 1))) for i in range(c["jobs"])]
        return {"bytes": sum(b for b, _ in got), "flops": sum(f for _, f in got)}
    if c["op"] == "exact":
        # one relaxation (an add and a min) per stage [u, v) x GPU count x position of the stage among the
        # GPUs of the largest template [x stages before it], before and after some slowest stage
        L, M, G = c["L"], c["M"], c["n_max"] * c["M"]
        stages = L * (L + 1) // 2 * M
        depth = min(L, G, c["nb"]) if c["staged"] else 1
        return {"bytes": 8 * L * (2 * M + 2) + 8 * (c["n_max"] - c["n_min"] + 1), "flops": 2 * 2 * stages * G * depth}
    if c["op"] == "reconf":
        N = c["n_hi"] + c["f"] * c["n0"]
        steps = -(-(N - (c["f"] + 1) * c["n0"] + 1) // c["burst"])
        return {"bytes": c["trajectories"] * (4 * steps * (c["burst"] + 1) + 4 * (c["pipelines"] + 8)),
                "flops": c["trajectories"] * steps * c["pipelines"]}
    p, (_, total) = c["n_hi"] - c["n0"] + 1, plan_count(c["n0"], c["n_hi"], c["f"])
    if c["op"] == "enumerate":
        p, (_, total) = p - 1, plan_count(c["n0"], c["n_hi"], c["f"], c["n_hi"] - 1)
    moved = 2 * p if c["op"] == "enumerate" else 6 * p + 28
    return {"bytes": total * moved, "flops": total * p}


def tolerance(case):
    return "exact"
