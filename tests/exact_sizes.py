"""csrc/oob_exact_sizes.h compiled for the host."""
import ctypes as C
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_08125_amd", "csrc")
WRAPPERS = r"""
#include "oob_exact_sizes.h"
using namespace oob_exact;
extern "C" {
// first index at which the quotient is wrong, -1: none
int wrong_quotient(int M) {
    for (int i = 0; i < 256 * M; ++i) if (quot(i, recip(M)) != i / M) return i;
    return -1;
}
// LDS of k_exact_eval for each accepted n_max of (L, M), one template and all of them, against the tables of its largest
// slowest stage, the bands as wide as the sides: the smallest surplus in doubles over all that take the LDS path
// (1 << 30: none does); -2 for a shape whose times have to stay exact in doubles and that has no tables in LDS.
int smallest_surplus(int L, int M) {
    size_t tables = 0; // covers next to the stage, both W, one one-node table, by the layers before it
    for (int P = 0; P <= L - 1; ++P) {
        const int S = L - 1 - P, most = P > S ? P : S;
        const size_t n = (size_t)(L - 1) * M + band_size(P, P) + band_size(S, S) + (size_t)(most + 1) * (M + 1);
        tables = n > tables ? n : tables;
    }
    int least = 1 << 30;
    for (int n = 1; n * M <= 4096; ++n)
        for (int count : {1, n}) {
            const EvalLds e = eval_lds(L, M, n, count, 1, false);
            if (e.bytes == 0) { if (in_doubles(L, M, n, count)) return -2; else continue; }
            if (e.bytes > kLdsLimit - kLdsStatic) return -1;
            const long long pool = (long long)(e.bytes / 8) - (long long)eval_fixed(L, M, n, count, 1, e.sums, e.pad);
            const long long surplus = pool - (long long)tables;
            if (surplus < least) least = (int)surplus;
        }
    return least;
}
// whether the tables of (L, M, n_max) for all templates leave out the ends of the stages; -1: no tables in LDS
int sums(int L, int M, int n_max) {
    const EvalLds e = eval_lds(L, M, n_max, n_max, 1, false);
    return e.bytes ? e.sums : -1;
}
// whether the rows of the profile of (L, M, n_max) are padded in the evaluation
int padded(int L, int M, int n_max) { return eval_lds(L, M, n_max, n_max, 1, false).pad; }
// LDS of a launch: what it asks for, whether that is announced.  kernel 0: k_exact_prep of the fast path, 1: k_exact_bounds, 2: k_exact_eval
// (one template, without stage counts); 0: no such launch
size_t launch(int kernel, int L, int M, int counts, int *announced) {
    size_t n = 0;
    if (kernel == 0) n = prep_lds(L, M, in_doubles(L, M, 1, 1)).bytes;
    if (kernel == 1) { const int mus = bound_mus(L, M, counts); n = mus ? 8 * bound_doubles(L, M, mus, bound_pad(L, M, mus)) : 0; }
    if (kernel == 2) n = eval_lds(L, M, 1, 1, 1, false).bytes;
    *announced = beyond_default(n, kernel ? kLdsStatic : kPrepStatic);
    return n;
}
// offsets in the workspace of a job that takes the LDS path: times and stages of the list, its bounds, the leftovers
void offsets(int L, int M, int n_max, int counts, int staged, size_t *at) {
    const Layout y = layout(L, M, n_max, true, bound_mus(L, M, counts), staged);
    at[0] = y.ctau; at[1] = y.cuvd; at[2] = y.lb; at[3] = y.over;
}
}
"""
HEAD = ("ncand", "bucket", "nbuckets", "alive", "next", "done", "over", "narrow")  # first words of the workspace


def build(directory):
    src, lib = os.path.join(str(directory), "wrappers.cpp"), os.path.join(str(directory), "wrappers.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, "-o", lib, src], check=True)
    return C.CDLL(lib)


def offsets(sizes, L, M, n_max, counts=False, staged=False):
    at = (C.c_size_t * 4)()
    sizes.offsets(L, M, n_max, int(counts), int(staged), at)
    return dict(zip(("ctau", "cuvd", "lb", "over"), at))


def head(workspace):
    import torch

    return dict(zip(HEAD, workspace[:32].view(torch.int32).tolist()))


def static_lds():
    """Static LDS of the kernels of the exact minimum, the largest of every template, from the metadata of the library that is built."""
    import re
    import shutil
    import tempfile

    from paper_2309_08125_amd import build

    tools, sizes = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin"), {}
    with tempfile.TemporaryDirectory() as d:
        lib = shutil.copy(build.LIB, os.path.join(d, "lib.so"))
        subprocess.run([os.path.join(tools, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True, cwd=d)
        for name in os.listdir(d):
            if name.endswith("gfx950"):
                text = subprocess.run([os.path.join(tools, "llvm-readelf"), "--notes", os.path.join(d, name)], check=True, capture_output=True, text=True).stdout
                for n, symbol in re.findall(r"\.group_segment_fixed_size: (\d+)(?:(?!\.group_segment).)*?\.symbol: +(\S+)\.kd", text, re.S):
                    m = re.search(r"k_exact_(prep|bounds|eval)", symbol)
                    if m:
                        sizes[m[0]] = max(sizes.get(m[0], 0), int(n))
    return sizes
