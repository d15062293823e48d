"""The direct-to-LDS engine's barriers, from the assembly of kernels built here.

After a step's barrier the ring slot read in the step before is refilled, so no
wavefront may pass it with an LDS read of its own still pending.  In a loop the
compiler waits for a step's reads before the loop's end; where it unrolls the
steps (a constant K) only the engine's own wait keeps them in front of the
barrier."""
import re
import subprocess

import pytest

from paper_1506_05741_amd import build

# (T, BM, BN, ST, AKC, BKC, SETS, GRP, SPLIT, NARROW), K: constant K of more slices than the ring holds
KERNELS = [
    (("double", 64, 64, 3, "false", "false", 1, 1, "false", "false"), 128),
    (("double", 64, 32, 2, "true", "true", 1, 1, "false", "false"), 64),
    (("double", 32, 32, 3, "false", "false", 1, 1, "false", "true"), 100),
    (("double", 64, 64, 5, "false", "false", 2, 1, "true", "false"), 256),
    (("float", 64, 64, 3, "true", "false", 1, 1, "false", "false"), 256),
    (("float", 64, 32, 2, "true", "true", 2, 1, "false", "false"), 256),
    (("float", 64, 32, 3, "true", "true", 4, 1, "false", "false"), 384),
    (("float", 32, 32, 2, "true", "true", 1, 4, "false", "false"), 640),
]


def source():
    out = ['#include "gemm.h"', "using namespace gemm;"]
    for i, ((T, bm, bn, st, akc, bkc, sets, grp, split, narrow), K) in enumerate(KERNELS):
        out.append(f"""
__global__ __launch_bounds__(256) void probe{i}(const {T}* __restrict__ A, const {T}* __restrict__ B, {T}* __restrict__ C, int ld) {{
  typedef TFrag<{T}, {bm}, {bn}, 2, 2> F;
  __shared__ __attribute__((aligned(1024))) {T} lds[{st} * {grp} * ({bm} + {bn}) * tbk<{T}>()];
  F f[{sets}];
  for (int x = 0; x < {sets}; ++x) f[x].zero();
  for (int rep = 0; rep < 2; ++rep)
    t_gemm<{T}, {bm}, {bn}, 2, 2, {st}, {akc}, {bkc}, false, {sets}, {grp}, {split}, {narrow}>(
        f, A, ld, {bm}, B, ld, {bn}, 0, 0, rep * {K}, (rep + 1) * {K}, lds);
  for (int x = 0; x < {sets}; ++x)
    for (int m = 0; m < F::FM; ++m)
      for (int n = 0; n < F::FN; ++n)
        for (int r = 0; r < 4; ++r) C[(((x * F::FM + m) * F::FN + n) * 4 + r) * 256 + threadIdx.x] = f[x].c[m][n][r];
}}""")
    return "\n".join(out)


def kernels(asm):
    """(name, basic blocks in order, successors) of every function."""
    for name, body in re.findall(r"^(\w+):[^\n]*@\w+\n(.*?)^\.Lfunc_end", asm, re.M | re.S):
        blocks = [("", [])]
        for line in body.splitlines():
            t = line.split(";")[0].strip()
            label = re.match(r"(\.LBB\w+):", t)
            if label:
                blocks.append((label.group(1), []))
            elif t and not t.startswith("."):
                blocks[-1][1].append(t)
                if re.match(r"s_(c?branch|endpgm)", t):
                    blocks.append(("", []))
        index = {b[0]: i for i, b in enumerate(blocks) if b[0]}
        succ = []
        for i, (_, ins) in enumerate(blocks):
            last = ins[-1] if ins else ""
            jump = [index[last.split()[1]]] if re.match(r"s_c?branch", last) else []
            through = [] if re.match(r"s_(branch|endpgm)", last) or i + 1 == len(blocks) else [i + 1]
            succ.append(jump + through)
        yield name, [b[1] for b in blocks], succ


def reads_pending_at_barriers(blocks, succ):
    """The most LDS reads that can be pending at any s_barrier, by propagating
    the count of reads since the last sufficient wait along every path."""
    entry, work, worst = {0: 0}, [0], 0
    while work:
        b = work.pop()
        p = entry[b]
        for t in blocks[b]:
            wait = re.search(r"lgkmcnt\((\d+)\)", t)
            if t.startswith(("ds_read", "ds_load")):
                p = min(p + 1, 63)
            elif wait:
                p = min(p, int(wait.group(1)))
            elif t.startswith("s_barrier"):
                worst = max(worst, p)
        for s in succ[b]:
            if entry.get(s, -1) < p:
                entry[s] = p
                work.append(s)
    return worst


@pytest.fixture(scope="module")
def pending(tmp_path_factory):
    d = tmp_path_factory.mktemp("lds")
    (d / "probe.hip").write_text(source())
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-I", build.CSRC, str(d / "probe.hip"), "-o",
                    str(d / "probe.s")], check=True, capture_output=True)
    asm = (d / "probe.s").read_text()
    return {name: reads_pending_at_barriers(b, s) for name, b, s in kernels(asm)
            if any("load_lds" in t for blk in b for t in blk)}


@pytest.mark.parametrize("i", range(len(KERNELS)))
def test_no_lds_read_pending_at_a_barrier(pending, i):
    found = [v for name, v in pending.items() if f"probe{i}P" in name]
    assert found == [0]
