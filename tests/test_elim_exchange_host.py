"""Lanes that exchange values through LDS without a workgroup barrier (the 4 x 4
blocks of the diagonal tiles, the factor's tiles read back by columns) are
ordered for the compiler, not only by the hardware's in-order LDS (no GPU): in
the device code's intermediate form a wavefront or workgroup fence stands between
a store to LDS and the next load from it, and for the 4 x 4 blocks also between
the load and the next store."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_06834_amd", "csrc")

KERNELS = {
    "diagonal": """
extern "C" __global__ void diagonal(const double *in, double *out) {
  __shared__ double scr[64], rs[16];
  const int c = threadIdx.x & 15, q = threadIdx.x >> 4;
  const double *p = in + 4 * threadIdx.x;
  el::Diag<false> g(el::v4d{p[0], p[1], p[2], p[3]}, c, q);
  g.strip<0>(scr, rs, nullptr);
  g.strip<1>(scr, rs, nullptr);
  g.strip<2>(scr, rs, nullptr);
  g.strip<3>(scr, rs, nullptr);
  for (int v = 0; v < 4; ++v) out[64 * v + threadIdx.x] = g.e[v] + g.r[v];
}""",
    "factor": """
struct Out {
  static constexpr bool kOn = true;
  double *dst;
  __device__ void below(int I, int J, const el::v4d &l) {
    for (int v = 0; v < 4; ++v) dst[64 * v + threadIdx.x] = l[v];
  }
  __device__ void diagonal(int J, const el::v4d &l) {}
};
extern "C" __global__ __launch_bounds__(64) void factor(const double *in, double *out) {
  __shared__ el::Lds<2, 1> L;
  __shared__ int flag;
  el::Elim<2, 1> E(threadIdx.x);
  for (int s = 0; s < 3; ++s)
    for (int v = 0; v < 4; ++v) E.a[s][v] = in[256 * s + 64 * v + threadIdx.x];
  E.run<0, 0, false>(L, &flag, nullptr, nullptr, [](int) {}, Out{out});
}""",
}


def accesses(ir, kernel, what):
    """'load' and 'store' of the LDS objects whose names hold `what`, and 'fence',
    per basic block in order."""
    body = ir[ir.index("define", ir.index("\n", ir.index("target triple"))):]
    body = re.search(r"define [^\n]*@" + kernel + r"\([^\n]*\{\n(.*?)\n\}\n", body, re.S).group(1)
    of = {}   # the LDS object that an address is formed from

    def names(line):
        return " ".join(of.get(t, t) for t in re.findall(r"[%@][\w.$]+", line))

    blocks, cur = [], []
    for line in body.splitlines():
        m = re.match(r"\s*(%[\w.]+) = getelementptr.* ptr addrspace\(3\) ([%@][\w.$]+)", line)
        if m:
            of[m[1]] = of.get(m[2], m[2])
        if re.match(r"^[\w.\d]+:", line):
            blocks.append(cur)
            cur = []
        elif re.search(r"fence syncscope\(\"(wavefront|workgroup)\"\) acquire", line):
            cur.append("fence")
        elif " load " in line and "addrspace(3)" in line and what in names(line):
            cur.append("load")
        elif line.strip().startswith("store ") and "addrspace(3)" in line and what in names(line):
            cur.append("store")
    return blocks + [cur]


@pytest.mark.parametrize("kernel,what", [("diagonal", "scr"), ("factor", "")])
def test_fences_between_lds_stores_and_loads(kernel, what, tmp_path):
    from paper_2607_06834_amd import build as b
    src = tmp_path / (kernel + ".hip")
    src.write_text('#include "elim_dev.h"\n' + KERNELS[kernel])
    ll = tmp_path / (kernel + ".ll")
    subprocess.run([b.HIPCC, *b.FLAGS, "-Wno-unused-command-line-argument", "--cuda-device-only", "-S", "-emit-llvm", str(src),
                    "-o", str(ll)], check=True, capture_output=True)
    n = {"load": 0, "store": 0}
    for block in accesses(ll.read_text(), kernel, what):
        last = None
        for a in block:
            if a != "fence":
                n[a] += 1
                assert not (a == "load" and last == "store"), block
                assert not (what and a == "store" and last == "load"), block
            last = a
    assert n["load"] >= 4 and n["store"] >= 4
