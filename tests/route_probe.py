"""The kernel that csrc/qift_route.h chooses for a linear on codes, asked through a program compiled from that header."""
import functools
import os
import shutil
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_02823_amd", "csrc")
KERNELS = ["batch", "gemm_split", "gemm", "skinny", "skinny_split", "codes", "decode"]
PROBE = """
#include <cstdio>
#include "qift_route.h"
using namespace qift;
int main() {
  long w4, N, K, M, codes, ws;
  while (std::scanf("%ld %ld %ld %ld %ld %ld", &w4, &N, &K, &M, &codes, &ws) == 6)
    std::printf("%d %d %d %d\\n", (int)route::choose(w4, N, K, M, codes, ws), route::gemm_split_plan(w4, N, M, K).S,
                route::skinny_split_plan(w4, N, M, K).S, route::gemm_tile_tokens(w4, N, M));
}
"""


@functools.lru_cache(maxsize=None)
def _probe():
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    d = tempfile.TemporaryDirectory(prefix="qift_route")
    src, exe = os.path.join(d.name, "probe.cpp"), os.path.join(d.name, "probe")
    with open(src, "w") as f:
        f.write(PROBE)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, src, "-o", exe], check=True)
    return d, exe


def ask(queries):
    """list of (w4, N, K, M, codes fit LDS, workspace) -> list of (kernel, GEMM ranges, skinny ranges, tokens of the
    unsplit GEMM's tiles)."""
    out = subprocess.run([_probe()[1]], input="".join("%d %d %d %d %d %d\n" % tuple(q) for q in queries), text=True,
                         capture_output=True, check=True).stdout.splitlines()
    assert len(out) == len(queries)
    rows = [[int(v) for v in line.split()] for line in out]
    return [(KERNELS[r[0]], *r[1:]) for r in rows]
