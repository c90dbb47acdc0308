"""The counted waits of the tiled GEMM and of the batch linear, replayed on the CPU.

Both kernels keep direct-to-LDS loads in flight across steps and wait, where a step hands its buffer over, for
"all but the last n loads".  Loads return in the order they were sent, so the replay sends them in the kernels' order
and asks at each handover whether the next step's activations are among those that must have landed.  The
counts come from the header that the kernels are compiled with.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_02823_amd", "csrc")
# (tag, weight loads of a line group, steps of a group, activation loads of a step): k_gemm32 of 64, 96 and 128 tokens ...
GEMM = [(f"{f}-{32 * tc}", 8, ls, tc) for f, ls in (("w2", 4), ("w4", 2)) for tc in (2, 3, 4)]
# ... and k_batch of 1-4 row tiles and 16-64 tokens
BATCH = [(f"{f}-{rj}x{8 * na}", rj * 4, ls, na) for f, ls in (("w2", 4), ("w4", 2)) for rj in (1, 2, 3, 4)
         for na in (2, 4, 6, 8)]

PROBE = """
#include <cstdio>
#include "qift_waits.h"
using namespace qift::waits;
int main() {
  int NA, NW, LS;
  while (std::scanf("%d %d %d", &NA, &NW, &LS) == 3) {
    std::printf("%d", gemm32_prologue(NA, LS));
    for (int more = 0; more < 2; ++more)
      for (int q = 0; q < LS; ++q) std::printf(" %d", gemm32_handover(NA, NW, LS, q, more != 0));
    std::printf(" %d", batch_prologue(NA));
    for (int more = 0; more < 2; ++more)
      for (int q = 0; q < LS; ++q) std::printf(" %d", batch_step(NA, NW, LS, q, more != 0));
    std::printf("\\n");
  }
}
"""


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    """(NA, NW, LS) -> {"gemm": (prologue, [more][q]), "batch": ...}, as the kernels' compiler sees them."""
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    d = tmp_path_factory.mktemp("waits")
    (d / "probe.cpp").write_text(PROBE)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(d / "probe.cpp"), "-o", str(d / "probe")], check=True)
    keys = sorted({(na, nw, ls) for _, nw, ls, na in GEMM + BATCH})
    out = subprocess.run([str(d / "probe")], input="".join("%d %d %d\n" % k for k in keys), text=True,
                         capture_output=True, check=True).stdout
    table = {}
    for (na, nw, ls), line in zip(keys, out.splitlines()):
        v = [int(x) for x in line.split()]
        half = 1 + 2 * ls
        table[na, nw, ls] = {k: (p[0], (p[1:1 + ls], p[1 + ls:])) for k, p in (("gemm", v[:half]), ("batch", v[half:]))}
    assert len(table) == len(keys)
    return table


class Replay:
    """Loads sent in order; wait(n) leaves at most the last n outstanding."""

    def __init__(self):
        self.sent, self.landed, self.missing = [], 0, []

    def send(self, tag, n):
        self.sent += [tag] * n

    def wait(self, n):
        assert 0 <= n < 64, "six bits of vmcnt"
        self.landed = max(self.landed, len(self.sent) - n)

    def need(self, tag):
        last = len(self.sent) - self.sent[::-1].index(tag)   # one past its last load
        if last > self.landed:
            self.missing.append(tag)


def replay_gemm(prologue, handover, NA, NW, LS, KT):
    r = Replay()
    r.send(("W", 0), NW)
    for k in range(4):
        r.send(("A", k), NA)
    r.wait(prologue)
    r.need(("A", 0))

    def group(k0, more):
        for q in range(LS):
            k = k0 + q
            r.wait(handover[more][q])
            r.need(("A", k + 1))
            r.send(("A", k + 4), NA)

    kt, g = 0, 1
    while kt + LS < KT:
        r.send(("W", g), NW)
        group(kt, True)
        r.send(("W", g + 1), NW)
        group(kt + LS, True)
        kt, g = kt + 2 * LS, g + 2
    if kt < KT:
        group(kt, False)
    return r.missing


def replay_batch(prologue, step, NA, NW, LS, GT):
    r = Replay()
    r.send(("W", 0), NW)
    r.send(("W", 1), NW)
    for k in range(4):
        r.send(("A", k), NA)
    r.wait(prologue)
    r.need(("A", 0))

    def group(g, more):
        for q in range(LS):
            k = LS * g + q
            r.send(("A", k + 4), NA)
            r.wait(step[more][q])
            r.need(("A", k + 1))

    group(0, False)
    g = 1
    while g + 1 < GT:
        r.send(("W", g + 1), NW)
        group(g, True)
        r.send(("W", g + 2), NW)
        group(g + 1, True)
        g += 2
    if g < GT:
        group(g, False)
    return r.missing


@pytest.mark.parametrize("tag,NW,LS,NA", GEMM, ids=[c[0] for c in GEMM])
def test_tiled_gemm_waits(counts, tag, NW, LS, NA):
    prologue, handover = counts[NA, NW, LS]["gemm"]
    for KT in range(1, 40):
        assert replay_gemm(prologue, handover, NA, NW, LS, KT) == [], KT


@pytest.mark.parametrize("tag,NW,LS,NA", BATCH, ids=[c[0] for c in BATCH])
def test_batch_linear_waits(counts, tag, NW, LS, NA):
    prologue, step = counts[NA, NW, LS]["batch"]
    for GT in range(1, 20):
        assert replay_batch(prologue, step, NA, NW, LS, GT) == [], GT


@pytest.mark.parametrize("NA", [2, 3, 4])
def test_replay_finds_a_lax_wait(counts, NA):
    # W4's first step with a prologue that leaves A(1) in flight: two weight groups are counted there, one is sent
    _, handover = counts[NA, 8, 2]["gemm"]
    assert replay_gemm(3 * NA, handover, NA, 8, 2, 3) == [("A", 1)]
    assert replay_gemm(3 * NA, handover, NA, 8, 2, 2) == []        # one group: nothing else is sent
    # and any count of the loop that is one too large
    prologue, handover = counts[NA, 8, 4]["gemm"]
    for q in range(4):
        lax = (handover[0], [n + (i == q) for i, n in enumerate(handover[1])])
        assert replay_gemm(prologue, lax, NA, 8, 4, 12) != []
