// Counted waits of the linears that keep direct-to-LDS loads in flight across steps (k_gemm32, k_batch):
// how many of a wave's vector-memory loads may still be outstanding where a step hands its buffer over.
// Loads return in the order they were sent, so "at most n outstanding" means that all but the last n have
// landed.  A(k) are the NA loads of step k's activations, W(g) the NW loads of weight line group g (LS
// steps).  Host code too: the issue order is replayed against these counts without a GPU.
#pragma once

namespace qift {
namespace waits {

// k_gemm32.  Order: W(0) A(0) A(1) A(2) A(3) | per group g: W(g + 1), then per step k of it the handover
// of step k, then A(k + 4).  Before the first step the wait leaves A(2) and A(3) of groups of two steps, A(1) too of
// groups of four.  (Two steps are fewer than the three that the activations run ahead, so the handover of
// a group's first step counts two weight groups between A(k + 1) and now; at step 0 only one has been sent
// since A(1), so that one must have landed by then.)
constexpr int gemm32_prologue(int NA, int LS) { return (LS == 2 ? 2 : 3) * NA; }
// handover of step q of a group: A(k + 1) has landed, sent three steps earlier.  more: false in an odd last
// group, which sends no weights.
constexpr int gemm32_handover(int NA, int NW, int LS, int q, bool more) {
  if (!more) return 2 * NA;
  if (LS == 4) return q < 3 ? 2 * NA + NW : 2 * NA;
  return q == 0 ? 2 * NA + 2 * NW : 2 * NA + NW;
}

// k_batch.  Order: W(0) W(1) A(0) A(1) A(2) A(3) | group 0 | per group g >= 1: W(g + 1) unless it is the
// last of an even count; per step k: A(k + 4), then the wait for A(k + 1).  more: the group sent weights.
constexpr int batch_prologue(int NA) { return 3 * NA; }
constexpr int batch_step(int NA, int NW, int LS, int q, bool more) {
  return LS == 4 && q == 3 ? 3 * NA : 3 * NA + (more ? NW : 0);
}

// s_waitcnt operand: vmcnt(n) with expcnt and, unless lgkm0, lgkmcnt left alone
constexpr int encode(int n, bool lgkm0) { return (lgkm0 ? 0x0070 : 0x0F70) | (n & 15) | ((n >> 4) << 14); }
static_assert(encode(63, false) == 0xCF7F && encode(0, true) == 0x0070, "six bits of vmcnt");

}  // namespace waits
}  // namespace qift
