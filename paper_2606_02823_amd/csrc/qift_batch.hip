// Linear on codes for batches of up to 64 tokens: one pass over the weights, one launch.
//
// A workgroup owns 32 RJ weight rows and 32 TC tokens and cuts K into a slice per wave.  The waves share
// nothing until their partial sums meet in LDS at the end, so the loop has no barrier: a wave sends the
// activations of its own slice to its own LDS stages (direct-to-LDS loads of whole 128-byte rows, three
// steps ahead) and its packed weights straight to registers (128-byte lines, two line groups from the start),
// and waits only on its own load counter.  RJ is chosen so that the grid is about one workgroup per CU:
// the weights are read once, each CU reads the M x K codes once, and the time hardly grows with the tokens.
// What bounds it at these sizes is latency: launch, the first loads from HBM, a few steps (a 4096-k row is
// 32 steps over 4 or 8 waves), the sum of the slices, and the address unit, which takes 36 to 70 cycles for
// each kilobyte of codes or weights (busy 28-59 % of the time at K = 4096, 80 % at 11008 and 14336): so the loads of a step cover 16, 32, 48 or 64 tokens (NA; 4096 x 14336 at 16 tokens
// 11.5 -> 10.2 us against 32), and RJ is as large as the grid allows.  Eight waves where their registers allow (32 RJ TC
// accumulators each), four otherwise.  Four line groups of weights in flight instead of two measured slower
// (12288 x 4096 at 16 tokens 8.2 -> 9.1 us).
// us, before (skinny kernel, its split over K, the split GEMM) -> now: W4 12288 x 4096 at 37 tokens 19.0 ->
// 12.1, 22016 x 4096 23.5 -> 19.6; W2 6144 x 4096 at 64 11.9 -> 7.9, 4096 x 14336 15.7 -> 13.1 (without a
// workspace 29.8 -> 12.8), 28672 x 4096 at 24 17.7 -> 14.3 (its 29 MB take 5.6 us at a large copy's rate).
#include "qift_fwht.h"   // buffer-load helpers
#include "qift_internal.h"
#include "qift_mma.h"
#include "qift_waits.h"

#include <type_traits>

namespace qift {
namespace {

using namespace mma;

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kBK = 128;   // k per step
constexpr int kNS = 4;     // activation stages
template <int FMT>
constexpr int line_steps() { return FMT == FMT_W4 ? 2 : 4; }   // steps in 128 bytes of a weight row

// slot of 16-byte column c of activation row r (8 and 16 consecutive rows spread over the banks)
__device__ __forceinline__ int slot(int r, int c) { return c ^ (((r >> 1) & 7) ^ ((r & 1) << 2)); }

template <int FMT, int RJ, int NA, int NWV, bool SUMQ>
__global__ __launch_bounds__(64 * NWV, NWV / 4) void k_batch(const uint32_t* __restrict__ P,
                                                             const uint16_t* __restrict__ sw, int N, int K,
                                                             const int8_t* __restrict__ act,
                                                             const float* __restrict__ sx,
                                                             const int32_t* __restrict__ asum, int M,
                                                             uint16_t* __restrict__ y, int32_t* __restrict__ acc_out) {
  constexpr int NB = FMT == FMT_W4 ? 2 : 1, LS = line_steps<FMT>();
  // NA: direct-to-LDS loads of a step, 1 KB and 8 tokens each (tokens past them: whatever the stage holds,
  // in outputs that are not stored)
  constexpr int TC = (NA + 3) / 4;
  constexpr int NW = RJ * NB * LS;      // weight loads of a line group
  constexpr int BUF = 4096 * TC;        // bytes of a wave's stage
  __shared__ __align__(16) int8_t lds0[NWV * BUF];
  __shared__ __align__(16) int8_t lds1[NWV * BUF];
  __shared__ __align__(16) int8_t lds2[NWV * BUF];
  __shared__ __align__(16) int8_t lds3[NWV * BUF];
  __shared__ int s_sum[NWV][32 * TC];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, h = lane >> 5;
  const int n_base = blockIdx.x * (32 * RJ);
  const int m_base = blockIdx.y * (32 * TC);
  M = M - m_base < 32 * TC ? M - m_base : 32 * TC;   // tokens of this workgroup
  act += (int64_t)m_base * K;
  sx += m_base;
  if (asum) asum += m_base;
  y += (int64_t)m_base * N;
  if (acc_out) acc_out += (int64_t)m_base * N;
  const int64_t rowbytes = FMT == FMT_W4 ? (int64_t)K / 2 : (int64_t)K / 4;
  // the wave's slice of K: GT line groups from k0 on, of which the steps past Kend read zeros
  const int KA = (K + kBK - 1) / kBK, S = (KA + NWV - 1) / NWV;
  const int k0 = wave * S * kBK;
  const int Kend = k0 + S * kBK < K ? k0 + S * kBK : K;
  const int GT = k0 < K ? ((Kend - k0 + kBK - 1) / kBK + LS - 1) / LS : 0;

  float sxt[TC];
  int sqt[TC];
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    const int m = 32 * t + r32;
    sxt[t] = m < M ? sx[m] : 0.f;
    sqt[t] = 0;
    if constexpr (!SUMQ) sqt[t] = m < M ? asum[m] : 0;
  }

  // s_w of the output quads this wave stores (p = wave + NWV i of the RJ TC 4)
  constexpr int NQ = (RJ * TC * 4 + NWV - 1) / NWV;
  uint2 swq[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int p = wave + NWV * i, n0 = n_base + 32 * (p / (TC * 4)) + 8 * (p & 3) + 4 * h;
    uint32_t v[4] = {0, 0, 0, 0};
    if (n0 + 3 < N) {
      swq[i] = *reinterpret_cast<const uint2*>(sw + n0);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = n0 + r < N ? sw[n0 + r] : 0u;
      swq[i] = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
    }
  }

  const __amdgpu_buffer_rsrc_t wrs = dev::make_rsrc(P, (uint32_t)(N * rowbytes));
  uint32_t wbase[RJ];
#pragma unroll
  for (int j = 0; j < RJ; ++j) {
    const int n = n_base + 32 * j + r32;
    wbase[j] = n < N ? (uint32_t)(n * rowbytes) + (uint32_t)k0 / (FMT == FMT_W4 ? 2 : 4) + 16u * NB * h : dev::kOutOfRange;
  }
  auto load_w = [&](uint4 (&w)[LS][RJ][NB], int g) {   // line group g of the slice (past it: zeros, no traffic)
    const uint32_t go = (uint32_t)g * 128u;
#pragma unroll
    for (int q = 0; q < LS; ++q)
#pragma unroll
      for (int j = 0; j < RJ; ++j)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          w[q][j][b] = dev::bload16(wrs, (g < GT ? wbase[j] + go : dev::kOutOfRange) + 32u * NB * q + 16u * b);
    __builtin_amdgcn_sched_barrier(0);
  };
  // activations: load q takes tokens 8 q .. 8 q + 7 (lane l column l mod 8 of token 8 q + l / 8)
  const __amdgpu_buffer_rsrc_t ars = dev::make_rsrc(act, (uint32_t)M * (uint32_t)K);
  const int arow = lane >> 3;
  // slot(row, .) of row 8 q + arow: adding 8 to the row flips column bit 2, i.e. 64 bytes
  const int acol0 = 16 * slot(arow, lane & 7);
  auto issue_a = [&](int kt, int8_t* dst) {
    const int ko = k0 + kt * kBK;
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int row = 8 * q + arow, col = acol0 ^ (64 * (q & 1));
      const bool ok = row < M && col + ko < Kend;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ars, (__attribute__((address_space(3))) void*)(dst + wave * BUF + 1024 * q), 16,
                                               ok ? (uint32_t)row * (uint32_t)K + (uint32_t)(col + ko) : dev::kOutOfRange,
                                               0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  v16i acc[RJ][TC];
#pragma unroll
  for (int j = 0; j < RJ; ++j)
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[j][t][i] = 0;
  int boff[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) boff[s] = wave * BUF + r32 * kBK + 16 * slot(r32, 4 * h + s);
  v4i b[TC][4], bn[TC][4];
  int sq[TC];
#pragma unroll
  for (int t = 0; t < TC; ++t) sq[t] = 0;
  auto read_b = [&](v4i (&d)[TC][4], const int8_t* buf) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < TC; ++t) d[t][s] = *reinterpret_cast<const v4i*>(buf + 4096 * t + boff[s]);
  };
  // step kt: its operands are in b (their reads done), so its buffer takes the activations of step kt +
  // 4; the operands of step kt + 1 are read (out: loads that may still be in flight then) while the
  // MFMAs of step kt run
  auto step = [&](int kt, int8_t* own, const int8_t* nxt, const uint4 (&w)[RJ][NB], auto out) {
    constexpr int OUT = decltype(out)::value;
    issue_a(kt + kNS, own);
    __builtin_amdgcn_s_waitcnt(waits::encode(OUT, false));
    __builtin_amdgcn_sched_barrier(0);
    read_b(bn, nxt);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      v4i a[RJ];
#pragma unroll
      for (int j = 0; j < RJ; ++j) a[j] = decode_unit<FMT>(w[j], s);
#pragma unroll
      for (int t = 0; t < TC; ++t)
#pragma unroll
        for (int j = 0; j < RJ; ++j)
          acc[j][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[j], b[t][s], acc[j][t], 0, 0, 0);
      if constexpr (SUMQ) {
#pragma unroll
        for (int t = 0; t < TC; ++t)
          sq[t] = sum16_i8(make_uint4((uint32_t)b[t][s][0], (uint32_t)b[t][s][1], (uint32_t)b[t][s][2],
                                      (uint32_t)b[t][s][3]), sq[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int s = 0; s < 4; ++s) b[t][s] = bn[t][s];
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the reads of step kt + 1's operands are done
    __builtin_amdgcn_sched_barrier(0);
  };
  // The wait of step k is for the activations of step k + 1, sent at step k - 3: those of steps k + 2 .. k +
  // 4 and the weight group sent at this group's start stay in flight (qift_waits.h; W4's groups are two
  // steps, and the one sent at the start of the group before is in use by now).
#define QIFT_OUT(q, more) std::integral_constant<int, waits::batch_step(NA, NW, LS, q, more)>()
#define QIFT_GROUP4(k, w, more)                      \
  step(k, lds0, lds1, w[0], QIFT_OUT(0, more));      \
  step(k + 1, lds1, lds2, w[1], QIFT_OUT(1, more));  \
  step(k + 2, lds2, lds3, w[2], QIFT_OUT(2, more));  \
  step(k + 3, lds3, lds0, w[3], QIFT_OUT(3, more));
#define QIFT_GROUP2(k, b0, b1, b2, w, more)          \
  step(k, b0, b1, w[0], QIFT_OUT(0, more));          \
  step(k + 1, b1, b2, w[1], QIFT_OUT(1, more));
  if (GT > 0) {
    uint4 wa[LS][RJ][NB], wb[LS][RJ][NB];
    load_w(wa, 0);
    load_w(wb, 1);   // two groups from the start: most slices have no more
    issue_a(0, lds0);
    issue_a(1, lds1);
    issue_a(2, lds2);
    issue_a(3, lds3);
    __builtin_amdgcn_s_waitcnt(waits::encode(waits::batch_prologue(NA), false));
    __builtin_amdgcn_sched_barrier(0);
    read_b(b, lds0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (LS == 4) {
      QIFT_GROUP4(0, wa, false)
    } else {
      QIFT_GROUP2(0, lds0, lds1, lds2, wa, false)
    }
    int g = 1;
    for (; g + 1 < GT; g += 2) {
      load_w(wa, g + 1);
      if constexpr (LS == 4) {
        QIFT_GROUP4(4 * g, wb, true)
        load_w(wb, g + 2);
        QIFT_GROUP4(4 * g + 4, wa, true)
      } else {
        QIFT_GROUP2(2 * g, lds2, lds3, lds0, wb, true)
        load_w(wb, g + 2);
        QIFT_GROUP2(2 * g + 2, lds0, lds1, lds2, wa, true)
      }
    }
    // a last group with no weights to load after it (loads that no MFMA uses would be dropped by the
    // compiler, and must not be counted in flight)
    if (g < GT) {
      if constexpr (LS == 4) {
        QIFT_GROUP4(4 * g, wb, false)
      } else {
        QIFT_GROUP2(2 * g, lds2, lds3, lds0, wb, false)
      }
    }
  }
#undef QIFT_GROUP4
#undef QIFT_GROUP2
#undef QIFT_OUT

  // ---- the slices meet in LDS: tile (j, t) of wave w in buffer j, the lane's register quads 16 bytes apart
  // by 64 lanes; wave w then adds and stores the quads p = w (mod NWV) of the RJ TC 4
  static_assert(RJ <= 4, "a buffer per row tile");
  __builtin_amdgcn_s_waitcnt(0x0F70);   // every load into LDS has landed
  __syncthreads();
  auto tile_at = [&](int j) { return j == 0 ? lds0 : j == 1 ? lds1 : j == 2 ? lds2 : lds3; };
#pragma unroll
  for (int j = 0; j < RJ; ++j)
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<int4*>(tile_at(j) + wave * BUF + 4096 * t + 1024 * q + 16 * lane) =
            make_int4(acc[j][t][4 * q], acc[j][t][4 * q + 1], acc[j][t][4 * q + 2], acc[j][t][4 * q + 3]);
  if constexpr (SUMQ) {
#pragma unroll
    for (int t = 0; t < TC; ++t) {
      const int v = sq[t] + __shfl_xor(sq[t], 32);
      if (h == 0) s_sum[wave][32 * t + r32] = v;
    }
  }
  __syncthreads();
  if constexpr (SUMQ) {
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int w4 = 0; w4 < NWV; ++w4) sqt[t] += s_sum[w4][32 * t + r32];
  }
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int p = wave + NWV * i, jt = p >> 2, q = p & 3;   // wave-uniform
    if (p >= RJ * TC * 4) break;
    const int j = jt / TC, t = jt % TC;
    const int8_t* src = (j == 0 ? lds0 : j == 1 ? lds1 : j == 2 ? lds2 : lds3) + 4096 * t + 1024 * q + 16 * lane;
    v4i D = v4i{0, 0, 0, 0};
#pragma unroll
    for (int w4 = 0; w4 < NWV; ++w4) D += *reinterpret_cast<const v4i*>(src + w4 * BUF);
    const int m = 32 * t + r32, n0 = n_base + 32 * j + 8 * q + 4 * h;
    const float s_x = TC == 1 || t == 0 ? sxt[0] : sxt[TC - 1];
    const int s_q = TC == 1 || t == 0 ? sqt[0] : sqt[TC - 1];
    if (m < M && n0 < N) store4_sw<FMT>(D, m, n0, N, s_x, s_q, swq[i], y, acc_out);
  }
}

template <int FMT, int RJ, int NA, int NWV>
hipError_t launch_t(const uint32_t* P, const uint16_t* sw, int64_t N, int64_t K, const int8_t* act, const float* sx,
                    const int32_t* asum, int64_t M, uint16_t* y, int32_t* acc_out, hipStream_t s) {
  constexpr int TC = (NA + 3) / 4;
  const dim3 grid((unsigned)((N + 32 * RJ - 1) / (32 * RJ)), (unsigned)((M + 32 * TC - 1) / (32 * TC)));
  if (asum)
    hipLaunchKernelGGL((k_batch<FMT, RJ, NA, NWV, false>), grid, dim3(64 * NWV), 0, s, P, sw, (int)N, (int)K, act, sx,
                       asum, (int)M, y, acc_out);
  else
    hipLaunchKernelGGL((k_batch<FMT, RJ, NA, NWV, true>), grid, dim3(64 * NWV), 0, s, P, sw, (int)N, (int)K, act, sx,
                       asum, (int)M, y, acc_out);
  return hipGetLastError();
}

template <int FMT>
hipError_t launch_f(const uint32_t* P, const uint16_t* sw, int64_t N, int64_t K, const int8_t* act, const float* sx,
                    const int32_t* asum, int64_t M, uint16_t* y, int32_t* acc_out, hipStream_t s) {
  if (M < 1 || M > kBatchMaxM) return hipErrorInvalidValue;
  const int64_t rj = (N + 32 * 256 - 1) / (32 * 256);   // rows for about one workgroup per CU
  // up to 4096 rows two token tiles share the chip (4096 x 4096 at 64 tokens 7.4 -> 6.6 us, 4096 x 14336
  // 16.1 -> 13.1)
#define QIFT_B(RJ_, NA_, NWV_) launch_t<FMT, RJ_, NA_, NWV_>(P, sw, N, K, act, sx, asum, M, y, acc_out, s)
  if (M <= 16) {
    if (rj <= 1) return QIFT_B(1, 2, 8);
    if (rj == 2) return QIFT_B(2, 2, 8);
    if (rj == 3) return QIFT_B(3, 2, 4);
    return QIFT_B(4, 2, 4);
  }
  if (M <= 32 || N <= 4096) {
    if (rj <= 1) return QIFT_B(1, 4, 8);
    if (rj == 2) return QIFT_B(2, 4, 8);
    if (rj == 3) return QIFT_B(3, 4, 4);
    return QIFT_B(4, 4, 4);
  }
  if (M <= 48) {
    if (rj <= 1) return QIFT_B(1, 6, 4);
    if (rj == 2) return QIFT_B(2, 6, 4);
    if (rj == 3) return QIFT_B(3, 6, 4);
    return QIFT_B(4, 6, 4);
  }
  if (rj <= 1) return QIFT_B(1, 8, 4);
  if (rj == 2) return QIFT_B(2, 8, 4);
  if (rj == 3) return QIFT_B(3, 8, 4);
  return QIFT_B(4, 8, 4);
#undef QIFT_B
}

}  // namespace

hipError_t launch_batch(int fmt, const uint32_t* P, const uint16_t* sw, int64_t N, int64_t K, const int8_t* act,
                        const float* sx, const int32_t* asum, int64_t M, uint16_t* y, int32_t* acc_out, hipStream_t s) {
  switch (fmt) {
    case FMT_MNZ: return launch_f<FMT_MNZ>(P, sw, N, K, act, sx, asum, M, y, acc_out, s);
    case FMT_POT: return launch_f<FMT_POT>(P, sw, N, K, act, sx, asum, M, y, acc_out, s);
    case FMT_W4: return launch_f<FMT_W4>(P, sw, N, K, act, sx, asum, M, y, acc_out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qift
