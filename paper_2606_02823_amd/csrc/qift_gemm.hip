// Tiled GEMM on v_mfma_i32_32x32x32_i8 for prompts (M > 64 tokens), W2 and W4 weights.
#include "qift_fwht.h"   // buffer-load helpers
#include "qift_internal.h"
#include "qift_mma.h"
#include "qift_route.h"
#include "qift_waits.h"

#include <type_traits>

namespace qift {
namespace {

using namespace mma;

typedef int v16i __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v16i mfma32_i8(v4i a, v4i b, v16i c) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

constexpr int kBK = 128;                       // k per step
template <int FMT>
constexpr int wload16() { return FMT == FMT_W4 ? 2 : 1; }   // 16-byte loads per row tile, half wave and step
template <int FMT>
constexpr int line_steps() { return FMT == FMT_W4 ? 2 : 4; }   // steps in 128 bytes of a weight row

// What the weight operands of the MFMA hold.
//   kCodes    the raw codes: the exact correction needs the per-token code sums, which the caller gives (MNZ, W4)
//   kLevels   the levels, W4's times 16: no sums (PoT, and the others where none are given)
//   kLevels1  the levels of W4 as they are, where 16 times the accumulator may not fit int32 (K > 2^21)
enum Operand { kCodes, kLevels, kLevels1 };

// register r of the MFMA operand s of a lane's weights of one step
template <int FMT, int OP>
__device__ __forceinline__ int decode_part(const uint4 (&u)[FMT == FMT_W4 ? 2 : 1], int s, int r) {
  if constexpr (FMT == FMT_W4) {
    const uint4 h = u[s >> 1];
    const uint32_t w = (s & 1) ? (r < 2 ? h.z : h.w) : (r < 2 ? h.x : h.y);
    // nibble u = q + 8: in the upper half of a byte with its top bit flipped it is 16 q
    if constexpr (OP == kLevels) return (int)(((r & 1 ? w : w << 4) & 0xF0F0F0F0u) ^ 0x80808080u);
    const uint32_t c = (r & 1 ? w >> 4 : w) & 0x0F0F0F0Fu;
    // u + 120 stays within the byte, and is 128 + q
    return OP == kLevels1 ? (int)((c + 0x78787878u) ^ 0x80808080u) : (int)c;
  } else {
    const uint32_t w = s == 0 ? u[0].x : s == 1 ? u[0].y : s == 2 ? u[0].z : u[0].w;
    const uint32_t c = (w >> (2 * r)) & 0x03030303u;
    if constexpr (FMT == FMT_POT) return (int)__builtin_amdgcn_perm(0u, 0x0401FFFCu, c);   // {-4, -1, +1, +4}
    return OP == kCodes ? (int)c : (int)__builtin_amdgcn_perm(0u, 0x0301FFFDu, c);         // {-3, -1, +1, +3}
  }
}

// the accumulator from the MFMA sum D
template <int FMT, int OP>
__device__ __forceinline__ int finish(int D, int sum_q) {
  if constexpr (OP == kCodes) return finish_acc<FMT>(D, sum_q);
  else return FMT == FMT_W4 && OP == kLevels ? D >> 4 : D;
}

// slot of 16-byte column c of activation row r
__device__ __forceinline__ int slot(int r, int c) { return c ^ (((r >> 1) & 7) ^ ((r & 1) << 2)); }

// Tiles of 256 weight rows x 32 TC tokens, steps of 128 k.  Four waves, two workgroups to a CU; wave w owns
// weight rows [64 w, +64) (two 32-row MFMA tiles) and all the tokens: 2 TC accumulator tiles, whose 32-wide
// MFMA holds the int8 rate better than the 16-wide one (33 cycles per 65536 operations against 39).
//
// What bounds it: the chip's power.  The MFMAs alone, on registers of such codes, reach 3.2-3.5 POP/s here
// (the clock falls to about 1.8 GHz); with one LDS read to two MFMAs and the weights' decode 3.2.  So the
// design spends little on anything else: the packed weights go from memory straight to registers, decoded
// once per 32 TC tokens; the int8 activations go to LDS without passing registers; consecutive MFMAs share
// an operand; no instruction waits inside a step.
//   weights      a lane loads its rows' 128-byte lines (512 k of W2, 256 k of W4) one line ahead, in two
//                register sets; half wave h holds k = 128 q + 64 h .. + 63 of step q of the line.
//   activations  four LDS buffers, filled three steps ahead by direct-to-LDS loads.  The buffers are distinct
//                arrays, so the compiler sees that loads into one never alias reads from another and adds
//                no waits of its own.  Rows are 128 bytes; 16-byte column c of row r lies in slot(r, c),
//                which spreads 8 and 16 consecutive rows over the banks (5 % of LDS cycles conflict).
//   tiles        in the order of the XCDs: a workgroup's neighbours in its L2 share tokens and weights.
//   outputs      through LDS (the idle activation buffers), then whole rows of 512 bytes.
// At 2048 tokens, us before (256 x 64 tiles of 16-wide MFMAs, three workgroups to a CU) -> now: W2 28672 x
// 4096 221 -> 187 (2.57 POP/s), 4096 x 4096 40 -> 33, 4096 x 14336 105 -> 94; W4 253 -> 206, 49 -> 36, 137 ->
// 108.  At 512: W2 73 -> 56, 27.2 -> 17.3, 66.7 -> 51.
// Without per-token sums (the plain calls) the operands are the levels, so that none are needed: one byte permute a
// register for MNZ, nothing for W4.  (Sums added up in the loop spilled 28 registers of MNZ's 128-token
// instance, whose reloads drained the loads in flight: 4096 x 14336 at 2048 tokens 118 -> 103 us, with sums 95; 28672 x
// 4096 at 1024 tokens 125 -> 107.)
template <int FMT, int TC, int OP>
__global__ __launch_bounds__(256, 2) void k_gemm32(const uint32_t* __restrict__ P, const uint16_t* __restrict__ sw,
                                                     int N, int K, const int8_t* __restrict__ act,
                                                     const float* __restrict__ sx, const int32_t* __restrict__ asum,
                                                     int M, int tiles_n, int tiles_m, uint16_t* __restrict__ y,
                                                     int32_t* __restrict__ acc_out) {
  constexpr int BM = 32 * TC;
  constexpr int NB = wload16<FMT>(), LS = line_steps<FMT>();
  constexpr int NA = BM * kBK / 4096;   // direct-to-LDS loads per wave and step
  constexpr int NW = 2 * NB * LS;       // weight loads per wave and line group
  __shared__ __align__(16) int8_t lds0[BM * kBK];
  __shared__ __align__(16) int8_t lds1[BM * kBK];
  __shared__ __align__(16) int8_t lds2[BM * kBK];
  __shared__ __align__(16) int8_t lds3[BM * kBK];

  __shared__ __align__(16) float s_sx[BM];
  __shared__ __align__(16) int s_sum[BM];
  __shared__ __align__(16) uint16_t s_sw[256];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, h = lane >> 5;
  // tile of this workgroup: consecutive tiles of one XCD (workgroups go round the 8 XCDs) share weights
  // and tokens in its L2
  int tn, tm;
  {
    const int T = tiles_n * tiles_m;
    const int id = blockIdx.x, x = id & 7, base = T >> 3, rem = T & 7;
    const int tile = x * base + (x < rem ? x : rem) + (id >> 3);
    constexpr int GT = 8;
    const int grp = tile / (GT * tiles_n), first = grp * GT;
    const int width = tiles_m - first < GT ? tiles_m - first : GT;
    const int in = tile - grp * GT * tiles_n;
    tn = in / width;
    tm = first + in - tn * width;
  }
  const int n_base = tn * 256 + wave * 64;
  const int m_base = tm * BM;
  const int64_t rowbytes = FMT == FMT_W4 ? (int64_t)K / 2 : (int64_t)K / 4;
  const int KT = (K + kBK - 1) / kBK;

  const __amdgpu_buffer_rsrc_t wrs = dev::make_rsrc(P, (uint32_t)(N * rowbytes));
  uint32_t wbase[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = n_base + 32 * j + r32;
    wbase[j] = n < N ? (uint32_t)(n * rowbytes) + 16u * NB * h : dev::kOutOfRange;
  }
  auto load_w = [&](uint4 (&w)[LS][2][NB], int kt) {   // the 128 bytes from step kt on
    const uint32_t ko = (uint32_t)kt * (32u * NB);
#pragma unroll
    for (int q = 0; q < LS; ++q)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int b = 0; b < NB; ++b) w[q][j][b] = dev::bload16(wrs, wbase[j] + ko + 32u * NB * q + 16u * b);
  };
  const int mrows = M - m_base < BM ? M - m_base : BM;
  const __amdgpu_buffer_rsrc_t ars = dev::make_rsrc(act + (int64_t)m_base * K, (uint32_t)(mrows * K));
  uint32_t abase[NA];
  int acol[NA];
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    const int row = 8 * (NA * wave + q) + (lane >> 3);
    acol[q] = 16 * slot(row, lane & 7);
    abase[q] = row < mrows ? (uint32_t)(row * K + acol[q]) : dev::kOutOfRange;
  }
  auto issue_a = [&](int kt, int8_t* dst, int q) {
    const int ko = kt * kBK;
    uint32_t off = abase[q] + (uint32_t)ko;
    if (acol[q] + ko >= K) off = dev::kOutOfRange;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        ars, (__attribute__((address_space(3))) void*)(dst + 1024 * (NA * wave + q)), 16, off, 0, 0, 0);
  };

  v16i acc[2][TC];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int t = 0; t < TC; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[j][t][i] = 0;

  int boff[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) boff[s] = r32 * kBK + 16 * slot(r32, 4 * h + s);

  // One step of 16 pairs of MFMAs (pair i = 4 s + t: operand s of the lane's weights against token tile
  // t, both row tiles).  Pair i reads the token operand of pair i + 3 and decodes a quarter of the
  // weight operands of s + 1, so neither is waited for; the barrier that hands the buffers over comes
  // after pair 12, when this wave's operand reads of the step are done, and the last pairs already
  // read the next step's buffer.
  v4i a[2], an[2], bq[4];
  auto read_b = [&](const int8_t* tileb, int i) {
    const uint4 bb = *reinterpret_cast<const uint4*>(tileb + 32 * kBK * (i % TC) + boff[i / TC]);
    return v4i{(int)bb.x, (int)bb.y, (int)bb.z, (int)bb.w};
  };
  auto step = [&](const int8_t* cur, int8_t* own, const int8_t* nxt, const uint4 (&w)[2][NB],
                  const uint4 (&wnx)[2][NB], int kt, auto outstanding) {
    constexpr int NP = 4 * TC, OUT = decltype(outstanding)::value;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int s = i / TC, t = i % TC;
      const v4i b = bq[i & 3];
      // the last two pairs read three operands of the next step
      if (i + 3 < NP) bq[(i + 3) & 3] = read_b(cur, i + 3);
      if (i == NP - 2) {
        bq[0] = read_b(nxt, 0);
        bq[1] = read_b(nxt, 1);
      }
      if (i == NP - 1) bq[2] = read_b(nxt, 2);
      const int j0 = t & 1;   // consecutive MFMAs share an operand
      acc[j0][t] = mfma32_i8(a[j0], b, acc[j0][t]);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 4 * t / TC; r < 4 * (t + 1) / TC; ++r)
          an[j][r] = s < 3 ? decode_part<FMT, OP>(w[j], s + 1, r) : decode_part<FMT, OP>(wnx[j], 0, r);
      if (i >= NP - 2) {
#pragma unroll
        for (int q = 0; q < NA; ++q)
          if ((q >= (NA + 1) / 2) == (i == NP - 1)) issue_a(kt + 4, own, q);
      }
      acc[1 - j0][t] = mfma32_i8(a[1 - j0], b, acc[1 - j0][t]);
      if (t == TC - 1) {
        a[0] = an[0];
        a[1] = an[1];
      }
      __builtin_amdgcn_sched_barrier(0);
      if (i == NP - 3) {
        __builtin_amdgcn_s_waitcnt(waits::encode(OUT, true));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto issue_all = [&](int kt, int8_t* dst) {
#pragma unroll
    for (int q = 0; q < NA; ++q) issue_a(kt, dst, q);
  };

  // scales and sums of the tile for the epilogue (their loads go out before the tile's)
  const float sx_pre = tid < mrows ? sx[m_base + tid] : 0.f;
  int sum_pre = 0;
  if constexpr (OP == kCodes) sum_pre = tid < mrows ? asum[m_base + tid] : 0;
  const uint16_t sw_pre = tn * 256 + tid < N ? sw[tn * 256 + tid] : (uint16_t)0;
  __builtin_amdgcn_sched_barrier(0);
  uint4 wa[LS][2][NB], wb[LS][2][NB];
  load_w(wa, 0);
  issue_all(0, lds0);
  issue_all(1, lds1);
  issue_all(2, lds2);
  issue_all(3, lds3);
  if (tid < BM) {
    s_sx[tid] = sx_pre;
    if constexpr (OP == kCodes) s_sum[tid] = sum_pre;
  }
  s_sw[tid] = sw_pre;
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(waits::encode(waits::gemm32_prologue(NA, LS), true));
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < 3; ++i) bq[i] = read_b(lds0, i);
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) a[j][r] = decode_part<FMT, OP>(wa[0][j], 0, r);
  // A line group of W2 is four steps, of W4 two (whose buffers rotate over two groups).  The handover of
  // step k waits for the activations of step k + 1, sent three steps earlier: those of steps k + 2 and
  // k + 3 and the weight loads sent since stay in flight (qift_waits.h).
#define QIFT_OUT(q, more) std::integral_constant<int, waits::gemm32_handover(NA, NW, LS, q, more)>()
#define QIFT_GROUP4(k, w, wn, more)                                    \
  step(lds0, lds0, lds1, w[0], w[1], k, QIFT_OUT(0, more));            \
  step(lds1, lds1, lds2, w[1], w[2], k + 1, QIFT_OUT(1, more));        \
  step(lds2, lds2, lds3, w[2], w[3], k + 2, QIFT_OUT(2, more));        \
  step(lds3, lds3, lds0, w[3], wn[0], k + 3, QIFT_OUT(3, more));
#define QIFT_GROUP2(k, b0, b1, b2, w, wn, more)                        \
  step(b0, b0, b1, w[0], w[1], k, QIFT_OUT(0, more));                  \
  step(b1, b1, b2, w[1], wn[0], k + 1, QIFT_OUT(1, more));
  auto load_w_here = [&](uint4 (&w)[LS][2][NB], int kt) {
    load_w(w, kt);
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = 0;
  for (; kt + LS < KT; kt += 2 * LS) {
    load_w_here(wb, kt + LS);
    if constexpr (LS == 4) {
      QIFT_GROUP4(kt, wa, wb, true)
      load_w_here(wa, kt + 2 * LS);
      QIFT_GROUP4(kt + 4, wb, wa, true)
    } else {
      QIFT_GROUP2(kt, lds0, lds1, lds2, wa, wb, true)
      load_w_here(wa, kt + 2 * LS);
      QIFT_GROUP2(kt + 2, lds2, lds3, lds0, wb, wa, true)
    }
  }
  // an odd last group, with no weights to load after it (a load of weights that no MFMA uses would be
  // dropped by the compiler, and must not be counted in flight)
  if (kt < KT) {
    if constexpr (LS == 4) {
      QIFT_GROUP4(kt, wa, wa, false)
    } else {
      QIFT_GROUP2(kt, lds0, lds1, lds2, wa, wa, false)
    }
  }
#undef QIFT_GROUP4
#undef QIFT_GROUP2
#undef QIFT_OUT
  __builtin_amdgcn_s_waitcnt(0x0F70);   // the loads past K have landed before a buffer is reused
  __syncthreads();

  float sxt[TC];
  int sqt[TC];
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    sxt[t] = s_sx[32 * t + r32];
    sqt[t] = 0;
    if constexpr (OP == kCodes) sqt[t] = s_sum[32 * t + r32];
  }
  // D of tile (j, t): register 4 q + i of lane (token r32, half h) is row 32 j + 8 q + 4 h + i
  if (acc_out == nullptr) {
    // through LDS: token tile t in buffer t as rows of 256 outputs (32 chunks of 8, chunk c of token m in
    // slot c ^ m), then 16-byte stores of whole rows
    // (8 TC tokens' rows to a buffer)
    auto row_at = [&](int t, int r) -> int8_t* {
      constexpr int RB = BM / 4;   // rows of outputs that a buffer holds
      const int b = 32 * t / RB, row = 32 * t + r - b * RB;
      int8_t* lo = b == 0 ? lds0 : b == 1 ? lds1 : b == 2 ? lds2 : lds3;
      int8_t* hi = b == 0 ? lds1 : b == 1 ? lds2 : lds3;
      return row < RB ? lo + 512 * row : hi + 512 * (row - RB);
    };
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint2 swq = *reinterpret_cast<const uint2*>(s_sw + 64 * wave + 32 * j + 8 * q + 4 * h);
        const uint16_t s4[4] = {(uint16_t)(swq.x & 0xFFFFu), (uint16_t)(swq.x >> 16), (uint16_t)(swq.y & 0xFFFFu),
                                (uint16_t)(swq.y >> 16)};
#pragma unroll
        for (int t = 0; t < TC; ++t) {
          uint32_t o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = epilogue(finish<FMT, OP>(acc[j][t][4 * q + i], sqt[t]), sxt[t], s4[i]);
          const int c = 8 * wave + 4 * j + q;
          *reinterpret_cast<uint2*>(row_at(t, r32) + 16 * (c ^ r32) + 8 * h) =
              make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
        }
      }
    __syncthreads();
    const int nt = N - tn * 256 < 256 ? N - tn * 256 : 256;   // rows of the tile below N
    if ((N & 7) == 0) {
      const int c = tid & 31;
      if (8 * c < nt) {
#pragma unroll
        for (int t = 0; t < TC; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 8 * i + (tid >> 5), m = m_base + 32 * t + r;
            const uint4 d = *reinterpret_cast<const uint4*>(row_at(t, r) + 16 * (c ^ r));
            if (m < M) *reinterpret_cast<uint4*>(y + (int64_t)m * N + tn * 256 + 8 * c) = d;
          }
      }
    } else if (tid < nt) {   // rows of y at any alignment: one output a thread, a token at a time
#pragma unroll
      for (int t = 0; t < TC; ++t)
        for (int r = 0; r < 32; ++r) {
          const int m = m_base + 32 * t + r;
          if (m < M)
            y[(int64_t)m * N + tn * 256 + tid] =
                *reinterpret_cast<const uint16_t*>(row_at(t, r) + 16 * ((tid >> 3) ^ r) + 2 * (tid & 7));
        }
    }
    return;
  }
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    const int m = m_base + 32 * t + r32;
    if (m < M) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          // (the accumulators as they are: PoT's form of the store)
          store4_sw<FMT_POT>(v4i{finish<FMT, OP>(acc[j][t][4 * q], sqt[t]), finish<FMT, OP>(acc[j][t][4 * q + 1], sqt[t]),
                                 finish<FMT, OP>(acc[j][t][4 * q + 2], sqt[t]), finish<FMT, OP>(acc[j][t][4 * q + 3], sqt[t])},
                             m, n_base + 32 * j + 8 * q + 4 * h, N, sxt[t], 0,
                             *reinterpret_cast<const uint2*>(s_sw + 64 * wave + 32 * j + 8 * q + 4 * h), y, acc_out);
    }
  }
}

template <int FMT, int TC, int OP>
hipError_t launch_t(const uint32_t* P, const uint16_t* sw, int64_t N, int64_t K, const int8_t* act, const float* sx,
                    const int32_t* asum, int64_t M, uint16_t* y, int32_t* acc_out, hipStream_t s) {
  const int tn = (int)((N + 255) / 256), tm = (int)((M + 32 * TC - 1) / (32 * TC));
  const dim3 grid((unsigned)tn * (unsigned)tm);
  hipLaunchKernelGGL((k_gemm32<FMT, TC, OP>), grid, dim3(256), 0, s, P, sw, (int)N, (int)K, act, sx, asum, (int)M, tn, tm,
                     y, acc_out);
  return hipGetLastError();
}

template <int FMT>
hipError_t launch_f(const uint32_t* P, const uint16_t* sw, int64_t N, int64_t K, const int8_t* act, const float* sx,
                    const int32_t* asum, int64_t M, uint16_t* y, int32_t* acc_out, hipStream_t s) {
  const int tokens = route::gemm_tile_tokens(FMT == FMT_W4, N, M);
#define QIFT_G(TC_, OP_) launch_t<FMT, TC_, OP_>(P, sw, N, K, act, sx, asum, M, y, acc_out, s)
#define QIFT_GT(OP_) (tokens == 128 ? QIFT_G(4, OP_) : tokens == 96 ? QIFT_G(3, OP_) : QIFT_G(2, OP_))
  if constexpr (FMT != FMT_POT)
    if (asum) return QIFT_GT(kCodes);
  // 16 x 8 x 7 x K stays below 2^31
  if constexpr (FMT == FMT_W4)
    if (K > (1 << 21)) return QIFT_G(2, kLevels1);
  return QIFT_GT(kLevels);
#undef QIFT_GT
#undef QIFT_G
}

}  // namespace

hipError_t launch_gemm32(int fmt, const uint32_t* P, const uint16_t* sw, int64_t N, int64_t K, const int8_t* act,
                         const float* sx, const int32_t* asum, int64_t M, uint16_t* y, int32_t* acc_out, hipStream_t s) {
  switch (fmt) {
    case FMT_MNZ: return launch_f<FMT_MNZ>(P, sw, N, K, act, sx, asum, M, y, acc_out, s);
    case FMT_POT: return launch_f<FMT_POT>(P, sw, N, K, act, sx, asum, M, y, acc_out, s);
    case FMT_W4: return launch_f<FMT_W4>(P, sw, N, K, act, sx, asum, M, y, acc_out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qift
