// Online Hadamard rotation + per-token symmetric INT4 quantization.
//
// Per token (Sec. 3.1; Sec. 4.1 "Quantization configuration"):
//   X = (I_{K/b} (x) H_b) x  exactly,  A = max|X|,
//   q = sign(X) min(7, rne(7|X| / (cA))),  s_x = cA / (7 sqrt(b)),  sum = sum q.
//
// Tokens of K <= 12288 with blocks b <= 4096 (k_act_tokens): a persistent
// grid of 256-thread workgroups, each walking tokens blockIdx.x, + gridDim.x,
// ... (for tokens of up to two 4096-element tiles with the next token's fp16
// loads in flight while the current one is rotated).  Each thread keeps 16 consecutive elements of every 4096-element
// tile of the token in fp64 registers (the whole token stays on chip until
// its absmax is known); the butterflies run in registers (quad DPP for index
// bits 4-5 of blocks up to 64) with LDS exchanges between groups of four
// index bits; values are quantized in the layout the transform ends in,
// their codes scattered into the exchange buffer in natural order and copied
// out with 16-byte stores.  The block exponent is a template constant for
// common block sizes.
//
// Larger tokens (k_rotate_quant_act): one 512-thread workgroup per token,
// returning to the natural layout before quantizing.  See qift_fwht.h for
// the exactness argument and the rounding decision.
//
// Few tokens of several tiles, and any number of four-tile tokens (k_act_wide): one workgroup per
// token of G groups of four waves, the groups rotating their tiles at once (each group with its own
// exchange buffer and wave barrier), one workgroup barrier for the token's max, each group quantizing
// its own tiles.  The same transform and rounding as above, so the codes, scales and sums are the
// same.
//   Up to kActWideMaxM tokens the chip has room for a group per tile, and a token's latency is that
//   of one tile instead of NTILES (down's 14336-wide input at 16 tokens: the tiles one after another
//   took about 10 us, at once 6.9).
//   Beyond, latency between the exchanges bounds the kernel, so what counts is waves per SIMD: a
//   four-tile token in one group of waves holds 128 fp64 registers' worth of values per thread (199
//   VGPRs, 2 waves per SIMD), in two groups of two tiles half of that (117, 4 waves).  14336 wide,
//   b = 2048, 2048 tokens: 45.4 us in one group, 39.0 in two, 50.6 in four (a fourth of whose last
//   tile is padding that holds a whole group); 512 tokens: 14.5, 13.3, 15.0; 257: 12.5, 11.4, 12.8.
//   Three tiles stay with k_act_tokens there: a second group would rotate one tile while the first
//   does two (11008 wide, 2048 tokens: 23.4 us against 28.5), and so do two (8192: 18.8 against
//   18.6 to 19.1).
#include "qift_fwht.h"
#include "qift_internal.h"

namespace qift {
namespace {

// tokens up to which all of a token's tiles are rotated at once, one to a group of waves
constexpr int64_t kActWideMaxM = 256;

template <int NT, int NTILES, bool BF16>
__global__ __launch_bounds__(NT) void k_rotate_quant_act(const uint16_t* __restrict__ x, int64_t K, int L,
                                                         int num, int den, double denom,
                                                         int8_t* __restrict__ act_q,
                                                         float* __restrict__ act_scale,
                                                         int32_t* __restrict__ act_sum) {
  using S = dev::Tile<NT, 16>;
  __shared__ double lds[S::LDS_DOUBLES];
  __shared__ double red_d[NT / 64];
  __shared__ int red_i[NT / 64];
  const int64_t m = blockIdx.x;
  int sum_q;
  float scale;
  dev::quant_token<NT, NTILES, BF16>(x + m * K, K, L, num, den, denom, lds, red_d, red_i, act_q + m * K,
                                   sum_q, scale);
  if (threadIdx.x == 0) {
    if (act_sum) act_sum[m] = sum_q;
    act_scale[m] = scale;
  }
}

template <int NTILES, int LC, bool BF16>
__global__ __launch_bounds__(256) void k_act_tokens(const uint16_t* __restrict__ x, int M, int64_t K, int L,
                                                    int num, int den, double denom, int8_t* __restrict__ act_q,
                                                    float* __restrict__ act_scale, int32_t* __restrict__ act_sum) {
  using S = dev::Tile<256, 16>;
  static_assert(NTILES * S::T <= S::LDS_DOUBLES * 8, "the codes of a token fit in the exchange buffer");
  __shared__ double xch[S::LDS_DOUBLES];
  __shared__ double red_d[4];
  __shared__ int red_i[4];
  const int t = threadIdx.x;
  dev::BlockSync sync;
  int8_t* codes = reinterpret_cast<int8_t*>(xch);   // natural-order codes, once the transform is done
  int m = blockIdx.x;                               // gridDim.x <= M
  // tokens of up to two tiles keep the next token's loads in flight; longer ones need those registers
  constexpr bool kPrefetch = NTILES <= 2;
  dev::TokenRaw<NTILES> raw;
  dev::load_token_raw<256, NTILES>(raw, x + (int64_t)m * K, K);
  for (; m < M; m += gridDim.x) {
    dev::TokenRaw<NTILES> cur = raw;
    if (kPrefetch && m + (int)gridDim.x < M)
      dev::load_token_raw<256, NTILES>(raw, x + (int64_t)(m + gridDim.x) * K, K);
    __syncthreads();   // the previous token's codes have been copied out and its partial sums read
    const double A = dev::quant_token_group<NTILES, LC, false, dev::BlockSync, BF16>(cur, K, L, num, den, xch, xch,
                                                                                   red_d, red_i, sync, codes);
    __syncthreads();   // codes and partial sums are in LDS
#pragma unroll
    for (int tau = 0; tau < NTILES; ++tau) {
      const int64_t base = (int64_t)tau * S::T + 16 * t;
      if (base < K) *reinterpret_cast<uint4*>(act_q + (int64_t)m * K + base) = *reinterpret_cast<const uint4*>(codes + base);
    }
    if (t == 0) {
      act_scale[m] = (float)((A * (double)num) / denom);
      if (act_sum) act_sum[m] = red_i[0] + red_i[1] + red_i[2] + red_i[3];
    }
    if (!kPrefetch && m + (int)gridDim.x < M)
      dev::load_token_raw<256, NTILES>(raw, x + (int64_t)(m + gridDim.x) * K, K);
  }
}

// One workgroup of G groups of four waves per token, TPG tiles to a group one after another (G TPG >=
// NTILES).
template <int NTILES, int G, int LC, bool BF16>
__global__ __launch_bounds__(256 * G) void k_act_wide(const uint16_t* __restrict__ x, int64_t K, int L, int num,
                                                      int den, double denom, int8_t* __restrict__ act_q,
                                                      float* __restrict__ act_scale, int32_t* __restrict__ act_sum,
                                                      int wait_limit, uint32_t* __restrict__ err) {
  using S = dev::Tile<256, 16>;
  constexpr int TPG = (NTILES + G - 1) / G;
  extern __shared__ __align__(16) double xch_all[];   // G exchange buffers of S::LDS_DOUBLES
  __shared__ double red_d[4 * G];
  __shared__ int red_i[4 * G];
  __shared__ unsigned ctr[G];
  const int gi = threadIdx.x >> 8, t = threadIdx.x & 255, lane = t & 63, w = t >> 6;
  if (threadIdx.x < G) ctr[threadIdx.x] = 0u;
  __syncthreads();
  dev::GroupSync<4> gs{ctr + gi, 0u, wait_limit, err};
  const int m = blockIdx.x;
  const int Lc = LC > 0 ? LC : L;
  double* xch = xch_all + gi * S::LDS_DOUBLES;
  // tiles gi + G i of token m: 16 consecutive elements per thread (zeros past K)
  const __amdgpu_buffer_rsrc_t r = dev::make_rsrc(x + (int64_t)m * K, (uint32_t)(K * 2));
  uint4 raw[TPG][2];
  int64_t base[TPG];
#pragma unroll
  for (int i = 0; i < TPG; ++i) {
    base[i] = (int64_t)(gi + G * i) * S::T + 16 * t;
    const uint32_t off = base[i] < K ? (uint32_t)(base[i] * 2) : dev::kOutOfRange;
    raw[i][0] = dev::bload16(r, off);
    raw[i][1] = dev::bload16(r, off + 16);
  }
  double v[TPG][16];
  int wend = 0;
  double amax = 0.0;
#pragma unroll
  for (int i = 0; i < TPG; ++i) {
    dev::unpack16<BF16>(v[i], raw[i]);
    if (i > 0 && Lc > 6) gs();   // the previous tile's exchange reads are done
    wend = dev::fwht_tile_s<256, 16, false>(v[i], xch, t, Lc, gs);
#pragma unroll
    for (int e = 0; e < 16; ++e) amax = fmax(amax, fabs(v[i][e]));
  }
  amax = dev::wave_max(amax);
  if (lane == 0) red_d[4 * gi + w] = amax;
  __syncthreads();   // every group's maxima are in
  double A = red_d[0];
#pragma unroll
  for (int k = 1; k < 4 * G; ++k) A = fmax(A, red_d[k]);
  const dev::QuantParams p = dev::make_qparams(A, num, den);
  int q[TPG][16];
  int qs = 0;
#pragma unroll
  for (int i = 0; i < TPG; ++i) {
    dev::quant16(v[i], p, q[i]);
#pragma unroll
    for (int e = 0; e < 16; ++e) qs += q[i][e];
  }
  // the codes in natural order through the group's exchange buffer (its exchange reads are done
  // once every wave of the group has passed the wave barrier), then 16 bytes per thread and tile
  gs();
  int8_t* codes = reinterpret_cast<int8_t*>(xch);
#pragma unroll
  for (int i = 0; i < TPG; ++i) {
    if (wend == 0) dev::store_codes<0>(codes + i * S::T, q[i], t);
    else if (wend == 4) dev::store_codes<4>(codes + i * S::T, q[i], t);
    else dev::store_codes<8>(codes + i * S::T, q[i], t);
  }
  gs();
#pragma unroll
  for (int i = 0; i < TPG; ++i)
    if (base[i] < K)
      *reinterpret_cast<uint4*>(act_q + (int64_t)m * K + base[i]) =
          *reinterpret_cast<const uint4*>(codes + i * S::T + 16 * t);
  qs = dev::wave_sum(qs);
  if (lane == 0) red_i[4 * gi + w] = qs;
  __syncthreads();
  if (threadIdx.x == 0) {
    act_scale[m] = (float)((A * (double)num) / denom);
    if (act_sum) {
      int sum = 0;
#pragma unroll
      for (int k = 0; k < 4 * G; ++k) sum += red_i[k];
      act_sum[m] = sum;
    }
  }
}

template <int NTILES, int G, int LC, bool BF16>
hipError_t launch_wide_l(const uint16_t* x, int64_t M, int64_t K, int L, int num, int den, double denom, int8_t* q,
                         float* sc, int32_t* sum, hipStream_t s) {
  constexpr size_t shmem = (size_t)G * dev::Tile<256, 16>::LDS_DOUBLES * 8;
  // the dynamic LDS this instance takes (the kernel's static LDS comes on top of it)
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_act_wide<NTILES, G, LC, BF16>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((k_act_wide<NTILES, G, LC, BF16>), dim3((unsigned)M), dim3(256 * G), shmem, s, x, K, L, num,
                     den, denom, q, sc, sum, wait_limit(), device_error_word());
  return hipGetLastError();
}

template <int NTILES, int LC, bool BF16>
hipError_t launch_tokens_l(const uint16_t* x, int64_t M, int64_t K, int L, int num, int den, double denom,
                           int8_t* q, float* sc, int32_t* sum, hipStream_t s) {
  // persistent grid: every workgroup that fits on the chip at once (queried once per instance)
  static const int resident = [] {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(&k_act_tokens<NTILES, LC, BF16>),
                                                     256, 0) != hipSuccess || per_cu < 1)
      per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 256;
    return per_cu * cus;
  }();
  const unsigned grid = (unsigned)(M < resident ? M : resident);
  hipLaunchKernelGGL((k_act_tokens<NTILES, LC, BF16>), dim3(grid), dim3(256), 0, s, x, (int)M, K, L, num, den, denom, q,
                     sc, sum);
  return hipGetLastError();
}

// block exponents compiled as constants: 12, 11, 8 and 6; anything else at run time
template <int NTILES, int G, bool BF16>
hipError_t launch_wide(const uint16_t* x, int64_t M, int64_t K, int L, int num, int den, double denom, int8_t* q,
                       float* sc, int32_t* sum, hipStream_t s) {
  switch (L) {
    case 12: return launch_wide_l<NTILES, G, 12, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
    case 11: return launch_wide_l<NTILES, G, 11, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
    case 8: return launch_wide_l<NTILES, G, 8, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
    case 6: return launch_wide_l<NTILES, G, 6, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
    default: return launch_wide_l<NTILES, G, 0, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
  }
}

template <int NTILES, bool BF16>
hipError_t launch_tokens(const uint16_t* x, int64_t M, int64_t K, int L, int num, int den, double denom,
                         int8_t* q, float* sc, int32_t* sum, hipStream_t s) {
  if constexpr (NTILES > 1) {
    if (M <= kActWideMaxM) return launch_wide<NTILES, NTILES, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
  }
  if constexpr (NTILES > 3) {
    return launch_wide<NTILES, 2, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
  } else {
    switch (L) {
      case 12: return launch_tokens_l<NTILES, 12, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
      case 11: return launch_tokens_l<NTILES, 11, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
      case 8: return launch_tokens_l<NTILES, 8, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
      case 6: return launch_tokens_l<NTILES, 6, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
      default: return launch_tokens_l<NTILES, 0, BF16>(x, M, K, L, num, den, denom, q, sc, sum, s);
    }
  }
}

template <int NT, bool BF16>
hipError_t launch_nt(const uint16_t* x, int64_t M, int64_t K, int L, int num, int den, double denom,
                     int8_t* q, float* sc, int32_t* sum, hipStream_t s) {
  const int64_t T = 16 * NT;
  const int nt = (int)((K + T - 1) / T);
  const dim3 grid((unsigned)M), block(NT);
  switch (nt) {
    case 1: hipLaunchKernelGGL((k_rotate_quant_act<NT, 1, BF16>), grid, block, 0, s, x, K, L, num, den, denom, q, sc, sum); break;
    case 2: hipLaunchKernelGGL((k_rotate_quant_act<NT, 2, BF16>), grid, block, 0, s, x, K, L, num, den, denom, q, sc, sum); break;
    case 3: hipLaunchKernelGGL((k_rotate_quant_act<NT, 3, BF16>), grid, block, 0, s, x, K, L, num, den, denom, q, sc, sum); break;
    case 4: hipLaunchKernelGGL((k_rotate_quant_act<NT, 4, BF16>), grid, block, 0, s, x, K, L, num, den, denom, q, sc, sum); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

double act_denominator(int block, int clip_den) {
  // the fixed divisor of the per-token scale, (den * 7) * sqrt(b), rounded in that order
  return ((double)clip_den * 7.0) * sqrt((double)block);
}

template <bool BF16>
hipError_t launch_rqa(const uint16_t* x, int64_t M, int64_t K, int block, int clip_num, int clip_den, int8_t* act_q,
                      float* act_scale, int32_t* act_sum, hipStream_t s) {
  const int L = dev::ilog2c(block);
  const double denom = act_denominator(block, clip_den);
  if (block <= 4096 && K <= 4 * 4096) {
    switch ((K + 4095) / 4096) {
      case 1: return launch_tokens<1, BF16>(x, M, K, L, clip_num, clip_den, denom, act_q, act_scale, act_sum, s);
      case 2: return launch_tokens<2, BF16>(x, M, K, L, clip_num, clip_den, denom, act_q, act_scale, act_sum, s);
      case 3: return launch_tokens<3, BF16>(x, M, K, L, clip_num, clip_den, denom, act_q, act_scale, act_sum, s);
      default: return launch_tokens<4, BF16>(x, M, K, L, clip_num, clip_den, denom, act_q, act_scale, act_sum, s);
    }
  }
  return launch_nt<512, BF16>(x, M, K, L, clip_num, clip_den, denom, act_q, act_scale, act_sum, s);
}

hipError_t launch_rotate_quant_act(const uint16_t* x, int64_t M, int64_t K, int block, int clip_num,
                                   int clip_den, int8_t* act_q, float* act_scale, int32_t* act_sum,
                                   hipStream_t s, bool bf16) {
  return bf16 ? launch_rqa<true>(x, M, K, block, clip_num, clip_den, act_q, act_scale, act_sum, s)
              : launch_rqa<false>(x, M, K, block, clip_num, clip_den, act_q, act_scale, act_sum, s);
}

}  // namespace qift
