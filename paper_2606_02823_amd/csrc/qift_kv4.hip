// KV4: the asymmetric 4-bit key/value cache of the W2A4/KV4 setting (Sec. 3.3 Eq. (15) with the
// Sec. 4.1 configuration: clipping ratio 0.95 for keys and values) and one decode step of
// grouped-query attention that reads it.
//
// Quantizer (k_kv4_quant): 16 lanes per group of 128 values (one token's key or value vector of
// one KV head), lane j holding values 8j .. 8j + 7 (one 16-byte load, one 4-byte store of their
// codes), 4 groups per wave and step.  In fp32, in this order, rounding
// half to even:
//   x_max = c max(max x, 0), x_min = c min(min x, 0) with c = fp32(0.95),
//   s = (x_max - x_min) / 15 (1 for a group of zeros), z = round(-x_min / s),
//   q = clip(round(x / s) + z, 0, 15),   reconstruction s (q - z).
// Codes are packed two per byte, value 2i in the low nibble of byte i: the cache holds 64 bytes
// of codes, an fp32 scale and a zero-point byte per token and KV head.
//
// Decode attention (k_kv4_attn, then a merge kernel: k_kv4_merge_regs or k_kv4_merge): for query head h and KV head h / G (G = Hq / Hkv),
//   out_h = sum_t softmax_t(q_h . k_t / sqrt(d)) v_t.
// Workgroup (chunk, kv, b) covers 256 cached tokens for the G query heads of one KV head and
// writes its unnormalized partial output with the chunk's maximum score and sum of exponentials;
// the merge kernel combines the chunks.  The reconstruction is folded into the sums:
//   q . k_t = s_t sum_i (code_{t,i} - z_t) q_i,
//   sum_t p_t v_t = sum_t (p_t s_t) code_t - sum_t p_t s_t z_t,
// so both phases run on the f16 MFMA with the codes as exact fp16 operands: the key phase codes x
// queries (16 tokens x 32 dimensions per instruction), the value phase P = p s (split into two fp16
// parts) x codes (16 heads x 32 tokens x 16 dimensions), its operands read from LDS with the 4-bit
// transposing read.  A workgroup issues all its loads first and waits on HBM once.  What a workgroup
// spends after its loads bounds the kernel (its vector instructions took 66 % of the cycles, and six
// workgroups share a CU), so scores, weights and statistics go through LDS 16 bytes a lane and the
// reductions through DPP: B = 16, T = 4096, 32 / 8 heads 26.4 -> 23.9 us with the merge (3.0 TB/s; 14 us at a
// large copy's rate), B = 1 9.0 -> 8.0.
#include "qift_fwht.h"
#include "qift_internal.h"

namespace qift {
namespace {

constexpr int kD = 128;         // head dimension
constexpr int kChunk = 256;     // cached tokens per workgroup

typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

// Eight 4-bit codes of a word (nibble n at bits 4n) as MFMA fp16 operands without conversion: a code
// masked in place within a 16-bit half is an exact fp16 subnormal, code 2^-24 (bits 0-3 of the half)
// or code 2^-20 (bits 4-7).  Element e is nibble kNib[e]; elements with e & 2 carry the 2^-20 kind,
// so the other operand's element e takes a factor 1/16 there and the product sums are 2^-24 times
// the code sums.  The f16 MFMA sums products of subnormal inputs less precisely than those of
// normal ones (measured on gfx950: about 9e-7 against 6e-8 of the sum of |products|), which the
// value phase can afford (its error is linear in the output) and the scores cannot.
constexpr int kNib[8] = {0, 4, 1, 5, 2, 6, 3, 7};
__device__ __forceinline__ v8h codes_f16(uint32_t w) {
  const uint32_t w8 = w >> 8;
  const uint4 h = {w & 0x000F000Fu, w & 0x00F000F0u, w8 & 0x000F000Fu, w8 & 0x00F000F0u};
  return __builtin_bit_cast(v8h, h);
}

// Eight 4-bit codes of one group minus its zero-point z, as exact normal fp16 values: a byte
// permute puts each code below an 0x64 byte (the fp16 value 1024 + code) and a packed subtraction
// of 1024 + z leaves code - z.  Element e is nibble kNibK[e] of the word.
constexpr int kNibK[8] = {0, 2, 4, 6, 1, 3, 5, 7};
__device__ __forceinline__ v8h codes_minus_z(uint32_t w, v2h base) {
  const uint32_t lo = w & 0x0F0F0F0Fu, hi = (w >> 4) & 0x0F0F0F0Fu;   // byte m: nibble 2m / 2m + 1
  const uint32_t k64 = 0x64646464u;
  // selector bytes 0-3 pick from the second operand, 4-7 from the first (all 0x64)
  const uint32_t s01 = 0x04010400u, s23 = 0x04030402u;
  const v2h h0 = __builtin_bit_cast(v2h, __builtin_amdgcn_perm(k64, lo, s01)) - base;   // nibbles 0, 2
  const v2h h1 = __builtin_bit_cast(v2h, __builtin_amdgcn_perm(k64, lo, s23)) - base;   // nibbles 4, 6
  const v2h h2 = __builtin_bit_cast(v2h, __builtin_amdgcn_perm(k64, hi, s01)) - base;   // nibbles 1, 3
  const v2h h3 = __builtin_bit_cast(v2h, __builtin_amdgcn_perm(k64, hi, s23)) - base;   // nibbles 5, 7
  return v8h{h0[0], h0[1], h1[0], h1[1], h2[0], h2[1], h3[0], h3[1]};
}

// Reductions by DPP moves within rows of 16 lanes (every lane gets its row's result) and lane reads across
// the four rows: a few cycles a step, where a shuffle through LDS takes about a hundred.
#define QIFT_DPP_B32(x, CTRL) __builtin_amdgcn_update_dpp(x, x, CTRL, 0xf, 0xf, false)
template <typename Op>
__device__ __forceinline__ int row_reduce(int x, Op op) {
  x = op(x, QIFT_DPP_B32(x, 0xb1));    // quad_perm [1,0,3,2]
  x = op(x, QIFT_DPP_B32(x, 0x4e));    // quad_perm [2,3,0,1]
  x = op(x, QIFT_DPP_B32(x, 0x141));   // row_half_mirror
  return op(x, QIFT_DPP_B32(x, 0x140));   // row_mirror
}

template <typename Op>
__device__ __forceinline__ float wave_reduce(float x, Op op) {   // every lane gets the wave's result
  const int r = row_reduce(__float_as_int(x), [&](int a, int b) {
    return __float_as_int(op(__int_as_float(a), __int_as_float(b)));
  });
  auto row = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(r, l)); };
  return op(op(row(0), row(16)), op(row(32), row(48)));
}
__device__ __forceinline__ float max_op(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float add_op(float a, float b) { return a + b; }

__device__ __forceinline__ v2h pk_max(v2h a, v2h b) { return __builtin_elementwise_max(a, b); }

// d / 15 correctly rounded for a finite d >= 0 that is 0 or far above the subnormals (the values here are
// fp16 times 0.95): the quotient by the rounded reciprocal, then one correction (checked against the
// division for every fp32 mantissa).
__device__ __forceinline__ float div15(float d) {
  constexpr float y = 1.0f / 15.0f;
  const float q = d * y;
  return d == INFINITY ? d : fmaf(fmaf(-q, 15.0f, d), y, q);
}

// Bound by its arithmetic: 25 vector instructions a value took 85 % of the cycles (3.3 TB/s at 524288
// groups).  So the maxima run on packed fp16 pairs (max x and max -x in one register through the row
// moves), the reciprocal is the hardware's approximation (the residual test decides as before), one
// running maximum of the residuals replaces a test per value, and the codes are packed by bytes.
// 524288 groups, 170 MB: 52.4 -> 44.4 us (3.8 TB/s), 65536: 8.8 -> 7.4.
__global__ __launch_bounds__(256) void k_kv4_quant(const uint16_t* __restrict__ x, int64_t groups,
                                                   uint8_t* __restrict__ codes, float* __restrict__ scales,
                                                   uint8_t* __restrict__ zeros, int per) {
  const int lane = threadIdx.x & 63, j = lane & 15;
  const int64_t quads = (groups + 3) / 4;
  // the next step's values are loaded while this step's are quantized
  auto load = [&](int64_t wq) {   // lanes of a missing group run along with zeros (the row moves need them)
    const int64_t grp = wq * 4 + (lane >> 4);
    uint4 u = {0u, 0u, 0u, 0u};
    if (grp < groups) u = reinterpret_cast<const uint4*>(x + grp * kD)[j];
    return u;
  };
  // per steps of 16 consecutive groups to a workgroup
  int64_t wq = ((int64_t)blockIdx.x * per) * 4 + (threadIdx.x >> 6);
  uint4 next = load(wq);
  for (int i = 0; i < per && wq < quads; ++i, wq += 4) {
    const int64_t grp = wq * 4 + (lane >> 4);
    const uint4 u = next;
    if (i + 1 < per) next = load(wq + 4);
    const v2h h[4] = {__builtin_bit_cast(v2h, u.x), __builtin_bit_cast(v2h, u.y), __builtin_bit_cast(v2h, u.z),
                      __builtin_bit_cast(v2h, u.w)};
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)h[e >> 1][e & 1];
    // (max x, max -x) of the lane, then of its group's 16 lanes
    const v2h hx = pk_max(pk_max(h[0], h[1]), pk_max(h[2], h[3]));
    const v2h hn = pk_max(pk_max(-h[0], -h[1]), pk_max(-h[2], -h[3]));
    const v2h both = pk_max(v2h{hx[0], hn[0]}, v2h{hx[1], hn[1]});
    const v2h ext = __builtin_bit_cast(v2h, row_reduce(__builtin_bit_cast(int, both), [](int a, int b) {
                                         return __builtin_bit_cast(int, pk_max(__builtin_bit_cast(v2h, a), __builtin_bit_cast(v2h, b)));
                                       }));
    const float c = 0.95f;
    const float x_max = fmaxf((float)ext[0], 0.f) * c, x_min = fminf(-(float)ext[1], 0.f) * c;
    float s = div15(x_max - x_min);
    if (s == 0.f) s = 1.f;
    // rint of the rounded quotient v / s without the division where it is clear: q0 = rint(v r), r the
    // approximate reciprocal, is that value when the residual v - q0 s lies inside half a step by more
    // than both roundings (|v / s| < 32 here); otherwise (a wave-uniform branch, rarely taken) divide.
    // The zero-point is decided the same way.
    const float inv = __builtin_amdgcn_rcpf(s);
    float qf[8];
    float z = rintf(-x_min * inv);
    float res = fabsf(fmaf(-z, s, -x_min));
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      qf[e] = rintf(v[e] * inv);
      res = fmaxf(res, fabsf(fmaf(-qf[e], s, v[e])));
    }
    const float half = (0.5f - 0x1p-16f) * s;
    if (__any(!(res < half))) {
      z = rintf(-x_min / s);
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[e] = rintf(v[e] / s);
    }
    z = fminf(fmaxf(z, 0.f), 15.f);
    // codes as bytes, even values and odd ones, then two to a byte: values 8j .. 8j + 7
    uint32_t even = 0, odd = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float q = fminf(fmaxf(qf[e] + z, 0.f), 15.f);
      if (e & 1) odd = __builtin_amdgcn_cvt_pk_u8_f32(q, e >> 1, odd);
      else even = __builtin_amdgcn_cvt_pk_u8_f32(q, e >> 1, even);
    }
    if (grp < groups) {
      reinterpret_cast<uint32_t*>(codes + grp * (kD / 2))[j] = even | (odd << 4);
      if (j == 0) {
        scales[grp] = s;
        zeros[grp] = (uint8_t)z;
      }
    }
  }
}

// partial record of one (b, kv, chunk, g): kD unnormalized output sums, then the chunk's maximum
// score m and sum of exp(score - m)
constexpr int kPart = kD + 2;

template <int G>
__global__ __launch_bounds__(256) void k_kv4_attn(const uint16_t* __restrict__ q, int Hq, int Hkv, int64_t T,
                                                  const uint8_t* __restrict__ kc, const float* __restrict__ ks,
                                                  const uint8_t* __restrict__ kz, const uint8_t* __restrict__ vc,
                                                  const float* __restrict__ vs, const uint8_t* __restrict__ vz,
                                                  float* __restrict__ part, int nchunks, int head_major,
                                                  uint16_t* __restrict__ y) {
  constexpr int Gp = G < 4 ? 4 : G;      // heads per value-phase output row, padded to a float4
  __shared__ __attribute__((aligned(16))) float pr[G][kChunk];   // scores, then P_t f_g (below)
  __shared__ __attribute__((aligned(16))) float sz[4][kChunk];   // key scale, key zero-point, value scale, value zero-point
  __shared__ float stat[G][4];           // m, l, Z, 2^24 / f_g
  // value codes, 64 bytes per token with the 16-byte slots of row r XOR-swizzled by (r / 4) mod 4
  // (the transposed reads below then hit 32 distinct banks per 16 lanes); once a wave has read its
  // 64 rows it reuses them for its partial sums [dimension][Gp]
  __shared__ __attribute__((aligned(16))) uint32_t vl[kChunk * (kD / 8)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunk = blockIdx.x, kv = blockIdx.y;
  const int64_t b = blockIdx.z;
  const int64_t t0 = (int64_t)chunk * kChunk;
  const int nt = (int)(T - t0 < kChunk ? T - t0 : kChunk);   // tokens of this chunk
  // cache row of token t: row0 + t rs, rows ordered [B][T][Hkv] (token-major) or [B][Hkv][T]
  const uint32_t rs = head_major ? 1u : (uint32_t)Hkv;
  const int64_t row0 = head_major ? ((int64_t)b * Hkv + kv) * T : (b * T) * Hkv + kv;
  const uint32_t rows = (uint32_t)(T * rs);    // T Hkv 64 < 2^31: checked by the host, so 32-bit
  const uint32_t rc = (uint32_t)t0 * rs;       // offsets below cannot wrap
  const __amdgpu_buffer_rsrc_t kcr = dev::make_rsrc(kc + row0 * (kD / 2), rows * (kD / 2));
  const __amdgpu_buffer_rsrc_t vcr = dev::make_rsrc(vc + row0 * (kD / 2), rows * (kD / 2));
  const __amdgpu_buffer_rsrc_t ksr = dev::make_rsrc(ks + row0, rows * 4u);
  const __amdgpu_buffer_rsrc_t vsr = dev::make_rsrc(vs + row0, rows * 4u);
  const __amdgpu_buffer_rsrc_t kzr = dev::make_rsrc(kz + row0, rows);
  const __amdgpu_buffer_rsrc_t vzr = dev::make_rsrc(vz + row0, rows);

  // ---- every load of the chunk is issued before any is used, so a workgroup waits on HBM once.
  // Range-checked buffer loads return zeros for tokens past T (their weights are zeroed below).
  // Thread tid: scale and zero-point of token t0 + tid, key and value.
  float own[4];
  {
    const bool ok = tid < nt;
    const uint32_t r = rc + (uint32_t)tid * rs;
    own[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ksr, ok ? 4u * r : dev::kOutOfRange, 0, 0));
    own[1] = (float)__builtin_amdgcn_raw_buffer_load_b8(kzr, ok ? r : dev::kOutOfRange, 0, 0);
    own[2] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vsr, ok ? 4u * r : dev::kOutOfRange, 0, 0));
    own[3] = (float)__builtin_amdgcn_raw_buffer_load_b8(vzr, ok ? r : dev::kOutOfRange, 0, 0);
  }
  // Key phase operands, lane (c, kg) = (lane mod 16, lane / 16): the A operand of tile i is 16
  // tokens' codes, a lane loading the 16 bytes of dimensions 32 kg .. + 31 of token 64 wave + 16 i + c,
  // word st holding dimensions 32 kg + 8 st + n in nibble n; the B operand holds the G queries
  // (columns >= G zero) with element e of k-step st = dimension 32 kg + 8 st + kNibK[e] (the MFMA
  // pairs A and B element by element within a lane group).
  // (branch-free range-checked loads: a branch here would make the compiler wait for every load
  // issued so far before the code loads below are issued)
  const int c = lane & 15, kg = lane >> 4;
  const __amdgpu_buffer_rsrc_t qr = dev::make_rsrc(q + (b * Hq + (int64_t)kv * G) * kD, G * kD * 2u);
  uint4 qu[4];
#pragma unroll
  for (int st = 0; st < 4; ++st)
    qu[st] = dev::bload16(qr, c < G ? 2u * (c * kD + 32 * kg + 8 * st) : dev::kOutOfRange);
  uint4 kw[4];
#pragma unroll
  for (int tile = 0; tile < 4; ++tile) {
    const int tl = 64 * wave + 16 * tile + c;
    kw[tile] = dev::bload16(kcr, tl < nt ? (rc + (uint32_t)tl * rs) * (kD / 2) + 16u * kg : dev::kOutOfRange);
  }
  // Value codes of the wave's 64 tokens: load u, lane l takes 16-byte slot l mod 4 of token
  // 64 wave + 16 u + l / 4 (it goes to LDS before the value phase).
  uint4 vq[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int tl = 64 * wave + 16 * u + (lane >> 2);
    vq[u] = dev::bload16(vcr, tl < nt ? (rc + (uint32_t)tl * rs) * (kD / 2) + 16u * (lane & 3) : dev::kOutOfRange);
  }

  v8h qb[4];
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const v8h qraw = __builtin_bit_cast(v8h, qu[st]);
#pragma unroll
    for (int e = 0; e < 8; ++e) qb[st][e] = qraw[kNibK[e]];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) sz[i][tid] = own[i];
  __syncthreads();

  // ---- scores on the f16 MFMA: per 16 tokens, D[token][head] = sum over the 128 dimensions of
  // (code - z_t) x query (4 MFMAs of 32 dimensions, every operand exact); q . k_t = s_t D.
  {
    const float rsd = 1.0f / sqrtf((float)kD);
#pragma unroll
    for (int tile = 0; tile < 4; ++tile) {
      const uint32_t ww[4] = {kw[tile].x, kw[tile].y, kw[tile].z, kw[tile].w};
      const _Float16 zb = (_Float16)(1024.0f + sz[1][64 * wave + 16 * tile + c]);   // exact: z <= 15
      const v2h base = {zb, zb};
      v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 4; ++st)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(codes_minus_z(ww[st], base), qb[st], acc, 0, 0, 0);
      // D: lane (c, kg) holds tokens 16 tile + 4 kg + i of head c (four at a time to LDS; a row of pr past
      // the G heads does not exist)
      const int t4 = 64 * wave + 16 * tile + 4 * kg;
      v4f sc = *reinterpret_cast<const v4f*>(&sz[0][t4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[i] = sc[i] * acc[i] * rsd;
      if (nt < kChunk) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[i] = t4 + i < nt ? sc[i] : -INFINITY;
      }
      if (c < G) *reinterpret_cast<v4f*>(&pr[c][t4]) = sc;
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = 64 * wave + 16 * u + (lane >> 2);   // (row / 4) mod 4 = (lane / 16) mod 4
    *reinterpret_cast<uint4*>(&vl[row * (kD / 8) + 4 * ((lane & 3) ^ ((lane >> 4) & 3))]) = vq[u];
  }
  __syncthreads();

  // ---- the chunk's softmax statistics, one wave per head: m, l = sum_t e_t with e_t = exp(score_t
  // - m), and for the value phase P_t = e_t s_t and Z = sum_t P_t z_t.  pr receives P_t f_g with f_g
  // the power of two that puts the chunk's largest P in [2^14, 2^15): the value phase splits it into
  // two fp16 parts without overflow and with the small terms far above the fp16 subnormal range.
  for (int g = wave; g < G; g += 4) {
    // lane l takes tokens 4 l .. 4 l + 3 (one 16-byte access per array)
    static_assert(kChunk == 256, "four tokens a lane");
    v4f v = *reinterpret_cast<const v4f*>(&pr[g][4 * lane]);
    const v4f vs4 = *reinterpret_cast<const v4f*>(&sz[2][4 * lane]), vz4 = *reinterpret_cast<const v4f*>(&sz[3][4 * lane]);
    const float m = wave_reduce(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), max_op);
    float l = 0.f, zs = 0.f, pm = __FLT_MIN__;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = expf(v[i] - m);   // 0 for tokens past T (-infinity)
      const float P = e * vs4[i];
      v[i] = P;
      pm = fmaxf(pm, P);
      l += e;
      zs = fmaf(P, vz4[i], zs);
    }
    l = wave_reduce(l, add_op);
    zs = wave_reduce(zs, add_op);
    pm = wave_reduce(pm, max_op);
    const int ex = ilogbf(pm);   // pm normal: P of the top token is its scale s > 0
    const float f = ldexpf(1.0f, 14 - ex);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] *= f;
    *reinterpret_cast<v4f*>(&pr[g][4 * lane]) = v;
    if (lane == 0) {
      stat[g][0] = m;
      stat[g][1] = l;
      stat[g][2] = zs;
      stat[g][3] = ldexpf(1.0f, 10 + ex);   // 2^24 / f
    }
  }
  __syncthreads();

  // ---- values on the f16 MFMA: D[head][dim] = sum over the wave's 64 tokens of A[head][token]
  // B[token][dim], A = P f (rows >= G zero) as an fp16 high part plus an fp16 low part (two MFMAs,
  // 2^-22 relative), B = the codes.  The transposing LDS read gives lane (i, kg) = (lane mod 16,
  // lane / 16) the 16 codes of dimension 16 dt + i for tokens 64 wave + 16 kg + 0 .. 15 (the rows
  // that the 16 lanes of its group address), nibble n for token n.  B element e is the code of
  // token kNib[e] of the word (codes_f16), and the A element it meets carries 1/16 where e & 2:
  // D = 2^-24 sum_t P_t f code_t.  Z is subtracted when the partial is written.
  {
    const int i16 = lane & 15, kg = lane >> 4;
    v8h ahi[2], alo[2];
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      float pv[8];
      if (i16 < G) {
        const float4 x0 = *reinterpret_cast<const float4*>(&pr[i16][64 * wave + 16 * kg + 8 * st]);
        const float4 x1 = *reinterpret_cast<const float4*>(&pr[i16][64 * wave + 16 * kg + 8 * st + 4]);
        pv[0] = x0.x; pv[1] = x0.y; pv[2] = x0.z; pv[3] = x0.w;
        pv[4] = x1.x; pv[5] = x1.y; pv[6] = x1.z; pv[7] = x1.w;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[e] = 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const float x = (e & 2) ? pv[kNib[e]] * 0.0625f : pv[kNib[e]];
        const float y = (e & 2) ? pv[kNib[e + 1]] * 0.0625f : pv[kNib[e + 1]];
        const v2h h = __builtin_bit_cast(v2h, __builtin_amdgcn_cvt_pkrtz(x, y));
        const v2h r = __builtin_bit_cast(v2h, __builtin_amdgcn_cvt_pkrtz(x - (float)h[0], y - (float)h[1]));
        ahi[st][e] = h[0];
        ahi[st][e + 1] = h[1];
        alo[st][e] = r[0];
        alo[st][e + 1] = r[1];
      }
    }
    const int row = 64 * wave + 16 * kg + i16;   // the row this lane addresses
    v4f acc[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      const uint32_t off = row * (kD / 8) + 4 * ((dt >> 1) ^ ((row >> 2) & 3)) + 2 * (dt & 1);
      const v2i t = __builtin_amdgcn_ds_read_tr4_b64_v2i32((__attribute__((address_space(3))) v2i*)(vl + off));
      acc[dt] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        const v8h bv = codes_f16(st ? (uint32_t)t.y : (uint32_t)t.x);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi[st], bv, acc[dt], 0, 0, 0);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(alo[st], bv, acc[dt], 0, 0, 0);
      }
    }
    // D lane (i16, kg) holds heads 4 kg .. 4 kg + 3 of dimension 16 dt + i16; the wave's own rows
    // take them (its transposed reads above are done: a wave's LDS operations complete in order)
    if (4 * kg < G) {
      float* red = reinterpret_cast<float*>(vl) + 64 * wave * (kD / 8);
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
        *reinterpret_cast<v4f*>(&red[(16 * dt + i16) * Gp + 4 * kg]) = acc[dt];
    }
  }
  __syncthreads();
  float* out = part + ((((int64_t)b * Hkv + kv) * nchunks + chunk) * G) * kPart;
  const float* red = reinterpret_cast<const float*>(vl);
  constexpr int kWaveRed = 64 * (kD / 8);   // floats per wave's region
  for (int i = tid; i < G * kD; i += 256) {
    const int g = i / kD, dd = i % kD, o = dd * Gp + g;
    const float sum = (red[o] + red[kWaveRed + o]) + (red[2 * kWaveRed + o] + red[3 * kWaveRed + o]);
    const float o_dd = sum * stat[g][3] - stat[g][2];
    // a cache of one chunk needs no merge: its weight is 1 (250 tokens of four sequences: 8.3 -> 5.3 us)
    if (nchunks == 1) y[(b * Hq + (int64_t)kv * G + g) * kD + dd] = __half_as_ushort(__float2half_rn(o_dd / stat[g][1]));
    else out[g * kPart + dd] = o_dd;
  }
  if (nchunks > 1 && tid < G) {
    out[tid * kPart + kD] = stat[tid][0];
    out[tid * kPart + kD + 1] = stat[tid][1];
  }
}

// out[b][kv G + g][:] = sum_c e^(m_c - M) part_c / sum_c e^(m_c - M) l_c,  M = max_c m_c.
// Up to NC chunks: thread dd loads its value and every chunk's m and l at once (independent loads,
// one wait on memory), then reduces in registers.
template <int G, int NC>
__global__ __launch_bounds__(kD) void k_kv4_merge_regs(const float* __restrict__ part, int Hq, int Hkv, int nchunks,
                                                       uint16_t* __restrict__ y) {
  const int dd = threadIdx.x;
  const int kv = blockIdx.x / G, g = blockIdx.x % G;
  const int64_t b = blockIdx.y;
  const float* base = part + (((int64_t)b * Hkv + kv) * nchunks) * G * kPart + g * kPart;
  const int64_t cstride = (int64_t)G * kPart;
  float pv[NC], mv[NC], lv[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const bool ok = c < nchunks;   // chunks past the count: weight 0
    const float* r = base + (ok ? c : 0) * cstride;
    pv[c] = r[dd];
    mv[c] = ok ? r[kD] : -INFINITY;
    lv[c] = r[kD + 1];
  }
  float M = mv[0];
#pragma unroll
  for (int c = 1; c < NC; ++c) M = fmaxf(M, mv[c]);
  float acc = 0.f, L = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const float e = c < nchunks ? expf(mv[c] - M) : 0.f;
    acc = fmaf(pv[c], e, acc);
    L = fmaf(lv[c], e, L);
  }
  y[(b * Hq + (int64_t)kv * G + g) * kD + dd] = __half_as_ushort(__float2half_rn(acc / L));
}

// More chunks: workgroup (kv G + g, b) of S x 128 threads (S = blockDim.x / 128 <= kMergeSlices).
// Slice j takes batches of kMergeBatch chunks (chunks j kMergeBatch + i, then S kMergeBatch further
// on, ...), each batch's values and statistics loaded at once (one wait on memory per batch) and
// folded into the slice's running maximum and sums; the slices' results are rescaled to the common
// maximum through LDS.
constexpr int kMergeSlices = 8;
constexpr int kMergeBatch = 16;
template <int G>
__global__ __launch_bounds__(kMergeSlices * kD) void k_kv4_merge(const float* __restrict__ part, int Hq, int Hkv,
                                                                 int nchunks, uint16_t* __restrict__ y) {
  __shared__ float sacc[kMergeSlices][kD];
  __shared__ float sm[kMergeSlices], sl[kMergeSlices];
  const int S = blockDim.x / kD;
  const int tid = threadIdx.x, dd = tid % kD, slice = tid / kD;
  const int kv = blockIdx.x / G, g = blockIdx.x % G;
  const int64_t b = blockIdx.y;
  const float* base = part + (((int64_t)b * Hkv + kv) * nchunks) * G * kPart + g * kPart;
  const int64_t cstride = (int64_t)G * kPart;
  float m = -INFINITY, acc = 0.f, L = 0.f;
  for (int c0 = slice * kMergeBatch; c0 < nchunks; c0 += S * kMergeBatch) {
    float pv[kMergeBatch], mv[kMergeBatch], lv[kMergeBatch];
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      const bool ok = c0 + i < nchunks;      // chunks past the count: weight 0
      const float* r = base + (ok ? c0 + i : c0) * cstride;
      pv[i] = r[dd];
      mv[i] = ok ? r[kD] : -INFINITY;
      lv[i] = r[kD + 1];
    }
    float mb = mv[0];                        // chunk c0 exists: mb and the new maximum are finite
#pragma unroll
    for (int i = 1; i < kMergeBatch; ++i) mb = fmaxf(mb, mv[i]);
    const float mn = fmaxf(m, mb);
    const float sc = expf(m - mn);           // 0 for the first batch (m = -inf)
    acc *= sc;
    L *= sc;
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      const float e = c0 + i < nchunks ? expf(mv[i] - mn) : 0.f;
      acc = fmaf(pv[i], e, acc);
      L = fmaf(lv[i], e, L);
    }
    m = mn;
  }
  sacc[slice][dd] = acc;
  if (dd == 0) {
    sm[slice] = m;
    sl[slice] = L;
  }
  __syncthreads();
  if (tid < kD) {
    float M = sm[0];
    for (int j = 1; j < S; ++j) M = fmaxf(M, sm[j]);
    float a = 0.f, l = 0.f;
    for (int j = 0; j < S; ++j) {
      const float e = expf(sm[j] - M);       // 0 for a slice without chunks (sm = -inf, M finite)
      a = fmaf(sacc[j][tid], e, a);
      l = fmaf(sl[j], e, l);
    }
    y[(b * Hq + (int64_t)kv * G + g) * kD + tid] = __half_as_ushort(__float2half_rn(a / l));
  }
}

template <int G>
hipError_t launch_attn_g(const uint16_t* q, int64_t B, int Hq, int Hkv, int64_t T, const uint8_t* kc,
                         const float* ks, const uint8_t* kz, const uint8_t* vc, const float* vs,
                         const uint8_t* vz, uint16_t* y, float* part, int head_major, hipStream_t s) {
  const int nchunks = (int)((T + kChunk - 1) / kChunk);
  hipLaunchKernelGGL((k_kv4_attn<G>), dim3((unsigned)nchunks, (unsigned)Hkv, (unsigned)B), dim3(256), 0, s, q, Hq,
                     Hkv, T, kc, ks, kz, vc, vs, vz, part, nchunks, head_major, y);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nchunks == 1) return e;
  const dim3 mgrid((unsigned)(Hkv * G), (unsigned)B);
  if (nchunks <= 8) {
    hipLaunchKernelGGL((k_kv4_merge_regs<G, 8>), mgrid, dim3(kD), 0, s, part, Hq, Hkv, nchunks, y);
  } else if (nchunks <= 16) {
    hipLaunchKernelGGL((k_kv4_merge_regs<G, 16>), mgrid, dim3(kD), 0, s, part, Hq, Hkv, nchunks, y);
  } else if (nchunks <= 32) {
    hipLaunchKernelGGL((k_kv4_merge_regs<G, 32>), mgrid, dim3(kD), 0, s, part, Hq, Hkv, nchunks, y);
  } else {
    // slices of kMergeBatch chunks, at most kMergeSlices
    const int want = (nchunks + kMergeBatch - 1) / kMergeBatch;
    const int slices = want > kMergeSlices ? kMergeSlices : want;
    hipLaunchKernelGGL((k_kv4_merge<G>), dim3((unsigned)(Hkv * G), (unsigned)B), dim3(slices * kD), 0, s, part, Hq,
                       Hkv, nchunks, y);
  }
  return hipGetLastError();
}

}  // namespace

size_t kv4_attention_workspace(int64_t B, int64_t Hq, int64_t T) {
  const int64_t nchunks = (T + kChunk - 1) / kChunk;
  return (size_t)(B * Hq * nchunks * kPart) * sizeof(float);
}

hipError_t launch_kv4_quant(const uint16_t* x, int64_t groups, uint8_t* codes, float* scales, uint8_t* zeros,
                            hipStream_t s) {
  // Four steps to a workgroup where there are enough workgroups (their loads run ahead, and whole lines of
  // scales and zero-points come from one L2: 524288 groups 46.0 -> 44.4 us, 1048576 84.0 -> 79.0), else one
  // (131072: 12.8 us against 13.2; 4096: 2.3 against 3.7).
  const int per = groups < 262144 ? 1 : 4;
  hipLaunchKernelGGL(k_kv4_quant, dim3((unsigned)((groups + 16 * per - 1) / (16 * per))), dim3(256), 0, s, x, groups,
                     codes, scales, zeros, per);
  return hipGetLastError();
}

hipError_t launch_kv4_attention(const uint16_t* q, int64_t B, int Hq, int Hkv, int64_t T, int head_major,
                                const uint8_t* kc, const float* ks, const uint8_t* kz, const uint8_t* vc,
                                const float* vs, const uint8_t* vz, uint16_t* y, void* ws, hipStream_t s) {
  float* part = static_cast<float*>(ws);
  switch (Hq / Hkv) {
    case 1: return launch_attn_g<1>(q, B, Hq, Hkv, T, kc, ks, kz, vc, vs, vz, y, part, head_major, s);
    case 2: return launch_attn_g<2>(q, B, Hq, Hkv, T, kc, ks, kz, vc, vs, vz, y, part, head_major, s);
    case 4: return launch_attn_g<4>(q, B, Hq, Hkv, T, kc, ks, kz, vc, vs, vz, y, part, head_major, s);
    case 8: return launch_attn_g<8>(q, B, Hq, Hkv, T, kc, ks, kz, vc, vs, vz, y, part, head_major, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qift
