// Which kernel a linear on codes runs, and with which split over K: host arithmetic on sizes alone (no HIP),
// so that the rules can be read and tested in one place.
//
// Every line below is where one kernel's time crosses another's, measured on the grid of 15 row counts from 64
// to 40960, 12 K from 256 to 20480 and 20 token counts from 5 to 64, W2 (MNZ) and W4, weights streamed from
// HBM.  Figures are us, as kernel / the one it is compared with, rows x K at tokens.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace qift {

constexpr int64_t kBatchMaxM = 64;     // batch kernel (qift_batch.hip)
constexpr int64_t kCodesMaxM = 16;     // decode kernel on codes: one MFMA column block of tokens
constexpr int64_t kSkinnyMaxM = 64;    // skinny kernel (qift_skinny.hip)
constexpr int64_t kSkinnyMaxK = 16384;
constexpr int64_t kSkSplitMaxM = 47;   // its split over K (beyond, the batch kernel is always faster)
constexpr int kSkSlices = 8;           // its K-slice waves

namespace route {

// ---- GEMM split over K: tiles of 256 rows x 64 tokens, S ranges of us steps (256 k, W4 128).
// Where the tiles are few (4096 x 14336 at 65-512 tokens: 16 x ceil(M / 64) tiles, each a chain of 56 W2
// or 112 W4 steps whose loads are not hidden): S ranges of at least 4 W2 or 8 W4 steps (1024 k), about 512
// workgroups and no more than are resident at once.  W4 takes at least three ranges (two measured no
// faster).  From 33 tokens on (W4 24) wide (N >= 16384) and long (N >= 4096, K > 4096) linears have a plan too.
struct GemmSplit {
  int S = 1, us = 0;
};

inline GemmSplit gemm_split_plan(bool w4, int64_t N, int64_t M, int64_t K) {
  GemmSplit p;
  const int64_t bk = w4 ? 128 : 256, min_steps = w4 ? 8 : 4, min_s = w4 ? 3 : 2;
  const int64_t KT = (K + bk - 1) / bk, tiles = ((N + 255) / 256) * ((M + 63) / 64);
  p.us = (int)KT;
  const bool wide = M >= (w4 ? 24 : 33) && (N >= 16384 || (N >= 4096 && K > 4096));
  if (M <= 64 && !wide) return p;
  int64_t S = (512 + tiles - 1) / tiles;
  if (S > 512 / tiles) S = 512 / tiles;
  if (S > KT / min_steps) S = KT / min_steps;
  if (S < min_s) return p;
  p.us = (int)((KT + S - 1) / S);
  p.S = (int)((KT + p.us - 1) / p.us);   // every range holds at least one step
  return p;
}

// ---- tiles of the unsplit GEMM: 256 rows x 128, 96 or 64 tokens.
// A CU runs one or two workgroups (512 at once on the chip); times of a tile alone on its CU and of two there, at
// K = 4096 in us: whole rounds of two and then the rest decide.  128-token tiles spend the least on weights, 64-token
// tiles fill the chip from half as many tokens on (4096 x 4096 at 400 tokens 16.7 against 25.1), and 96-token
// tiles save the second tile that few CUs would take: 9000 x 7168 at 900 tokens 63.9 against 76.2 and 74.0 (65.9 for the
// former 64-token tiles of the 16-wide MFMA, three to a CU).  Over 1584 sizes within 0.1 % of the best tile on average.
inline int64_t tile_cost(int64_t tiles, int one, int two) {
  const int64_t rest = tiles % 512;
  return tiles / 512 * two + (rest == 0 ? 0 : rest <= 256 ? one : two);
}
inline int gemm_tile_tokens(bool w4, int64_t N, int64_t M) {
  const int64_t tn = (N + 255) / 256;
  const int64_t c128 = tile_cost(tn * ((M + 127) / 128), w4 ? 29 : 27, w4 ? 54 : 46);
  const int64_t c96 = tile_cost(tn * ((M + 95) / 96), w4 ? 26 : 22, w4 ? 46 : 38);
  const int64_t c64 = tile_cost(tn * ((M + 63) / 64), w4 ? 23 : 17, w4 ? 40 : 30);
  return c128 <= c96 && c128 <= c64 ? 128 : c96 <= c64 ? 96 : 64;
}

// ---- skinny linear split over K (W2): T = 4 tiles of 16 rows per workgroup, S ranges of us 256-k units,
// chosen for about one workgroup per CU with at most two units per slice; S = 0 for K <= 4096 (the codes
// per workgroup are few enough: measured faster unsplit) and when a linear has tiles enough without.
struct SkSplit {
  int T = 0, S = 0, us = 0, np = 0;
};

inline SkSplit skinny_split_plan(bool w4, int64_t N, int64_t M, int64_t K) {
  SkSplit p;
  if (w4 || M < 1 || M > kSkSplitMaxM || K > kSkinnyMaxK || N < 1 || K < 1) return p;
  const int T = 4;
  const int64_t tiles = (N + 15) / 16, gx = (tiles + T - 1) / T;
  const int ut = (int)((K + 255) / 256);
  if (ut <= 16) return p;
  int S = (int)((256 + gx / 2) / gx);
  if (S < 2) return p;
  const int min_s = (ut + kSkSlices * 2 - 1) / (kSkSlices * 2);   // at most two units per slice
  if (S < min_s) S = min_s;
  if (S > ut) S = ut;
  const int us = (ut + S - 1) / S;
  p.T = T;
  p.us = us;
  p.S = (ut + us - 1) / us;   // every range holds at least one unit
  p.np = (int)((N + 3) / 4 * 4);
  if (p.S < 2) p.S = 0;
  return p;
}

// ---- the kernels
enum Kernel {
  kBatch,         // up to 64 tokens, K cut into a slice per wave (qift_batch.hip)
  kGemmSplit,     // tiled GEMM split over K, with a workspace
  kGemm,          // tiled GEMM (qift_gemm.hip)
  kSkinny,        // up to 64 tokens, K <= 16384: one pass over the weights
  kSkinnySplit,   // the same split over K, with a workspace, up to 32 tokens
  kCodes,         // up to 16 tokens whose codes fit LDS
  kDecode,        // up to 16 tokens otherwise
};

// The batch kernel.  Its time hardly grows with the tokens, so it is the faster from some count on.  It puts 32 to
// 128 rows on a CU, one workgroup at a time: past 32768 rows a second round begins, nearly empty at first.
// gs: a split GEMM is there to take, ss: the skinny split, codes_fit: the decode kernel on codes.
inline bool take_batch(bool w4, int64_t N, int64_t K, int64_t M, bool gs, bool ss, bool codes_fit) {
  if (M < 5 || M > kBatchMaxM) return false;
  if (M > kCodesMaxM) {
    // two rounds: W2 40960 x 4096 at 33 34.9 / 20.3 (the GEMM), W4 at 48 43.3 / 28.5; where the others' passes
    // over the codes are long it is still ahead up to 32 tokens (W2 x 8192 at 24 0.85, W4 x 5120 at 17 0.82,
    // W2 70000 x 4096 at 30 0.89)
    if (N > 32768)
      return M <= 32 && !gs && K <= kSkinnyMaxK && (K > (w4 ? 4096 : 8191) || (K >= 4096 && M >= (w4 ? 30 : 28)));
    // a K that the skinny kernel does not take: against the GEMM (4096 x 20480 at 24: 14.7 / 70) always,
    // against its split W2 up to 8192 rows (12288 x 20480 at 33: 1.15 of it, 8192 x 28672 at 52: 1.08), W4 up
    // to 4096 and from 33
    if (K > kSkinnyMaxK) return !(gs && (N >= 12288 || (N > 6144 && K > 24576) || (w4 && (N > 4096 || M < 33))));
    // long K with a split GEMM: W4 4096 x 11008 at 24 1.12 of it, at 33 0.96, x 16384 at 33 1.09; W4 28672
    // x 14336 at 33 1.12, W2 22016 x 11008 at 33 1.08 but 0.93 at 64
    if (gs && w4 && N <= 4096 && K > 8192) return M >= 33 && K < 16384;
    if (gs && M >= 33 && K > 8192 && (w4 ? N > 24576 : N > 16384 && M < 48)) return false;
    // and W4 where the split fills the CUs once while the row tiles leave a third of them idle (just past 4096
    // and 8192 rows: 5120 x 13824 at 33 20.7 / 16.9, 9000 x 7168 at 26 17.8 / 16.3)
    if (gs && w4 && N > 4096 && K > 6144) {
      const int64_t rj = (N + 8191) / 8192, own = (N + 32 * rj - 1) / (32 * rj);
      const int64_t split = (N + 255) / 256 * gemm_split_plan(w4, N, M, K).S;
      if (own <= 170 && split >= 224 && split <= 272) return false;
    }
    if (N >= 16384) {
      // against the tiled GEMM: W2 of more than 24576 rows is its (28672 x 4096 at 64: 20.2 / 19.9)
      if (M >= 33) return K >= 2048 && (w4 || N <= 24576);
      // a short K leaves a wave a few steps: 16384 x 2048 at 17 8.4 / 5.9, 28672 x 2048 at 24 10.3 / 9.1; three
      // row tiles (16385-24576 rows) pay from there on (W2 22016 x 2048), W4 from 24 tokens
      return K >= (N > 16384 && N <= 24576 ? 2048 : 3072) && (M >= 24 || K > 3072 || (N > 16384 && (K >= 3072 || !w4)));
    }
    if (M >= 48) return K >= 2048;   // W4 4096 x 2048 at 48 6.0 / 5.7, at 32 4.8 / 5.2
    if (K < 4096) return false;
    if (N > 4096) return true;       // 12288 x 4096 at 17 8.3 / 8.7, W4 at 64 12.5 / 23.4
    // up to 4096 rows from 24 tokens (4096 x 4096 at 24 6.3 / 6.5, at 17 6.2 / 5.9); just past 4096 k, where a
    // slice is a line group and a piece, from 28 (1000 x 5120 at 17 1.17, at 24 1.07), W4 of up to
    // 1024 rows from 33 (777 x 6208 at 32 1.08);
    // long ones at once, W4 only small ones (3072 x 11008 at 17 1.18, at 28 1.03; 2560 x 9728 at 21 1.08).  The skinny split is the faster
    // for very long K (1000 x 14336 at 17 11.1 / 8.9) and around 2048 rows (2048 x 11008 at 17 1.09)
    // (from 33 tokens on only with few rows: 1000 x 14336 at 33 11.3 / 10.2)
    if (ss && M > 32) return K < 12288 || N <= 128 || N > 2560;
    if (ss)
      return K <= 8192 ? M >= 24 || K > 4096 : N <= 128 || (K < 12288 && (N < 1024 || N > 2560));
    if (K > 8192) return M >= 28 || !w4 || (N <= 2048 && N * K <= (int64_t(24) << 20));
    return M >= (K > 4096 && K < 8192 && !gs ? (w4 && N <= 1024 ? 33 : 28) : 24) || (K == 8192 && !w4);
  }
  // 5-16 tokens: the decode kernel on codes.  Wide and long (16384 x 8192, whose one 16-row tile per
  // workgroup takes four rounds: 13.4 / 23.4 at 9, W4 20.6 / 29.3 at 12)
  // (a second round: 40960 x 11008 at 5 1.14, W4 40960 x 5120 at 12 1.11; 57344 x 8192 at 5 44.6 / 56.7)
  if (N > 32768) return K > 4096 && M >= (!w4 ? (N >= 49152 ? 5 : 6) : K >= 8192 ? 9 : 15);
  if (N >= 16384 && K > 4096) return !w4 || M >= 9;
  // W4 from 15 tokens, wide (28672 x 4096 20.1 / 22.2) or at most 4096 rows of a whole number of line groups
  // a slice (4096 x 11008 11.2 / 13.6, 4096 x 4096 6.3 / 6.5 at 16, but x 5120 1.05-1.16, 300 x 4096 1.14)
  if (w4 && K >= 4096 && M >= 15 && (N >= 16384 || (N <= 4096 && (K >= 8192 || (K == 4096 && N > 512))))) return true;
  // where the codes exceed the decode kernel's LDS the skinny split (1000 x 14336 at 16: 9.5 / 8.2)
  if (ss && K >= 12288 && N > 128 && N <= 4096) return false;
  // W2 of at most 16384 rows from 12 tokens (at 16: 6144 x 4096 5.7 / 7.3, 4096 5.5 / 6.4, 12288 7.9 / 8.3), 4097-8192
  // rows from 9 (at 9 6144 x 4096 0.90, 12288 x 5120 0.82), few rows just past 4096 k from 13 (300 x 5120 at 12 1.09, 777 x 6208 at 13 0.85)
  if (!w4 && K >= 4096 && N <= 16384)
    if (M >= (N > 4096 && N <= 8192 ? 9 : N <= 4096 && K > 4096 && K < 8192 ? 13 : 12)) return true;
  // without a split the decode kernels that read the codes from memory (4096 x 14336 at 16 10.2 / 14.5)
  return !codes_fit && M >= (w4 ? 12 : 9) && !ss;
}

// ws: a workspace is given (the two split kernels need one).
inline Kernel choose(bool w4, int64_t N, int64_t K, int64_t M, bool codes_fit, bool ws) {
  const bool gs = ws && gemm_split_plan(w4, N, M, K).S > 1;
  const bool ss = ws && !(M <= kCodesMaxM && codes_fit) && skinny_split_plan(w4, N, M, K).S > 0;
  if (take_batch(w4, N, K, M, gs, ss, codes_fit)) return kBatch;
  // From 33 tokens on a wide linear that the batch kernel leaves runs the tiled GEMM rather than the skinny
  // kernel, whose workgroups each read all M x K codes (28672 x 4096 at 33 / 64 tokens: W2 22.9 -> 17.3 / 28.2 ->
  // 18.6), unsplit unless K is long; 16384 rows are still one round of the skinny kernel's (x 1024 at 33: GEMM
  // 8.1 / 6.8)
  const bool wide = N >= 16384 && M >= 33 && (K >= 2048 || N > 16384);
  if (gs) {
    if (M <= kSkinnyMaxM) {
      if (!(wide && K < 8192)) return kGemmSplit;
    } else {
      // What the split pays for (the second pass, 4-5 us, and the partial sums) grows with the tiles, what it gains
      // with K: it is the faster up to a number of tiles that grows with K.  W2, split over unsplit at 4096 k
      // 0.9 to 64 tiles and 1.1 from 72 on, 5120 1.0 at 72, 7168 1.0 at 108, 8192 1.0 at 128, 11008 1.0 at 156,
      // 14336 0.95 at 162 and 1.07 at 172, 20480 1.0 from 176 on; two ranges only (K <= 2816) 1.0 at 8 and 1.1 at 24.  W4 4096 k 0.95 at 80
      // and 1.0 at 96, 5120 1.0 at 120, 7168 and 8192 1.0 at 144, longer ones wherever there is a plan.
      const int64_t tiles = ((N + 255) / 256) * ((M + 63) / 64);
      const int64_t most = w4 ? (K >= 11008 ? tiles : K / 46 < 150 ? K / 46 : 150)
                              : K <= 2816 ? 8 : K <= 8192 ? K / 64 : 128 + (K - 8192) / 128;
      if (tiles <= most) return kGemmSplit;
    }
  }
  if (M > kSkinnyMaxM || (wide && (!gs || K < 8192))) return kGemm;
  if (M > kCodesMaxM) return K > kSkinnyMaxK ? kGemm : ss ? kSkinnySplit : kSkinny;
  // codes beyond LDS (16 tokens of K = 14336): with a workspace the skinny linear split over K, else the
  // decode kernels that read them from memory (faster there than the skinny kernel unsplit)
  return codes_fit ? kCodes : ss ? kSkinnySplit : kDecode;
}

}  // namespace route
}  // namespace qift
