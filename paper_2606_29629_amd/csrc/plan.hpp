// Arithmetic of the launches that needs no GPU (no HIP in here: the host tests
// compile it by itself).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace tri {

constexpr int kBK = 64;  // k per GEMM k-tile

constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }

// Row stride of fp32 planes with N columns: the epilogues write columns in
// groups of four.
constexpr int plane_ld(int N) { return cdiv(N, 4) * 4; }

// Tiles of the final partial round: total % CUs, or all of them when the
// GEMM has fewer tiles than CUs.
constexpr int tail_tiles(int total, int G) {
  return total > G ? total % G : (total == G ? 0 : total);
}

constexpr int kMaxTailSplit = 8;  // K-parts of a tail tile, at most

// How a GEMM of M x N x K runs: on 256 x 256 tiles, the last partial round of
// them whole (split 1), in `split` K-parts, or as 128-row halves (split 0), or
// on 128 x 256 tiles, or on 128 x 128 tiles, all of them split in K where they
// would fill less than half of the CUs.  The choice is
// the least of the forms' estimated times: rounds of workgroups (one per CU)
// of KT k-tiles, plus per round the fill and the epilogue, plus for a K-split
// the partials written and read back and one more launch.  The constants are
// measured at clocks the small GEMMs hold (per k-tile: 256 x 256 1.05 us, 128 x
// 256 0.74 us, 128 x 128 0.60 us).  Waiting for a k-tile's loads (64, 48, 32 KB)
// sets them, not LDS: in the ragged and the mixed prefill the waves of these forms
// wait for 26 to 44% of their cycles, LDS is active for 15 to 30% of the CUs' and the
// MFMA pipes for 19 to 67%, and the K-parts of down draw 6 to 7 TB/s from beyond L2.
// The largest tile does the most per byte, so the small ones only pay where they
// fill more of the CUs.
struct GemmPlan {
  int bm, bn, split;
};
constexpr float kUs256 = 1.05f, kUs128x256 = 0.74f, kUs128 = 0.60f;  // us per k-tile
constexpr float kUsRound256 = 12.f, kUsRound128x256 = 8.f, kUsRound128 = 6.f;  // us per round
constexpr float kUsLaunch = 5.f;         // one more launch
constexpr float kPartialMbPerUs = 4.2f;  // fp32 partials, written or read

// N: weight rows (gate and up for SwiGLU); have_tail: there is room for partials;
// G: CUs.
inline GemmPlan gemm_plan(int M, int N, int K, bool swiglu, bool have_tail, bool routed, int G) {
  const int kt = K / kBK;
  const int cols256 = cdiv(N, 256), t256 = cdiv(M, 256) * cols256;
  GemmPlan best{256, 256, 1};
  float cost = cdiv(t256, G) * (kt * kUs256 + kUsRound256);
  auto offer = [&](float c, GemmPlan p) {
    if (c < cost) {
      cost = c;
      best = p;
    }
  };
  const int rem = tail_tiles(t256, G);
  const float rounds = (t256 - rem) / G * (kt * kUs256 + kUsRound256);
  // The rows of a mixture of experts go on to its router, where a near tie
  // makes another sum order another choice of experts (measured: about one
  // token in 2000, a tenth of the rms in its output).  Whole tiles sum in one
  // order whatever their form, so K is not cut for the estimate's small gains,
  // only where a last round after whole ones (or alone, with a K past 8192) is
  // so empty that the cut pays.  Cut against whole, us (rows, in t parts): 8192 x
  // 8192 4200 t = 8 433 / 507, 4500 t = 4 469 / 502; 10240 x 8192 3400 t = 5 446 /
  // 488; 18432 x 4096 4500 t = 8 540 / 564, 5500 t = 5 649 / 659; 4096 x 16384 300 t =
  // 8 79 / 116, 900 t = 4 131 / 129; at a K of 2048 it is even: 5120 x 2048 3100 t = 8
  // 90 / 78, 3500 95 / 98, 6500 148 / 157, 3700 t = 5 107 / 100.
  if (routed && have_tail) {
    if (rem > 0 && (t256 > G || K > 8192)) {
      int t = std::min(G / rem, kMaxTailSplit);
      while (t > 1 && (t - 1) * cdiv(kt, t) >= kt) --t;
      if (t > 4 || (t == 4 && K > 4096)) return {256, 256, t};
    }
    have_tail = false;
  }
  if (rem > 0) {
    offer(rounds + cdiv(2 * rem, G) * (kt * kUs128x256 + kUsRound128x256) +
              (t256 > rem ? kUsLaunch : 0.f),
          {256, 256, 0});
    if (have_tail && !swiglu)
      for (int t = 2; t <= kMaxTailSplit && t * rem <= G && (t - 1) * cdiv(kt, t) < kt; ++t)
        offer(rounds + cdiv(kt, t) * kUs256 + kUsRound256 + 2 * kUsLaunch +
                  2 * rem * t * 0.262f * M / (cdiv(M, 256) * 256) / kPartialMbPerUs,
              {256, 256, t});
  }
  offer(cdiv(cdiv(M, 128) * cols256, G) * (kt * kUs128x256 + kUsRound128x256), {128, 256, 1});
  const int t128 = cdiv(M, 128) * cdiv(N, 128);
  offer(cdiv(t128, G) * (kt * kUs128 + kUsRound128), {128, 128, 1});
  if (have_tail && !swiglu)
    for (int t = 2; t <= kMaxTailSplit && t * t128 <= G && (t - 1) * cdiv(kt, t) < kt; ++t)
      offer(cdiv(kt, t) * kUs128 + kUsRound128 + 2 * kUsLaunch +
                2 * t128 * t * 0.0655f * M / (cdiv(M, 128) * 128) / kPartialMbPerUs,
            {128, 128, t});
  return best;
}

// Bytes of a residual [M, ld] (bf16) that a tile of `rows` rows at (row0, col0)
// may read, counted from its first element: its valid rows, and in the last of
// them nothing past the row's end (for the last row, the tensor's).
constexpr int resid_range_bytes(int M, int ld, int row0, int col0, int rows) {
  const int valid = rows < M - row0 ? rows : M - row0;
  return (valid * ld - col0) * 2;
}

// Most rows with which a projection of N weight rows over K runs as a weight
// stream (gemm_stream.hip); beyond them it takes the skinny tiles, split in K.
// paired: SwiGLU and q/k/v, whose blocks hold 32 weight rows instead of 16.
//
// A stream's workgroup walks the whole K alone, so a narrow matrix with a long
// K has too few of them, and the more rows the longer each k-tile takes; the
// skinny tiles pay a second launch, but split K over all CUs.  Measured (skinny
// against stream, us): wide, 3584 x 18944 at 12 / 16 rows 31.1 / 31.2 against
// 30.6 / 33.0, 4096 x 16384 at 16 34.7 against 31.8; narrow, 1024 x 4096 at 5 / 16
// rows 8.4 / 8.7 against 6.7 / 7.7, 1024 x 8192 9.9 / 10.2 against 9.8 / 12.0, 1024 x
// 16384 12.5 / 12.8 against 16.8 / 21.2, 2048 x 8192 12.4 / 12.6 against 12.5 / 13.9;
// paired (a layer's stage), gate/up 1024 x 8192 11.8 / 12.4 against 15.0 / 17.7, 2048
// x 4096 11.8 / 11.9 against 10.6 / 12.3, q/k/v 1024 x 6144 13.9 / 14.0 against 14.7
// / 16.9, 768 x 4096 13.0 / 12.9 against 11.3 / 12.7.
constexpr int kStreamMaxRows = 16;
constexpr int stream_rows(int N, int K, bool paired) {
  const bool wide = N >= (paired ? 4096 : 3072);
  const int most = wide ? (1 << 18) / K : (paired ? 164000 : 215000) / K - 24;
  return most < 0 ? 0 : most < kStreamMaxRows ? most : kStreamMaxRows;
}

// Rows per tile of the grouped expert GEMMs, by the mean rows per expert and by
// whether a tile per expert and column (128 columns of ffn in gate/up, 256 of
// hidden in down, the wider pass) is all one round of the G CUs: then 32-row
// tiles, two workgroups per CU, last a little longer, and 128-row tiles last as
// long as they fit in the round, counting a fifth more rows than the mean.
//
// Both passes at a mean of so many rows, us, for 128 experts of 768 x 2048 (E), 64 of
// 1536 x 2048 (F), 32 of 1024 x 2048 (T), 8 of 2048 x 4096 (W):
//   32 / 128 rows    16  E 230 / 231, F 226 / 226, T 85 / 99   24  E 248 / 240, F 254 / 231,
//                    T 99 / 100   32  E 309 / 244, F 320 / 235, T 103 / 102   48  E 411 / 255
//   128 / 256 rows   96  E 292 / 293, F 268 / 273   104  E 326 / 290, F 315 / 279   192  E 389
//                    / 343, F 393 / 320, T 153 / 131
//   in one round     W 160  130 / 142, 208  139 / 156 (256 rows leave half the CUs idle)
inline int moe_tile_rows(int n_pairs, int n_experts, int hidden, int ffn, int G) {
  const int64_t pairs = n_pairs, E = n_experts;
  const int64_t cols = std::max(cdiv(ffn, 128), cdiv(hidden, 256));
  if (pairs <= (E * cols <= G ? 24 : 20) * E) return 32;
  if (pairs < 100 * E) return 128;
  if (pairs >= 224 * E) return 256;
  const int64_t tiles = (pairs * 6 / 5 + 128 * E - 1) / (128 * E);  // per expert and column
  return E * cols * tiles <= G ? 128 : 256;
}

// A launch holds fewer than 2^32 threads per grid dimension: of the jobs
// first .. n - 1 with `threads` threads each, the end of those that fit in one
// launch together (at least one: a job that does not fit fails as it would alone).
constexpr int64_t kMaxGridThreads = ((int64_t)1 << 32) - 256;
constexpr int jobs_of_launch(const int64_t* threads, int first, int n) {
  int64_t sum = threads[first];
  int end = first + 1;
  while (end < n && sum + threads[end] <= kMaxGridThreads) sum += threads[end++];
  return end;
}

}  // namespace tri
