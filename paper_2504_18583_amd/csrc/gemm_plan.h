// Tile plans of the skinny GEMM (passes of up to kMaxRows rows): which strips
// per workgroup, wavefronts and input ranges a weight takes, and which of these
// the kernel is compiled for.  Plain C++: the planner, the launcher and the
// plans' test share it.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdlib>

namespace pard {

enum Epi { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };

// A split input dimension: tile counters and fp32 partial tiles.
constexpr int kSplitCounters = 4096;
constexpr size_t kSplitPartFloats = (size_t)4 << 20;
// LDS of a workgroup's wavefront partials: four wavefronts of 7 strips and 4
// row tiles.
constexpr size_t kGemmLdsMax = 112 * 1024;
constexpr int kLmStrips = 8;   // strips per lm_head workgroup at up to 48 lm rows

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Prefill of n rows in passes of at most pass_rows (a multiple of 128, at least
// 512): as few passes as that takes, of even lengths in units of 128 rows, so
// that none is a few rows that stream all weights (with two passes or more the
// shortest has over 128).  The first row of pass i of n_chunks; i = n_chunks: n.
inline int prefill_chunks(int n, int pass_rows) { return ceil_div(n, pass_rows); }
inline int prefill_chunk_begin(int n, int n_chunks, int i) {
  const long long units = ceil_div(n, 128);
  return (int)std::min<long long>(n, (units * i + n_chunks - 1) / n_chunks * 128);
}

// The (epilogue, row tiles, strips) that k_gemm is compiled for: launch_gemm
// instantiates these and nothing else, and a plan may name no other.
constexpr bool gemm_instance(int epi, int mt, int S) {
  if (mt < 1 || mt > 4) return false;
  switch (S) {
    case 1: case 2: return true;
    case 4: return epi == EPI_SWIGLU || epi == EPI_LOGITS || (epi == EPI_QKV && mt == 1);
    case 7: return epi == EPI_SWIGLU;
    case 8: return (epi == EPI_LOGITS && mt <= 3) || (epi == EPI_SWIGLU && mt == 1);
    case 9: case 10: return epi == EPI_SWIGLU && mt == 1;
  }
  return false;
}

// What launch_gemm accepts: a compiled instance whose LDS fits, tiles that cover
// the strips (only gate/up workgroups of 8+ strips may be ragged), every input
// range non-empty, and the counters and partial tiles of a split within their
// buffers.
inline bool gemm_launchable(int epi, int mt, int S, int nw, int n_strips, int kb_total, int n_tiles, int ksplit,
                            int kb_split) {
  if (!gemm_instance(epi, mt, S) || nw < 4 || nw > 8 || (size_t)nw * S * mt * 1024 > kGemmLdsMax) return false;
  if (n_tiles < 1 || (size_t)n_tiles * S < (size_t)n_strips || (size_t)(n_tiles - 1) * S >= (size_t)n_strips) return false;
  if (n_tiles * S != n_strips && !(epi == EPI_SWIGLU && mt == 1 && S >= 8)) return false;
  if (ksplit < 1 || kb_split < 1 || (size_t)(ksplit - 1) * kb_split >= (size_t)kb_total ||
      (size_t)ksplit * kb_split < (size_t)kb_total)
    return false;
  return ksplit == 1 || (n_tiles <= kSplitCounters && (size_t)n_tiles * ksplit * S * mt * 256 <= kSplitPartFloats);
}

// Tile plan of one skinny GEMM: S strips per workgroup, nw wavefronts splitting
// the input dimension.  nw and ksplit, and with them the order of a sum, depend
// only on the weight shape: a row's result does not depend on how many other
// rows its pass has.
struct GemmPlan {
  int n_strips = 0, kb_total = 0;
  int nw = 4;   // one wavefront per SIMD: more waves per workgroup measured slower at every decode shape
  int ksplit = 1;   // input ranges of the skinny GEMM
};

inline int pick_S(int epi, int n_strips, int mt) {
  // residual GEMMs: one strip per workgroup up to 256 strips (one round), two
  // beyond (a tile is also one entry of the row sums that the next normalised
  // GEMM adds up: resid_ss_tiles)
  if (epi == EPI_RESID) return (n_strips > 256 && n_strips % 2 == 0) ? 2 : 1;
  // lm_head: eight strips per workgroup (four at 49 rows and more), fewer for
  // small vocabularies until the workgroups cover the CUs (41 rows, 4096-wide
  // hidden: 8016 strips 242 us at 2 per workgroup, 202 at 4, 194 at 8; 57 rows
  // 264, 220, 228; 256 strips, 41 rows: 16.1 at 2, 13.4 at 1).  Eight also where
  // they are one round that leaves up to a quarter of the CUs out (9 rows: 1536
  // strips 31.7 at 8, 34.3 at 4; 2000, a vocabulary of 32000, 41.9 and 43.2; 1024
  // 27.5 and 21.7; 41 rows: 1536 39.0 and 41.8, 2000 45.1 and 45.7)
  if (epi == EPI_LOGITS) {
    int s = mt <= 3 ? kLmStrips : 4;
    while (s > 1 && (n_strips % s || n_strips / s < (s == kLmStrips ? 192 : 256))) s >>= 1;
    return s;
  }
  if (mt == 1) {
    // decode rows: the fewest strips per workgroup that cover the weight in
    // one round of at most 256 workgroups (one per CU), so each CU reads the
    // activation rows once; from 8 strips on the last workgroup may hold
    // fewer.  Measured (gemm_counters, 9 rows): gate/up 8B 1792 strips 7 per
    // workgroup, 37.7 us (54 at 1); Qwen2.5-7B 2368 strips 10, 43.5 us
    // against 57.1 at 2, 50.0 at 4, 56.0 at 8 and 60.5 at 9; 1B 1024 strips
    // 4, 13.7 us against 14.7 at 2 and 19.7 at 1; Qwen2.5-0.5B 608 strips 4,
    // 7.2 us against 8.1 at 2 and 9.3 at 1; QKV 8B 384 strips 2 (12.4 us
    // against 14.1 at 1), Qwen2.5-7B 288 strips 2 (12.2 against 14.8).
    for (int s : {1, 2, 4, 7, 8, 9, 10}) {
      if (s >= 7 && epi != EPI_SWIGLU) break;
      if ((s >= 8 || n_strips % s == 0) && ceil_div(n_strips, s) <= 256) return s;
    }
  }
  if (epi == EPI_SWIGLU && mt == 1) {
    // wider weights: the strips-per-workgroup count that divides the strips
    // and fills the 256 CUs most evenly; among equally even ones, the one
    // closest to two rounds of workgroups
    int best = 1, best_d = 1 << 30;
    double best_u = 0.0;
    for (int s : {7, 4, 2, 1}) {
      if (n_strips % s) continue;
      const int tiles = n_strips / s;
      const double u = (double)tiles / (ceil_div(tiles, 256) * 256);
      const int d = std::abs(tiles - 512);
      if (u > best_u + 1e-9 || (u > best_u - 1e-9 && d < best_d)) {
        best_u = u;
        best_d = d;
        best = s;
      }
    }
    return best;
  }
  // 17 to 64 rows: the activations a workgroup reads (1 KiB per row tile and
  // k-block, against S KiB of weights) come from the XCD's L2, so wider tiles
  // read less of them; one round of workgroups where that is possible.  Measured
  // (us at 41 rows, rotating weight copies): gate/up 8B 1792 strips 56 at 2, 44
  // at 4, 41 at 7; 1B 1024 strips 17.9 at 2, 16.3 at 4, 23.6 at 8; Qwen2.5-7B
  // 2368 strips 65 at 2, 55 at 4, 70 at 8; QKV 8B 384 strips 21.4 at 1, 18.2 at 2,
  // Qwen2.5-7B 288 strips 18.6 and 15.7, 1B 192 strips 9.2 and 11.8.  Two strips
  // where they are one round by themselves (512 strips x 64 k-blocks, 25 / 41 / 57
  // rows: 10.2 / 11.7 / 13.5 at 2, 12.6 / 15.0 / 17.4 at 4), and with two row
  // tiles where four would leave a second round half empty or more (25 rows, 128
  // k-blocks: 1056 strips 32.6 at 2, 35.8 at 4; 1376 36.3, 37.5; 1536 37.6, 38.3;
  // 1664 46.5, 38.7; at 41 rows 1376 42.1, 41.1).
  int s = 1;
  if (epi == EPI_QKV && n_strips > 256) s = 2;
  if (epi == EPI_SWIGLU) {
    if (n_strips > 1024 && n_strips <= 1792 && n_strips % 7 == 0) return 7;
    s = n_strips <= 512 || (mt == 2 && n_strips > 1024 && n_strips <= 1536) ? 2 : 4;
  }
  while (s > 1 && n_strips % s) s >>= 1;
  return s;
}

inline GemmPlan plan_gemm(int epi, int n_pad, int k_pad) {
  GemmPlan p;
  p.n_strips = n_pad / 16;
  p.kb_total = k_pad / 32;
  // A long, narrow residual GEMM (the 1B down projection: 128 strips x 256
  // k-blocks) fills only half the CUs with one workgroup per strip; two input
  // ranges per strip measured 11.8 against 13.6 us.  Shorter or wider shapes
  // measured slower split (the partial-tile exchange adds ~2 us of tail).  From
  // 17 rows on two strips over two ranges would serve the 8B and 7B down
  // projections better (8B: 27.3 -> 26.1 us at 25 rows, 39.4 -> 34.4 at 57; four
  // conversations' step 2 %), but a row would then be summed in another order
  // than in a pass of fewer rows.
  if (epi == EPI_RESID && p.n_strips <= 128 && p.kb_total >= 256) p.ksplit = 2;
  return p;
}

inline GemmPlan plan_o(int n_pad, int k_pad) {
  GemmPlan p = plan_gemm(EPI_RESID, n_pad, k_pad);
  // one strip per workgroup: eight partial sums over the input, as the O units
  // fused into the QKV + attention launch form, so a row's O-projection is
  // summed in the same order whether or not its pass runs fused (the unfused
  // launch measured 8.3 -> 10.9 us at the 8B shape for it, 10.6 -> 13.1 at 25 rows;
  // 16k-context 8B/1B step 4.53 -> 4.57 ms)
  if (pick_S(EPI_RESID, p.n_strips, 1) == 1) p.nw = 8;
  return p;
}

// Tiles that write row sums of squares per residual GEMM of a pass served by
// the skinny GEMM (its consumers' ss_tiles).
inline int resid_ss_tiles(const GemmPlan& p) { return p.n_strips / pick_S(EPI_RESID, p.n_strips, 1); }

}  // namespace pard
