// Skinny bf16 GEMM for decode-sized row counts, on gfx950 MFMA.
//
//   Y[r, n] = sum_k A[r, k] * W[n, k]            (W block-packed, A fp16)
//
// Decode streams every weight once per forward (Sec. 2.1: decoding is bound by
// reloading the weights), so the kernel is organised around the weight
// stream.  A workgroup owns S strips (16 output columns each) over the whole
// input dimension (the grid's last gate/up workgroup of 8-10 strips may own
// fewer, so that one round of workgroups covers the weight); its NW wavefronts
// split the input dimension, each one
// streaming its slice of the strips' 1 KiB blocks (one 16-byte load per lane,
// directly in the 16x16x32 MFMA B-operand layout) through a double-buffered
// register pipeline and accumulating MT 16x16 fp32 tiles.  Activation rows
// (<= 16*MT) are the A operand, in fp16; the weights (bf16 values kept in fp16
// encoding) feed v_mfma_f32_16x16x32_f16 directly.
//
// The wavefront partials are summed in LDS in wave order, so results are
// deterministic; the split depends only on the weight shape, so a row's sums do
// not depend on the pass's row count.  No workgroup ever waits for another one.
//
// Shapes with few strips also split the input dimension over the grid's y
// dimension (P contiguous ranges of k-blocks), so that narrow GEMMs still
// occupy every CU and one activation fragment feeds several strips.  Each
// workgroup stores its fp32 partial tile and counts itself in on the tile's
// counter; the last of the P to arrive adds the P partials in range order
// (the same order whichever workgroup is last) and runs the epilogue, then
// resets the counter for the next launch.
//
// Epilogues fuse the surrounding element-wise work of a Llama block:
//   EPI_QKV     RMSNorm row scale (A holds x*g in fp16, written by the
//               producer; 1/rms comes from the producer's per-tile sums of
//               squares), bias, rotate-half RoPE on Q/K, Q to an fp16 buffer,
//               K (16-key MFMA fragments) and V (32-key blocks, transposed)
//               to the fp16 cache.
//   EPI_RESID   x += Y (O-projection, down-projection), plus fp16(x * g_next)
//               and per-tile row sums of squares for the next normalised GEMM.
//   EPI_SWIGLU  RMSNorm row scale, h = silu(gate) * up, fp16 (each strip
//               holds 8 gate and the 8 matching up columns).
//   EPI_LOGITS  final RMSNorm scale, fp32 logits and per-tile (max, argmax).
// k_lm_tail then reduces the tiles per row (lowest id on ties) and runs the
// step tail: candidates for a draft pass; greedy prefix acceptance, KV
// rollback and next-pass staging for a verify pass.
#include "attn_tile.h"
#include "gemm_util.h"
#include "pard_internal.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <map>

namespace pard {
namespace {

// Wavefront reductions and scan in a fixed order (results do not depend on timing).
// They stay in the VALU (DPP moves, then the lane swaps): through LDS shuffles
// they were most of a sampled step's tail.
__device__ __forceinline__ float wave_sum(float v) { return attn::sum4g(sum16(v)); }
// The best (value, index) of the wavefront, in every lane.
__device__ __forceinline__ void wave_best(float& bv, int& bi) {
  best16(bv, bi);
  auto swap = [&](const auto v, const auto i) {
    bv = __uint_as_float(v[0]);
    bi = (int)i[0];
    if (better(__uint_as_float(v[1]), (int)i[1], bv, bi)) { bv = __uint_as_float(v[1]); bi = (int)i[1]; }
  };
  swap(__builtin_amdgcn_permlane16_swap(__float_as_uint(bv), __float_as_uint(bv), false, false),
       __builtin_amdgcn_permlane16_swap((unsigned)bi, (unsigned)bi, false, false));
  swap(__builtin_amdgcn_permlane32_swap(__float_as_uint(bv), __float_as_uint(bv), false, false),
       __builtin_amdgcn_permlane32_swap((unsigned)bi, (unsigned)bi, false, false));
}
__device__ __forceinline__ float wave_incl_scan(float v, int lane) {
  for (int off = 1; off < 64; off <<= 1) {
    const float o = __shfl_up(v, off);
    if (lane >= off) v += o;
  }
  return v;
}

// Input iterations per wavefront that a fused gate/up tile may take from LDS.
constexpr int kGuPreMax = 8;

// One workgroup tile of the skinny GEMM: strips [tile*S, tile*S + S) over the
// input range `split` of n_split, computed by the first nw wavefronts of the
// workgroup; red is the [nw][S*MT*256] float LDS of the wave reduction.  With
// FUSED (the QKV GEMM of a launch that also carries the attention reading its
// output) the Q / K / V stores are device-scope, so that workgroups on other
// XCDs of the same launch read them after the count-in.  With PM = 1 (the gate/up
// tile of such a launch: one row tile, one input range, four wavefronts) the
// first `pre` iterations of each wavefront take their weights from LDS, the
// first pre_d of them from pre_lds and the rest from pre_stat (gu_preload put
// them there; the caller has waited for its loads), the
// first global weight stages are requested before the tile waits for the O
// workers (fc), and the activations and row sums they wrote in this launch
// are read at device scope (one acquire fence per workgroup measured 8B/1B
// 3.511 ms against 3.456, one per wavefront 3.757), and h is stored at device
// scope.  With PM = 2 (the down projection of such a launch, one strip per
// tile) the first weight stages are requested before the tile waits for every
// gate/up tile (fc), and h and the residual x, written in this launch, are
// read at device scope.  The arithmetic and its order are those of the
// unfused tile.
template <int MT, int S, int EPI, bool FUSED = false, int PM = 0>
__device__ __forceinline__ void gemm_tile(const GemmArgs& p, const int tile, const unsigned split, const int n_split,
                                          const int nw, float* red, const FuseCtl* fc = nullptr,
                                          const uint32_t* pre_lds = nullptr, const int pre = 0,
                                          const uint32_t* pre_stat = nullptr, const int pre_d = 0,
                                          const int red_stride = 0) {
  static_assert(PM != 1 || (MT == 1 && EPI == EPI_SWIGLU && S < 8), "preloaded tiles: one row tile of gate/up, not ragged");
  static_assert(PM != 2 || (MT == 1 && EPI == EPI_RESID && S == 1), "fused down tiles: one row tile, one strip");
  constexpr int NE = S * MT * 256;   // elements of one workgroup tile
  constexpr int NJ = S * MT;         // elements per thread in the epilogue (first 256 threads)
  // k-blocks per pipeline stage: 8 KiB of W per wave (smaller for prefill-sized row counts)
  constexpr int U = MT >= 3 ? (S <= 2 ? 2 : 1) : MT == 2 && S == 1 ? 4 : ((8 / S) > 0 ? 8 / S : 1);
  __shared__ float rs_s[MT * 16];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform per wavefront

  // input range of this workgroup: k-blocks [kb0, kb0 + kb_n)
  const int kb0 = split * p.kb_split;
  const int kb_n = min(p.kb_split, p.kb_total - kb0);
  // wave w streams k-blocks kb0 + w, kb0 + w + nw, ...: at any time the
  // workgroup reads nw consecutive k-blocks of each strip
  const int n_it = (kb_n - wave + nw - 1) / nw;

  f32x4 acc[S][MT];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[s][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Raw buffer loads: a per-matrix descriptor, a constant per-lane VGPR offset
  // and a scalar per-iteration offset, so the prefetch needs no VGPR address
  // arithmetic (which would otherwise force waits on in-flight loads), and
  // every access is bounds-checked by the hardware.
  // W is k-block-major: block (kb, strip) sits at (kb * n_strips + strip) KiB.
  // A gate/up workgroup of 8 or more strips may be the grid's last, with
  // fewer strips than S (ragged): its missing strips re-read its last strip
  // (cache hits) and store nothing.
  constexpr bool RAGGED = EPI == EPI_SWIGLU && MT == 1 && S >= 8;
  const int n_strips = p.n_strips;
  const int s_last = RAGGED ? min(S - 1, n_strips - 1 - tile * S) : S - 1;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.W), 0, (int)min((size_t)n_strips * p.kb_total * 1024, (size_t)0x7fffffff), kRsrcWord3);
  const int w_voff = (tile * S * 64 + lane) * 16;

  // Two register stages of U k-blocks each: loads of stage i+1 are in flight
  // while stage i feeds the MFMAs.  Iterations past the wave's range are
  // clamped (cache hits) and their A fragment is zeroed.
  u32x4 w0[U][S], a0[U][MT], w1[U][S], a1[U][MT];
  auto load_w = [&](u32x4 (&w)[U][S], int its) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kb = kb0 + wave + min(its + u, n_it - 1) * nw;
#pragma unroll
      for (int s = 0; s < S; ++s)
        w[u][s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, w_voff, (kb * n_strips + (RAGGED ? min(s, s_last) : s)) * 1024,
                                                        kCachePolicyNT);
    }
  };

  constexpr bool LM = EPI == EPI_LOGITS;              // rows are the pass's lm rows
  constexpr bool NORM = EPI != EPI_RESID;             // A is RMS-normalised: rows need 1/rms

  // 1/rms per row from the producer's per-tile sums of squares: 16 threads per
  // row and row tile, fixed summation order.  The loads of the first 256 tiles
  // are issued ahead of the weight stream (ss_issue) and summed just before
  // the first MFMAs (ss_finish): loads complete in issue order, so waiting for
  // them would otherwise also wait for every weight load in flight and empty
  // the pipeline.
  float ss_part[MT][16];
  auto ss_issue = [&](int mt, int row) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      // unconditional loads (a tile index past the end re-reads the last
      // tile and is dropped when summed), so none waits behind a branch
      const int q = (tid & 15) + 16 * u;
      if constexpr (PM)   // written by the O workers of this launch: device scope
        ss_part[mt][u] = __hip_atomic_load(p.ss_in + (size_t)row * p.ss_stride + min(q, p.ss_tiles - 1),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        ss_part[mt][u] = p.ss_in[(size_t)row * p.ss_stride + min(q, p.ss_tiles - 1)];
    }
  };
  auto ss_finish = [&](int mt, int row) {
    float t = 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) t += (tid & 15) + 16 * u < p.ss_tiles ? ss_part[mt][u] : 0.f;
    for (int q0 = (tid & 15) + 256; q0 < p.ss_tiles; q0 += 256) {
      float part[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int q = q0 + 16 * u;
        if constexpr (PM)
          part[u] = q < p.ss_tiles ? __hip_atomic_load(p.ss_in + (size_t)row * p.ss_stride + q, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT) : 0.f;
        else
          part[u] = q < p.ss_tiles ? p.ss_in[(size_t)row * p.ss_stride + q] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) t += part[u];
    }
    t += __shfl_xor(t, 8);
    t += __shfl_xor(t, 4);
    t += __shfl_xor(t, 2);
    t += __shfl_xor(t, 1);
    if ((tid & 15) == 0) rs_s[mt * 16 + ((tid & 255) >> 4)] = 1.0f / sqrtf(t * p.inv_k + p.eps);
  };
  // thread tid (< 256) of the epilogue owns, for j = s*MT + mt, element
  // (row, col) below; its epilogue operands are fetched while the weights stream
  const bool epi = tid < 256;
  const int ew = tid >> 6;
  const int rsub = (lane >> 4) * 4 + ew;
  const int csub = lane & 15;

  // Per-lane reads of the pass descriptor are issued first, for the same
  // reason: lm source rows (A fragment rows, row-scale rows) and, for QKV, the
  // position and sequence slot of each epilogue row.  Entries past the pass
  // are read (in bounds) but never used.
  const FwdDesc* dp = p.desc;
  int lm_a[MT], e_pos[MT], e_slot[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    lm_a[mt] = LM ? dp->lm_src[mt * 16 + (lane & 15)] : 0;
    e_pos[mt] = EPI == EPI_QKV ? dp->pos[mt * 16 + rsub] : 0;
    e_slot[mt] = EPI == EPI_QKV ? dp->slot[mt * 16 + rsub] : 0;
  }
  int ss_row[MT];                                     // the row whose sums this thread adds, per row tile
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int r = mt * 16 + ((tid & 255) >> 4);
    ss_row[mt] = LM ? dp->lm_src[r] : r;
  }
  // rows of a pass's activations need no descriptor (rows past the pass read
  // unused sums and are never stored)
  if constexpr (NORM && !LM && !PM) {
    if (tid < 256) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) ss_issue(mt, ss_row[mt]);
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // The weight stream does not depend on the pass: its first stage is in
  // flight before the pass descriptor's scalar fields are read.  It is loaded
  // unconditionally (a wave with no k-block of its own, n_it = 0, reads the
  // range's last one and never uses it): a branch around it would make every
  // later wait on an earlier load wait for the whole stage too.
  const int its0 = PM == 1 ? pre : 0;   // the first iteration streamed from memory
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int kb = kb0 + min(wave + min(its0 + u, max(n_it - 1, 0)) * nw, kb_n - 1);
#pragma unroll
    for (int s = 0; s < S; ++s)
      w0[u][s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, w_voff, (kb * n_strips + (RAGGED ? min(s, s_last) : s)) * 1024,
                                                       kCachePolicyNT);
  }
  __builtin_amdgcn_sched_barrier(0);

  const int row_count = LM ? dp->n_lm : dp->n_rows;
  if constexpr (LM) {                             // lm rows read their source row's sums
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt * 16 + ((tid & 255) >> 4) >= row_count) ss_row[mt] = 0;
    if (tid < 256) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) ss_issue(mt, ss_row[mt]);
    }
  }

  // A fragment of this lane: row (lane % 16) of each M tile, 8 columns at
  // 8*(lane/16); A is k-blocked, so k-block kb of all rows is one contiguous
  // run at kb * act_rows * 64 bytes.  Rows past the pass get an offset
  // beyond the buffer: the hardware returns zeros for them without a memory
  // access.  lm rows read their source row.
  const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.A), 0, p.act_rows * p.lda * 2, kRsrcWord3);
  constexpr int kOutOfRange = 0x7FFFFFF0;
  int a_voff[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int r = mt * 16 + (lane & 15);
    const int src = r < row_count ? (LM ? lm_a[mt] : r) : 0;
    a_voff[mt] = r < row_count ? src * 64 + (lane >> 4) * 16 : kOutOfRange;
  }
  auto load_a = [&](u32x4 (&a)[U][MT], int its) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kb = kb0 + wave + min(its + u, n_it - 1) * nw;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        a[u][mt] = __builtin_amdgcn_raw_buffer_load_b128(ars, a_voff[mt], kb * (p.act_rows * 64),
                                                         PM ? attn::kCachePolicyDevice : 0);
    }
  };
  auto load = [&](u32x4 (&w)[U][S], u32x4 (&a)[U][MT], int its) {
    load_w(w, its);
    load_a(a, its);
  };

  float e0[NJ], e1[NJ];
  float2 e2[NJ];
  auto prefetch_epilogue = [&]() {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int s = j / MT, mt = j % MT;
      const int row = mt * 16 + rsub;
      const int n = (tile * S + s) * 16 + csub;
      e0[j] = 0.f;
      e1[j] = 0.f;
      e2[j] = float2{1.f, 0.f};
      if constexpr (EPI == EPI_RESID) {
        if (epi && row < row_count) {
          if constexpr (PM == 2)   // written by the O workers of this launch
            e0[j] = __hip_atomic_load(p.x + (size_t)row * p.ldx + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          else
            e0[j] = p.x[(size_t)row * p.ldx + n];
          e1[j] = p.g_next[n];
        }
      } else if constexpr (EPI == EPI_QKV) {
        if (epi && p.bias) e0[j] = p.bias[n];
        if (epi && row < row_count && n < p.q_dim + p.kv_dim)
          e2[j] = p.rope[(size_t)e_pos[mt] * (p.hd / 2) + ((n % p.hd) >> 1)];
      }
    }
  };
  auto compute = [&](const u32x4 (&w)[U][S], const u32x4 (&a)[U][MT], int its) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = its + u < n_it;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const u32x4 av = live ? a[u][mt] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int s = 0; s < S; ++s)
          acc[s][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, av),
                                                              __builtin_bit_cast(f16x8, w[u][s]), acc[s][mt], 0, 0, 0);
      }
    }
  };

  // sched_barrier keeps the compiler from sinking the prefetch next to its use
  if constexpr (PM == 2) {
    int its = 0;
    load_w(w1, its + U);                                // the second stage, before the wait
    __builtin_amdgcn_sched_barrier(0);
    attn::fuse_wait_on<kFuseLanes>(fc->counters + 3 * kFuseLanes * kFuseStride, fc->gu_tiles, fc->err);
    load_a(a0, its);
    load_a(a1, its + U);
    __builtin_amdgcn_sched_barrier(0);
    prefetch_epilogue();
    __builtin_amdgcn_sched_barrier(0);
    while (its + 2 * U < n_it) {
      compute(w0, a0, its);
      __builtin_amdgcn_sched_barrier(0);
      load(w0, a0, its + 2 * U);
      __builtin_amdgcn_sched_barrier(0);
      compute(w1, a1, its + U);
      __builtin_amdgcn_sched_barrier(0);
      load(w1, a1, its + 3 * U);
      __builtin_amdgcn_sched_barrier(0);
      its += 2 * U;
    }
    compute(w0, a0, its);
    if (its + U < n_it) compute(w1, a1, its + U);     // uniform
  } else if constexpr (PM == 1) {
    int its = pre;
    load_w(w1, its + U);                                // the second stage, before the wait
    __builtin_amdgcn_sched_barrier(0);
    attn::fuse_wait_on<kFuseLanes>(fc->counters + 2 * kFuseLanes * kFuseStride, fc->n_odone, fc->err);
    if (tid < 256) ss_issue(0, ss_row[0]);
    load_a(a0, its);
    load_a(a1, its + U);
    // A of the preloaded iterations (iterations past `pre` re-read the last
    // one and are never used)
    u32x4 ap[kGuPreMax];
#pragma unroll
    for (int i = 0; i < kGuPreMax; ++i)
      ap[i] = __builtin_amdgcn_raw_buffer_load_b128(ars, a_voff[0], (kb0 + wave + min(i, max(pre - 1, 0)) * nw) *
                                                    (p.act_rows * 64), attn::kCachePolicyDevice);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 256) ss_finish(0, ss_row[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kGuPreMax; ++i) {
      if (i < pre) {                                    // uniform
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const uint32_t* wb = i < pre_d ? pre_lds + ((wave * pre_d + i) * S + s) * 256
                                         : pre_stat + ((wave * (pre - pre_d) + i - pre_d) * S + s) * 256;
          const u32x4 wl = *reinterpret_cast<const u32x4*>(wb + lane * 4);
          acc[s][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, ap[i]),
                                                             __builtin_bit_cast(f16x8, wl), acc[s][0], 0, 0, 0);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    while (its + 2 * U < n_it) {
      compute(w0, a0, its);
      __builtin_amdgcn_sched_barrier(0);
      load(w0, a0, its + 2 * U);
      __builtin_amdgcn_sched_barrier(0);
      compute(w1, a1, its + U);
      __builtin_amdgcn_sched_barrier(0);
      load(w1, a1, its + 3 * U);
      __builtin_amdgcn_sched_barrier(0);
      its += 2 * U;
    }
    compute(w0, a0, its);
    if (its + U < n_it) compute(w1, a1, its + U);     // uniform
  } else if (n_it > 0) {
    int its = 0;
    load_a(a0, its);
    __builtin_amdgcn_sched_barrier(0);
    load(w1, a1, its + U);
    __builtin_amdgcn_sched_barrier(0);
    prefetch_epilogue();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NORM) {
      if (tid < 256) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) ss_finish(mt, ss_row[mt]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // One exit per pair of stages, at the loop's top: with an exit between
    // the two halves the compiler's wait at the top covered every load in
    // flight (draining the pipeline once per pair); with one exit it waits
    // only for the stage it computes.  The last two stages are computed after
    // the loop (loads past the range are clamped: at most one stage of them).
    while (its + 2 * U < n_it) {
      compute(w0, a0, its);
      __builtin_amdgcn_sched_barrier(0);
      load(w0, a0, its + 2 * U);
      __builtin_amdgcn_sched_barrier(0);
      compute(w1, a1, its + U);
      __builtin_amdgcn_sched_barrier(0);
      load(w1, a1, its + 3 * U);
      __builtin_amdgcn_sched_barrier(0);
      its += 2 * U;
    }
    compute(w0, a0, its);
    if (its + U < n_it) compute(w1, a1, its + U);     // uniform
  } else {
    if constexpr (NORM) {
      if (tid < 256) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) ss_finish(mt, ss_row[mt]);
      }
    }
    prefetch_epilogue();
  }

  // ---- workgroup reduction over the NW input-dimension slices (wave order) ----
  const int rs = red_stride > 0 ? red_stride : NE;    // floats between the wavefronts' partial tiles
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wave * rs + ((s * MT + mt) * 4 + i) * 64 + lane] = acc[s][mt][i];

  __syncthreads();

  // the first four wavefronts run the epilogue; all waves stay until the end
  // so that every barrier below is reached by the whole workgroup
  float v[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * 256 + (tid & 255);
    float t = red[e];
    for (int w = 1; w < nw; ++w) t += red[w * rs + e];
    v[j] = t;
  }

  // ---- split input dimension: the last workgroup of the tile to finish sums the partials ----
  // Partials are stored and loaded at device scope (written through to, and
  // read from, the level shared by all XCDs), so the count needs no cache
  // write-back or invalidation: each wavefront waits until its stores are
  // complete before the workgroup counts itself in.
  if (n_split > 1) {
    __shared__ int last_s;
    float* part = p.part + (size_t)tile * n_split * NE;
    if (epi) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        __hip_atomic_store(part + (size_t)split * NE + j * 256 + tid, v[j], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    if (tid == 0) {
      const int prev = __hip_atomic_fetch_add(p.counters + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_s = prev == n_split - 1;
      if (prev == n_split - 1) __hip_atomic_store(p.counters + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last_s) return;    // uniform over the workgroup
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int e = j * 256 + (tid & 255);
      float t = 0.f;
      for (int q = 0; q < n_split; ++q)
        t += __hip_atomic_load(part + (size_t)q * NE + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      v[j] = t;
    }
  }

  [[maybe_unused]] bool bad = false;
  if constexpr (EPI == EPI_QKV) {
    if (!epi) return;   // no barrier follows in this epilogue
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int s = j / MT, mt = j % MT;
      const int row = mt * 16 + rsub;
      const int n = (tile * S + s) * 16 + csub;
      float y = v[j] * rs_s[row] + e0[j];            // + bias
      // rotary partner column (n ^ 1) is in lane l ^ 1 (DPP quad swap)
      const float partner = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, y), 0xB1, 0xF,
                                                                               0xF, false));
      if (row < row_count) {
        const int pos = e_pos[mt];
        const size_t cache = (size_t)e_slot[mt] * p.kv_seq_stride;
        if (n < p.q_dim + p.kv_dim) {
          const float2 cs = e2[j];                     // rotary (cos, sin) of (pos, pair)
          y = (n & 1) ? (y * cs.x + partner * cs.y) : (y * cs.x - partner * cs.y);
        }
        const uint16_t b = f16_flagged(y, bad);
        uint16_t* dst;
        if (n < p.q_dim) {
          dst = p.out + (size_t)row * p.ld_out + n;
        } else if (n < p.q_dim + p.kv_dim) {
          const int c = n - p.q_dim;
          dst = p.kc + cache + (size_t)(c / p.hd) * p.cap * p.hd + k_index(pos, c % p.hd, p.hd);
        } else {
          const int c = n - p.q_dim - p.kv_dim;
          const size_t blk = (size_t)(c / p.hd) * (p.cap / 32) + (pos >> 5);
          dst = p.vc + cache + (blk * p.hd + (c % p.hd)) * 32 + v_slot(pos & 31);
        }
        if constexpr (FUSED)
          __hip_atomic_store(dst, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          *dst = b;
      }
    }
    flag_range(bad, p.ovf);
  } else if constexpr (EPI == EPI_RESID) {
    if (!epi) return;   // no barrier follows in this epilogue
    float sq[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sq[mt] = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int s = j / MT, mt = j % MT;
      const int row = mt * 16 + rsub;
      const int n = (tile * S + s) * 16 + csub;
      if (row < row_count) {
        const size_t o = (size_t)row * p.ldx + n;
        const float xn = e0[j] + v[j];                 // residual + projection
        p.x[o] = xn;
        p.xg[act_index(row, n, p.act_rows)] = f16_flagged(xn * e1[j], bad);
        sq[mt] += xn * xn;
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float t = sum16(sq[mt]);
      if (csub == 0) p.ss_out[(size_t)(mt * 16 + rsub) * p.ss_stride + tile] = t;
    }
    flag_range(bad, p.ovf);
  } else if constexpr (EPI == EPI_SWIGLU) {
    // a strip holds 8 gate columns then the 8 up columns of the same features:
    // the up value of column csub < 8 is in lane ^ 8 (same row)
    if (!epi) return;   // whole wavefronts; no barrier follows in this epilogue
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int row = mt * 16 + rsub;
        const float gt = v[s * MT + mt] * rs_s[row];
        // lane l ^ 8 of the row of 16 (DPP row rotate by 8)
        const float up = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, gt), 0x128, 0xF,
                                                                            0xF, false));
        const float h = gt / (1.0f + expf(-gt)) * up;
        const int f = (tile * S + s) * 8 + csub;
        if (csub < 8 && row < row_count && s <= s_last) {
          if constexpr (PM == 1)   // read by the down tiles of this launch: device scope
            __hip_atomic_store(p.out + act_index(row, f, p.act_rows), f16_flagged(h, bad), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          else
            p.out[act_index(row, f, p.act_rows)] = f16_flagged(h, bad);
        }
      }
    flag_range(bad, p.ovf);
  } else {  // EPI_LOGITS
    // (max, argmax) of a row's S*16 columns: over the strips in registers, then
    // over the row's 16 lanes with DPP moves
    if (!epi) return;   // whole wavefronts; no barrier follows in this epilogue
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = mt * 16 + rsub;
      float bv = -INFINITY;
      int bi = INT_MAX;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int n = (tile * S + s) * 16 + csub;
        const float val = v[s * MT + mt] * rs_s[row];
        if (row < row_count) p.logits[(size_t)row * p.vocab + n] = val;
        if (better(val, n, bv, bi)) { bv = val; bi = n; }
      }
      best16(bv, bi);
      if (csub == 0 && row < row_count) {
        p.amax_val[(size_t)row * p.amax_stride + tile] = bv;
        p.amax_idx[(size_t)row * p.amax_stride + tile] = bi;
      }
      if (p.samp_k > 0.f) {         // sampling: the tile's softmax weight relative to its max
        float sw = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s) sw += __builtin_amdgcn_exp2f((v[s * MT + mt] * rs_s[row] - bv) * p.samp_k);
        sw = sum16(sw);
        if (csub == 0 && row < row_count) p.amax_sum[(size_t)row * p.amax_stride + tile] = sw;
      }
    }
  }
}

template <int MT, int S, int EPI>
__global__ __launch_bounds__(512) void k_gemm(const GemmArgs p) {
  extern __shared__ float red[];     // [NW][NE]
  gemm_tile<MT, S, EPI>(p, blockIdx.x, blockIdx.y, gridDim.y, blockDim.x >> 6, red);
}

// O-projection units of a fused decode-layer launch (one row tile, EPI_RESID,
// one strip per unit, the whole input range): NU units of this worker
// starting at strip u0.  Wavefront v of the eight holds k-blocks v, v + 8, ...
// (KI of them; past the input range it re-reads the last one and never uses
// it).  Every weight block is requested before the wait for the attention
// workgroups, so the weights stream while the attention runs; the attention
// output (written in this launch) is then read at device scope.  The eight
// wavefront partials are summed in wave order, then the residual epilogue of
// gemm_tile: x += Y, fp16(x * g_next) and the strip's row sums of squares.
template <int KI, int NU, bool GUF, class Pre>
__device__ __forceinline__ void o_units(const GemmArgs& p, const FuseCtl& f, const int u0, float* red, Pre&& preload) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_strips = p.n_strips, kb_total = p.kb_total;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.W), 0, (int)min((size_t)n_strips * kb_total * 1024, (size_t)0x7fffffff), kRsrcWord3);
  u32x4 wv[NU][KI];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int kb = min(wave + 8 * i, kb_total - 1);
#pragma unroll
    for (int j = 0; j < NU; ++j)
      wv[j][i] = __builtin_amdgcn_raw_buffer_load_b128(wrs, ((u0 + j) * 64 + lane) * 16, kb * n_strips * 1024,
                                                       kCachePolicyNT);
  }
  __builtin_amdgcn_sched_barrier(0);
  preload();                                         // gate/up weights into LDS, behind the O weights
  __builtin_amdgcn_sched_barrier(0);
  // epilogue element of this thread: unit ej, row rsub, column csub of the
  // strip (the MFMA output layout; threads < 256 * NU)
  const int row_count = p.desc->n_rows;
  const bool epi = tid < 256 * NU;
  const int ej = min(tid >> 8, NU - 1);
  const int rsub = (lane >> 4) * 4 + ((tid & 255) >> 6), csub = lane & 15;
  const int n = (u0 + ej) * 16 + csub;
  float x_old = 0.f, g = 0.f;
  if (epi && rsub < row_count) {
    x_old = p.x[(size_t)rsub * p.ldx + n];
    g = p.g_next[n];
  }
  __builtin_amdgcn_sched_barrier(0);
  attn::fuse_wait_on<1>(f.counters + (kFuseLanes + blockIdx.x % kFuseLanes) * kFuseStride, f.n_cons, f.err);
  __builtin_amdgcn_sched_barrier(0);
  // A fragment of this lane: row lane % 16, 8 columns at 8 * (lane / 16) of
  // each k-block; rows past the pass read zeros without a memory access
  constexpr int kOutOfRange = 0x7FFFFFF0;
  const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.A), 0, p.act_rows * p.lda * 2, kRsrcWord3);
  const int a_voff = (lane & 15) < row_count ? (lane & 15) * 64 + (lane >> 4) * 16 : kOutOfRange;
  u32x4 av[KI];
#pragma unroll
  for (int i = 0; i < KI; ++i)
    av[i] = __builtin_amdgcn_raw_buffer_load_b128(ars, a_voff, min(wave + 8 * i, kb_total - 1) * (p.act_rows * 64),
                                                  attn::kCachePolicyDevice);
  f32x4 acc[NU];
#pragma unroll
  for (int j = 0; j < NU; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const u32x4 a = wave + 8 * i < kb_total ? av[i] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < NU; ++j)
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, wv[j][i]),
                                                      acc[j], 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < NU; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[(wave * NU + j) * 256 + i * 64 + lane] = acc[j][i];
  __syncthreads();
  if (!epi) return;   // whole wavefronts; no barrier follows
  float v = red[ej * 256 + (tid & 255)];
  for (int w = 1; w < 8; ++w) v += red[(w * NU + ej) * 256 + (tid & 255)];
  float sq = 0.f;
  bool bad = false;
  if (rsub < row_count) {
    const float xn = x_old + v;                      // residual + projection
    if constexpr (GUF)   // read by the down tiles of this launch: device scope
      __hip_atomic_store(p.x + (size_t)rsub * p.ldx + n, xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      p.x[(size_t)rsub * p.ldx + n] = xn;
    const uint16_t h = f16_flagged(xn * g, bad);
    if constexpr (GUF)   // read by the gate/up tiles of this launch: device scope
      __hip_atomic_store(p.xg + act_index(rsub, n, p.act_rows), h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      p.xg[act_index(rsub, n, p.act_rows)] = h;
    sq = xn * xn;
  }
  const float t = sum16(sq);
  if (csub == 0) {
    if constexpr (GUF)
      __hip_atomic_store(p.ss_out + (size_t)rsub * p.ss_stride + u0 + ej, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      p.ss_out[(size_t)rsub * p.ss_stride + u0 + ej] = t;
  }
  flag_range(bad, p.ovf);
}

// The O units of worker w (see FuseCtl), if it has any; `preload` runs once
// in any case (after the O weight requests when there are units).  With GUF
// (gate/up in the launch) a worker with units counts itself in once its
// stores are complete.
template <int KI, bool GUF, class Pre>
__device__ __forceinline__ void o_part(const GemmArgs& p, const FuseCtl& f, const int w, float* red, Pre&& preload) {
  if (w < f.o_two) {
    o_units<KI, 2, GUF>(p, f, 2 * w, red, preload);
  } else if (f.o_two + w < f.o_units) {
    o_units<KI, 1, GUF>(p, f, f.o_two + w, red, preload);
  } else {
    preload();
    return;
  }
  if constexpr (GUF) {
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);          // this wavefront's stores are complete
    __syncthreads();
    if (threadIdx.x == 0)
      __hip_atomic_fetch_add(f.counters + (2 * kFuseLanes + blockIdx.x % kFuseLanes) * kFuseStride, 1,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Gate/up weights of tile `tile` for input iterations [i0, i1) of
// wavefronts 0-3 (k-blocks w + 4i, as gemm_tile streams them), loaded
// straight into LDS (1 KiB blocks, lane-ordered) with no registers held:
// iterations below pre_d at dyn [w][i][strip], the others (STAT) at stat
// [w][i - pre_d][strip] for a workgroup of `pre` iterations; called by
// wavefronts 0-3, each for its own blocks.  Every load's LDS target derives
// from one LDS object, so the compiler's LDS-DMA waits stay precise.
template <int S, bool STAT>
__device__ __forceinline__ void gu_preload(const GemmArgs& p, const int tile, const int i0, const int i1,
                                           const int pre, const int pre_d, uint32_t* dyn, uint32_t* stat) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.W), 0, (int)min((size_t)p.n_strips * p.kb_total * 1024, (size_t)0x7fffffff), kRsrcWord3);
  const int voff = (tile * S * 64 + lane) * 16;
  for (int i = i0; i < min(i1, pre_d); ++i) {
    const int kb = wave + 4 * i;                     // < kb_total: pre <= kb_total / 4 (host)
#pragma unroll
    for (int s = 0; s < S; ++s)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          wrs, (__attribute__((address_space(3))) void*)(dyn + ((wave * pre_d + i) * S + s) * 256), 16, voff,
          (kb * p.n_strips + s) * 1024, 0, kCachePolicyNT);
  }
  if constexpr (STAT) {
    for (int i = max(i0, pre_d); i < i1; ++i) {
      const int kb = wave + 4 * i;
#pragma unroll
      for (int s = 0; s < S; ++s)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            wrs, (__attribute__((address_space(3))) void*)(stat + ((wave * (pre - pre_d) + i - pre_d) * S + s) * 256),
            16, voff, (kb * p.n_strips + s) * 1024, 0, kCachePolicyNT);
    }
  }
}

// Static LDS of the one-launch layer: the attention arrays of its attention
// workgroups, and in the others (and in those after their attention) the last
// preloaded gate/up iterations (two).
template <int HD, int SG>
union FusedStatLds {
  attn::AttnLds<HD, 1> attn;
  uint32_t pre[SG > 0 ? 2 * 4 * SG * 256 : 4];
};

// Decode passes over contexts of one attention chunk: the QKV GEMM, the
// attention that reads its output and (OKI > 0) the O-projection of the
// attention output in one launch.  Workgroups [0, n_tiles) are GEMM tiles
// (wavefronts 0-3 compute, 4-7 only take part in the workgroup's barriers);
// each stores its Q / K / V at device scope, waits for its stores, and counts
// itself in.  The next n_cons workgroups are the attention workgroups of
// k_attn's single-chunk plan (KV head, query group, sequence): the first pair
// of key tiles, when it precedes the pass, is requested before they wait for
// every GEMM tile; Q and the keys of the pass are then read at device scope.
// With O units their output is stored at device scope and they count
// themselves in; O-projection workers (the QKV workgroups once their tile is
// done, and o_extra workgroups after the attention ones) request their
// weights, wait for every attention workgroup and finish their units
// (o_part).  The counters: FuseCtl.  All workgroups of the launch are
// co-resident (the host checks the grid against the device's occupancy), a
// phase waits only for earlier phases, and every wait is bounded
// (attn::fuse_wait_on), so every wait ends.
template <int MT, int S, int HD, int OKI, int SG, int SD>
__global__ __launch_bounds__(512) void k_qkv_attn(const GemmArgs g, const AttnArgs a, const FuseCtl f,
                                                  const GemmArgs o, const GemmArgs gu, const GemmArgs dn) {
  static_assert(SG == 0 || (MT == 1 && OKI > 0), "gate/up joins only launches with O units");
  static_assert(SD == 0 || (SD == 1 && SG > 0), "the down projection joins only launches with gate/up");
  // [0, gu_lds): reductions (GEMM tiles [4][S * MT * 256], O units [8][2][256],
  // down tiles [4][256]); from gu_lds: preloaded gate/up weights, whose first
  // block of each wavefront later holds that wavefront's gate/up partial tile
  extern __shared__ float red[];
  __shared__ FusedStatLds<HD, SG> stat_sm;
  attn::AttnLds<HD, 1>& attn_sm = stat_sm.attn;
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  uint32_t* pre_lds = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(red) + f.gu_lds);
  uint32_t* stat_lds = stat_sm.pre;
  const bool gu_tile = SG > 0 && b < f.gu_tiles;          // uniform
  const int pre = b < g.n_tiles ? f.gu_pre_q : f.gu_pre;
  const int pre_d = pre - min(pre, f.gu_stat);            // the rest go into stat_sm
  auto preload = [&]() {
    if constexpr (SG > 0) {
      if (gu_tile && tid < 256) gu_preload<SG, true>(gu, b, 0, pre, pre, pre_d, pre_lds, stat_lds);
    }
  };
  if (b < g.n_tiles) {
    if (tid < 256) {
      gemm_tile<MT, S, EPI_QKV, true>(g, b, 0, 1, 4, red);
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);      // this wavefront's stores are complete
    } else {
      __syncthreads();                              // the tile's reduction barrier
    }
    __syncthreads();
    if (tid == 0)
      __hip_atomic_fetch_add(f.counters + (b % kFuseLanes) * kFuseStride, 1, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (OKI > 0) o_part<OKI, (SG > 0)>(o, f, f.o_extra + b, red, preload);
  } else if (b - g.n_tiles < f.n_cons) {
    const int i = b - g.n_tiles;
    const int kvh = i % a.n_kv, qg = (i / a.n_kv) % a.n_qblocks;
    const unsigned z = i / (a.n_kv * a.n_qblocks);
    attn::attn_tile<HD, 1, 2 * kAttnWaves, true>(a, kvh, qg, z, f, attn_sm);
    if constexpr (OKI > 0) {
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);      // this wavefront's output stores are complete
      __syncthreads();
      if (tid < kFuseLanes)   // every counter: each poller reads the one of its XCD
        __hip_atomic_fetch_add(f.counters + (kFuseLanes + tid) * kFuseStride, 1, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    // the gate/up preload only now: issued earlier it competes with the QKV
    // weights that the attention waits for (SG > 0 implies OKI > 0: the
    // barrier above ended the attention's use of stat_sm)
    if constexpr (SG > 0) {
      if (gu_tile && tid < 256) gu_preload<SG, true>(gu, b, 0, pre, pre, pre_d, pre_lds, stat_lds);
    }
  } else {
    if constexpr (OKI > 0) o_part<OKI, (SG > 0)>(o, f, b - g.n_tiles - f.n_cons, red, preload);
  }
  if constexpr (SG > 0) {
    if (gu_tile) {
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);      // this wavefront's preloaded weights are in LDS
      if (tid < 256) {
        // the tile's reduction in each wavefront's own first block of the
        // dynamic preload area (read only by that wavefront, before it)
        gemm_tile<1, SG, EPI_SWIGLU, false, 1>(gu, b, 0, 1, 4, reinterpret_cast<float*>(pre_lds), &f, pre_lds, pre,
                                               stat_lds, pre_d, max(pre_d, 1) * SG * 256);
      } else {                                      // the tile's two barriers
        attn::fuse_wait_on<kFuseLanes>(f.counters + 2 * kFuseLanes * kFuseStride, f.n_odone, f.err);
        __syncthreads();
      }
      if constexpr (SD > 0) {                       // h of this tile complete: count in
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        if (tid == 0)
          __hip_atomic_fetch_add(f.counters + (3 * kFuseLanes + b % kFuseLanes) * kFuseStride, 1, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if constexpr (SD > 0) {
    if (b < f.d_tiles) {                            // uniform: unit b = (strip, input range)
      const int P = dn.ksplit;
      if (tid < 256) {
        gemm_tile<1, 1, EPI_RESID, false, 2>(dn, b / P, b % P, P, 4, red, &f);
      } else {                                      // the tile's barriers
        attn::fuse_wait_on<kFuseLanes>(f.counters + 3 * kFuseLanes * kFuseStride, f.gu_tiles, f.err);
        __syncthreads();
        if (P > 1) {                                // the partial-tile exchange's two
          __syncthreads();
          __syncthreads();
        }
      }
    }
  }
}

__device__ void commit_verify(const TailArgs& p, const PassSeq& ps, int a, int bonus, const int* res);

// Decode-state update of one sequence once the argmax of its lm rows is
// known (one thread).  Draft: store the candidates, commit only the real rows
// (the mask rows are never committed).  Vanilla draft pass (one of K per
// step, eq. 3): one more candidate, every row committed.  Verify: longest
// agreeing prefix a (eq. 2), bonus t_a, L_t += a + 1, emit the a + 1 tokens;
// in vanilla mode the draft cache keeps the candidates that agree.
__device__ void seq_tail(const TailArgs& p, const PassSeq& ps, const int* res) {
  SeqState* s = p.states + ps.slot;
  if (p.tail == TAIL_PREFILL) {
    s->bonus = res[0];
    s->t[0] = res[0];
    s->pending[0] = res[0];
    s->n_pending = 1;
  } else if (p.tail == TAIL_DRAFT) {
    const int k = s->k;
    for (int i = 0; i < k; ++i) s->cand[i] = res[i];
    s->L[1] = ps.pos0 + ps.n_real;
  } else if (p.tail == TAIL_VSD_DRAFT) {
    s->cand[s->j] = res[0];
    ++s->j;
    s->L[1] = ps.pos0 + ps.n_real;
  } else if (p.tail == TAIL_VERIFY) {
    const int k = s->k;
    int a = 0;
    while (a < k && s->cand[a] == res[a]) ++a;      // longest agreeing prefix
    commit_verify(p, ps, a, res[a], res);
  }
}

// Verify step of one sequence with a accepted candidates and the step's last
// token (greedy: the target's argmax t_a; sampling: the residual or bonus
// draw): L_t += a + 1, emit c_1..c_a and the last token, count the step.
__device__ void commit_verify(const TailArgs& p, const PassSeq& ps, int a, int bonus, const int* res) {
  SeqState* s = p.states + ps.slot;
  {
    const int k = s->k;
    for (int i = 0; i <= k; ++i) s->t[i] = res[i];
    s->a = a;
    s->bonus = bonus;
    s->L[0] = ps.pos0 + a + 1;                     // keep pending + accepted rows
    if (s->vsd && k > 0) {
      // the draft cache holds the pending token and c_1..c_{k-1}; it keeps
      // those that agree, and the tokens after them become pending
      const int keep = min(a, k - 1);
      s->L[1] = ps.pos0 + 1 + keep;
      int n = 0;
      for (int i = keep; i < a; ++i) s->pending[n++] = s->cand[i];
      s->pending[n++] = bonus;
      s->n_pending = n;
      s->j = 0;
    } else {
      for (int i = 0; i < a; ++i) s->pending[i] = s->cand[i];
      s->pending[a] = bonus;
      s->n_pending = a + 1;
    }
    if (p.out_tokens) {                             // emitted: c_1..c_a, then the bonus
      int* out = p.out_tokens + (size_t)ps.slot * p.out_cap;
      for (int i = 0; i <= a; ++i) {
        if (s->n_out < p.out_cap) out[s->n_out] = i < a ? s->cand[i] : bonus;
        ++s->n_out;
      }
    }
    ++s->steps;
    ++s->draw;
    ++s->accept_hist[a];
  }
}

// Rows of one sequence in the pass that follows
//   a draft pass (PARD), or the last vanilla draft pass of a step: the verify
//     pass, [pending, c_1..c_k] at L_t;
//   an earlier vanilla draft pass: the next one, the candidate just drafted;
//   a verify pass with k > 0: the next draft pass, the pending tokens at L_d
//     followed (PARD) by k-1 mask rows, lm rows from the last pending row on;
//   a verify pass with k = 0: the next plain target step.
__device__ bool to_verify(int after, const SeqState& s) {
  return after == TAIL_DRAFT || (after == TAIL_VSD_DRAFT && s.j >= s.k);
}

__device__ void next_rows(int after, const SeqState& s, int* n_rows, int* n_real, int* pos0, int* lm_first,
                          int* lm_rows) {
  const int k = s.k;
  if (to_verify(after, s)) {
    *n_rows = k + 1; *n_real = k + 1; *pos0 = s.L[0]; *lm_first = 0; *lm_rows = k + 1;
  } else if (after == TAIL_VSD_DRAFT) {
    *n_rows = 1; *n_real = 1; *pos0 = s.L[1]; *lm_first = 0; *lm_rows = 1;
  } else if (k > 0 && s.vsd) {
    *n_rows = s.n_pending; *n_real = s.n_pending; *pos0 = s.L[1]; *lm_first = s.n_pending - 1; *lm_rows = 1;
  } else if (k > 0) {
    *n_rows = s.n_pending + k - 1; *n_real = s.n_pending; *pos0 = s.L[1]; *lm_first = s.n_pending - 1; *lm_rows = k;
  } else {
    *n_rows = 1; *n_real = 1; *pos0 = s.L[0]; *lm_first = 0; *lm_rows = 1;
  }
}

__device__ int next_id(int after, const SeqState& s, int i) {
  if (to_verify(after, s)) return i == 0 ? s.bonus : s.cand[i - 1];
  if (after == TAIL_VSD_DRAFT) return s.cand[s.j - 1];
  if (s.k > 0) return i < s.n_pending ? s.pending[i] : s.mask_id;
  return s.bonus;
}

// Stages the next pass of the step for the sequences of the current pass, in
// the same order (run by a whole workgroup).  With drop_done, sequences that
// have written all requested tokens leave the batch.  The current pass's
// sequence list is read before anything is written, so the next descriptor
// may be the current one (plain target steps).
__device__ void stage_next(const TailArgs& p, bool drop_done) {
  __shared__ int sl[kMaxPassSeqs], r0[kMaxPassSeqs + 1], l0[kMaxPassSeqs + 1];
  __shared__ int n_next_s;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int after = p.tail;
  if (tid == 0) {
    const int n_cur = p.desc->n_seq;
    int n = 0, rows = 0, lm = 0;
    for (int j = 0; j < n_cur; ++j) {
      const int slot = p.desc->seq[j].slot;
      const SeqState& s = p.states[slot];
      if (drop_done && after == TAIL_VERIFY && s.n_out >= s.n_target) {
        // its logits are overwritten by the passes that follow without it
        p.lm_map[slot] = int2{0, 0};
        if (p.lm_map_draft) p.lm_map_draft[slot] = int2{0, 0};
        continue;
      }
      int nr, nreal, pos0, lmf, lmr;
      next_rows(after, s, &nr, &nreal, &pos0, &lmf, &lmr);
      sl[n] = slot;
      r0[n] = rows;
      l0[n] = lm;
      rows += nr;
      lm += lmr;
      ++n;
    }
    r0[n] = rows;
    l0[n] = lm;
    n_next_s = n;
  }
  __syncthreads();
  const int n = n_next_s;
  FwdDesc* nd = p.next_desc;
  for (int j = tid; j < n; j += nth) {
    const SeqState& s = p.states[sl[j]];
    PassSeq q{};
    int lmf;
    next_rows(after, s, &q.n_rows, &q.n_real, &q.pos0, &lmf, &q.lm_rows);
    q.slot = sl[j];
    q.row0 = r0[j];
    q.lm0 = l0[j];
    nd->seq[j] = q;
  }
  // rows and lm rows: a thread finds its sequence by binary search over the
  // row offsets
  for (int r = tid; r < r0[n]; r += nth) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (r0[mid] <= r) lo = mid; else hi = mid - 1;
    }
    const SeqState& s = p.states[sl[lo]];
    int nr, nreal, pos0, lmf, lmr;
    next_rows(after, s, &nr, &nreal, &pos0, &lmf, &lmr);
    const int i = r - r0[lo];
    nd->ids[r] = next_id(after, s, i);
    nd->pos[r] = pos0 + i;
    nd->slot[r] = sl[lo];
    if (i >= lmf && i < lmf + lmr) nd->lm_src[l0[lo] + i - lmf] = r;
  }
  if (tid == 0) {
    nd->n_rows = r0[n];
    nd->n_seq = n;
    nd->n_lm = l0[n];
    nd->linear = 0;
  }
}

// Second argmax pass and step tail.  Workgroup j serves sequence j of the
// pass: wave w reduces its lm rows w, w+16, ... over the tiles, 16
// independent loads per lane in flight at a time; then one thread updates
// the sequence's decode state.  A single-sequence pass also stages the next
// pass here; batched passes stage it in k_stage.
// ---- speculative sampling (temperature T; samp_k = log2(e) / T) ----
// A row's distribution is softmax(z / T).  The LM GEMM left, per tile of
// tile_w columns, the tile's max m_t and s_t = sum 2^((z - m_t) k); the row's
// max M and normaliser S = sum_t s_t 2^((m_t - M) k) follow.  A token is
// drawn by inverse CDF in token-id order: the smallest x whose cumulative
// weight exceeds u S.  All sums run in a fixed order.

__device__ __forceinline__ float tile_weight(float m, float s, float M, float k) {
  return m == -INFINITY ? 0.f : s * __builtin_amdgcn_exp2f((m - M) * k);
}

constexpr int kScanBatch = 8;       // blocks of 64 tiles whose loads are in flight together
constexpr int kResidBlock = 256;    // vocabulary entries per wavefront block of the residual draw (4 per lane)
constexpr int kMaxResidBlocks = kMaxSampleVocab / kResidBlock;

// Tile weights of blocks b0 .. b0 + kScanBatch*64 of lm row lmr, lane-strided (coalesced).
__device__ __forceinline__ void tile_block_weights(const TailArgs& p, int lmr, int b0, float M, int lane,
                                                   float (&w)[kScanBatch]) {
  const float* mv = p.amax_val + (size_t)lmr * p.n_tiles;
  const float* sv = p.amax_sum + (size_t)lmr * p.n_tiles;
#pragma unroll
  for (int u = 0; u < kScanBatch; ++u) {
    const int t = b0 + 64 * u + lane;
    w[u] = t < p.n_tiles ? tile_weight(mv[t], sv[t], M, p.samp_k) : 0.f;
  }
}

// S of lm row `lmr` with maximum M (one wavefront): the blocks' sums in block
// order.
__device__ float row_sum(const TailArgs& p, int lmr, float M, int lane) {
  float acc = 0.f;
  for (int b0 = 0; b0 < p.n_tiles; b0 += 64 * kScanBatch) {
    float w[kScanBatch];
    tile_block_weights(p, lmr, b0, M, lane, w);
#pragma unroll
    for (int u = 0; u < kScanBatch; ++u) acc += wave_sum(w[u]);
  }
  return acc;
}

// Draw from lm row `lmr` with uniform u (one wavefront; every lane returns the
// token): the block of 64 tiles where the running sum (the same block sums in
// the same order as S) passes u S, the tile inside it, then the column.
__device__ int wave_sample(const TailArgs& p, int lmr, float M, float S, float u, int lane) {
  const float k = p.samp_k, target = u * S;
  float carry = 0.f, rem = 0.f;
  int tsel = -1;
  for (int b0 = 0; b0 < p.n_tiles && tsel < 0; b0 += 64 * kScanBatch) {
    float w[kScanBatch];
    tile_block_weights(p, lmr, b0, M, lane, w);
#pragma unroll
    for (int v = 0; v < kScanBatch; ++v) {
      if (tsel >= 0) break;                          // uniform
      const float tot = wave_sum(w[v]);
      if (carry + tot > target) {                    // uniform
        const float incl = wave_incl_scan(w[v], lane);
        const uint64_t hit = __ballot(w[v] > 0.f && carry + incl > target);
        const uint64_t nz = __ballot(w[v] > 0.f);
        const int l = hit ? __ffsll((unsigned long long)hit) - 1 : 63 - __clzll((long long)nz);
        tsel = b0 + 64 * v + l;
        rem = target - (carry + __shfl(incl - w[v], l));
      }
      carry += tot;
    }
  }
  if (tsel < 0) {          // u S rounded up to S: the last tile with weight, its last column
    for (int b = (p.n_tiles - 1) / 64 * 64; b >= 0 && tsel < 0; b -= 64) {
      const int t = b + lane;
      const float w = t < p.n_tiles ? tile_weight(p.amax_val[(size_t)lmr * p.n_tiles + t],
                                                  p.amax_sum[(size_t)lmr * p.n_tiles + t], M, k) : 0.f;
      const uint64_t nz = __ballot(w > 0.f);
      if (nz) tsel = b + 63 - __clzll((long long)nz);
    }
    if (tsel < 0) return 0;
    rem = INFINITY;
  }
  // columns of the chosen tile, 64 at a time (one per lane), running sum in column order
  int x = -1, last = -1;
  float ccarry = 0.f;
  for (int c0 = 0; c0 < p.tile_w && x < 0; c0 += 64) {
    const int col = tsel * p.tile_w + c0 + lane;
    float w = 0.f;
    if (c0 + lane < p.tile_w && col < p.vocab)
      w = __builtin_amdgcn_exp2f((p.logits[(size_t)lmr * p.vocab + col] - M) * k);
    const float cincl = wave_incl_scan(w, lane);
    const uint64_t chit = __ballot(w > 0.f && ccarry + cincl > rem);
    const uint64_t cnz = __ballot(w > 0.f);
    if (chit) x = c0 + __ffsll((unsigned long long)chit) - 1;
    if (cnz) last = c0 + 63 - __clzll((long long)cnz);
    ccarry += __shfl(cincl, 63);
  }
  if (x < 0) x = last < 0 ? 0 : last;   // rounding: the tile's last column with weight
  return tsel * p.tile_w + x;
}

// Residual draw at a rejected position: weights max(0, p(x) - q(x)) over the
// vocabulary, p from the target row zp (M_p, S_p), q from the draft row zq
// (M_q, S_q).  Block g holds entries [256 g, 256 g + 256), 4 per lane.  Whole
// workgroups: resid_sums leaves the sums of its share of the blocks (wavefront
// w of workgroup `part` of n_part: blocks 16 part + w, + 16 n_part, ..) in LDS
// or, where several workgroups share the row, in memory; resid_pick scans all
// block sums in order and the chosen block inside (-1 when the residual has no
// mass, only through rounding).
struct Resid {
  const float *zp, *zq;
  float Mp, Mq, k, ip, iq;
  int V;
  __device__ __forceinline__ void entries(int g, int lane, float (&r)[4]) const {
    const int x0 = g * kResidBlock + 4 * lane;     // V is a multiple of 16: a lane's 4 entries are all in range or not
    if (x0 < V) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(zp + x0);
      const f32x4 b = *reinterpret_cast<const f32x4*>(zq + x0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        r[e] = fmaxf(__builtin_amdgcn_exp2f((a[e] - Mp) * k) * ip - __builtin_amdgcn_exp2f((b[e] - Mq) * k) * iq, 0.f);
    } else {
      r[0] = r[1] = r[2] = r[3] = 0.f;
    }
  }
};

__device__ void resid_sums(const Resid& q, int part, int n_part, float* part_s, float* part_g) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, step = 16 * n_part;
  const int n_blocks = (q.V + kResidBlock - 1) / kResidBlock;
  for (int g0 = 16 * part + wave; g0 < n_blocks; g0 += step * kScanBatch) {
    float r[kScanBatch][4];
#pragma unroll
    for (int v = 0; v < kScanBatch; ++v) {
      const int g = g0 + step * v;
      if (g < n_blocks) q.entries(g, lane, r[v]);
      else r[v][0] = r[v][1] = r[v][2] = r[v][3] = 0.f;
    }
#pragma unroll
    for (int v = 0; v < kScanBatch; ++v) {
      const int g = g0 + step * v;
      if (g >= n_blocks) break;                      // uniform
      const float t = wave_sum(((r[v][0] + r[v][1]) + r[v][2]) + r[v][3]);
      if (lane == 0) {
        if (n_part > 1)      // read by another workgroup of this launch: device scope
          __hip_atomic_store(part_g + g, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          part_s[g] = t;
      }
    }
  }
}

__device__ int resid_pick(const Resid& q, float u, const float* part_s, int* pick_s) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n_blocks = (q.V + kResidBlock - 1) / kResidBlock;
  __syncthreads();
  if (wave == 0) {
    float total = 0.f;
    for (int g0 = 0; g0 < n_blocks; g0 += 64) total += wave_sum(g0 + lane < n_blocks ? part_s[g0 + lane] : 0.f);
    int x_sel = -1;
    if (total > 0.f) {
      const float target = u * total;
      float carry = 0.f, rem = INFINITY;
      int gsel = -1;
      for (int g0 = 0; g0 < n_blocks && gsel < 0; g0 += 64) {
        const float w = g0 + lane < n_blocks ? part_s[g0 + lane] : 0.f;
        const float tot = wave_sum(w);
        if (carry + tot > target) {
          const float incl = wave_incl_scan(w, lane);
          const uint64_t hit = __ballot(w > 0.f && carry + incl > target);
          const uint64_t nz = __ballot(w > 0.f);
          const int l = hit ? __ffsll((unsigned long long)hit) - 1 : 63 - __clzll((long long)nz);
          gsel = g0 + l;
          rem = target - (carry + __shfl(incl - w, l));
        }
        carry += tot;
      }
      if (gsel < 0) {      // u * total rounded up to total: the last block with mass
        for (int g = n_blocks - 1; g >= 0; --g)
          if (part_s[g] > 0.f) { gsel = g; break; }
      }
      if (gsel < 0) gsel = 0;   // not reached: total > 0 means some block has mass
      // inside the block: lane sums in lane order, then the lane's 4 entries
      float r[4];
      q.entries(gsel, lane, r);
      const float ls = ((r[0] + r[1]) + r[2]) + r[3];
      const float incl = wave_incl_scan(ls, lane);
      const uint64_t hit = __ballot(ls > 0.f && incl > rem);
      const uint64_t nz = __ballot(ls > 0.f);
      const int l = hit ? __ffsll((unsigned long long)hit) - 1 : (nz ? 63 - __clzll((long long)nz) : 0);
      if (lane == l) {
        float acc = incl - ls;
        int last = -1;
        for (int e = 0; e < 4; ++e) {
          if (r[e] > 0.f) last = e;
          if (x_sel < 0 && hit && r[e] > 0.f && acc + r[e] > rem) x_sel = gsel * kResidBlock + 4 * lane + e;
          acc += r[e];
        }
        if (x_sel < 0) x_sel = gsel * kResidBlock + 4 * lane + (last < 0 ? 0 : last);
        pick_s[0] = x_sel;
      }
      if (!nz && lane == 0) pick_s[0] = -1;
    } else if (lane == 0) {
      pick_s[0] = -1;
    }
  }
  __syncthreads();
  return pick_s[0];
}

// Phase clock of the fused loop (one thread): at the start of a step tail the
// verify phase ends (target pass up to its lm_head); at the end of the tail --
// after the next pass is staged -- the draft phase (draft pass and tail) or the
// accept phase (verify tail) ends, and a verify tail records the step's end.
__device__ void clock_tail_start(const TailArgs& p) {
  if (p.tail != TAIL_VERIFY) return;
  const unsigned long long t = wall_clock64();
  // (device scope: the tail may end in another workgroup)
  __hip_atomic_store(&p.clock->tail_start, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  p.clock->verify_ticks += t - p.clock->pass_start[0];
}
__device__ void clock_tail_end(const TailArgs& p) {
  const unsigned long long t = wall_clock64();
  PhaseClock* c = p.clock;
  if (p.tail == TAIL_DRAFT || p.tail == TAIL_VSD_DRAFT) {
    c->draft_ticks += t - c->pass_start[1];
  } else if (p.tail == TAIL_VERIFY) {
    c->accept_ticks += t - __hip_atomic_load(&c->tail_start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    c->step_end[c->n_steps % kStepRing] = t;
    ++c->n_steps;
  }
}

__global__ __launch_bounds__(1024) void k_lm_tail(const TailArgs p) {
  __shared__ int res_s[kMaxK + 1];
  __shared__ float Ms[kMaxK + 1], Ss[kMaxK + 1];   // sampling: the rows' maxima and normalisers
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const FwdDesc* dp = p.desc;
  const int sj = blockIdx.x;
  if (sj >= dp->n_seq) return;                    // uniform: the whole block leaves
  // block 0 keeps the clock; with several sequences k_stage (the kernel after
  // this one) ends the phase
  const int part = blockIdx.y, n_part = gridDim.y;   // workgroups of a sequence (sampled verify passes)
  const bool clock = p.clock && blockIdx.x == 0;
  if (clock && part == 0 && tid == 0) clock_tail_start(p);
  const PassSeq ps = dp->seq[sj];
  const int rows = min(ps.lm_rows, kMaxK + 1);
  const bool sampling =
      p.samp_k > 0.f && (p.tail == TAIL_PREFILL || p.tail == TAIL_DRAFT || p.tail == TAIL_VERIFY);
  for (int r = wave; r < rows; r += 16) {
    float bv = -INFINITY;
    int bi = INT_MAX;
    const float* vals = p.amax_val + (size_t)(ps.lm0 + r) * p.n_tiles;
    const int* idxs = p.amax_idx + (size_t)(ps.lm0 + r) * p.n_tiles;
    for (int t0 = lane; t0 < p.n_tiles; t0 += 64 * 16) {
      float xv[16];
      int xi[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int t = t0 + 64 * u;
        xv[u] = t < p.n_tiles ? vals[t] : -INFINITY;
        xi[u] = t < p.n_tiles ? idxs[t] : INT_MAX;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (better(xv[u], xi[u], bv, bi)) { bv = xv[u]; bi = xi[u]; }
    }
    wave_best(bv, bi);
    const float S = sampling ? row_sum(p, ps.lm0 + r, bv, lane) : 0.f;
    if (lane == 0) {
      res_s[r] = (bi >= 0 && bi < p.vocab) ? bi : 0;
      Ms[r] = bv;
      Ss[r] = S;
    }
  }
  __syncthreads();
  if (!sampling) {
    if (tid == 0) {
      for (int r = 0; r < rows; ++r) p.result[ps.lm0 + r] = res_s[r];
      p.lm_map[ps.slot] = int2{ps.lm0, rows};
      seq_tail(p, ps, res_s);
    }
  } else {
    // speculative sampling: draft candidates and the first token are drawn
    // from their rows; a verify pass runs the keep tests in order and draws
    // the step's last token from the residual (first rejection) or from the
    // bonus row (all kept)
    __shared__ float part_s[kMaxResidBlocks];
    __shared__ int pick_s[2], a_s, tok_s, last_s;
    SeqState* st = p.states + ps.slot;
    const int draw = st->draw;
    if (p.tail == TAIL_DRAFT || p.tail == TAIL_PREFILL) {
      const int purpose = p.tail == TAIL_PREFILL ? PURPOSE_FIRST : PURPOSE_DRAFT;
      for (int r = wave; r < rows; r += 16) {
        const int x = wave_sample(p, ps.lm0 + r, Ms[r], Ss[r], sample_uniform(p.seed, ps.slot, draw, r, purpose), lane);
        if (lane == 0) res_s[r] = x;
      }
      if (p.tail == TAIL_DRAFT && tid < min(rows, kMaxK)) {   // the draft's rows, for the keep tests
        st->qM[tid] = Ms[tid];
        st->qS[tid] = Ss[tid];
      }
      __syncthreads();
      if (tid == 0) {
        for (int r = 0; r < rows; ++r) p.result[ps.lm0 + r] = res_s[r];
        p.lm_map[ps.slot] = int2{ps.lm0, rows};
        seq_tail(p, ps, res_s);
      }
    } else {   // TAIL_VERIFY
      const int k = st->k;
      if (wave == 0) {
        // keep test of position j in lane j (k <= 32); a = the first position not kept
        const int2 dm = p.lm_map_draft[ps.slot];   // this slot's rows of the draft's last pass
        bool keep = true;
        if (lane < k) {
          const int x = st->cand[lane];
          const float pz = p.logits[(size_t)(ps.lm0 + lane) * p.vocab + x];
          const float qz = p.q_logits[(size_t)(dm.x + lane) * p.vocab + x];
          const float pp = __builtin_amdgcn_exp2f((pz - Ms[lane]) * p.samp_k) / Ss[lane];
          const float qq = __builtin_amdgcn_exp2f((qz - st->qM[lane]) * p.samp_k) / st->qS[lane];
          keep = sample_uniform(p.seed, ps.slot, draw, lane, PURPOSE_KEEP) * qq < pp;
        }
        const uint64_t rejected = __ballot(!keep);
        if (lane == 0) a_s = rejected ? __ffsll((unsigned long long)rejected) - 1 : k;
      }
      __syncthreads();
      const int a = a_s;
      const float u = sample_uniform(p.seed, ps.slot, draw, a, PURPOSE_LAST);
      Resid q{};
      if (a < k) {
        const int2 dm = p.lm_map_draft[ps.slot];
        q = Resid{p.logits + (size_t)(ps.lm0 + a) * p.vocab, p.q_logits + (size_t)(dm.x + a) * p.vocab, Ms[a], st->qM[a],
                  p.samp_k, 1.0f / Ss[a], 1.0f / st->qS[a], p.vocab};
        resid_sums(q, part, n_part, part_s, p.resid_part + (size_t)sj * kMaxResidBlocks);
      }
      // The row's workgroups count themselves in, with their sums and their reads
      // of the state complete; the last one goes on alone.
      if (n_part > 1) {
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        if (tid == 0) {
          const int prev = __hip_atomic_fetch_add(p.counters + sj, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          last_s = prev == n_part - 1;
          if (prev == n_part - 1) __hip_atomic_store(p.counters + sj, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!last_s) return;                          // uniform over the workgroup
        if (a < k)
          for (int g = tid; g < (p.vocab + kResidBlock - 1) / kResidBlock; g += 1024)
            part_s[g] = __hip_atomic_load(p.resid_part + (size_t)sj * kMaxResidBlocks + g, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
      }
      const int tok = a < k ? resid_pick(q, u, part_s, pick_s) : -1;
      if (tok < 0) {                                // bonus row (or a residual without mass)
        if (wave == 0) {
          const int x = wave_sample(p, ps.lm0 + a, Ms[a], Ss[a], u, lane);
          if (lane == 0) tok_s = x;
        }
      } else if (tid == 0) {
        tok_s = tok;
      }
      __syncthreads();
      if (tid == 0) {
        for (int r = 0; r < rows; ++r) p.result[ps.lm0 + r] = res_s[r];
        p.lm_map[ps.slot] = int2{ps.lm0, rows};
        commit_verify(p, ps, a, tok_s, res_s);
      }
    }
  }
  if (gridDim.x == 1 && p.next_desc) {
    __syncthreads();
    stage_next(p, false);
  }
  if (clock && (gridDim.x == 1 || !p.next_desc)) {
    __syncthreads();
    if (tid == 0) clock_tail_end(p);
  }
}

__global__ __launch_bounds__(256) void k_stage(const TailArgs p) {
  stage_next(p, true);
  if (p.clock) {
    __syncthreads();
    if (threadIdx.x == 0) clock_tail_end(p);
  }
}

template <int EPI, int MT, int S>
hipError_t launch_one(int nw, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  const size_t lds = (size_t)nw * S * MT * 256 * sizeof(float);
  if (lds > 64 * 1024) {   // (wide tiles of several row tiles: above the default limit)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm<MT, S, EPI>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (ev.start) {
    hipExtLaunchKernelGGL(k_gemm<MT, S, EPI>, dim3(a.n_tiles, a.ksplit), dim3(64 * nw), (uint32_t)lds, st, ev.start, ev.stop,
                          0u, a);
  } else {
    k_gemm<MT, S, EPI><<<dim3(a.n_tiles, a.ksplit), dim3(64 * nw), lds, st>>>(a);
  }
  return hipGetLastError();
}

template <int EPI, int MT, int S>
hipError_t launch_if(int nw, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  if constexpr (gemm_instance(EPI, MT, S)) return launch_one<EPI, MT, S>(nw, a, st, ev);
  return hipErrorInvalidValue;
}

template <int EPI, int MT>
hipError_t launch_s(int S, int nw, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  switch (S) {
    case 1: return launch_if<EPI, MT, 1>(nw, a, st, ev);
    case 2: return launch_if<EPI, MT, 2>(nw, a, st, ev);
    case 4: return launch_if<EPI, MT, 4>(nw, a, st, ev);
    case 7: return launch_if<EPI, MT, 7>(nw, a, st, ev);
    case 8: return launch_if<EPI, MT, 8>(nw, a, st, ev);
    case 9: return launch_if<EPI, MT, 9>(nw, a, st, ev);
    case 10: return launch_if<EPI, MT, 10>(nw, a, st, ev);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t launch_mt(int mt, int S, int nw, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  switch (mt) {
    case 1: return launch_s<EPI, 1>(S, nw, a, st, ev);
    case 2: return launch_s<EPI, 2>(S, nw, a, st, ev);
    case 3: return launch_s<EPI, 3>(S, nw, a, st, ev);
    case 4: return launch_s<EPI, 4>(S, nw, a, st, ev);
  }
  return hipErrorInvalidValue;
}

// What launch_qkv_attn_any does for a shape: launch it, or report its
// co-resident workgroups (at `pre` preloaded gate/up iterations) or the
// largest `pre` its LDS holds.
struct FuseQuery {
  enum { LAUNCH, CAPACITY, PRE_MAX } what = LAUNCH;
  int pre = 0;
  int result = 0;
};

template <int MT, int S, int OKI, int SG>
constexpr size_t fuse_red_bytes() {   // (a fused down tile's [4][256] fits below the O units'; the gate/up
                                       // tile reduces in the preload area)
  return std::max((size_t)4 * S * MT * 256, OKI > 0 ? (size_t)8 * 2 * 256 : (size_t)0) * sizeof(float);
}

template <int MT, int S, int HD, int OKI, int SG, int SD>
hipError_t launch_qkv_attn_one(const GemmArgs& g, const AttnArgs& a, const FuseCtl& f, const GemmArgs& o,
                               const GemmArgs& gu, const GemmArgs& dn, hipStream_t st, LaunchEvents ev,
                               FuseQuery& q) {
  constexpr size_t red = fuse_red_bytes<MT, S, OKI, SG>();
  constexpr size_t iter = (size_t)4 * SG * 1024;            // one preloaded iteration
  // preloaded iterations that the attention arrays' static LDS holds (the
  // last ones of each workgroup; the attention workgroups load them there
  // after their attention)
  constexpr int stat_fit = SG > 0 ? (int)(sizeof(FusedStatLds<HD, SG>) / std::max<size_t>(iter, 1)) : 0;
  auto kern = k_qkv_attn<MT, S, HD, OKI, SG, SD>;
  const int pre = q.what == FuseQuery::LAUNCH ? std::max(f.gu_pre, f.gu_pre_q) : q.pre;
  // (at least one iteration's room: the gate/up tile's reduction)
  const size_t lds = red + (SG > 0 ? (size_t)std::max(pre - std::min(pre, stat_fit), 1) * iter : 0);
  if (q.what != FuseQuery::LAUNCH) {
    int dev = 0;
    hipDeviceProp_t prop;
    hipFuncAttributes attr;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess ||
        hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(kern)) != hipSuccess)
      return hipErrorInvalidValue;
    const size_t room = (size_t)prop.maxSharedMemoryPerMultiProcessor;
    if (q.what == FuseQuery::PRE_MAX) {
      const size_t used = attr.sharedSizeBytes + red;
      q.result = SG > 0 && room > used ? (int)std::min<size_t>(kGuPreMax, (room - used) / iter + stat_fit) : 0;
      return hipSuccess;
    }
    if (attr.sharedSizeBytes + lds > room) return hipErrorInvalidValue;
    int per_cu = 0;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(room - attr.sharedSizeBytes)) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 512, lds) != hipSuccess)
      return hipErrorInvalidValue;
    q.result = per_cu * prop.multiProcessorCount;
    return hipSuccess;
  }
  FuseCtl fl = f;
  fl.gu_lds = (int)red;
  fl.gu_stat = stat_fit;
  const int grid = g.n_tiles + f.n_cons + f.o_extra;
  if (ev.start) {
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(512), (uint32_t)lds, st, ev.start, ev.stop, 0u, g, a, fl, o, gu, dn);
  } else {
    kern<<<grid, 512, lds, st>>>(g, a, fl, o, gu, dn);
  }
  return hipGetLastError();
}

template <int MT, int S, int HD>
hipError_t launch_qkv_attn_oki(int oki, int sg, int sd, const GemmArgs& g, const AttnArgs& a, const FuseCtl& f,
                               const GemmArgs& o, const GemmArgs& gu, const GemmArgs& dn, hipStream_t st,
                               LaunchEvents ev, FuseQuery& q) {
  if (oki == 0 && sg == 0 && sd == 0) return launch_qkv_attn_one<MT, S, HD, 0, 0, 0>(g, a, f, o, gu, dn, st, ev, q);
  if constexpr (MT == 1) {
    switch (oki * 1000 + sg * 10 + sd) {
      case 8000: return launch_qkv_attn_one<MT, S, HD, 8, 0, 0>(g, a, f, o, gu, dn, st, ev, q);
      case 8040: return launch_qkv_attn_one<MT, S, HD, 8, 4, 0>(g, a, f, o, gu, dn, st, ev, q);
      case 8070: return launch_qkv_attn_one<MT, S, HD, 8, 7, 0>(g, a, f, o, gu, dn, st, ev, q);
      case 8041: return launch_qkv_attn_one<MT, S, HD, 8, 4, 1>(g, a, f, o, gu, dn, st, ev, q);
      case 8071: return launch_qkv_attn_one<MT, S, HD, 8, 7, 1>(g, a, f, o, gu, dn, st, ev, q);
      case 16000: return launch_qkv_attn_one<MT, S, HD, 16, 0, 0>(g, a, f, o, gu, dn, st, ev, q);
      case 16040: return launch_qkv_attn_one<MT, S, HD, 16, 4, 0>(g, a, f, o, gu, dn, st, ev, q);
      case 16070: return launch_qkv_attn_one<MT, S, HD, 16, 7, 0>(g, a, f, o, gu, dn, st, ev, q);
      case 16041: return launch_qkv_attn_one<MT, S, HD, 16, 4, 1>(g, a, f, o, gu, dn, st, ev, q);
      case 16071: return launch_qkv_attn_one<MT, S, HD, 16, 7, 1>(g, a, f, o, gu, dn, st, ev, q);
    }
  }
  return hipErrorInvalidValue;
}

template <int MT, int S>
hipError_t launch_qkv_attn_hd(int hd, int oki, int sg, int sd, const GemmArgs& g, const AttnArgs& a,
                              const FuseCtl& f, const GemmArgs& o, const GemmArgs& gu, const GemmArgs& dn,
                              hipStream_t st, LaunchEvents ev, FuseQuery& q) {
  if (hd == 64) return launch_qkv_attn_oki<MT, S, 64>(oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
  if (hd == 128) return launch_qkv_attn_oki<MT, S, 128>(oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
  return hipErrorInvalidValue;
}

hipError_t launch_qkv_attn_any(int mt, int S, int hd, int oki, int sg, int sd, const GemmArgs& g, const AttnArgs& a,
                               const FuseCtl& f, const GemmArgs& o, const GemmArgs& gu, const GemmArgs& dn,
                               hipStream_t st, LaunchEvents ev, FuseQuery& q) {
  switch (mt * 4 + S) {
    case 1 * 4 + 1: return launch_qkv_attn_hd<1, 1>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 1 * 4 + 2: return launch_qkv_attn_hd<1, 2>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 2 * 4 + 1: return launch_qkv_attn_hd<2, 1>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 2 * 4 + 2: return launch_qkv_attn_hd<2, 2>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 3 * 4 + 1: return launch_qkv_attn_hd<3, 1>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 3 * 4 + 2: return launch_qkv_attn_hd<3, 2>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 4 * 4 + 1: return launch_qkv_attn_hd<4, 1>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
    case 4 * 4 + 2: return launch_qkv_attn_hd<4, 2>(hd, oki, sg, sd, g, a, f, o, gu, dn, st, ev, q);
  }
  return hipErrorInvalidValue;
}

// k-blocks per wavefront of the fused O units for an O weight of kb k-blocks
// (0: no fused O; -1: unsupported)
int o_ki(int kb) { return kb == 0 ? 0 : kb <= 64 ? 8 : kb <= kFuseOMaxKb ? 16 : -1; }

}  // namespace

// Shape key of the fused launch queries (cached: the answers do not change,
// and nothing is asked during a graph capture once the engine has warmed up).
static int64_t fuse_key(int kind, int mt, int S, int head_dim, int oki, int sg, int sd, int pre) {
  return (((((((int64_t)kind * 8 + mt) * 4 + S) * 256 + head_dim) * 32 + oki) * 16 + sg) * 4 + sd) * 16 + pre;
}

static int fuse_query(int kind, int mt, int S, int head_dim, int oki, int sg, int sd, int pre) {
  static std::map<int64_t, int> cache;   // 0 or more: the answer; -1: unsupported
  const int64_t key = fuse_key(kind, mt, S, head_dim, oki, sg, sd, pre);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  FuseQuery q;
  q.what = kind == 0 ? FuseQuery::CAPACITY : FuseQuery::PRE_MAX;
  q.pre = pre;
  int r = -1;
  if (launch_qkv_attn_any(mt, S, head_dim, oki, sg, sd, GemmArgs{}, AttnArgs{}, FuseCtl{}, GemmArgs{}, GemmArgs{},
                          GemmArgs{}, nullptr, LaunchEvents{}, q) == hipSuccess)
    r = q.result;
  cache[key] = r;
  return r;
}

int qkv_attn_capacity(int mt, int S, int head_dim, int o_kb, int gu_S, int gu_pre, int d_S) {
  const int oki = o_ki(o_kb);
  if (mt < 1 || mt > 4 || S < 1 || S > 2 || (head_dim != 64 && head_dim != 128) || oki < 0 || (oki > 0 && mt != 1) ||
      (gu_S != 0 && gu_S != 4 && gu_S != 7) || (gu_S > 0 && (oki == 0 || gu_pre < 1 || gu_pre > kGuPreMax)) ||
      (d_S != 0 && (d_S != 1 || gu_S == 0)))
    return 0;
  const int r = fuse_query(0, mt, S, head_dim, oki, gu_S, d_S, gu_S > 0 ? gu_pre : 0);
  return r > 0 ? r : 0;
}

int qkv_attn_gu_pre_max(int S, int head_dim, int o_kb, int gu_S, int d_S) {
  const int oki = o_ki(o_kb);
  if (S < 1 || S > 2 || (head_dim != 64 && head_dim != 128) || oki <= 0 || (gu_S != 4 && gu_S != 7) ||
      (d_S != 0 && d_S != 1))
    return 0;
  const int r = fuse_query(1, 1, S, head_dim, oki, gu_S, d_S, 0);
  return r > 0 ? r : 0;
}

hipError_t launch_qkv_attn(int mt, int S, int head_dim, const GemmArgs& g, const AttnArgs& a, const FuseCtl& f,
                           const GemmArgs* o, const GemmArgs* gu, int gu_S, const GemmArgs* dn, hipStream_t st,
                           LaunchEvents ev) {
  // the GEMM tiles cover the strips exactly, one input range; the attention
  // part is the single-chunk plan with one query tile per workgroup
  if (g.n_tiles < 1 || g.ksplit != 1 || g.kb_split < g.kb_total || (size_t)g.n_tiles * S != (size_t)g.n_strips)
    return hipErrorInvalidValue;
  if (!a.wide || a.n_splits != 1 || a.nqt != 1 || a.split_len % 128 || a.n_seq < 1 || a.n_seq > kMaxPassSeqs)
    return hipErrorInvalidValue;
  if (!f.counters || !f.err || f.n_prod != g.n_tiles || f.n_cons != a.n_kv * a.n_qblocks * a.n_seq)
    return hipErrorInvalidValue;
  int oki = 0;
  const int workers = f.o_extra + f.n_prod;
  if (o) {
    // one row tile; O units: one strip each over one input range, every
    // worker with two units an extra workgroup
    oki = o_ki(o->kb_total);
    if (mt != 1 || oki <= 0 || o->n_strips != f.o_units || f.o_units < 1 || f.o_extra < 0 || f.o_two < 0 ||
        f.o_two > f.o_extra || f.o_units > workers + f.o_two || o->act_rows != a.act_rows || !o->A || !o->x ||
        !o->xg || !o->g_next || !o->ss_out || o->desc != a.desc)
      return hipErrorInvalidValue;
  } else if (f.o_units != 0 || f.o_extra != 0) {
    return hipErrorInvalidValue;
  }
  const int grid = g.n_tiles + f.n_cons + f.o_extra;
  if (gu) {
    // gate/up: needs the O units; tiles of gu_S strips cover the weight
    // exactly, one per workgroup of the grid at most; four wavefronts;
    // preloaded iterations within every wavefront's range
    if (!o || (gu_S != 4 && gu_S != 7) || gu->n_tiles != f.gu_tiles || f.gu_tiles < 1 || f.gu_tiles > grid ||
        (size_t)gu->n_tiles * gu_S != (size_t)gu->n_strips || gu->ksplit != 1 || gu->kb_split < gu->kb_total ||
        f.gu_pre < 1 || f.gu_pre_q < 0 || f.gu_pre > kGuPreMax || f.gu_pre_q > f.gu_pre || f.gu_pre > gu->kb_total / 4 ||
        f.n_odone != std::min(workers, f.o_units - f.o_two) || gu->act_rows != a.act_rows || gu->desc != a.desc ||
        gu->A != o->xg || gu->ss_in != o->ss_out)
      return hipErrorInvalidValue;
  } else if (f.gu_tiles != 0) {
    return hipErrorInvalidValue;
  }
  if (dn) {
    // down: needs gate/up; one strip per tile, one or two input ranges (each
    // unit, a tile's range, one workgroup of the grid at most); its input is
    // gate/up's output, its residual and outputs the O workers'
    if (!gu || dn->n_tiles * dn->ksplit != f.d_tiles || f.d_tiles < 1 || f.d_tiles > grid ||
        dn->n_tiles != dn->n_strips || dn->ksplit < 1 || dn->ksplit > 2 || dn->kb_split < 1 ||
        (dn->ksplit - 1) * dn->kb_split >= dn->kb_total || dn->ksplit * dn->kb_split < dn->kb_total ||
        dn->A != gu->out || dn->x != o->x || dn->xg != o->xg || dn->ss_out != o->ss_out || !dn->g_next ||
        dn->act_rows != a.act_rows || dn->desc != a.desc)
      return hipErrorInvalidValue;
    if (dn->ksplit > 1 && (!dn->part || !dn->counters || dn->n_tiles > kSplitCounters ||
                           (size_t)dn->n_tiles * dn->ksplit * 256 > kSplitPartFloats))
      return hipErrorInvalidValue;
  } else if (f.d_tiles != 0) {
    return hipErrorInvalidValue;
  }
  const int cap = qkv_attn_capacity(mt, S, head_dim, o ? o->kb_total : 0, gu ? gu_S : 0, gu ? f.gu_pre : 0,
                                    dn ? 1 : 0);
  if (cap <= 0 || grid > cap) return hipErrorInvalidValue;
  FuseQuery q;
  return launch_qkv_attn_any(mt, S, head_dim, oki, gu ? gu_S : 0, dn ? 1 : 0, g, a, f, o ? *o : GemmArgs{},
                             gu ? *gu : GemmArgs{}, dn ? *dn : GemmArgs{}, st, ev, q);
}

hipError_t launch_gemm(int epi, int mt, int S, int nw, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  if (!gemm_launchable(epi, mt, S, nw, a.n_strips, a.kb_total, a.n_tiles, a.ksplit, a.kb_split) ||
      (a.ksplit > 1 && (!a.part || !a.counters)))
    return hipErrorInvalidValue;
  switch (epi) {
    case EPI_QKV: return launch_mt<EPI_QKV>(mt, S, nw, a, st, ev);
    case EPI_RESID: return launch_mt<EPI_RESID>(mt, S, nw, a, st, ev);
    case EPI_SWIGLU: return launch_mt<EPI_SWIGLU>(mt, S, nw, a, st, ev);
    case EPI_LOGITS: return launch_mt<EPI_LOGITS>(mt, S, nw, a, st, ev);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_tail(const TailArgs& a, int n_seq, hipStream_t st) {
  if (n_seq < 1 || n_seq > kMaxPassSeqs) return hipErrorInvalidValue;
  // A sampled verify pass draws from a whole row of the vocabulary: one
  // workgroup per 16 blocks of it (one per wavefront), up to 32 per sequence and
  // 512 in all (152064 entries, one sequence, K = 12: a step's draft and verify
  // tails 88 us with one workgroup and reductions through shuffles, 48 now; a
  // vocabulary of 4096 is 16 blocks)
  int n_part = 1;
  if (a.samp_k > 0.f && a.tail == TAIL_VERIFY) {
    if (!a.resid_part || !a.counters) return hipErrorInvalidValue;
    n_part = std::max(1, std::min({(a.vocab + 16 * kResidBlock - 1) / (16 * kResidBlock), 32, 512 / n_seq}));
  }
  k_lm_tail<<<dim3(n_seq, n_part), 1024, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_stage(const TailArgs& a, hipStream_t st) {
  k_stage<<<1, 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace pard
