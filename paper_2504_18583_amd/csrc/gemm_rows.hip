// Row-block GEMM: passes of more than kMaxRows rows (prefill chunks and
// batched decode passes), where the GEMMs are dense contractions.
//
//   Y[r, n] = sum_k A[r, k] * W[n, k]        (W block-packed fp16, A fp16)
//
// A workgroup of CG wavefronts owns MB*16 rows x CG*NS strips (16 columns
// each) over one input range; every wavefront has all MB row tiles and its own
// NS strips.
//   * A passes through LDS, shared by the wavefronts: LDS-DMA loads (no
//     registers held) into a ring of four units of two k-blocks, three units
//     ahead, each 16 x 32 block stored in MFMA operand order (lane-linear
//     reads, no bank conflicts).
//   * W is read from memory straight into the MFMA operand registers, four
//     k-blocks ahead.
//   * A row tile's fragment register is refilled for the next k-block as soon
//     as its MFMAs are issued, so one fragment set is enough and the LDS reads
//     spread over the MFMAs.
// One barrier per unit (two k-blocks).  A unit's loads go out in one fixed
// order, so the wait before the barrier leaves the newer loads in flight, and
// the loop over whole rings has no branch (with one, every wait at the join
// covers all LDS reads in flight).
//
// Against the earlier form (A through registers into a two-deep LDS buffer, one
// 144 x 256 tile per CU), gate/up of the 8B shape in kernel traces of whole
// calls (profiles/prefill_8b_kernel_trace.txt and the batch-32 traces): the 288
// rows of 32 conversations' steps 92.3 -> 80.8 us (837 TFLOP/s), a 517-row prompt
// 176 -> 141 us (862), an 8192-row prompt 170 us for each 512-row chunk, which was
// the longest (709), -> 929 us for each 4096-row one (1036; torch's fp16 matmul
// at 8192^3: 1150).
//
// Blocks are numbered so that the row blocks of one column tile run on the
// same XCD at about the same time (the hardware deals block i to XCD i % 8):
// the later blocks' weight reads then hit that XCD's L2 rather than HBM.
// Narrow GEMMs split the input dimension (ksplit > 1) to fill the chip; each
// split writes fp32 partial tiles and k_gemm_rows_red adds them in split
// order and runs the epilogue, so results are deterministic.
//
// Epilogues: as in the skinny GEMM.  Stores of 2 bytes straight from the
// accumulator layout cost as much as a narrow GEMM, so QKV and the residual go
// through a transpose within quads of lanes (8 and 16 bytes a lane) and gate/up
// through LDS (stand-alone launches at 4096 rows: QKV 8B 272 -> 204 us, O 165 ->
// 144, 1B QKV 111 -> 69; the 8B QKV of a 517-row prompt, with its earlier split's
// reduction, 72 -> 49 us in the traces).
#include "attn_tile.h"
#include "gemm_util.h"
#include "pard_internal.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <type_traits>

namespace pard {
namespace {

// Tile variants: MB row tiles, CG wavefronts of NS strips, and the time of one
// k-block in us with one and with two workgroups on a CU, which the plan's cost
// model uses (plan_rows).
struct Variant {
  int mb, cg, ns;
  float us1, us2;      // us2 = 0: one workgroup per CU
};
constexpr Variant kVariants[] = {
    {8, 8, 2, 0.42f, 0.f},       // 128 x 256 in eight wavefronts: prefill chunks
    {9, 8, 2, 0.53f, 0.f},       // 144 x 256 in eight wavefronts: 32 conversations' nine rows
    {9, 4, 2, 0.30f, 0.58f},     // 144 x 128: narrow weights
    {8, 4, 2, 0.26f, 0.56f},     // 128 x 128
    {6, 4, 2, 0.26f, 0.44f},     // 96 x 128: few rows
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

// Compile-time loop: f(integral_constant<int, I>) for I in [B, E).  The row
// tiles of an accumulator are walked this way so that every index is a
// constant whatever the loop body's size: the accumulators then stay in
// registers (a rolled loop would index them dynamically, in scratch memory).
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// 4 x 4 transpose within each quad of lanes: lane q holds rows 0..3 of column
// q and gets columns 0..3 of row q (two exchanges, with lane q ^ 1 and q ^ 2).
// The epilogues use it to read and write 8 and 16 bytes a lane: one memory
// instruction where the accumulator layout takes four.
__device__ __forceinline__ f32x4 quad_transpose(f32x4 a, int lane) {
  const auto xor1 = [](float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false)); };
  const auto xor2 = [](float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false)); };
  const bool odd = lane & 1, hi = lane & 2;
  const float r = xor1(odd ? a[0] : a[1]), r2 = xor1(odd ? a[2] : a[3]);
  // row (q & 1) and row 2 + (q & 1), columns (q & 2) and the next
  const float p0 = odd ? r : a[0], p1 = odd ? a[1] : r;
  const float q0 = odd ? r2 : a[2], q1 = odd ? a[3] : r2;
  const float s0 = xor2(hi ? p0 : q0), s1 = xor2(hi ? p1 : q1);
  return f32x4{hi ? s0 : p0, hi ? s1 : p1, hi ? q0 : s0, hi ? q1 : s1};
}

// Four values as fp16, flagged as f16_flagged does.
__device__ __forceinline__ uint2 pack4_flagged(float a, float b, float c, float d, bool& bad) {
  const uint32_t h0 = f16_flagged(a, bad), h1 = f16_flagged(b, bad), h2 = f16_flagged(c, bad), h3 = f16_flagged(d, bad);
  return uint2{h0 | (h1 << 16), h2 | (h3 << 16)};
}

// 1/rms of R*T/16 rows (T threads) from the producer's per-tile sums of
// squares (fixed order), 16 threads per row: every row's loads of 64 tiles are
// in flight together.
template <bool LM, int R>
__device__ __forceinline__ void rows_scales(const GemmArgs& p, const FwdDesc* dp, int row0, int n, int row_count,
                                            float* rs_s) {
  const int tid = threadIdx.x, step = blockDim.x >> 4;
  int src[R];
  float t[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int gr = row0 + (tid >> 4) + step * k;
    src[k] = gr < row_count ? (LM ? dp->lm_src[gr] : gr) : 0;
    t[k] = 0.f;
  }
  for (int q0 = tid & 15; q0 < p.ss_tiles; q0 += 64) {
    float part[R][4];
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + 16 * u;
        part[k][u] = q < p.ss_tiles ? p.ss_in[(size_t)src[k] * p.ss_stride + q] : 0.f;
      }
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
      for (int u = 0; u < 4; ++u) t[k] += part[k][u];
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    float v = t[k];
    v += __shfl_xor(v, 8);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 1);
    const int r = (tid >> 4) + step * k;
    if ((tid & 15) == 0 && r < n) rs_s[r] = 1.0f / sqrtf(v * p.inv_k + p.eps);
  }
}

// Epilogue of one wavefront's accumulators: MBW row tiles from row `row0` of
// the pass (rs_s: their scales), strips strip0 .. strip0 + NS - 1.  Lane l
// holds, for row tile mt and strip s, column (strip*16 + l%16) of rows
// mt*16 + 4*(l/16) + i.  ent: this wavefront's entry in the per-row outputs
// (row sums of squares, argmax).  o_lds: NS KiB of this wavefront's LDS.
template <int EPI, int MBW, int NS>
__device__ __forceinline__ void rows_epilogue(const GemmArgs& p, const FwdDesc* dp, f32x4 (&acc)[MBW][NS], int strip0,
                                              int ent, int row0, int row_count, int lane, const float* rs_s,
                                              u32x4* o_lds) {
  const int c16 = lane & 15, g4 = lane >> 4;
  [[maybe_unused]] bool bad = false;
  if constexpr (EPI == EPI_QKV) {
    // a linear pass is one sequence's consecutive positions
    const bool linear = dp->linear != 0;
    const int lin_pos = dp->seq[0].pos0, lin_slot = dp->seq[0].slot;
    const int tr = g4 * 4 + (c16 & 3), tc = (c16 >> 2) * 4;   // this lane's row and first column once transposed
    static_for<0, MBW>([&](auto mtc) __attribute__((always_inline)) {
      constexpr int mt = decltype(mtc)::value;
      if (row0 + mt * 16 >= row_count) return;       // uniform
      const int r = row0 + mt * 16 + tr, rc = min(r, row_count - 1);
      const int pos = linear ? lin_pos + rc : dp->pos[rc];
      const size_t cache = (size_t)(linear ? lin_slot : dp->slot[rc]) * p.kv_seq_stride;
      const float sc = rs_s[mt * 16 + tr];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int n0 = (strip0 + s) * 16;            // (Q, K and V begin at multiples of head_dim)
        if (strip0 + s >= p.n_strips) continue;      // uniform
        if (n0 < p.q_dim + p.kv_dim) {               // uniform: Q or K, four columns of one row
          const int n = n0 + tc;
          f32x4 y = quad_transpose(acc[mt][s], lane) * sc;
          if (p.bias) y += *reinterpret_cast<const f32x4*>(p.bias + n);
          const f32x4 cs = *reinterpret_cast<const f32x4*>(p.rope + (size_t)pos * (p.hd / 2) + ((n % p.hd) >> 1));
          const float a0 = y[0] * cs[0] - y[1] * cs[1], a1 = y[1] * cs[0] + y[0] * cs[1];
          const float a2 = y[2] * cs[2] - y[3] * cs[3], a3 = y[3] * cs[2] + y[2] * cs[3];
          bool bad_r = false;
          const uint2 v = pack4_flagged(a0, a1, a2, a3, bad_r);
          if (r < row_count) {
            bad |= bad_r;
            const int c = n - p.q_dim;
            uint16_t* dst = n0 < p.q_dim ? p.out + (size_t)r * p.ld_out + n
                                         : p.kc + cache + (size_t)(c / p.hd) * p.cap * p.hd + k_index(pos, c % p.hd, p.hd);
            *reinterpret_cast<uint2*>(dst) = v;
          }
        } else {                                     // V: one column of four rows
          const int n = n0 + c16, c = n - p.q_dim - p.kv_dim;
          const float bias = p.bias ? p.bias[n] : 0.f;
          const int rl = mt * 16 + g4 * 4, r0 = row0 + rl;
          const size_t head = (size_t)(c / p.hd) * (p.cap / 32);
          float y[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) y[i] = acc[mt][s][i] * rs_s[rl + i] + bias;
          if (linear && !(lin_pos & 3) && r0 + 3 < row_count) {
            // four consecutive keys from a multiple of four on are contiguous
            const int ps = lin_pos + r0;
            *reinterpret_cast<uint2*>(p.vc + (size_t)lin_slot * p.kv_seq_stride +
                                      ((head + (ps >> 5)) * p.hd + (c % p.hd)) * 32 + v_slot(ps & 31)) =
                pack4_flagged(y[0], y[1], y[2], y[3], bad);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (r0 + i < row_count) {
                const int ps = linear ? lin_pos + r0 + i : dp->pos[r0 + i];
                const size_t at = (size_t)(linear ? lin_slot : dp->slot[r0 + i]) * p.kv_seq_stride;
                p.vc[at + ((head + (ps >> 5)) * p.hd + (c % p.hd)) * 32 + v_slot(ps & 31)] = f16_flagged(y[i], bad);
              }
          }
        }
      }
    });
    flag_range(bad, p.ovf);
  } else if constexpr (EPI == EPI_RESID) {
    const int tr = g4 * 4 + (c16 & 3), tc = (c16 >> 2) * 4;   // this lane's row and first column once transposed
    static_for<0, MBW>([&](auto mtc) __attribute__((always_inline)) {
      constexpr int mt = decltype(mtc)::value;
      if (row0 + mt * 16 >= row_count) return;       // uniform
      const int r = row0 + mt * 16 + tr;
      float sq = 0.f;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int n = (strip0 + s) * 16 + tc;
        if (strip0 + s >= p.n_strips) continue;      // uniform
        const f32x4 y = quad_transpose(acc[mt][s], lane);
        if (r < row_count) {
          f32x4* xp = reinterpret_cast<f32x4*>(p.x + (size_t)r * p.ldx + n);
          const f32x4 g = *reinterpret_cast<const f32x4*>(p.g_next + n);
          const f32x4 xn = *xp + y;                  // residual + projection
          *xp = xn;
          *reinterpret_cast<uint2*>(p.xg + act_index(r, n, p.act_rows)) =
              pack4_flagged(xn[0] * g[0], xn[1] * g[1], xn[2] * g[2], xn[3] * g[3], bad);
          sq += xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3];
        }
      }
      // the row's four lanes (c16, c16 ^ 4, ..): DPP row rotates by 4 and 8
      sq += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(sq), 0x124, 0xF, 0xF, false));
      sq += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(sq), 0x128, 0xF, 0xF, false));
      if (c16 < 4 && r < row_count && strip0 < p.n_strips) p.ss_out[(size_t)r * p.ss_stride + ent] = sq;
    });
    flag_range(bad, p.ovf);
  } else if constexpr (EPI == EPI_SWIGLU) {
    // 8 gate columns then the 8 up columns of the same features per strip: the
    // wavefront's strips are NS*8 consecutive features (16 bytes a strip and
    // row) of one k-block of h.  Four row tiles at a time are assembled in LDS
    // and written with 16-byte stores (2-byte stores straight from the
    // accumulator layout made the epilogue as long as a 4096-wide GEMM).
    constexpr int G = 4;
    static_for<0, (MBW + G - 1) / G>([&](auto gc) __attribute__((always_inline)) {
      constexpr int m0 = decltype(gc)::value * G, m1 = m0 + G < MBW ? m0 + G : MBW;
      if (row0 + m0 * 16 >= row_count) return;       // uniform
      static_for<m0, m1>([&](auto mtc) __attribute__((always_inline)) {
        constexpr int mt = decltype(mtc)::value;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int rl = mt * 16 + g4 * 4 + i, lr = rl - m0 * 16;
            const float gt = acc[mt][s][i] * rs_s[rl];
            // the up value of lane l < 8 is in lane l + 8 of its row of 16 (DPP row rotate by 8)
            const float up = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, gt), 0x128,
                                                                                0xF, 0xF, false));
            // silu(g) = g / (1 + e^-g), with the hardware exp2 and reciprocal
            const float h = gt * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-gt * attn::kLog2e)) * up;
            bool bad_h = false;
            const uint16_t hb = f16_flagged(h, bad_h);
            bad |= bad_h && c16 < 8 && row0 + rl < row_count && strip0 + s < p.n_strips;
            // lane pairs pack two values into one dword (DPP quad swap);
            // chunks are swizzled by (row / 4) % NS so the rows of one store
            // land in different banks
            const uint32_t pair =
                (uint32_t)hb | ((uint32_t)__builtin_amdgcn_mov_dpp((int)hb, 0xB1, 0xF, 0xF, false) << 16);
            if (c16 < 8 && !(c16 & 1))
              reinterpret_cast<uint32_t*>(o_lds)[(lr * NS + (s ^ ((lr >> 2) & (NS - 1)))) * 4 + (c16 >> 1)] = pair;
          }
        }
      });
      for (int e = lane; e < (m1 - m0) * 16 * NS; e += 64) {
        const int lr = e / NS, c = e % NS, r = row0 + m0 * 16 + lr;
        const u32x4 v = o_lds[lr * NS + (c ^ ((lr >> 2) & (NS - 1)))];
        if (r < row_count && strip0 + c < p.n_strips)
          *reinterpret_cast<u32x4*>(p.out + act_index(r, (strip0 + c) * 8, p.act_rows)) = v;
      }
    });
    flag_range(bad, p.ovf);
  } else {  // EPI_LOGITS
    static_for<0, MBW>([&](auto mtc) __attribute__((always_inline)) {
      constexpr int mt = decltype(mtc)::value;
      if (row0 + mt * 16 >= row_count || strip0 >= p.n_strips) return;   // uniform
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rl = mt * 16 + g4 * 4 + i, r = row0 + rl;
        float bv = -INFINITY;
        int bi = INT_MAX;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int n = (strip0 + s) * 16 + c16;
          if (strip0 + s >= p.n_strips) continue;    // uniform
          const float val = acc[mt][s][i] * rs_s[rl];
          if (r < row_count) p.logits[(size_t)r * p.vocab + n] = val;
          if (better(val, n, bv, bi)) { bv = val; bi = n; }
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) {
          const float ov = __shfl_xor(bv, off);
          const int oi = __shfl_xor(bi, off);
          if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if (c16 == 0 && r < row_count) {
          p.amax_val[(size_t)r * p.amax_stride + ent] = bv;
          p.amax_idx[(size_t)r * p.amax_stride + ent] = bi;
        }
        if (p.samp_k > 0.f) {       // sampling: the entry's softmax weight relative to its max
          float sw = 0.f;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            if (strip0 + s >= p.n_strips) continue;  // uniform
            sw += __builtin_amdgcn_exp2f((acc[mt][s][i] * rs_s[rl] - bv) * p.samp_k);
          }
#pragma unroll
          for (int off = 8; off > 0; off >>= 1) sw += __shfl_xor(sw, off);
          if (c16 == 0 && r < row_count) p.amax_sum[(size_t)r * p.amax_stride + ent] = sw;
        }
      }
    });
  }
}

// Block id -> (column tile, input split, row block), row blocks fastest and
// consecutive ids on one XCD.
__device__ __forceinline__ void rows_block(const GemmArgs& p, int* tile, int* ks, int* mb) {
  const int G = gridDim.x, bid = blockIdx.x;
  const int per = G / 8, rem = G % 8, xcd = bid % 8, slot = bid / 8;
  const int lid = xcd * per + min(xcd, rem) + slot;
  *mb = lid % p.m_blocks;
  const int rest = lid / p.m_blocks;
  *ks = rest % p.ksplit;
  *tile = rest / p.ksplit;
}

// One 1 KiB block of A (16 rows x 32 columns, each lane its 16 bytes) straight
// into LDS.
__device__ __forceinline__ void lds_load(__amdgpu_buffer_rsrc_t rs, u32x4* dst, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

// s_waitcnt vmcnt(n) with the other counters not waited for.
constexpr int vm_wait(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70 | 0xF00; }

// Workgroup barrier for LDS filled by LDS-DMA: the caller has waited for its
// own loads, and no access may move across.  (__syncthreads would wait for
// every load in flight.)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int EPI, int MB, int CG, int NS>
__global__ __launch_bounds__(64 * CG, 2) void k_gemm_rows(const GemmArgs p) {
  constexpr int D = 4;                         // weight k-blocks in flight
  constexpr int NQ = (MB + CG - 1) / CG;       // A blocks per wavefront and k-block
  constexpr int ND = 2 * NQ, NWL = 2 * NS;     // A and W loads per wavefront and unit
  constexpr bool LM = EPI == EPI_LOGITS;       // rows are the pass's lm rows
  // the ring: four arrays of their own (the compiler's waits before an LDS
  // read cover the loads into that array only)
  __shared__ __attribute__((aligned(16))) u32x4 s0[2 * MB * 64], s1[2 * MB * 64], s2[2 * MB * 64], s3[2 * MB * 64];
  __shared__ float rs_s[MB * 16];
  static_assert(EPI != EPI_SWIGLU || CG * NS * 64 <= 2 * MB * 64, "the SwiGLU staging fits one ring array");

  int tile, ks, mb;
  rows_block(p, &tile, &ks, &mb);
  const FwdDesc* dp = p.desc;
  const int row_count = LM ? dp->n_lm : dp->n_rows;
  const int row0 = mb * MB * 16;
  if (row0 >= row_count) return;                     // uniform: the whole block leaves
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kb0 = ks * p.kb_total / p.ksplit, kb1 = (ks + 1) * p.kb_total / p.ksplit;
  const int n_kb = kb1 - kb0;                        // >= 1 (host: ksplit <= kb_total)

  // W: this wavefront's strips, block (kb, strip) at (kb * n_strips + strip)
  // KiB; strips past the weight's last one (only in the last column tile) read
  // zeros or neighbouring weights: their columns are never stored
  const int strip0 = (tile * CG + wave) * NS;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.W), 0, (int)min((size_t)p.n_strips * p.kb_total * 1024, (size_t)0x7fffffff),
      kRsrcWord3);
  const int w_voff = (strip0 * 64 + lane) * 16;

  // A: block mt of a k-block holds rows mt*16 .., lane l row l % 16, columns
  // 8 * (l / 16) ..; rows past the pass re-read its last one and are never
  // stored.  Wavefront w loads blocks w, w + CG, .. (past MB: the last one
  // again, the same bytes to the same place)
  const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.A), 0, p.act_rows * p.lda * 2, kRsrcWord3);
  int a_voff[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int gr = min(row0 + min(wave + CG * i, MB - 1) * 16 + (lane & 15), row_count - 1);
    a_voff[i] = (LM ? dp->lm_src[gr] : gr) * 64 + (lane >> 4) * 16;
  }
  // (indices past the range are clamped: cache hits, never multiplied)
  auto load_a = [&](u32x4* buf, int u) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int kb = kb0 + min(2 * u + s, n_kb - 1);
#pragma unroll
      for (int i = 0; i < NQ; ++i)
        lds_load(ars, buf + (s * MB + min(wave + CG * i, MB - 1)) * 64, a_voff[i], kb * (p.act_rows * 64));
    }
  };
  u32x4 wr[D][NS], av[MB];
  auto load_w = [&](int slot, int it) {
    const int kb = kb0 + min(it, n_kb - 1);
#pragma unroll
    for (int s = 0; s < NS; ++s)
      wr[slot][s] = __builtin_amdgcn_raw_buffer_load_b128(wrs, w_voff, (kb * p.n_strips + s) * 1024, 0);
  };
  auto fence = [&]() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };

  f32x4 acc[MB][NS];
#pragma unroll
  for (int mt = 0; mt < MB; ++mt)
#pragma unroll
    for (int s = 0; s < NS; ++s) acc[mt][s] = f32x4{0.f, 0.f, 0.f, 0.f};

  // the loads of the three units before the first, in the loop's order
  load_a(s0, 0);
  fence();
  load_a(s1, 1);
  fence();
  load_w(0, 0);
  fence();
  load_w(1, 1);
  fence();
  load_a(s2, 2);
  fence();
  load_w(2, 2);
  fence();
  load_w(3, 3);
  fence();
  __builtin_amdgcn_s_waitcnt(vm_wait(2 * ND + 2 * NWL));   // this wavefront's loads of unit 0
  lds_barrier();
#pragma unroll
  for (int mt = 0; mt < MB; ++mt) av[mt] = s0[mt * 64 + lane];
  // Unit u (ring phase ph): k-blocks 2u, 2u + 1.  On entry av holds k-block
  // 2u's fragments.  The wait and the barrier make unit u + 1 complete in LDS;
  // unit u + 3 goes where unit u - 1 was (last read before the barrier before
  // this one).  checked: k-blocks past the range are not multiplied.
  auto unit = [&](int u, int ph, const u32x4* cur, const u32x4* nxt, u32x4* dst, auto checked)
                  __attribute__((always_inline)) {
    fence();
    __builtin_amdgcn_s_waitcnt(vm_wait(ND + 2 * NWL));
    lds_barrier();
    load_a(dst, u + 3);
    fence();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int it = 2 * u + s, slot = (2 * ph + s) & 3;
      if (!decltype(checked)::value || it < n_kb) {  // uniform
#pragma unroll
        for (int mt = 0; mt < MB; ++mt) {
#pragma unroll
          for (int st = 0; st < NS; ++st)
            acc[mt][st] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, av[mt]),
                                                                 __builtin_bit_cast(f16x8, wr[slot][st]), acc[mt][st],
                                                                 0, 0, 0);
          fence();
          av[mt] = (s == 0 ? cur : nxt)[((s == 0 ? MB : 0) + mt) * 64 + lane];
          fence();
        }
      }
      load_w(slot, it + D);
      fence();
    }
  };
  constexpr std::integral_constant<bool, false> whole{};
  constexpr std::integral_constant<bool, true> checked{};
  int u = 0;
  for (; 2 * u + 8 <= n_kb; u += 4) {
    unit(u, 0, s0, s1, s3, whole);
    unit(u + 1, 1, s1, s2, s0, whole);
    unit(u + 2, 2, s2, s3, s1, whole);
    unit(u + 3, 3, s3, s0, s2, whole);
  }
  if (2 * u < n_kb) {
    unit(u, 0, s0, s1, s3, checked);
    unit(u + 1, 1, s1, s2, s0, checked);
    unit(u + 2, 2, s2, s3, s1, checked);
    unit(u + 3, 3, s3, s0, s2, checked);
  }

  if (p.ksplit > 1) {
    // partial tiles of this split: block (split, row tile, strip) of 256
    // floats in lane order (coalesced)
    float* part = p.part + ((size_t)ks * p.m_blocks * MB + mb * MB) * p.n_strips * 256;
    static_for<0, MB>([&](auto mtc) __attribute__((always_inline)) {
      constexpr int mt = decltype(mtc)::value;
      if (row0 + mt * 16 >= row_count) return;       // uniform
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (strip0 + s < p.n_strips)                 // uniform
          *reinterpret_cast<f32x4*>(part + ((size_t)mt * p.n_strips + strip0 + s) * 256 + lane * 4) = acc[mt][s];
    });
    // (the clamped loads still in flight land before the workgroup gives its LDS back)
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    return;
  }
  // the clamped loads still in flight must not land in LDS that the epilogue
  // reuses
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  if constexpr (EPI != EPI_RESID) rows_scales<LM, (MB * 16 * 16 + 64 * CG - 1) / (64 * CG)>(p, dp, row0, MB * 16, row_count, rs_s);
  __syncthreads();
  rows_epilogue<EPI, MB, NS>(p, dp, acc, strip0, tile * CG + wave, row0, row_count, lane, rs_s, s0 + wave * NS * 64);
}

// Sum of the input splits of k_gemm_rows in split order, then the epilogue.
// One workgroup per 16-row tile and 16 strips (wavefront w: strips 4w ..);
// each thread has the loads of up to 8 splits in flight at a time.
template <int EPI>
__global__ __launch_bounds__(256) void k_gemm_rows_red(const GemmArgs p, int row_tiles) {
  constexpr int NS = 4;
  constexpr bool LM = EPI == EPI_LOGITS;
  __shared__ float rs_s[16];
  __shared__ __attribute__((aligned(16))) u32x4 o_lds[EPI == EPI_SWIGLU ? 4 * NS * 64 : 1];
  const int mt = blockIdx.y;
  const FwdDesc* dp = p.desc;
  const int row_count = LM ? dp->n_lm : dp->n_rows;
  if (mt * 16 >= row_count) return;                 // uniform
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int strip0 = (blockIdx.x * 4 + wave) * NS;
  const size_t split = (size_t)row_tiles * p.n_strips * 256;
  const float* base = p.part + (size_t)mt * p.n_strips * 256 + lane * 4;
  int at[NS];                                        // (strips past the weight re-read its last one)
#pragma unroll
  for (int s = 0; s < NS; ++s) at[s] = min(strip0 + s, p.n_strips - 1) * 256;
  f32x4 sum[1][NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) sum[0][s] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < p.ksplit; k0 += 8) {
    f32x4 v[8][NS];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (k0 + u < p.ksplit) v[u][s] = *reinterpret_cast<const f32x4*>(base + (k0 + u) * split + at[s]);
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (k0 + u < p.ksplit) sum[0][s] += v[u][s];
  }
  if constexpr (EPI != EPI_RESID) {
    rows_scales<LM, 1>(p, dp, mt * 16, 16, row_count, rs_s);
    __syncthreads();
  }
  rows_epilogue<EPI, 1, NS>(p, dp, sum, strip0, strip0 / NS, mt * 16, row_count, lane, rs_s,
                            EPI == EPI_SWIGLU ? o_lds + wave * NS * 64 : nullptr);
}

template <int EPI, int V>
hipError_t launch_variant(const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  constexpr Variant v = kVariants[V];
  const int grid = a.n_tiles * a.m_blocks * a.ksplit;
  auto kern = k_gemm_rows<EPI, v.mb, v.cg, v.ns>;
  if (ev.start) {
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(64 * v.cg), 0u, st, ev.start, a.ksplit > 1 ? nullptr : ev.stop, 0u, a);
  } else {
    kern<<<grid, 64 * v.cg, 0, st>>>(a);
  }
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_epi(int variant, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  hipError_t e = hipErrorInvalidValue;
  switch (variant) {
    case 0: e = launch_variant<EPI, 0>(a, st, ev); break;
    case 1: e = launch_variant<EPI, 1>(a, st, ev); break;
    case 2: e = launch_variant<EPI, 2>(a, st, ev); break;
    case 3: e = launch_variant<EPI, 3>(a, st, ev); break;
    case 4: e = launch_variant<EPI, 4>(a, st, ev); break;
  }
  if (e != hipSuccess || a.ksplit == 1) return e;
  const int row_tiles = a.m_blocks * kVariants[variant].mb;
  const dim3 grid((a.n_strips + 15) / 16, row_tiles);
  if (ev.start) {
    hipExtLaunchKernelGGL(k_gemm_rows_red<EPI>, grid, dim3(256), 0u, st, nullptr, ev.stop, 0u, a, row_tiles);
  } else {
    k_gemm_rows_red<EPI><<<grid, 256, 0, st>>>(a, row_tiles);
  }
  return hipGetLastError();
}

}  // namespace

// The variant and input split with the least modelled time at the typical row
// count: a launch's fixed cost and that of each round of workgroups over the
// 256 CUs (fill and epilogue), the k-blocks of these rounds at the variant's time
// with one or two workgroups on a CU, no less than the weights' reading, and for
// a split its fp32 partial tiles, written and read.  The constants are fitted to
// 195 measured (shape, rows) points of the 8B, 1B, Qwen2.5-7B and 0.5B layers at
// 72 to 4096 rows, all variants and splits each: the chosen plan is 1.7 % slower
// than the fastest one measured on average (15 % at most); constants estimated
// from a few shapes of the earlier epilogues: 6.4 %.
// The grid covers max_rows.
RowsPlan plan_rows(int n_strips, int kb_total, int max_rows, int typ_rows) {
  constexpr float kLaunchUs = 5.8f, kRoundUs = 1.2f, kWeightBytesPerUs = 5.3e6f, kPartBytesPerUs = 2.1e6f;
  RowsPlan best;
  float best_us = 0.f;
  const int typ = std::max(1, std::min(typ_rows, max_rows));
  for (int v = 0; v < kNumVariants; ++v) {
    const Variant& k = kVariants[v];
    const int n_tiles = (n_strips + k.cg * k.ns - 1) / (k.cg * k.ns);
    const int blocks = (typ + k.mb * 16 - 1) / (k.mb * 16), max_blocks = (max_rows + k.mb * 16 - 1) / (k.mb * 16);
    for (int ksplit = 1; ksplit <= std::min(12, std::max(1, kb_total / 8)); ++ksplit) {
      if (ksplit > 1 && (size_t)ksplit * max_blocks * k.mb * n_strips * 256 > kRowsPartTotal) break;
      const int per_cu = (n_tiles * blocks * ksplit + 255) / 256;
      const float rounds = k.us2 > 0.f ? (per_cu / 2) * k.us2 + (per_cu % 2) * k.us1 : per_cu * k.us1;
      float us = std::max(per_cu * kRoundUs + rounds * ((kb_total + ksplit - 1) / ksplit),
                          n_strips * (float)kb_total * 1024.f / kWeightBytesPerUs);
      us += kLaunchUs;
      if (ksplit > 1) us += ksplit * (float)((typ + 15) / 16) * n_strips * 1024.f / kPartBytesPerUs;
      if (best.variant < 0 || us < best_us) {
        best_us = us;
        best.variant = v;
        best.n_tiles = n_tiles;
        best.m_blocks = max_blocks;
        best.ksplit = ksplit;
        best.ent_strips = ksplit > 1 ? 4 : k.ns;
        best.entries = (n_strips + best.ent_strips - 1) / best.ent_strips;
      }
    }
  }
  return best;
}

hipError_t launch_gemm_rows(int epi, int variant, const GemmArgs& a, hipStream_t st, LaunchEvents ev) {
  if (variant < 0 || variant >= kNumVariants) return hipErrorInvalidValue;
  const Variant& v = kVariants[variant];
  if (a.n_tiles < 1 || a.m_blocks < 1 || a.ksplit < 1 || a.ksplit > a.kb_total || a.n_strips < 1) return hipErrorInvalidValue;
  if (a.n_tiles * v.cg * v.ns < a.n_strips || (a.ksplit > 1 && !a.part)) return hipErrorInvalidValue;
  if ((size_t)a.n_tiles * a.m_blocks * a.ksplit >= (1u << 31) || a.m_blocks * v.mb > 65535) return hipErrorInvalidValue;
  // A is addressed with 32-bit byte offsets
  if ((size_t)a.act_rows * a.lda * 2 >= ((size_t)1 << 31)) return hipErrorInvalidValue;
  if (a.ksplit > 1 && (size_t)a.ksplit * a.m_blocks * v.mb * a.n_strips * 256 > kRowsPartTotal) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_QKV: return launch_epi<EPI_QKV>(variant, a, st, ev);
    case EPI_RESID: return launch_epi<EPI_RESID>(variant, a, st, ev);
    case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(variant, a, st, ev);
    case EPI_LOGITS: return launch_epi<EPI_LOGITS>(variant, a, st, ev);
  }
  return hipErrorInvalidValue;
}

}  // namespace pard
