// Causal attention of a prefill chunk: one sequence's consecutive rows (more
// than kMaxRows) against its fp16 KV cache, on gfx950 MFMA.
//
// A workgroup of four wavefronts owns one KV head and 64*NQ (row,
// head-in-group) query pairs, 16*NQ of them per wavefront, and walks all keys
// up to its last row's position in stages of 64.  The arithmetic of a tile is
// k_attn's: S^T = K Q^T, base-2 online softmax in fp32, O^T += V^T P^T, the
// S^T accumulator being P^T's operand once packed to fp16.
//   * K and V pass through LDS, shared by the wavefronts: LDS-DMA loads into
//     two stage buffers, the next stage in flight during the current one.  K is
//     cached in operand order; V's lanes fetch their own 16 bytes of the
//     transposed block, so every LDS read is lane-linear.
//   * Q stays in registers; a fragment read from LDS feeds NQ MFMAs.
//   * The running maximum is only raised (and O rescaled) when a score exceeds
//     it by more than 2^kLazy: probabilities then reach 2^kLazy at most, which
//     fp16 holds at full relative precision, and O / l does not depend on the
//     maximum used.
//   * The softmax sums stay per lane until the end.
// Bound: the softmax's VALU work (at head_dim 128 about as long as the MFMAs,
// at 64 twice); two wavefronts per SIMD overlap one's softmax with the other's
// MFMAs.  Workgroups with the most keys start first.
//
// One layer of the 8B attention (head_dim 128) at 4096 rows from position 0:
// k_attn 648 us (212 TFLOP/s), this 154 (894); at position 4096 1070 -> 432
// (955).  The 1B draft's (head_dim 64): 489 -> 91 (758), 771 -> 255 (808).  In the
// trace of an 8192-token prompt (profiles/prefill_8b_kernel_trace.txt), a layer's
// attention in 512-row chunks by k_attn with its merges 1427 us, here in two
// 4096-row chunks 549; the draft's 869 and 351; 517 rows: 23.9 -> 12.2 and 11.9 ->
// 8.6.
#include "attn_tile.h"
#include "pard_internal.h"

namespace pard {
namespace {

using namespace attn;

constexpr int kStageKeys = 64;
constexpr float kLazy = 8.f;

template <int HD, int NQ>
__global__ __launch_bounds__(256, 2) void k_attn_prefill(const AttnArgs p) {
  constexpr int QW = 16 * NQ;                      // query pairs per wavefront
  constexpr int KS = HD / 32;                      // 32-dim steps of Q.K
  constexpr int DB = HD / 16;                      // 16-dim blocks of the output
  constexpr int FR = HD / 16;                      // 1 KiB fragments of 32 keys (K or V)
  // a stage: K of keys 0..31, K of keys 32..63, V, V; two arrays of their own
  // (the compiler's waits before an LDS read cover the loads into that array
  // only)
  __shared__ __attribute__((aligned(16))) u32x4 b0[4 * FR * 64], b1[4 * FR * 64];

  const int kvh = blockIdx.x, qg = gridDim.y - 1 - blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, g4 = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = p.n_heads / p.n_kv;
  const PassSeq d = p.desc->seq[0];
  const int n_qh = d.n_rows * group;
  const int qh0 = qg * 4 * QW;
  if (qh0 >= n_qh) return;                         // uniform: the whole block leaves

  // this wavefront's K or V half: wavefronts 0, 1 load K, 2, 3 V, the odd ones
  // the stage's second 32 keys
  const size_t cache = (size_t)d.slot * p.kv_seq_stride + (size_t)kvh * p.cap * HD;
  const uint16_t* const half = (wave < 2 ? p.kc : p.vc) + cache;
  const int voff = wave < 2 ? lane * 16 : c16 * 64 + g4 * 16;
  const int last32 = p.cap / 32 - 1;
  // (blocks past the cache re-read its last one: those keys are masked)
  auto load = [&](u32x4* buf, int st) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = kv_tile_rsrc<HD>(half, min(st * 2 + (wave & 1), last32));
#pragma unroll
    for (int j = 0; j < FR; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void*)(buf + (wave * FR + j) * 64), 16, voff, j * 1024, 0, 0);
  };
  load(b0, 0);

  // Q fragments (B operand): pair t*16 + c16, dims ks*32 + 8*g4 ..; pairs past
  // the pass repeat its last one and are not stored
  const int qw0 = qh0 + wave * QW;
  u32x4 q[NQ][KS];
  int qpos[NQ];
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    const int qh = min(qw0 + t * 16 + c16, n_qh - 1), row = qh / group, head = kvh * group + qh % group;
    qpos[t] = d.pos0 + row;
    const uint16_t* src = p.q + (size_t)(d.row0 + row) * p.ldq + head * HD + g4 * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[t][ks] = *reinterpret_cast<const u32x4*>(src + ks * 32);
  }
  const int pos_first = d.pos0 + min(qw0, n_qh - 1) / group;              // of this wavefront's pairs
  const int pos_last = d.pos0 + min(qw0 + QW - 1, n_qh - 1) / group;
  const int n_st = (d.pos0 + min(qh0 + 4 * QW - 1, n_qh - 1) / group) / kStageKeys + 1;   // the workgroup's stages

  float m[NQ], l[NQ];
  f32x4 o[NQ][DB];
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    m[t] = -INFINITY;
    l[t] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[t][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float scale2 = p.scale * kLog2e;           // scores in base 2

  auto stage = [&](int st, const u32x4* cur, u32x4* nxt) __attribute__((always_inline)) {
    // this wavefront's loads of the stage are in LDS and its reads of the other
    // buffer are done; after the barrier, everyone's
    __builtin_amdgcn_s_waitcnt(0x0070);            // vmcnt(0) lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (st + 1 < n_st) load(nxt, st + 1);          // uniform
    __builtin_amdgcn_sched_barrier(0);
    const int key0 = st * kStageKeys;
    if (key0 > pos_last) return;                   // uniform: all keys are past this wavefront's rows
    f32x4 s[NQ][4];
#pragma unroll
    for (int t = 0; t < NQ; ++t)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) s[t][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const u32x4 kf = cur[(kb * KS + ks) * 64 + lane];
#pragma unroll
        for (int t = 0; t < NQ; ++t)
          s[t][kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kf),
                                                            __builtin_bit_cast(f16x8, q[t][ks]), s[t][kb], 0, 0, 0);
      }
    if (key0 + kStageKeys - 1 > pos_first) {       // uniform: the stages around the diagonal
#pragma unroll
      for (int t = 0; t < NQ; ++t)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (key0 + kb * 16 + g4 * 4 + i > qpos[t]) s[t][kb][i] = -INFINITY;
    }
    bool raise = false;
    float mx[NQ];
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      float v = fmaxf(s[t][0][0], s[t][0][1]);
#pragma unroll
      for (int i = 2; i < 16; i += 2) v = fmaxf(fmaxf(v, s[t][i / 4][i % 4]), s[t][i / 4][i % 4 + 1]);
      mx[t] = v * scale2;
      raise |= mx[t] > m[t] + kLazy;
    }
    if (__any(raise)) {                            // uniform
#pragma unroll
      for (int t = 0; t < NQ; ++t) {
        // (the first stage holds key 0, which every row sees: m is finite from there on)
        const float mr = max4g(mx[t]);
        const float m_new = mr > m[t] + kLazy ? mr : m[t];   // (each row by itself, whatever its neighbours do)
        const float corr = __builtin_amdgcn_exp2f(m[t] - m_new);
        m[t] = m_new;
        l[t] *= corr;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[t][db] *= corr;
      }
    }
    u32x4 pf[NQ][2];
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        float pv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(fmaf(s[t][kb][i], scale2, -m[t]));
          l[t] += pv[i];
        }
        pf[t][kb >> 1][(kb & 1) * 2] = pack_f16x2(pv[0], pv[1]);
        pf[t][kb >> 1][(kb & 1) * 2 + 1] = pack_f16x2(pv[2], pv[3]);
      }
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const u32x4 vf = cur[((2 + tt) * FR + db) * 64 + lane];
#pragma unroll
        for (int t = 0; t < NQ; ++t)
          o[t][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, vf),
                                                            __builtin_bit_cast(f16x8, pf[t][tt]), o[t][db], 0, 0, 0);
      }
  };
  int st = 0;
  for (; st + 2 <= n_st; st += 2) {
    stage(st, b0, b1);
    stage(st + 1, b1, b0);
  }
  if (st < n_st) stage(st, b0, b1);

  // lane (c16, g4) holds dims db*16 + 4*g4 .. +3 of pair t*16 + c16
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    const float inv = 1.0f / sum4g(l[t]);
    const int qh = qw0 + t * 16 + c16;
    if (qh < n_qh) {
      const int row = qh / group, head = kvh * group + qh % group;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const f32x4 v = o[t][db] * inv;
        *reinterpret_cast<uint2*>(p.out + act_index(d.row0 + row, head * HD + db * 16 + g4 * 4, p.act_rows)) =
            uint2{pack_f16x2(v[0], v[1]), pack_f16x2(v[2], v[3])};
      }
    }
  }
}

template <int HD>
hipError_t launch_hd(const AttnArgs& a, hipStream_t st) {
  const dim3 grid(a.n_kv, a.n_qblocks);
  if (a.nqt == 1) {
    k_attn_prefill<HD, 1><<<grid, 256, 0, st>>>(a);
  } else if (HD == 128 && a.nqt == 2) {
    k_attn_prefill<128, 2><<<grid, 256, 0, st>>>(a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// Which chunks take this kernel, and with how many query tiles per wavefront
// (0: k_attn with key chunks instead).  Measured (us; 8B attention: head_dim
// 128, 32 heads over 8 KV heads, unless stated):
//   * k_attn shares a 48-pair workgroup's keys among its wavefronts, so keys are
//     read from cache four times as often, but it splits a long context: it is
//     ahead for few rows at a long context (65 rows at 4096: 21 against 52; 257
//     rows, 136 workgroups here, at 16000: 167 against 201).  From 160
//     workgroups on (517 rows, 264: 258 against 322 at 16000, 73 against 106 at
//     4096), or where the chunk itself is at least half of the context (517
//     rows at 0: 12 against 29), this kernel is.
//   * Two tiles per wavefront halve the LDS reads per MFMA, but need two
//     workgroups per CU of about the same length: from 768 workgroups on (4096
//     rows at 0: 154 against 169 with one), or from 448 on where most keys
//     precede the chunk (2048 rows at 4096: 181 against 201; at 0, where the
//     workgroups' lengths differ: 53 against 51).  Three tiles: 152 and 226.  At
//     head_dim 64 the softmax bounds both (4096 rows: 92 against 91).
int attn_prefill_tiles(int head_dim, int n_kv, int qpairs, int rows, int l_bound) {
  const auto wgs = [&](int nq) { return (qpairs + 64 * nq - 1) / (64 * nq) * n_kv; };
  const bool own = l_bound <= 2 * rows;            // the chunk is at least half of the context
  if (wgs(1) < 160 && !own) return 0;
  return head_dim == 128 && wgs(2) >= (own ? 768 : 448) ? 2 : 1;
}

hipError_t launch_attn_prefill(int head_dim, const AttnArgs& a, hipStream_t st) {
  if (a.n_seq != 1 || a.n_splits != 1 || a.n_qblocks < 1 || a.n_qblocks > 65535) return hipErrorInvalidValue;
  if (head_dim == 64) return launch_hd<64>(a, st);
  if (head_dim == 128) return launch_hd<128>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace pard
