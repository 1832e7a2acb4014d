// Grouped-query causal attention of a short block of query rows against the
// fp16 KV cache (the draft pass with its mask rows, the verify pass, prefill
// chunks of few rows over long contexts), on gfx950 MFMA.  Q, K, V, the
// probabilities and the output are fp16 (10-bit mantissa: bf16 scores drift past
// the logit tolerance at 8B width).
//
// A workgroup serves one sequence of the pass, one KV head, one group of 16*NQ
// (row, head-in-group) query pairs -- for decode passes every pair of the KV
// head, so each key is read once per pass -- and one chunk of split_len keys
// (256 keys, two 32-key tiles per wavefront; passes over long contexts and of
// many sequences take longer chunks, multiples of 128 keys, so that their grid
// stays within one workgroup per CU: k_attn_chunk).  Its four wavefronts take the
// chunk's tiles round-robin; per tile a wavefront computes
//   S^T[key][q] = K[key] . Q[q]          (v_mfma_f32_16x16x32_f16, K as A,
//                                          Q as B, accumulated over head_dim)
//   O^T[dim][q] += V^T[dim][key] P^T[key][q]
// with an online softmax (running max m, sum l, fp32, base 2) in between.  The
// S^T accumulator of lane l holds keys 4g..4g+3 (and 16+4g..) for query l%16,
// g = l/16, which is exactly the B-operand fragment P^T needs once packed to
// fp16; the V cache stores each 32-key block transposed ([dim][key]) with those
// eight keys of group g contiguous, and the K cache stores each 16-key block as
// ready A fragments, so every K or V fragment is one contiguous 1 KiB
// wavefront load.  Q fragments are staged once in LDS.
//
// Scores are causal by absolute position: key j is visible to the query at
// position pos0 + row iff j <= pos0 + row.  Mask rows of the draft pass are
// ordinary causal rows (Sec. 3.1, eq. 7: candidate k is conditioned on the
// prefix and the k-1 mask tokens before it).
//
// The wavefronts are merged in LDS in wave order.  With several chunks each
// workgroup writes (o, m, l) and a merge kernel combines them in a fixed order
// (k_attn_merge_few in chunk order for up to 16 chunks, k_attn_merge over lanes
// for more).
// All reductions have a fixed order, chunk boundaries sit at fixed multiples
// of split_len, the kernel follows from the chunks alone and a query's
// arithmetic does not depend on which other pairs share its workgroup: results
// are deterministic, and a query's result depends on the other rows of the pass
// only through the chunk length (fixed up to kAttnWideMaxKeys; past it, it
// follows from the number of sequences and query groups).  Chunks past a query's
// position contribute exact zeros.
#include "attn_tile.h"

namespace pard {
namespace {

using namespace attn;

// One workgroup per (KV head, query group, sequence x key chunk).
template <int HD, int NQ, int NW>
__global__ __launch_bounds__(64 * NW) void k_attn(const AttnArgs p) {
  __shared__ AttnLds<HD, NQ> sm;
  attn_tile<HD, NQ, NW, false>(p, blockIdx.x, blockIdx.y, blockIdx.z, FuseCtl{}, sm);
}

// The same attention without the fused launch's needs, for passes whose keys
// come in chunks (batched decode, long contexts): one workgroup per (KV head,
// query group, sequence x key chunk), four wavefronts that take the chunk's
// 32-key tiles round-robin.  Each wavefront's K and V tiles pass through its own
// LDS by LDS-DMA -- the next K requested once this tile's scores are computed,
// the next V once its values are multiplied -- and Q stays in registers, so that
// two workgroups fit a CU and overlap each other's start, waits and merge (k_attn
// holds two tiles in registers: one wavefront per SIMD).  The running maximum is
// raised as in k_attn_prefill.
constexpr float kLazy = 8.f;

template <int HD, int NQ, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_attn_chunk(const AttnArgs p) {
  constexpr int QP = 16 * NQ;        // query pairs per workgroup
  constexpr int KS = HD / 32;        // 32-dim steps of Q.K
  constexpr int DB = HD / 16;        // 16-dim blocks of the output
  constexpr int FR = HD / 16;        // 1 KiB fragments of 32 keys (K or V)
  constexpr int OS = HD + 4;         // row stride of the merge's output tiles in LDS
  constexpr int REC = QP * HD + 2 * QP;   // floats of one chunk record: o [QP][HD], m [QP], l [QP]
  // K and V tiles of the wavefronts (two arrays: the compiler's waits before an
  // LDS read cover the loads into that array only); then each an output tile of
  // the merge
  constexpr int NB = std::max(NW * FR * 64, NW / 4 * QP * OS / 4);
  __shared__ __attribute__((aligned(16))) u32x4 k_s[NB], v_s[NB];
  __shared__ float m_s[NW / 2][QP], l_s[NW / 2][QP];

  const int kvh = blockIdx.x, qg = blockIdx.y;
  const int sj = blockIdx.z / p.n_splits, ch = blockIdx.z % p.n_splits;
  const int tid = threadIdx.x, lane = tid & 63, g4 = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = p.n_heads / p.n_kv;
  if (sj >= p.desc->n_seq) return;                 // uniform: the whole block leaves
  const PassSeq d = p.desc->seq[sj];
  const int L_end = d.pos0 + d.n_rows;
  const int n_qh = d.n_rows * group;
  if (qg * QP >= n_qh) return;                     // uniform
  const int k_begin = ch * p.split_len;            // multiple of 128
  if (k_begin >= L_end) return;                    // uniform: chunk beyond the context
  const int k_end = min(L_end, k_begin + p.split_len);
  const int n_t = (k_end - k_begin + 31) / 32;
  const int n_my = (n_t - wave + NW - 1) / NW;     // (none: the wavefront loads nothing and adds nothing)

  const size_t cache = (size_t)d.slot * p.kv_seq_stride + (size_t)kvh * p.cap * HD;
  u32x4* const kw = k_s + wave * FR * 64;
  u32x4* const vw = v_s + wave * FR * 64;
  auto load = [&](const uint16_t* head, u32x4* dst, int voff, int it) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rs = kv_tile_rsrc<HD>(head, (k_begin >> 5) + wave + NW * it);
#pragma unroll
    for (int j = 0; j < FR; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(dst + j * 64), 16, voff,
                                               j * 1024, 0, 0);
  };
  auto load_k = [&](int it) __attribute__((always_inline)) { load(p.kc + cache, kw, lane * 16, it); };
  auto load_v = [&](int it) __attribute__((always_inline)) { load(p.vc + cache, vw, c16 * 64 + g4 * 16, it); };

  // Q fragments (B operand): pair t*16 + c16, dims ks*32 + 8*g4 ..; pairs past
  // the group repeat its last one and are not stored
  u32x4 q[NQ][KS];
  int qpos[NQ];
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    const int qh = min(qg * QP + t * 16 + c16, n_qh - 1), row = qh / group, head = kvh * group + qh % group;
    qpos[t] = d.pos0 + row;
    const uint16_t* src = p.q + (size_t)(d.row0 + row) * p.ldq + head * HD + g4 * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[t][ks] = *reinterpret_cast<const u32x4*>(src + ks * 32);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (n_my > 0) {                                  // uniform
    load_k(0);
    load_v(0);
  }

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

  for (int it = 0; it < n_my; ++it) {
    const int key0 = k_begin + (wave + NW * it) * 32;
    // this tile's K is in LDS (the FR loads after it are its V's)
    __builtin_amdgcn_s_waitcnt(0x0F70 | FR);
    asm volatile("" ::: "memory");
    f32x4 s[NQ][2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int t = 0; t < NQ; ++t) s[t][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const u32x4 kf = kw[(kb * KS + ks) * 64 + lane];
#pragma unroll
        for (int t = 0; t < NQ; ++t)
          s[t][kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kf),
                                                            __builtin_bit_cast(f16x8, q[t][ks]), s[t][kb], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): K has been read
    if (it + 1 < n_my) load_k(it + 1);             // uniform
    __builtin_amdgcn_sched_barrier(0);
    if (key0 + 31 > d.pos0 || key0 + 31 >= k_end) {   // uniform: tiles that reach a query's position or the end
#pragma unroll
      for (int t = 0; t < NQ; ++t)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = key0 + kb * 16 + g4 * 4 + i;
            if (key >= k_end || key > qpos[t]) s[t][kb][i] = -INFINITY;
          }
    }
    bool raise = false;
    float mx[NQ];
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      float v = fmaxf(s[t][0][0], s[t][0][1]);
#pragma unroll
      for (int i = 2; i < 8; i += 2) v = fmaxf(fmaxf(v, s[t][i / 4][i % 4]), s[t][i / 4][i % 4 + 1]);
      mx[t] = v * scale2;
      raise |= mx[t] > m[t] + kLazy;
    }
    if (__any(raise)) {                            // uniform
#pragma unroll
      for (int t = 0; t < NQ; ++t) {
        const float mr = max4g(mx[t]);
        const float m_new = mr > m[t] + kLazy ? mr : m[t];   // (each row by itself, whatever its neighbours do)
        // (a row that has seen no key yet keeps m = -inf, o = l = 0)
        const float corr = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[t] - m_new);
        m[t] = m_new;
        l[t] *= corr;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[t][db] *= corr;
      }
    }
    u32x4 pf[NQ];
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      const float m_use = m[t] == -INFINITY ? 0.f : m[t];   // keeps 2^(-inf - m) = 0 well defined
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        float pv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(fmaf(s[t][kb][i], scale2, -m_use));
          l[t] += pv[i];
        }
        pf[t][kb * 2] = pack_f16x2(pv[0], pv[1]);
        pf[t][kb * 2 + 1] = pack_f16x2(pv[2], pv[3]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // this tile's V (the loads after it are the next tile's K, if there is one)
    if (it + 1 < n_my) __builtin_amdgcn_s_waitcnt(0x0F70 | FR);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const u32x4 vf = vw[db * 64 + lane];
#pragma unroll
      for (int t = 0; t < NQ; ++t)
        o[t][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, vf), __builtin_bit_cast(f16x8, pf[t]),
                                                          o[t][db], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): V has been read
    if (it + 1 < n_my) load_v(it + 1);             // uniform
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- merge the wavefronts: the upper half into the lower until two are left,
  // then these two ----
#pragma unroll
  for (int t = 0; t < NQ; ++t) l[t] = sum4g(l[t]);
  __syncthreads();                                 // all tiles are done with k_s and v_s
  // lane (c16, g4) holds dims db*16 + 4*g4 .. +3 of pair t*16 + c16
  auto tile = [&](int slot) { return reinterpret_cast<float*>(slot & 1 ? v_s : k_s) + (slot >> 1) * QP * OS; };
  auto publish = [&](int slot) {
    float* ob = tile(slot);
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      if (g4 == 0) {
        m_s[slot][t * 16 + c16] = m[t];
        l_s[slot][t * 16 + c16] = l[t];
      }
#pragma unroll
      for (int db = 0; db < DB; ++db)
        *reinterpret_cast<f32x4*>(ob + (t * 16 + c16) * OS + db * 16 + g4 * 4) = o[t][db];
    }
  };
#pragma unroll
  for (int half = NW / 2; half >= 2; half /= 2) {
    if (wave >= half && wave < 2 * half) publish(wave - half);
    __syncthreads();
    if (wave < half) {
      const float* ob = tile(wave);
#pragma unroll
      for (int t = 0; t < NQ; ++t) {
        const float mb = m_s[wave][t * 16 + c16], lb = l_s[wave][t * 16 + c16];
        const float mn = fmaxf(m[t], mb);
        const float mu = mn == -INFINITY ? 0.f : mn;
        const float sa = __builtin_amdgcn_exp2f(m[t] - mu), sb = __builtin_amdgcn_exp2f(mb - mu);
        l[t] = l[t] * sa + lb * sb;
        m[t] = mn;
#pragma unroll
        for (int db = 0; db < DB; ++db)
          o[t][db] = o[t][db] * sa + *reinterpret_cast<const f32x4*>(ob + (t * 16 + c16) * OS + db * 16 + g4 * 4) * sb;
      }
    }
    __syncthreads();
  }
  if (wave < 2) publish(wave);
  __syncthreads();
  float* rec = p.part + (((size_t)(sj * p.n_kv + kvh) * p.n_qblocks + qg) * p.n_splits + ch) * REC;   // this chunk's record
  const float *o0 = tile(0), *o1 = tile(1);
  // each thread finishes 8 consecutive dims of one pair: one 16-byte fp16 store
  // (or two 16-byte fp32 stores of the chunk record)
  for (int e = tid; e < QP * HD / 8; e += 64 * NW) {
    const int qi = e / (HD / 8), d0 = (e % (HD / 8)) * 8;
    const float M = fmaxf(m_s[0][qi], m_s[1][qi]), M_use = M == -INFINITY ? 0.f : M;
    const float s0 = __builtin_amdgcn_exp2f(m_s[0][qi] - M_use), s1 = __builtin_amdgcn_exp2f(m_s[1][qi] - M_use);
    const float L = l_s[0][qi] * s0 + l_s[1][qi] * s1;
    const f32x4 a = *reinterpret_cast<const f32x4*>(o0 + qi * OS + d0) * s0 + *reinterpret_cast<const f32x4*>(o1 + qi * OS + d0) * s1;
    const f32x4 b = *reinterpret_cast<const f32x4*>(o0 + qi * OS + d0 + 4) * s0 +
                    *reinterpret_cast<const f32x4*>(o1 + qi * OS + d0 + 4) * s1;
    if (p.n_splits == 1) {
      const int qh = qg * QP + qi;
      if (qh < n_qh) {
        const int row = qh / group, head = kvh * group + qh % group;
        const float inv = 1.0f / L;
        store_f16x8(p.out + act_index(d.row0 + row, head * HD + d0, p.act_rows), a * inv, b * inv);
      }
    } else {
      *reinterpret_cast<f32x4*>(rec + qi * HD + d0) = a;
      *reinterpret_cast<f32x4*>(rec + qi * HD + d0 + 4) = b;
      if (d0 == 0) {
        rec[QP * HD + qi] = M;
        rec[QP * HD + QP + qi] = L;
      }
    }
  }
}

// Combine a few key chunks of k_attn (passes with many sequences or query
// groups and short contexts) in chunk order.  Grid (kv head, query group,
// sequence x kMergeParts): per-query (max, sum) first, then each thread merges
// 8 consecutive dims of one pair with the loads of 4 chunks in flight at a
// time.
constexpr int kMergeParts = 8;

template <int HD, int NQ>
__global__ __launch_bounds__(256) void k_attn_merge_few(const AttnArgs p) {
  constexpr int QP = 16 * NQ;
  constexpr int REC = QP * HD + 2 * QP;
  __shared__ float Ms[QP], Linv[QP];
  const int kvh = blockIdx.x, qg = blockIdx.y, tid = threadIdx.x;
  const int sj = blockIdx.z / kMergeParts, part = blockIdx.z % kMergeParts;
  const int group = p.n_heads / p.n_kv;
  if (sj >= p.desc->n_seq) return;                 // uniform
  const PassSeq d = p.desc->seq[sj];
  const int L_end = d.pos0 + d.n_rows;
  const int n_qh = d.n_rows * group;
  if (qg * QP >= n_qh) return;                     // uniform
  const int n_act = min(p.n_splits, (L_end + p.split_len - 1) / p.split_len);
  const float* base = p.part + ((size_t)(sj * p.n_kv + kvh) * p.n_qblocks + qg) * p.n_splits * REC;
  if (tid < QP) {
    // the (m, l) of up to 8 chunks are requested together
    float mv[8], lv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int sx = min(u, n_act - 1);
      mv[u] = base[(size_t)sx * REC + QP * HD + tid];
      lv[u] = base[(size_t)sx * REC + QP * HD + QP + tid];
    }
    float M = -INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < n_act) M = fmaxf(M, mv[u]);
    for (int s = 8; s < n_act; ++s) M = fmaxf(M, base[(size_t)s * REC + QP * HD + tid]);
    const float M_use = M == -INFINITY ? 0.f : M;
    float L = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < n_act) L += lv[u] * __builtin_amdgcn_exp2f(mv[u] - M_use);
    for (int s = 8; s < n_act; ++s)
      L += base[(size_t)s * REC + QP * HD + QP + tid] *
           __builtin_amdgcn_exp2f(base[(size_t)s * REC + QP * HD + tid] - M_use);
    Ms[tid] = M_use;
    Linv[tid] = 1.0f / L;
  }
  __syncthreads();
  constexpr int NV = QP * HD / 8;                  // 8-dim vectors of the group
  constexpr int PER = (NV + kMergeParts - 1) / kMergeParts;
  for (int e = part * PER + tid; e < min(NV, (part + 1) * PER); e += 256) {
    const int q = e / (HD / 8), d0 = (e % (HD / 8)) * 8;
    const int qh = qg * QP + q;
    if (qh >= n_qh) continue;
    const float M = Ms[q];
    f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f}, b = a;
    for (int s0 = 0; s0 < n_act; s0 += 4) {
      f32x4 va[4], vb[4];
      float mv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int sx = min(s0 + u, n_act - 1);
        const float* r = base + (size_t)sx * REC;
        va[u] = *reinterpret_cast<const f32x4*>(r + q * HD + d0);
        vb[u] = *reinterpret_cast<const f32x4*>(r + q * HD + d0 + 4);
        mv[u] = r[QP * HD + q];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s0 + u < n_act) {
          const float sc = __builtin_amdgcn_exp2f(mv[u] - M);
          a += va[u] * sc;
          b += vb[u] * sc;
        }
    }
    const int row = qh / group, head = kvh * group + qh % group;
    store_f16x8(p.out + act_index(d.row0 + row, head * HD + d0, p.act_rows), a * Linv[q], b * Linv[q]);
  }
}

// Combine many key chunks of k_attn (long contexts).  One workgroup per (KV
// head, query group, sequence, 16 output vectors of 8 dims), so that the
// chunks spread over many workgroups and lanes.  (With few chunks its many
// small workgroups cost more than they save: batch-32 step 15.8 -> 16.7 ms.)  The chunks are dealt round-robin over
// lanes, every lane folds its chunks in chunk order with all of its loads in
// flight together, and lanes are combined in a fixed tree order: the result
// is deterministic and no lane waits on more than one round of loads for
// contexts up to 16 x kAttnChunk x 8 keys.
//   (1) per query pair of the workgroup: the running (max, sum) of its chunks'
//       (m, l) over lanes, then the combination over lanes (wavefront
//       shuffles, then the wavefronts in order);
//   (2) per output vector: 16 lanes add o_chunk * 2^(m_chunk - M), then a
//       shuffle tree; lane 0 stores o / L.
constexpr int kMergeFewChunks = 16;   // up to this many chunks: k_attn_merge_few
constexpr int kMergeVecs = 16;     // 8-dim output vectors per workgroup
constexpr int kMergeLanes = 16;    // lanes (chunk subsets) per vector

// (m, l) of two partial softmax sums combined: the larger max is kept and the
// other sum rescaled (an empty part has m = -inf, l = 0).
__device__ __forceinline__ void ml_combine(float& m, float& l, float m2, float l2) {
  const float M = fmaxf(m, m2);
  const float Mu = M == -INFINITY ? 0.f : M;
  l = l * __builtin_amdgcn_exp2f(m - Mu) + l2 * __builtin_amdgcn_exp2f(m2 - Mu);
  m = M;
}

template <int HD, int NQ>
constexpr int merge_parts() { return (16 * NQ * HD / 8 + kMergeVecs - 1) / kMergeVecs; }

template <int HD, int NQ>
__global__ __launch_bounds__(256) void k_attn_merge(const AttnArgs p) {
  constexpr int QP = 16 * NQ;
  constexpr int REC = QP * HD + 2 * QP;
  constexpr int VPQ = HD / 8;                      // output vectors per query pair
  constexpr int NPAIR = (kMergeVecs + VPQ - 1) / VPQ;   // pairs a workgroup touches (1 or 2)
  constexpr int TPP = 256 / NPAIR;                 // step (1) lanes per pair: whole wavefronts
  constexpr int WPP = TPP / 64;
  constexpr int PARTS = merge_parts<HD, NQ>();
  static_assert(VPQ % kMergeVecs == 0 || kMergeVecs % VPQ == 0, "vectors of a workgroup cover whole pairs");
  __shared__ float wm_s[4], wl_s[4], M_s[NPAIR], Linv_s[NPAIR];
  const int kvh = blockIdx.x, qg = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int sj = blockIdx.z / PARTS, part = blockIdx.z % PARTS;
  const int group = p.n_heads / p.n_kv;
  if (sj >= p.desc->n_seq) return;                 // uniform
  const PassSeq d = p.desc->seq[sj];
  const int L_end = d.pos0 + d.n_rows;
  const int n_qh = d.n_rows * group;
  if (qg * QP >= n_qh) return;                     // uniform
  const int n_act = min(p.n_splits, (L_end + p.split_len - 1) / p.split_len);
  const float* base = p.part + ((size_t)(sj * p.n_kv + kvh) * p.n_qblocks + qg) * p.n_splits * REC;
  const int v0 = part * kMergeVecs;                // first output vector of the workgroup
  const int q0 = v0 / VPQ;                         // its first pair

  // (1) (max, sum) of pair q0 + tid / TPP over its chunks
  {
    const int pi = tid / TPP, ln = tid % TPP;
    const int q = min(q0 + pi, QP - 1);
    float m = -INFINITY, l = 0.f;
    for (int s0 = ln; s0 < n_act; s0 += 4 * TPP) {
      float mv[4], lv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int sx = min(s0 + u * TPP, n_act - 1);
        mv[u] = base[(size_t)sx * REC + QP * HD + q];
        lv[u] = base[(size_t)sx * REC + QP * HD + QP + q];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s0 + u * TPP < n_act) ml_combine(m, l, mv[u], lv[u]);
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const float m2 = __shfl_xor(m, off), l2 = __shfl_xor(l, off);
      // lower lane first: both lanes hold the same combination
      if (lane & off) { float mm = m2, ll = l2; ml_combine(mm, ll, m, l); m = mm; l = ll; }
      else ml_combine(m, l, m2, l2);
    }
    if (lane == 0) { wm_s[tid >> 6] = m; wl_s[tid >> 6] = l; }
    __syncthreads();
    if (tid < NPAIR) {
      float M = wm_s[tid * WPP], L = wl_s[tid * WPP];
      for (int w = 1; w < WPP; ++w) ml_combine(M, L, wm_s[tid * WPP + w], wl_s[tid * WPP + w]);
      M_s[tid] = M == -INFINITY ? 0.f : M;
      Linv_s[tid] = 1.0f / L;
    }
    __syncthreads();
  }

  // (2) output vector v0 + tid / kMergeLanes
  const int v = v0 + tid / kMergeLanes, ln = tid % kMergeLanes;
  const int q = v / VPQ, d0 = (v % VPQ) * 8;
  const int qc = min(q, QP - 1);
  const float M = M_s[min(qc - q0, NPAIR - 1)];
  f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f}, b = a;
  for (int s0 = ln; s0 < n_act; s0 += 4 * kMergeLanes) {
    f32x4 va[4], vb[4];
    float mv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int sx = min(s0 + u * kMergeLanes, n_act - 1);
      const float* r = base + (size_t)sx * REC;
      va[u] = *reinterpret_cast<const f32x4*>(r + qc * HD + d0);
      vb[u] = *reinterpret_cast<const f32x4*>(r + qc * HD + d0 + 4);
      mv[u] = r[QP * HD + qc];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u * kMergeLanes < n_act) {
        const float sc = __builtin_amdgcn_exp2f(mv[u] - M);
        a += va[u] * sc;
        b += vb[u] * sc;
      }
  }
#pragma unroll
  for (int off = 1; off < kMergeLanes; off <<= 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // lower lane's value first, so both lanes of a pair hold the same sum
      const float a2 = __shfl_xor(a[i], off), b2 = __shfl_xor(b[i], off);
      a[i] = (lane & off) ? a2 + a[i] : a[i] + a2;
      b[i] = (lane & off) ? b2 + b[i] : b[i] + b2;
    }
  }
  const int qh = qg * QP + q;
  if (ln == 0 && q < QP && qh < n_qh) {
    const float li = Linv_s[min(qc - q0, NPAIR - 1)];
    const int row = qh / group, head = kvh * group + qh % group;
    store_f16x8(p.out + act_index(d.row0 + row, head * HD + d0, p.act_rows), a * li, b * li);
  }
}

template <int HD, int NQ>
hipError_t launch_hd_nq(const AttnArgs& a, hipStream_t st) {
  if constexpr (NQ == 1)
    if (a.wide) {                    // one chunk, 8 waves: no merge kernel
      k_attn<HD, 1, 2 * kAttnWaves><<<dim3(a.n_kv, a.n_qblocks, a.n_seq), dim3(128 * kAttnWaves), 0, st>>>(a);
      return hipGetLastError();
    }
  // Chunks of more than two tiles a wavefront take k_attn_chunk (us, 8B
  // attention: 32 sequences of 256-2048 keys, 9 rows each, 1024-key chunks 40.8
  // -> 36.3, 17 rows 64.0 -> 48.0; one sequence, 16384 keys, 640-key chunks 22.3
  // -> 21.4); shorter ones, whose two tiles k_attn requests at once, do not (4000
  // keys, 256-key chunks 13.3 against 14.9).  With one query tile, where two of
  // k_attn's wavefronts fit a SIMD, there is little between them (32 sequences,
  // one row 26.3 against 26.8), and the kernel, whose sums round differently,
  // must not depend on the pass's row count.
  const dim3 grid(a.n_kv, a.n_qblocks, a.n_seq * a.n_splits);
  // Whole contexts at head_dim 64 (a workgroup per CU or fewer, whose tiles are
  // half as long) run eight wavefronts: 32 sequences of 256-2048 keys in a
  // model's step 31 -> 26 us; at head_dim 128 44 with either, and key chunks
  // are slower (16384 keys 22 -> 24).
  if (HD == 64 && a.split_len > kAttnChunk && a.n_splits == 1)
    k_attn_chunk<HD, NQ, HD == 64 ? 8 : 4><<<grid, dim3(512), 0, st>>>(a);
  else if (a.split_len > kAttnChunk) k_attn_chunk<HD, NQ, 4><<<grid, dim3(256), 0, st>>>(a);
  else k_attn<HD, NQ, kAttnWaves><<<grid, dim3(64 * kAttnWaves), 0, st>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_splits == 1) return e;
  if (a.n_splits <= kMergeFewChunks)
    k_attn_merge_few<HD, NQ><<<dim3(a.n_kv, a.n_qblocks, a.n_seq * kMergeParts), dim3(256), 0, st>>>(a);
  else
    k_attn_merge<HD, NQ><<<dim3(a.n_kv, a.n_qblocks, a.n_seq * merge_parts<HD, NQ>()), dim3(256), 0, st>>>(a);
  return hipGetLastError();
}

template <int HD>
hipError_t launch_hd(const AttnArgs& a, hipStream_t st) {
  switch (a.nqt) {
    case 1: return launch_hd_nq<HD, 1>(a, st);
    case 2: return launch_hd_nq<HD, 2>(a, st);
    case 3: return launch_hd_nq<HD, 3>(a, st);
    case 4: if constexpr (HD == 64) return launch_hd_nq<HD, 4>(a, st); break;
  }
  return hipErrorInvalidValue;
}

}  // namespace

int attn_max_q_tiles(int head_dim) { return head_dim == 128 ? 3 : 4; }

size_t attn_part_floats(int head_dim, int nqt) { return (size_t)16 * nqt * head_dim + 2 * 16 * nqt; }

hipError_t launch_attention(int head_dim, const AttnArgs& a, hipStream_t st) {
  if (a.split_len % 128 || a.split_len <= 0) return hipErrorInvalidValue;
  if (a.nqt < 1 || a.nqt > attn_max_q_tiles(head_dim)) return hipErrorInvalidValue;
  if (a.n_seq < 1 || a.n_seq > kMaxPassSeqs || (size_t)a.n_seq * a.n_splits > 65535) return hipErrorInvalidValue;
  if (a.wide && (a.n_splits != 1 || a.nqt != 1)) return hipErrorInvalidValue;
  if (head_dim == 64) return launch_hd<64>(a, st);
  if (head_dim == 128) return launch_hd<128>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace pard
