// Conditional drop-token (COD) training-data processing (Sec. 3.2 eqs. 9-11,
// Alg. 1, App. B), one workgroup per sample.
//
// A sample of L tokens has n = L - 1 columns per subtask k = 1..K.  Subtask 1
// keeps every column (the real tokens).  Column j of subtask k >= 2 (a mask
// token at position j, label t_{j+1}) may be kept only if its whole context
// is kept -- j >= k - 1 and column j - 1 of subtask k - 1 kept -- and the
// subtask keeps min(#valid, floor(n * gamma_k + 1/2)) of the valid columns,
// gamma_k = max(r^{k-1}, r_min): those with the smallest (key, j), key a
// 24-bit SplitMix64 value of (seed, sample, k, j).  The kept columns of all
// subtasks are packed in subtask order, each in column order.
//
// The kept set of a subtask is a bit mask in LDS (one 64-bit word per 64
// columns): the next subtask's valid columns are that mask shifted by one.
// The smallest (key, j) are selected, not sorted: a histogram of the keys' top
// bits finds the bin in which the keep count is reached, and only the columns
// of that bin (a few) are ranked exactly.  The kept columns then go through an
// index list in LDS, so that the five output arrays are written by full
// wavefronts at consecutive addresses.
// Only integers and the float64 keep count decide anything, so results are
// bit-exact and independent of timing.
//
// What bounds it: with few samples the chain of the subtasks (four barriers
// each), with many the keys' 64-bit multiplications and the 20 output bytes per
// kept column.  Against a bitonic sort of the keys in LDS, per call: 48
// samples of 512-6000 tokens 917 -> 49 us, 4096 of 256-1024 (186 MB) 412 -> 87
// us (2.1 TB/s).
#include "pard_internal.h"

#include <algorithm>

namespace pard {
namespace {

constexpr int kCodMaxColumns = 8192;
constexpr int kCodKeyBits = 24;

// Inclusive sum over the wavefront's lanes: DPP row shifts inside each row of
// 16, then the rows' last lanes broadcast to the rows after them (a shuffle
// through LDS takes several times as long per step).
__device__ __forceinline__ int wave_incl_scan_int(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// NW wavefronts per sample.  Every wavefront scans the whole histogram by
// itself, so no barrier separates the scan from its result.
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_cod(const int32_t* __restrict__ tokens, const int64_t* tok_off,
                                                  const int64_t* out_off, CodArgs a, int p_max) {
  constexpr int T = 64 * NW;
  constexpr int kBinBits = NW == 1 ? 8 : NW == 2 ? 9 : 10;
  constexpr int kBins = 1 << kBinBits, kLaneBins = kBins / 64;
  constexpr int kShift = kCodKeyBits - kBinBits;     // key -> bin
  constexpr int kMaxWords = kCodMaxColumns / 64;
  static_assert(kMaxWords <= 128, "two mask words per lane in the position scan");
  // dynamic LDS (p_max: a multiple of 64): two column masks (the previous and
  // the current subtask's kept columns), the columns' keys, a column list
  extern __shared__ uint64_t mask_s[];
  uint32_t* key_s = reinterpret_cast<uint32_t*>(mask_s + 2 * (p_max / 64));
  uint16_t* list_s = reinterpret_cast<uint16_t*>(key_s + p_max);
  __shared__ __attribute__((aligned(16))) int hist_s[kBins];
  __shared__ int count_s;
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t t0 = tok_off[s];
  const int n = (int)(tok_off[s + 1] - t0) - 1;     // columns; the host checked 1 <= n <= kCodMaxColumns
  const int32_t* t = tokens + t0;
  const int64_t o0 = out_off[s];
  const int words = (n + 63) / 64;
  const uint64_t last_word = (n & 63) ? (1ull << (n & 63)) - 1 : ~0ull;
  uint64_t* prev = mask_s;
  uint64_t* cur = mask_s + p_max / 64;

  // Packed entries [at, at + count): the columns j_of(i), i < count, of subtask
  // k; each thread has four labels' loads in flight.
  auto pack = [&](int64_t at, int count, int k, auto j_of) {
    for (int i0 = tid; i0 < count; i0 += 4 * T) {
      int j[4], id[4], label[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        j[u] = j_of(min(i0 + u * T, count - 1));
        label[u] = t[j[u] + 1];
        id[u] = k == 1 ? t[j[u]] : a.mask_id;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * T;
        if (i < count) {
          a.ids[at + i] = id[u];
          a.labels[at + i] = label[u];
          a.pos[at + i] = j[u];
          a.section[at + i] = k;
          a.column[at + i] = j[u];
        }
      }
    }
  };

  pack(o0, n, 1, [](int i) { return i; });          // subtask 1: every real token
  for (int w = tid; w < words; w += T) prev[w] = w == words - 1 ? last_word : ~0ull;
  auto clear = [&]() {
    for (int b = tid; b < kBins / 4; b += T) reinterpret_cast<int4*>(hist_s)[b] = int4{0, 0, 0, 0};
    if (tid == 0) count_s = 0;
  };
  clear();
  __syncthreads();
  int written = n, kept = n;                        // packed columns; columns the last subtask kept
  const uint64_t z_sample = mix64(a.seed + ((uint64_t)s + 1) * kGamma);
  double gamma = 1.0;
  for (int k = 2; k <= a.k_max; ++k) {
    gamma *= a.r;
    const int target = (int)floor((double)n * fmax(gamma, a.r_min) + 0.5);
    const uint64_t z_k = mix64(z_sample + ((uint64_t)k + 1) * kGamma);
    // valid columns: the previous mask one column on (its bit j - 1 implies
    // j >= k - 1); the successor of the last column falls off the end
    const int n_valid = kept - (int)((prev[(n - 1) >> 6] >> ((n - 1) & 63)) & 1);
    const int keep = min(n_valid, target);
    if (keep <= 0) break;                            // uniform: nothing kept here, nor after
    auto valid_word = [&](int w) {
      const uint64_t v = (prev[w] << 1) | (w > 0 ? prev[w - 1] >> 63 : 0);
      return w == words - 1 ? v & last_word : v;
    };
    const bool select = keep < n_valid;              // uniform
    uint32_t key_max = 0;                            // the last kept (key, column)
    int col_max = 0;
    if (select) {
      for (int w = wave; w < words; w += NW) {
        const int j = w * 64 + lane;
        if ((valid_word(w) >> lane) & 1) {
          const uint32_t key = (uint32_t)(mix64(z_k + ((uint64_t)j + 1) * kGamma) >> 40);
          key_s[j] = key;
          atomicAdd(&hist_s[key >> kShift], 1);
        }
      }
      __syncthreads();
      // the bin in which the running count reaches `keep`: the lane that
      // crosses it, then the bin among the lane's
      int h[kLaneBins], sum = 0;
#pragma unroll
      for (int q = 0; q < kLaneBins / 4; ++q) {
        const int4 v = reinterpret_cast<const int4*>(hist_s)[lane * (kLaneBins / 4) + q];
        h[4 * q] = v.x;
        h[4 * q + 1] = v.y;
        h[4 * q + 2] = v.z;
        h[4 * q + 3] = v.w;
        sum += v.x + v.y + v.z + v.w;
      }
      const int incl = wave_incl_scan_int(sum);
      const uint64_t crossed = __ballot(incl >= keep);     // not empty: the total is n_valid
      const int owner = __ffsll((unsigned long long)crossed) - 1;
      int before = incl - sum, b = 0, in_bin = 0;
      bool done = false;
#pragma unroll
      for (int q = 0; q < kLaneBins; ++q) {
        done = done || before + h[q] >= keep;
        if (!done) {
          before += h[q];
          b = q + 1;
        }
      }
#pragma unroll
      for (int q = 0; q < kLaneBins; ++q) in_bin = b == q ? h[q] : in_bin;
      const int bin = __builtin_amdgcn_readlane(lane * kLaneBins + b, owner);
      const int limit = __builtin_amdgcn_readlane(keep - before, owner);   // columns the bin contributes (>= 1)
      in_bin = __builtin_amdgcn_readlane(in_bin, owner);
      if (limit == in_bin) {                         // uniform: the whole bin
        key_max = ((uint32_t)(bin + 1) << kShift) - 1;
        col_max = kCodMaxColumns;
      } else {
        // the bin's columns, in whatever order: the kept set ends with the one
        // that limit - 1 of them precede
        for (int w = wave; w < words; w += NW) {
          const int j = w * 64 + lane;
          if (((valid_word(w) >> lane) & 1) && (int)(key_s[j] >> kShift) == bin)
            list_s[atomicAdd(&count_s, 1)] = (uint16_t)j;
        }
        __syncthreads();
        for (int i0 = 0; i0 < in_bin; i0 += 64) {
          const int j = list_s[min(i0 + lane, in_bin - 1)];
          const uint32_t key = key_s[j];
          int rank = i0 + lane < in_bin ? 0 : kCodMaxColumns;
          for (int b0 = 0; b0 < in_bin; b0 += 64) {
            const int jo = list_s[min(b0 + lane, in_bin - 1)];
            const int ko = (int)key_s[jo];
            for (int q = 0; q < min(64, in_bin - b0); ++q) {
              const uint32_t kq = (uint32_t)__builtin_amdgcn_readlane(ko, q);
              const int jq = __builtin_amdgcn_readlane(jo, q);
              rank += kq < key || (kq == key && jq < j);
            }
          }
          const uint64_t hit = __ballot(rank == limit - 1);
          if (hit) {
            const int l = __ffsll((unsigned long long)hit) - 1;
            key_max = (uint32_t)__builtin_amdgcn_readlane((int)key, l);
            col_max = __builtin_amdgcn_readlane(j, l);
            break;
          }
        }
      }
    }
    for (int w = wave; w < words; w += NW) {
      uint64_t m = valid_word(w);
      if (select) {                                  // uniform
        const int j = w * 64 + lane;
        bool in = false;
        if ((m >> lane) & 1) {
          const uint32_t key = key_s[j];
          in = key < key_max || (key == key_max && j <= col_max);
        }
        m = __ballot(in);
      }
      if (lane == 0) cur[w] = m;
    }
    __syncthreads();
    // column list in column order: each wavefront scans the words' counts
    // (two words per lane) and lists its own words' columns
    {
      const int c0 = 2 * lane < words ? __popcll(cur[2 * lane]) : 0;
      const int c1 = 2 * lane + 1 < words ? __popcll(cur[2 * lane + 1]) : 0;
      const int base = wave_incl_scan_int(c0 + c1) - (c0 + c1);
      clear();                                       // (everyone is past this subtask's histogram)
      for (int w = wave; w < words; w += NW) {
        const int at = __builtin_amdgcn_readlane(base, w >> 1) + ((w & 1) ? __builtin_amdgcn_readlane(c0, w >> 1) : 0);
        const uint64_t m = cur[w];
        if ((m >> lane) & 1) list_s[at + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)(w * 64 + lane);
      }
    }
    __syncthreads();
    pack(o0 + written, keep, k, [&](int i) { return (int)list_s[i]; });
    written += keep;
    kept = keep;
    uint64_t* const swap = prev;
    prev = cur;
    cur = swap;
  }
  if (tid == 0) a.out_len[s] = written;
}

template <int NW>
hipError_t launch_cod_nw(const int32_t* tokens, const int64_t* tok_off, const int64_t* out_off, int n_samples,
                         int p_max, const CodArgs& a, hipStream_t st) {
  const size_t lds = (size_t)p_max * (2.0 / 8 + 4 + 2);
  k_cod<NW><<<n_samples, 64 * NW, lds, st>>>(tokens, tok_off, out_off, a, p_max);
  return hipGetLastError();
}

}  // namespace

int cod_max_columns() { return kCodMaxColumns; }

hipError_t launch_cod(const int32_t* tokens, const int64_t* tok_off, const int64_t* out_off, int n_samples,
                      int max_columns, const CodArgs& a, hipStream_t st) {
  if (n_samples < 1 || a.k_max < 1 || max_columns < 1 || max_columns > kCodMaxColumns) return hipErrorInvalidValue;
  const int p_max = (max_columns + 63) / 64 * 64;
  // Wavefronts per sample: about 4096 in all (four per SIMD), and at least one
  // per 512 columns up to 8 (long samples' LDS lets few workgroups share a
  // CU).  Measured, us per call at 1 / 2 / 4 / 8 / 16 wavefronts: 48 samples
  // of 512-6000 tokens 362 / 195 / 104 / 64 / 49; 256 of 256-1024 73 / 44 /
  // 31 / 25 / 25; 1024 of 256-1024 78 / 50 / 39 / 49 / 79; 4096 of 256-1024
  // 101 / 87 / 93 / 131 / 279; 16384 of 20-200 73 / 95 / 168 / 326 / 891;
  // 2000 of 4000-8193 1486 / 822 / 596 / 403 / 470.
  int nw = 1;
  while (nw < 16 && nw < std::max(4096 / n_samples, std::min(8, (p_max + 511) / 512))) nw *= 2;
  switch (nw) {
    case 1: return launch_cod_nw<1>(tokens, tok_off, out_off, n_samples, p_max, a, st);
    case 2: return launch_cod_nw<2>(tokens, tok_off, out_off, n_samples, p_max, a, st);
    case 4: return launch_cod_nw<4>(tokens, tok_off, out_off, n_samples, p_max, a, st);
    case 8: return launch_cod_nw<8>(tokens, tok_off, out_off, n_samples, p_max, a, st);
  }
  return launch_cod_nw<16>(tokens, tok_off, out_off, n_samples, p_max, a, st);
}

}  // namespace pard
