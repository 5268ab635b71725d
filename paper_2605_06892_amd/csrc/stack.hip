// Kernels of the multi-layer sampling loop that are not matrix products.
//
//   * gather_latent: the fp32 latent rows of the active tokens, converted to
//     the model dtype, as the compact input of the patch embedding (Section
//     2.3: only the active rows flow through the model).
//   * velocity_keys + rank_budgets / select_budgets: the group refresh. Group sizes are fixed
//     and membership follows a per-token velocity ranking (Section 2.2,
//     Appendix B): the key of a token is the squared L2 norm of its velocity,
//     a float64 sum of the exact squares in channel order, and its rank is
//     its position in ascending (key, token) order, keys compared as their
//     IEEE bit patterns (a total order on non-negative doubles; NaN keys are
//     made the canonical positive NaN, above every number). The n_1 lowest
//     ranks get budget s_1, the next n_2 get s_2, and so on.
//
//   * l1_rel_accumulate: strategy D (Appendix B, Eq. 7): per token, the sum
//     over the initial full-budget steps of |v_i - v_{i-1}|_1 / |v_i|_1, the
//     two L1 norms summed in float64 in channel order, one float64 division
//     per step; v_{i-1} is kept in a token-major copy.
//   * reorder_plan_kernel + permute_rows_kernel: token reordering (Section
//     2.5): non-baseline tokens first, then the baseline group, each part in
//     index order, and the row permutation that applies it to token-indexed
//     state (and inverts it at the end).
//   * row_rms_scale: 1 / sqrt(mean(h^2) + eps) of every compact hidden row, the
//     RMS normalization before each layer's Q/K/V projections and before the
//     velocity head. A per-row factor commutes with the projection, so the
//     normalized rows are never written: the GEMM epilogue scales its rows.
//
// All of them are small (N x C fp32 reads, N budgets, one read of the hidden
// state): one pass each, grid-stride loops; the ranking needs only the group
// boundaries, which one workgroup finds by histogram.
#include "common.h"

namespace hsa {
namespace {

constexpr int kThreads = 256;

int grid_for(long work) {
  long g = (work + kThreads - 1) / kThreads;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return (int)g;
}

// Each thread keeps kGatherU independent 16-byte row loads in flight before
// its stores; the latent rows are streamed once (nontemporal loads).
constexpr int kGatherU = 4;

template <bool BF16>
__global__ __launch_bounds__(kThreads) void gather_latent_vec(const f32x4* __restrict__ x,
                                                              const int32_t* __restrict__ idx,
                                                              int n_active, long n_tokens, int vpr,
                                                              void* __restrict__ xa) {
  const long total = (long)n_active * vpr;
  for (long e0 = blockIdx.x * (long)(kThreads * kGatherU) + threadIdx.x; e0 < total;
       e0 += (long)gridDim.x * kThreads * kGatherU) {
    f32x4 v[kGatherU];
#pragma unroll
    for (int u = 0; u < kGatherU; ++u) {
      const long e = e0 + (long)u * kThreads;
      v[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
      if (e < total) {
        const long j = e / vpr;
        const int c = (int)(e - j * vpr);
        const int t = idx[j];
        if (t >= 0 && t < n_tokens) v[u] = __builtin_nontemporal_load(x + (long)t * vpr + c);
      }
    }
#pragma unroll
    for (int u = 0; u < kGatherU; ++u) {
      const long e = e0 + (long)u * kThreads;
      if (e >= total) break;
      if constexpr (BF16)
        static_cast<bf16x4*>(xa)[e] = to_bf16x4(v[u]);
      else
        static_cast<f32x4*>(xa)[e] = v[u];
    }
  }
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void gather_latent_scalar(const float* __restrict__ x,
                                                                 const int32_t* __restrict__ idx,
                                                                 int n_active, long n_tokens,
                                                                 int channels,
                                                                 void* __restrict__ xa) {
  const long total = (long)n_active * channels;
  for (long e = blockIdx.x * (long)kThreads + threadIdx.x; e < total;
       e += (long)gridDim.x * kThreads) {
    const long j = e / channels;
    const int c = (int)(e - j * channels);
    const int t = idx[j];
    const float v = (t >= 0 && t < n_tokens) ? x[(long)t * channels + c] : 0.f;
    if constexpr (BF16)
      static_cast<bf16*>(xa)[e] = (bf16)v;
    else
      static_cast<float*>(xa)[e] = v;
  }
}

__device__ __forceinline__ double canonical_key(double acc) {
  return acc != acc ? __longlong_as_double(0x7FF8000000000000LL) : acc;
}

// bit pattern of a key, NaNs made the canonical positive NaN
__device__ __forceinline__ unsigned long long key_bits(unsigned long long k) {
  const unsigned long long e = 0x7FF0000000000000ull;
  return ((k & e) == e && (k & 0x000FFFFFFFFFFFFFull)) ? 0x7FF8000000000000ull : k;
}

// Strategy D accumulation, 16-byte rows. HBM-bound (12 bytes per value): one
// wave takes 32 tokens, whose rows are read (and v copied to v_prev) with
// coalesced 16-byte accesses, up to 64 channels at a time, and staged in LDS;
// then one lane per token and sum adds them in channel order, lanes 0-31 the
// numerators and 32-63 the denominators. At 17 KB of LDS nine such workgroups
// fit a CU, 73728 tokens on all, if three waves' registers fit a SIMD: unbounded, the
// compiler takes 254 (64 tokens on two waves that way: 22.9 us).
// One thread walking each row in global memory took 132 us at 75600 x 64, this
// takes 14.5 us (4.0 TB/s).
constexpr int kL1Tokens = 32, kL1Quads = 16;

__global__ __launch_bounds__(kWave, 3) void l1_rel_accumulate_vec(const f32x4* __restrict__ v,
                                                               f32x4* __restrict__ v_prev, long n,
                                                               int vpr, double* __restrict__ acc,
                                                               int first) {
  constexpr int LOADS = kL1Tokens * kL1Quads / kWave;
  __shared__ f32x4 a[kL1Tokens][kL1Quads + 1], b[kL1Tokens][kL1Quads + 1];
  const int lane = threadIdx.x, tok = lane % kL1Tokens;
  const long t0 = (long)blockIdx.x * kL1Tokens;
  const int rows = (int)min((long)kL1Tokens, n - t0);
  double sum = 0.0;  // lanes 0-31: |v - v_prev|_1 of token t0 + tok; 32-63: |v|_1
  for (int q0 = 0; q0 < vpr; q0 += kL1Quads) {
    const int w = min(kL1Quads, vpr - q0);
    f32x4 va[LOADS], vb[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int f = lane + i * kWave, r = f / w, q = f - r * w;
      if (r < rows) {
        const long e = (t0 + r) * vpr + q0 + q;
        va[i] = v[e];
        if (!first) vb[i] = v_prev[e];
      }
    }
    __syncthreads();  // the previous channels are no longer read
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int f = lane + i * kWave, r = f / w, q = f - r * w;
      if (r < rows) {
        v_prev[(t0 + r) * vpr + q0 + q] = va[i];
        if (!first) {
          a[r][q] = va[i];
          b[r][q] = vb[i];
        }
      }
    }
    __syncthreads();
    if (!first && tok < rows) {
      for (int q = 0; q < w; ++q) {
        const f32x4 x = a[tok][q];
        const f32x4 y = lane < kL1Tokens ? b[tok][q] : (f32x4){};
#pragma unroll
        for (int u = 0; u < 4; ++u) sum = sum + fabs((double)x[u] - (double)y[u]);
      }
    }
  }
  const double den = __shfl(sum, kL1Tokens + tok);
  if (lane < rows) acc[t0 + lane] = first ? 0.0 : acc[t0 + lane] + sum / den;
}

__global__ __launch_bounds__(kThreads) void l1_rel_accumulate(const float* __restrict__ v,
                                                              float* __restrict__ v_prev, long n,
                                                              int channels, double* __restrict__ acc,
                                                              int first) {
  for (long t = blockIdx.x * (long)kThreads + threadIdx.x; t < n; t += (long)gridDim.x * kThreads) {
    const float* row = v + t * channels;
    float* prev = v_prev + t * channels;
    if (first) {
      acc[t] = 0.0;
    } else {
      double num = 0.0, den = 0.0;
      for (int c = 0; c < channels; ++c) {
        const double a = row[c], b = prev[c];
        num = num + fabs(a - b);
        den = den + fabs(a);
      }
      acc[t] = acc[t] + num / den;
    }
    for (int c = 0; c < channels; ++c) prev[c] = row[c];
  }
}

// one thread per token; channel order is the summation order
__global__ __launch_bounds__(kThreads) void velocity_keys_vec(const f32x4* __restrict__ v, long n,
                                                              int vpr, double* __restrict__ keys) {
  for (long t = blockIdx.x * (long)kThreads + threadIdx.x; t < n; t += (long)gridDim.x * kThreads) {
    const f32x4* row = v + t * vpr;
    double acc = 0.0;
    for (int c = 0; c < vpr; ++c) {
      const f32x4 e = row[c];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double w = e[u];
        acc = acc + w * w;  // w * w is exact in float64
      }
    }
    keys[t] = canonical_key(acc);
  }
}

__global__ __launch_bounds__(kThreads) void velocity_keys_scalar(const float* __restrict__ v,
                                                                 long n, int channels,
                                                                 double* __restrict__ keys) {
  for (long t = blockIdx.x * (long)kThreads + threadIdx.x; t < n; t += (long)gridDim.x * kThreads) {
    const float* row = v + t * channels;
    double acc = 0.0;
    for (int c = 0; c < channels; ++c) {
      const double w = row[c];
      acc = acc + w * w;
    }
    keys[t] = canonical_key(acc);
  }
}

// Group assignment by selection. A token's group is the number of group
// boundaries (ranks end[0], end[1], ...) at or below its rank, so only the
// neighbourhoods of the at most 15 boundaries need ranks. One workgroup:
//   1. minimum and maximum key;
//   2. a histogram of the keys over kSelBins equal ranges of bit patterns from
//      minimum to maximum (LDS atomics), scanned: a bin with no boundary inside
//      has one group, whose budget replaces its count;
//   3. every token reads its bin's budget; the keys of the bins with a boundary
//      inside, a few dozen, are collected and ranked by comparing all pairs.
// Bins too full for that (an outlier that widens the range, or many equal
// keys) are divided again, all at once, first by key, from the least to the greatest
// one holds, then, among equal keys, by token index, around their boundaries
// until every boundary's element (key, token) is found; their keys are then compared
// with those elements. (One boundary after the other, 16 groups of keys of 16 values
// took 168 us at 5121 keys and 503 at 32760, where all pairs take 45 and 295; at once
// 38 and 171.)
// Steps 1 and 2 and the lookup of 3 use the upper halves of the keys (sign,
// exponent and 20 mantissa bits), which stay in registers for up to 81920
// tokens; whole keys are read again for the collected ones only. The bound is
// one CU's loads, LDS atomics and instruction fetches. Spreading the steps over
// CUs would take two or more further launches, at 3 us each.
// Comparing all pairs of keys on the whole chip took 297 us at 32760 tokens and
// 1110 us at 75600, this takes 16 and 31 us (keys without structure, 4 groups), 88 and
// 207 with all keys equal. It is slower than all pairs in one corner: 16 groups, and an
// outlier that puts all other keys, of a few values, into one bin (50 against 45 us at
// 5121 keys, 79 against 70 at 8193, 126 against 139 at 16384).
constexpr int kSelThreads = 1024, kSelBinBits = 13, kSelBins = 1 << kSelBinBits;
constexpr int kSelList = 1024;     // collected keys
constexpr int kSelBig = -64;       // histogram code of a bin too full for the list

// Few keys: all pairs, 16 tokens a workgroup, so 4096 keys give every CU one.
// All keys are in LDS and 64 slices of them count for each token, which takes
// 5.6 us a call at 1000 keys, 6.3 at 4096 and 10.2 at 5000 whatever the keys are
// (10.6, 35.5 and 43.8 with 64 tokens on four waves). select_budgets takes 8 to 10 us
// at 5121 keys without structure, but 22 to 50 if many are equal: the line lies where
// all pairs stop being about as fast as the former.
constexpr int kRankTokens = 16, kRankMax = 5120;
__global__ __launch_bounds__(kSelThreads) void rank_budgets(const unsigned long long* __restrict__ keys, int n,
                                                            GroupTable tab, int32_t* __restrict__ budget) {
  constexpr int kSlices = kSelThreads / kRankTokens;
  __shared__ unsigned long long key[kRankMax];
  __shared__ int partial[kSlices][kRankTokens];
  const int tid = threadIdx.x, tok = tid % kRankTokens, slice = tid / kRankTokens;
  const int t = blockIdx.x * kRankTokens + tok;
#pragma unroll
  for (int i = 0; i < kRankMax / kSelThreads; ++i) {
    const int e = tid + i * kSelThreads;
    if (e < n) key[e] = key_bits(keys[e]);
  }
  __syncthreads();
  const unsigned long long kt = key[min(t, n - 1)];
  int count = 0;
#pragma unroll 8
  for (int e = slice; e < n; e += kSlices) {
    const unsigned long long km = key[e];
    count += (km < kt) | ((km == kt) & (e < t));
  }
  partial[slice][tok] = count;
  __syncthreads();
  if (tid >= kWave) return;
  int r = 0;  // of the lanes' 16 slices, then of all four lanes of a token
#pragma unroll
  for (int w = 0; w < kSlices; w += kWave / kRankTokens) r += partial[w + slice][tok];
  r += __shfl_xor(r, 16);
  r += __shfl_xor(r, 32);
  if (slice > 0 || t >= n) return;
  int g = 0;
  while (g + 1 < tab.n && r >= tab.end[g]) ++g;
  budget[t] = tab.budget[g];
}

// KEYS: upper halves per thread in registers (0: read by each step)
template <int KEYS>
__global__ __launch_bounds__(kSelThreads) void select_budgets(const unsigned long long* __restrict__ keys,
                                                              int n, GroupTable tab,
                                                              int32_t* __restrict__ budget) {
  typedef unsigned long long u64;
  constexpr int kWaves = kSelThreads / kWave, kPer = kSelBins / kSelThreads;
  constexpr unsigned kNone = 0xFFFFFFFFu;  // no token: above every key's upper half
  // and a bin for no token in every lane: where the last rows of kSelThreads tokens are
  // empty, one bin would take all their atomics (35 us at 8193 keys, 15 with these)
  __shared__ __attribute__((aligned(16))) int hist[kSelBins + kWave];
  __shared__ u64 list_key[kSelList];
  __shared__ int list_tok[kSelList];
  __shared__ unsigned red_lo[kWaves], red_hi[kWaves];
  __shared__ int wave_total[kWaves];
  __shared__ int end_at[kMaxGroups], budget_of[kMaxGroups];
  __shared__ int bin_of[kMaxGroups], before_of[kMaxGroups], count_of[kMaxGroups], slot_of[kMaxGroups];
  __shared__ int slot_off[kMaxGroups + 1], slot_fill[kMaxGroups], slot_before[kMaxGroups], n_slots, n_big;
  __shared__ int bnd_group[kMaxGroups], bnd_range[kMaxGroups], n_bnd;
  __shared__ int sub_bin[kMaxGroups], sub_before[kMaxGroups], sub_count[kMaxGroups];
  __shared__ u64 key0[kMaxGroups + 1], key1[kMaxGroups], range_min[kMaxGroups], range_max[kMaxGroups], thr_key[kMaxGroups];
  __shared__ int key_bits_of[kMaxGroups], tok0[kMaxGroups + 1], tok_bits_of[kMaxGroups], thr_tok[kMaxGroups];
  __shared__ int range_first[kMaxGroups], range_before[kMaxGroups], range_count[kMaxGroups], range_off[kMaxGroups + 1];
  __shared__ int n_ranges, n_full, any_key;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int nb = tab.n - 1;  // boundaries
  // The most keys of one bin that are ranked. Dividing the bins takes four more
  // passes over all keys at least, 14 us at 5121 and 70 at 32760.
  const int cap = min(kSelList, max(256, n / 100));

  // upper half of the key of token t as it is stored, and of its key_bits
  auto load = [&](long t) -> unsigned { return reinterpret_cast<const unsigned*>(keys)[2 * min(t, (long)n - 1) + 1]; };
  auto top_bits = [&](unsigned hi, long t) -> unsigned {
    hi = t < n ? hi : kNone;
    if ((hi & 0x7FF00000u) == 0x7FF00000u && t < n)  // infinite or NaN
      return (unsigned)(key_bits(keys[t]) >> 32);
    return hi;
  };
  unsigned top[KEYS > 0 ? KEYS : 1];
  if constexpr (KEYS > 0) {
    // buffer loads, each through a resource over the keys from its row of
    // kSelThreads on: the address steps are scalar, and past the last token a load
    // returns 0, which top_bits replaces. (The range check covers the lane's offset
    // alone; a step in the scalar offset would pass it.)
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
      const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<u64*>(keys + i * kSelThreads), 0,
                                                        max(n - i * kSelThreads, 0) * 8, 0x00020000);
      top[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, tid * 8 + 4, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < KEYS; ++i) top[i] = top_bits(top[i], i * kSelThreads + tid);
  }
  // f(upper half, token) for every key of this thread
  auto each = [&](auto&& f) __attribute__((always_inline)) {
    if constexpr (KEYS > 0) {
#pragma unroll
      for (int i = 0; i < KEYS; ++i) f(top[i], (long)i * kSelThreads + tid);
    } else {
      constexpr int V = 16;
#pragma unroll 1
      for (long t0 = tid; t0 < n; t0 += (long)V * kSelThreads) {
        unsigned k[V];
#pragma unroll
        for (int i = 0; i < V; ++i) k[i] = load(t0 + (long)i * kSelThreads);
#pragma unroll
        for (int i = 0; i < V; ++i) f(top_bits(k[i], t0 + (long)i * kSelThreads), t0 + (long)i * kSelThreads);
      }
    }
  };
  // f(key bits, token), for the steps that only the division of full bins takes:
  // keys read again, or from hold_keys on held if a thread has few
  constexpr int V = 8;
  u64 held[KEYS == V ? V : 1];
  auto hold_keys = [&]() {
    if constexpr (KEYS == V) {
#pragma unroll
      for (int i = 0; i < V; ++i) held[i] = keys[min(tid + i * kSelThreads, n - 1)];
#pragma unroll
      for (int i = 0; i < V; ++i) held[i] = key_bits(held[i]);
    }
  };
  auto each_again = [&](auto&& f) __attribute__((always_inline)) {
    if constexpr (KEYS == V) {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (tid + i * kSelThreads < n) f(held[i], tid + i * kSelThreads);
    } else {
#pragma unroll 1
      for (long t0 = tid; t0 < n; t0 += (long)V * kSelThreads) {
        u64 k[V];
#pragma unroll
        for (int i = 0; i < V; ++i) k[i] = keys[min(t0 + (long)i * kSelThreads, (long)n - 1)];
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (t0 + (long)i * kSelThreads < n) f(key_bits(k[i]), (int)(t0 + (long)i * kSelThreads));
      }
    }
  };
  auto clear_hist = [&]() {
#pragma unroll
    for (int i = 0; i < kPer; ++i) hist[i * kSelThreads + tid] = 0;
    __syncthreads();
  };
  // Counts of this thread's kPer bins, and the keys before the first of them.
  auto scan_bins = [&](int (&c)[kPer]) -> int {
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      c[i] = hist[tid * kPer + i];
      sum += c[i];
    }
    int inc = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) wave_total[wave] = inc;
    __syncthreads();
    int p = inc - sum;
    for (int w = 0; w < wave; ++w) p += wave_total[w];
    return p;
  };
  // rank of list element i within the list elements a .. b-1
  auto rank_in = [&](int i, int a, int b) -> int {
    const u64 k = list_key[i];
    const int t = list_tok[i];
    int r = 0;
#pragma unroll 8
    for (int j = a; j < b; ++j) r += (list_key[j] < k) | ((list_key[j] == k) & (list_tok[j] < t));
    return r;
  };

  if (tid < kMaxGroups) {
    end_at[tid] = tid < nb ? (int)tab.end[tid] : 0;
    budget_of[tid] = tid <= nb ? tab.budget[tid] : 0;
    bin_of[tid] = -1;  // no bin has this boundary inside
    slot_fill[tid] = 0;
  }
  unsigned lo32 = kNone, hi32 = 0;  // hi32: one above the maximum
  each([&](unsigned k, long) {
    lo32 = min(lo32, k);
    hi32 = max(hi32, k + 1);
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo32 = min(lo32, (unsigned)__shfl_xor((int)lo32, o));
    hi32 = max(hi32, (unsigned)__shfl_xor((int)hi32, o));
  }
  if (lane == 0) {
    red_lo[wave] = lo32;
    red_hi[wave] = hi32;
  }
  clear_hist();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    lo32 = min(lo32, red_lo[w]);
    hi32 = max(hi32, red_hi[w]);
  }
  const int bits = hi32 - 1 > lo32 ? 32 - __clz(hi32 - 1 - lo32) : 0;
  const int shift32 = bits > kSelBinBits ? bits - kSelBinBits : 0;
  const u64 lo = (u64)lo32 << 32;  // the bins in whole keys
  const int shift = shift32 + 32;
  auto bin32 = [&](unsigned k) { return k == kNone ? (unsigned)(kSelBins + lane) : (k - lo32) >> shift32; };
  // the held keys become their bins: found once, and no lane mask of k == kNone per key stays live
  if constexpr (KEYS > 0) {
#pragma unroll
    for (int i = 0; i < KEYS; ++i) top[i] = bin32(top[i]);
  }
  auto bin_at = [&](unsigned k) { return KEYS > 0 ? k : bin32(k); };
  if (bits > 0) {
    each([&](unsigned k, long) { atomicAdd(&hist[bin_at(k)], 1); });
  } else if (tid == 0) {
    hist[0] = n;  // one bin, without an atomic per key on one address
  }

  {
    int c[kPer];
    int p = scan_bins(c), sum = 0, g0 = 0, g1 = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum += c[i];
    for (int g = 0; g < nb; ++g) {  // ascending: g0 at or below p, g1 below the end of this thread's bins
      const int e = end_at[g];
      g0 += e <= p;
      g1 += e <= p || e - p < sum;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) hist[tid * kPer + i] = budget_of[g0];
    if (g0 < g1) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        while (g0 < g1 && end_at[g0] <= p) ++g0;
        hist[tid * kPer + i] = budget_of[g0];
        for (int g = g0; g < g1 && end_at[g] - p < c[i]; ++g) {  // inside: keys of this bin on both sides
          bin_of[g] = tid * kPer + i;
          before_of[g] = p;
          count_of[g] = c[i];
        }
        p += c[i];
      }
    }
  }
  __syncthreads();
  if (tid < kWave) hist[kSelBins + tid] = kSelBig;  // no token: nothing to write
  if (tid == 0) {  // a slot of the list for every bin with a boundary inside
    int slots = 0, fill = 0, last = -1, big = 0;
    for (int g = 0; g < nb; ++g) {  // ascending ranks: equal bins are adjacent
      slot_of[g] = -1;
      if (bin_of[g] < 0) continue;
      if (last >= 0 && bin_of[last] == bin_of[g]) {
        slot_of[g] = slot_of[last];
      } else if (count_of[g] <= min(cap, kSelList - fill)) {
        slot_off[slots] = fill;
        slot_before[slots] = before_of[g];
        fill += count_of[g];
        hist[bin_of[g]] = -1 - slots;
        slot_of[g] = slots++;
      } else {
        hist[bin_of[g]] = kSelBig;
        big = 1;
      }
      last = g;
    }
    slot_off[slots] = fill;
    n_slots = slots;
    n_big = big;
  }
  __syncthreads();
  each([&](unsigned k, long t) {
    const int code = hist[bin_at(k)];
    if (code >= 0) {
      budget[t] = code;
    } else if (code != kSelBig) {
      const int at = slot_off[-1 - code] + atomicAdd(&slot_fill[-1 - code], 1);
      list_tok[at] = (int)t;
    }
  });
  __syncthreads();
  const int listed = slot_off[n_slots];
  for (int i = tid; i < listed; i += kSelThreads) list_key[i] = key_bits(keys[list_tok[i]]);
  __syncthreads();
  for (int i = tid; i < listed; i += kSelThreads) {
    int s = 0;
    while (i >= slot_off[s + 1]) ++s;
    const int r = slot_before[s] + rank_in(i, slot_off[s], slot_off[s + 1]);
    int group = 0;
    for (int g = 0; g < nb; ++g) group += end_at[g] <= r;
    budget[list_tok[i]] = budget_of[group];
  }
  if (!n_big) return;

  hold_keys();
  // The bins that did not fit. Their boundaries, j = 0 .. n_bnd-1 in order, and the
  // ranges these lie in, s = 0 .. n_ranges-1 in order: at first the bins, each keys
  // key0 .. key1 (less than 2^key_bits of them) of every token; among equal keys
  // (key_bits 0) tokens tok0 .. tok0 + 2^tok_bits - 1. Each round divides all ranges at
  // once.
  // Lane j of wave 0 keeps boundary j: new ranges from their boundaries' (id, equal for
  // boundaries of one range) and, for the first boundary of each, what it is.
  auto set_ranges = [&](bool bnd, int id, u64 k0, u64 k1, int kb, int t0, int tb, int before, int count) {
    const int prev = __shfl_up(bnd ? id : -1, 1);
    const bool lead = bnd && (lane == 0 || prev != id);
    const u64 leads = __ballot(lead);
    const int s = __popcll(leads & (2ull << lane) - 1) - 1, ranges = __popcll(leads);
    if (bnd) bnd_range[lane] = s;
    if (lane >= ranges && lane <= kMaxGroups) key0[lane] = ~0ull;  // above every key
    if (lead) {
      key0[s] = k0;
      key1[s] = k1;
      key_bits_of[s] = kb;
      tok0[s] = t0;
      tok_bits_of[s] = tb;
      range_first[s] = lane;
      range_before[s] = before;
      range_count[s] = count;
      range_min[s] = ~0ull;
      range_max[s] = 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const int c = lane < ranges ? range_count[lane] : 0;
    int inc = c;
#pragma unroll
    for (int o = 1; o < kMaxGroups; o <<= 1) {
      const int y = __shfl_up(inc, o);
      if (lane >= o) inc += y;
    }
    if (lane <= ranges) range_off[lane] = inc - c;
    const bool full = __any(c > kSelList / kMaxGroups), by_key = __any(lane < ranges && key_bits_of[lane] > 0);
    if (lane == 0) {
      n_ranges = ranges;
      n_full = full;
      any_key = by_key;
    }
  };
  if (wave == 0) {
    const bool big = lane < nb && bin_of[lane] >= 0 && slot_of[lane] < 0;
    const u64 bigs = __ballot(big);
    if (lane < kMaxGroups) thr_key[lane] = ~0ull;  // past n_bnd: above every key
    if (big) bnd_group[__popcll(bigs & (1ull << lane) - 1)] = lane;
    if (lane == 0) n_bnd = __popcll(bigs);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const bool bnd = lane < __popcll(bigs);
    const int g = bnd ? bnd_group[lane] : 0, bin = bin_of[g];
    const u64 k0 = lo + ((u64)bin << shift);
    set_ranges(bnd, bin, k0, k0 + ((1ull << shift) - 1), shift, 0, 32 - __clz(n), before_of[g], count_of[g]);
  }
  __syncthreads();
  // number of the pairs (k[i], t[i]) at or below (key, token), the pairs in ascending
  // order and past their number above every key; at most 2 top - 1 of them
  auto pairs_below = [](const u64* k, const int* t, int top, u64 key, int tok) {
    int j = 0;
    for (int step = top; step > 0; step >>= 1) {
      const u64 m = k[j + step - 1];
      if (m < key || (m == key && t[j + step - 1] <= tok)) j += step;
    }
    return j;
  };
  // f(range, key bits, token) for the keys inside a range
  auto each_inside = [&](auto&& f) __attribute__((always_inline)) {
    const int top = 1 << (31 - __clz(n_ranges));
    each_again([&](u64 k, int t) {
      const int s = pairs_below(key0, tok0, top, k, t) - 1;
      if (s < 0 || k > key1[s] || (key_bits_of[s] == 0 && (t - tok0[s]) >> tok_bits_of[s])) return;
      f(s, k, t);
    });
  };
  while (true) {
    if (any_key) {  // draw the key ranges in to their keys
      each_inside([&](int s, u64 k, int) {
        // few keys pass the first test, so few atomics meet
        if (k < __hip_atomic_load(&range_min[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
          atomicMin(&range_min[s], k);
        if (k > __hip_atomic_load(&range_max[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
          atomicMax(&range_max[s], k);
      });
      __syncthreads();
      if (tid < n_ranges && key_bits_of[tid] > 0) {
        const u64 a = range_min[tid], b = range_max[tid];
        key0[tid] = a;
        key1[tid] = b;
        key_bits_of[tid] = b > a ? 64 - __clzll(b - a) : 0;
      }
    }
    clear_hist();
    const int bin_bits = kSelBinBits - (n_ranges > 1 ? 32 - __clz(n_ranges - 1) : 0);  // bins of a range
    auto step_of = [&](int s) { return max((key_bits_of[s] > 0 ? key_bits_of[s] : tok_bits_of[s]) - bin_bits, 0); };
    each_inside([&](int s, u64 k, int t) {
      const int b = key_bits_of[s] > 0 ? (int)((k - key0[s]) >> step_of(s)) : (t - tok0[s]) >> step_of(s);
      atomicAdd(&hist[(s << bin_bits) + b], 1);
    });
    int c[kPer];
    const int p = scan_bins(c), s = tid * kPer >> bin_bits;  // this thread's bins are of one range
    int sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum += c[i];
    for (int j = s < n_ranges ? range_first[s] : n_bnd; j < n_bnd && bnd_range[j] == s; ++j) {
      int q = range_before[s] + p - range_off[s];
      const int e = end_at[bnd_group[j]];
      if (e < q || e - q >= sum) continue;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        if (e >= q && e - q < c[i]) {
          sub_bin[j] = (tid * kPer + i) - (s << bin_bits);
          sub_before[j] = q;
          sub_count[j] = c[i];
        }
        q += c[i];
      }
    }
    __syncthreads();
    if (wave == 0) {
      const bool bnd = lane < n_bnd;
      const int j = bnd ? lane : 0, r = bnd_range[j], b = sub_bin[j], sh = step_of(r), kb = key_bits_of[r];
      const u64 k0 = kb > 0 ? key0[r] + ((u64)b << sh) : key0[r];
      const u64 k1 = kb > 0 ? min(key1[r], k0 + ((1ull << sh) - 1)) : key1[r];
      const int t0 = kb > 0 ? 0 : tok0[r] + (b << sh), tb = kb > 0 ? 32 - __clz(n) : sh;
      const int before = sub_before[j], count = sub_count[j];
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // read before the ranges are replaced
      set_ranges(bnd, (r << kSelBinBits) + b, k0, k1, kb > 0 ? sh : 0, t0, tb, before, count);
    }
    __syncthreads();
    if (!n_full) break;
  }
  // all ranges fit the list: the element (key, token) of each boundary
  if (tid < kMaxGroups) slot_fill[tid] = 0;
  __syncthreads();
  each_inside([&](int s, u64 k, int t) {
    const int at = range_off[s] + atomicAdd(&slot_fill[s], 1);
    list_key[at] = k;
    list_tok[at] = t;
  });
  __syncthreads();
  for (int i = tid; i < range_off[n_ranges]; i += kSelThreads) {
    int s = 0;
    while (i >= range_off[s + 1]) ++s;
    const int r = range_before[s] + rank_in(i, range_off[s], range_off[s + 1]);
    for (int j = 0; j < n_bnd; ++j)
      if (end_at[bnd_group[j]] == r) {
        thr_key[j] = list_key[i];
        thr_tok[j] = list_tok[i];
      }
  }
  __syncthreads();
  const int top_bnd = 1 << (31 - __clz(n_bnd));
  each_again([&](u64 k, int t) {
    const int bin = (int)((k - lo) >> shift), j = pairs_below(thr_key, thr_tok, top_bnd, k, t);
    // behind a boundary of the token's bin, or before its first one; else the bin is none of these
    if (j > 0 && bin_of[bnd_group[j - 1]] == bin) budget[t] = budget_of[bnd_group[j - 1] + 1];
    else if (j < n_bnd && bin_of[bnd_group[j]] == bin) budget[t] = budget_of[bnd_group[j]];
  });
}

// Token reordering plan: one workgroup walks the budgets twice in chunks of
// 1024 x 16 tokens, a wave prefix sum per chunk giving each thread its output
// offsets; pass 0 places the non-baseline tokens (budget < T), pass 1 the
// baseline tokens (budget T) after all of them.
constexpr int kPlanThreads = 1024, kPlanPer = 16;

__global__ __launch_bounds__(kPlanThreads) void reorder_plan_kernel(const int32_t* __restrict__ budget,
                                                                    int n, int T,
                                                                    int32_t* __restrict__ perm,
                                                                    int32_t* __restrict__ n_lead) {
  __shared__ int wave_total[kPlanThreads / kWave];
  __shared__ int bad_any;
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  if (t == 0) bad_any = 0;
  __syncthreads();
  int bad = 0, base = 0, lead_total = 0;
  for (int pass = 0; pass < 2; ++pass) {
    base = pass == 0 ? 0 : lead_total;
    for (int c0 = 0; c0 < n; c0 += kPlanThreads * kPlanPer) {
      const int e0 = c0 + t * kPlanPer;
      unsigned mask = 0;
#pragma unroll
      for (int r = 0; r < kPlanPer; ++r) {
        if (e0 + r < n) {
          const int s = budget[e0 + r];
          const bool ok = s >= 1 && s <= T && T % s == 0;
          bad |= !ok;
          const bool pick = pass == 0 ? (ok && s < T) : (!ok || s == T);
          mask |= (pick ? 1u : 0u) << r;
        }
      }
      const int cnt = __popc(mask);
      int inc = cnt;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
      }
      if (lane == kWave - 1) wave_total[w] = inc;
      __syncthreads();
      int before = 0, total = 0;
#pragma unroll
      for (int i = 0; i < kPlanThreads / kWave; ++i) {
        const int v = wave_total[i];
        before += (i < w) ? v : 0;
        total += v;
      }
      int pos = base + before + inc - cnt;
      while (mask) {
        const int r = __builtin_ctz(mask);
        perm[pos++] = e0 + r;
        mask &= mask - 1;
      }
      base += total;
      __syncthreads();  // wave_total is rewritten by the next chunk
    }
    if (pass == 0) lead_total = base;
  }
  if (bad) atomicOr(&bad_any, 1);
  __syncthreads();
  if (t == 0) n_lead[0] = bad_any ? -1 : lead_total;
}

// dst row i <- src row perm[i] (or the inverse), 16-, 4- or 1-byte units
template <typename U>
__global__ __launch_bounds__(kThreads) void permute_rows_kernel(const U* __restrict__ src,
                                                                const int32_t* __restrict__ perm,
                                                                long n_rows, long units, bool inverse,
                                                                U* __restrict__ dst) {
  const long total = n_rows * units;
  for (long e = blockIdx.x * (long)kThreads + threadIdx.x; e < total; e += (long)gridDim.x * kThreads) {
    const long i = e / units, u = e - i * units;
    const long p = perm[i];
    if (p < 0 || p >= n_rows) continue;
    if (inverse)
      dst[p * units + u] = src[e];
    else
      dst[e] = src[p * units + u];
  }
}

// one wave per row, fp32 sum of squares
template <bool BF16>
__global__ __launch_bounds__(kThreads) void row_rms_scale(const void* __restrict__ x, int n_rows,
                                                          int d, float eps, bool vec,
                                                          float* __restrict__ scale) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * (kThreads / kWave) + (threadIdx.x >> 6);
  if (row >= n_rows) return;  // the whole wave leaves together
  float acc = 0.f;
  if constexpr (BF16) {
    const bf16* r = static_cast<const bf16*>(x) + row * d;
    if (vec) {
      for (int c = lane * 8; c < d; c += kWave * 8) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(r + c);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float f = (float)v[u];
          acc = fmaf(f, f, acc);
        }
      }
    } else {
      for (int c = lane; c < d; c += kWave) {
        const float f = (float)r[c];
        acc = fmaf(f, f, acc);
      }
    }
  } else {
    const float* r = static_cast<const float*>(x) + row * d;
    if (vec) {
      for (int c = lane * 4; c < d; c += kWave * 4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(r + c);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = fmaf(v[u], v[u], acc);
      }
    } else {
      for (int c = lane; c < d; c += kWave) acc = fmaf(r[c], r[c], acc);
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) scale[row] = 1.0f / sqrtf(acc / (float)d + eps);
}

}  // namespace

hipError_t launch_row_rms_scale(const void* x, bool bf16_in, int n_rows, int d, float eps,
                                float* scale, hipStream_t s) {
  if (n_rows <= 0 || d <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n_rows + kThreads / kWave - 1) / (kThreads / kWave));
  const bool vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0 && d % (bf16_in ? 8 : 4) == 0;
  if (bf16_in)
    hipLaunchKernelGGL(row_rms_scale<true>, dim3(blocks), dim3(kThreads), 0, s, x, n_rows, d, eps,
                       vec, scale);
  else
    hipLaunchKernelGGL(row_rms_scale<false>, dim3(blocks), dim3(kThreads), 0, s, x, n_rows, d,
                       eps, vec, scale);
  return hipGetLastError();
}

hipError_t launch_gather_latent(const float* x, const int32_t* idx, int n_active, long n_tokens,
                                int channels, bool out_bf16, void* xa, hipStream_t s) {
  if (n_active <= 0 || channels <= 0) return hipSuccess;
  const bool vec = channels % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(xa) & (out_bf16 ? 7 : 15)) == 0;
  if (vec) {
    const int vpr = channels / 4;
    const dim3 grid(grid_for(((long)n_active * vpr + kGatherU - 1) / kGatherU));
    if (out_bf16)
      hipLaunchKernelGGL(gather_latent_vec<true>, grid, dim3(kThreads), 0, s,
                         reinterpret_cast<const f32x4*>(x), idx, n_active, n_tokens, vpr, xa);
    else
      hipLaunchKernelGGL(gather_latent_vec<false>, grid, dim3(kThreads), 0, s,
                         reinterpret_cast<const f32x4*>(x), idx, n_active, n_tokens, vpr, xa);
  } else {
    const dim3 grid(grid_for((long)n_active * channels));
    if (out_bf16)
      hipLaunchKernelGGL(gather_latent_scalar<true>, grid, dim3(kThreads), 0, s, x, idx, n_active,
                         n_tokens, channels, xa);
    else
      hipLaunchKernelGGL(gather_latent_scalar<false>, grid, dim3(kThreads), 0, s, x, idx,
                         n_active, n_tokens, channels, xa);
  }
  return hipGetLastError();
}

hipError_t launch_reorder_plan(const int32_t* budget, int n, int T, int32_t* perm,
                               int32_t* n_lead, hipStream_t s) {
  hipLaunchKernelGGL(reorder_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, budget, n, T, perm,
                     n_lead);
  return hipGetLastError();
}

hipError_t launch_permute_rows(const void* src, const int32_t* perm, long n_rows, long row_bytes,
                               bool inverse, void* dst, hipStream_t s) {
  if (n_rows <= 0 || row_bytes <= 0) return hipSuccess;
  const uintptr_t a = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst);
  if (row_bytes % 16 == 0 && a % 16 == 0) {
    const long u = row_bytes / 16;
    hipLaunchKernelGGL(permute_rows_kernel<u32x4>, dim3(grid_for(n_rows * u)), dim3(kThreads), 0, s,
                       static_cast<const u32x4*>(src), perm, n_rows, u, inverse,
                       static_cast<u32x4*>(dst));
  } else if (row_bytes % 4 == 0 && a % 4 == 0) {
    const long u = row_bytes / 4;
    hipLaunchKernelGGL(permute_rows_kernel<uint32_t>, dim3(grid_for(n_rows * u)), dim3(kThreads), 0,
                       s, static_cast<const uint32_t*>(src), perm, n_rows, u, inverse,
                       static_cast<uint32_t*>(dst));
  } else {
    hipLaunchKernelGGL(permute_rows_kernel<uint8_t>, dim3(grid_for(n_rows * row_bytes)),
                       dim3(kThreads), 0, s, static_cast<const uint8_t*>(src), perm, n_rows,
                       row_bytes, inverse, static_cast<uint8_t*>(dst));
  }
  return hipGetLastError();
}

hipError_t launch_rank_budgets(const double* keys, long n_tokens, const GroupTable& tab,
                               int32_t* budget, hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  const auto* k = reinterpret_cast<const unsigned long long*>(keys);
  if (n_tokens <= kRankMax) {
    hipLaunchKernelGGL(rank_budgets, dim3((unsigned)((n_tokens + kRankTokens - 1) / kRankTokens)),
                       dim3(kSelThreads), 0, s, k, (int)n_tokens, tab, budget);
    return hipGetLastError();
  }
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSelThreads), 0, s, k, (int)n_tokens, tab, budget);
  };
  const long per = (n_tokens + kSelThreads - 1) / kSelThreads;  // keys per thread
  if (per <= 8) launch(select_budgets<8>);
  else if (per <= 32) launch(select_budgets<32>);
  else if (per <= 80) launch(select_budgets<80>);
  else launch(select_budgets<0>);
  return hipGetLastError();
}

hipError_t launch_l1_rel(const float* v, float* v_prev, long n_tokens, int channels, double* acc,
                         bool first, hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  const uintptr_t align = reinterpret_cast<uintptr_t>(v) | reinterpret_cast<uintptr_t>(v_prev);
  // Two threads a token, below the 2^32 of a launch. Rows of 4 channels are one load of the scalar
  // kernel's threads too, which need no LDS: 75600 x 4 3.6 us against 4.2 (2.6 against 3.6 the first
  // time), 10^6 x 4 18.7 against 26.3; but 75600 x 8 8.2 against 4.5.
  if (channels % 4 == 0 && channels > 4 && align % 16 == 0 && n_tokens <= INT32_MAX - kL1Tokens)
    hipLaunchKernelGGL(l1_rel_accumulate_vec, dim3((unsigned)((n_tokens + kL1Tokens - 1) / kL1Tokens)),
                       dim3(kWave), 0, s, reinterpret_cast<const f32x4*>(v),
                       reinterpret_cast<f32x4*>(v_prev), n_tokens, channels / 4, acc, first ? 1 : 0);
  else
    hipLaunchKernelGGL(l1_rel_accumulate, dim3(grid_for(n_tokens)), dim3(kThreads), 0, s, v, v_prev,
                       n_tokens, channels, acc, first ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_assign_budgets(const float* v, long n_tokens, int channels,
                                 const GroupTable& tab, double* keys, int32_t* budget,
                                 hipStream_t s) {
  if (n_tokens <= 0) return hipSuccess;
  if (channels % 4 == 0 && (reinterpret_cast<uintptr_t>(v) & 15) == 0)
    hipLaunchKernelGGL(velocity_keys_vec, dim3(grid_for(n_tokens)), dim3(kThreads), 0, s,
                       reinterpret_cast<const f32x4*>(v), n_tokens, channels / 4, keys);
  else
    hipLaunchKernelGGL(velocity_keys_scalar, dim3(grid_for(n_tokens)), dim3(kThreads), 0, s, v,
                       n_tokens, channels, keys);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_rank_budgets(keys, n_tokens, tab, budget, s);
}

}  // namespace hsa
