// fp32 active-query attention (Section 2.3, step 3) for fp32 workloads: each
// active query attends to all N cached key/value rows of its head.
//
// Both contractions run on the matrix cores in fp32 (v_mfma_f32_32x32x2_f32 or
// 16x16x4: fp32 products and sums, twice the rate of unpacked FMAs), which
// bound it: they are busy 61% of a launch of 2499 queries, 4999 rows and 12
// heads of 64, the softmax's VALU work taking most of the rest. One workgroup
// of 8 waves takes 32 (or 16) queries of one head and its waves split the
// cached rows (wave w takes the 32-key blocks w, w+8, ...), so that even a
// launch of few queries fills the SIMDs and no wave waits for another before
// the end, where the eight partial softmaxes are merged through LDS.
// Workgroups of one head are contiguous on one XCD, so the rows that every
// wave loads for itself stay in that XCD's L2.
//
// Per 32-key block, in one wave (32 queries; 16 are alike):
//   S^T = K Q^T     K rows are the A operand (lane: key l%32), the queries the
//                   B operand. The contraction order is free, so a lane reads
//                   runs of 4 channels (16 bytes) and step 4j + t of slot hi
//                   takes channel 8j + 4hi + t. Each lane then holds 16 scores
//                   of ONE query.
//   softmax         online; the maximum and the sum need one exchange between
//                   the lanes of one query. exp_neg is as exact as expf for
//                   x <= 0 and normal results, in half its instructions.
//   O^T += V^T P^T  step e takes the probabilities as they sit in the score
//                   registers (key row(e, slot)) and the matching rows of V;
//                   tile dt's row r is channel r*DT + dt, so a lane reads DT
//                   consecutive channels at once.
//
// Measured against one wave per (query, head) with FMAs and a serial walk over
// the keys: 682 queries, 1024 rows, 4 x 64 heads 285 -> 17 us; 2499 queries,
// 4999 rows, 12 x 64 heads 9083 -> 449 us (85 TFLOP/s); its error against
// float64 is 0.6 of the former's. Up to 4 rows of 64-wide heads and 8 of 128-wide
// it is the slower one (1 query, 1 row 4.1 against 3.0 us, 16 x 8 x 12 heads of 128
// 6.2 against 5.5): the launch, the trip through LDS and the merge; a single wave for such
// rows takes 3.8 and 6.3.
#include "common.h"

namespace hsa {
namespace {

constexpr int kWaves = 8;  // waves per workgroup, each on its own key blocks
constexpr int kThreads = kWaves * kWave;
constexpr int kKeys = 32;  // keys per block
constexpr int kMaxOffsetRow = 1 << 24;  // a block of rows up to this wide is addressed by 32-bit byte offsets

// fp32 rows are only 4-byte aligned
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// The W x W fp32 matrix instruction: 64/W contraction slots (lane / W), the
// result's column lane % W, its rows row(e, lane / W) for e < W*W/64.
template <int W>
struct Mfma;
template <>
struct Mfma<32> {
  typedef f32x16 acc;
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int e, int slot) { return (e >> 2) * 8 + slot * 4 + (e & 3); }
};
template <>
struct Mfma<16> {
  typedef f32x4 acc;
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int e, int slot) { return slot * 4 + e; }
};

// exp(x) for x <= 0 (NaN stays NaN): 2^t with t = fl(x log2 e), corrected by
// the remainder x - t ln 2, which is exact to below an ulp. Results under 2^-126,
// which v_exp_f32 flushes (expf does not), are 0: a key's weight of 1e-38 of the greatest.
__device__ __forceinline__ float exp_neg(float x) {
  const float c = x < -104.f ? -104.f : x;
  const float t = c * 1.44269504088896341f;
  const float e = __builtin_amdgcn_exp2f(t);
  const float u = fmaf(-t, -1.90465429995776804525e-09f, fmaf(-t, 0.693147182464599609375f, c));
  return fmaf(e, u, e);
}

// W: queries per workgroup
template <int DH, int W, bool SPLIT>
__global__ __launch_bounds__(kThreads) void attention_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, int n_q, int n_kv, int heads, int d, float scale, int n_qtiles,
    const float* __restrict__ k2, const float* __restrict__ v2, int n_split) {
  typedef typename Mfma<W>::acc Acc;
  constexpr int SL = kWave / W;        // contraction slots of one instruction
  constexpr int NE = W / SL;           // result registers per lane
  constexpr int KT = kKeys / W;        // key tiles of a block
  constexpr int DT = DH / W;           // channel tiles of O^T
  constexpr int J = DH / (4 * SL);     // 16-byte reads of a K or Q row per lane
  constexpr int CPR = DH / 4;          // 16-byte chunks per row
  constexpr int LD = kKeys * CPR / kWave;  // 16-byte loads per lane of a block's K rows
  constexpr int P = DH + 4;            // padded LDS row, floats
  constexpr bool kQLds = DH > 64 && W > 16;
  typedef float vrow __attribute__((ext_vector_type(DT)));
  // the same in a row of the merge buffer, whose stride of P floats is a multiple of 16 bytes and no more
  typedef vrow vrow_lds __attribute__((aligned(DT < 4 ? 4 * DT : 16)));
  static_assert(P * 4 % alignof(vrow_lds) == 0, "rows of the merge buffer are aligned for its stores");
  // per wave: its block's K rows, at the end its share of the output
  __shared__ __attribute__((aligned(16))) float buf[kWaves][kKeys * P];
  __shared__ float m_part[kWaves][W], l_part[kWaves][W];
  __shared__ __attribute__((aligned(16))) float q_lds[kQLds ? W * P : 4];

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform: scalar block addresses
  const int lw = lane % W, slot = lane / W;
  const int item = xcd_contiguous(blockIdx.x, n_qtiles * heads);
  const int h = item / n_qtiles, qt = item - h * n_qtiles;
  const long col0 = (long)h * DH;
  const float* kg = k + col0;
  const float* vg = v + col0;

  // this lane's query (rows past n_q repeat the last one and are not stored):
  // in registers, or where those hold the next block's K rows instead (32
  // queries of 128 channels) in LDS, the same for every wave
  f32x4 qf[kQLds ? 1 : J];
  {
    const float* qb = q + col0;
    if constexpr (kQLds) {
      for (int f = threadIdx.x; f < W * CPR; f += kThreads) {
        const int r = f / CPR, c = (f - r * CPR) * 4;
        *reinterpret_cast<f32x4*>(&q_lds[r * P + c]) =
            *reinterpret_cast<const f32x4u*>(qb + (long)min(qt * W + r, n_q - 1) * d + c);
      }
      __syncthreads();
    } else {
      const float* qr = qb + (long)min(qt * W + lw, n_q - 1) * d + slot * 4;
#pragma unroll
      for (int j = 0; j < J; ++j) qf[j] = *reinterpret_cast<const f32x4u*>(qr + j * 4 * SL);
    }
  }
  auto query = [&](int j) -> f32x4 {
    if constexpr (kQLds) return *reinterpret_cast<const f32x4*>(&q_lds[lw * P + j * 4 * SL + slot * 4]);
    else return qf[j];
  };

  // Maxima are of the products q.k and the scale follows the subtraction: the
  // exponents (q.k - m) scale are then at most 0 however large the products are. (With
  // q.k scale - fl(m scale) in one FMA they carry what rounding m scale lost, which is
  // over 88 and overflows the exponential from scores of about 1e9 on.)
  Acc acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = (Acc){};
  float m_run = -INFINITY, l_run = 0.f;

  // Rows n0 .. n0+31 of the keys or values are read through a buffer resource
  // at row n0 (uniform, so scalar), with the lane's byte offset and the row
  // step in the two offsets of the load: no address arithmetic per load. The
  // resource ends at row n_kv, and in the last block, where the step is part of the
  // lane's offset, the one that is range-checked, rows past it read as zeros: their
  // scores are masked, and 0 times a zero adds nothing to an output.
  auto first = [&](const float* a, const float* a2, int n0) {
    const float* b = (SPLIT && n0 >= n_split) ? a2 + (long)(n0 - n_split) * d + col0 : a + (long)n0 * d;
    const unsigned bytes = (unsigned)min(kKeys, n_kv - n0) * (unsigned)(d * 4) - (unsigned)(col0 * 4);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(b), 0, (int)bytes, 0x00020000);
  };
  auto by_row = [&](int n0) {
    return SPLIT && (d > kMaxOffsetRow || (n0 < n_split && n0 + kKeys > n_split));
  };
  const int row_bytes = d * 4;
  // C channels of row n0 + r + step, c floats into it (r and c per lane, step uniform)
  auto read = [&](auto* dst, const float* a, const float* a2, int n0, int r, int step, int c) {
    constexpr int C = sizeof(*dst) / 4;
    if (by_row(n0)) {
      const int n = min(n0 + r + step, n_kv - 1);
      const float* src = n >= n_split ? a2 + (long)(n - n_split) * d + col0 : a + (long)n * d;
      __builtin_memcpy(dst, src + c, sizeof(*dst));
      if (n0 + r + step >= n_kv) __builtin_memset(dst, 0, sizeof(*dst));
      return;
    }
    const auto rs = first(a, a2, n0);
    int vo = r * row_bytes + c * 4, so = step * row_bytes;
    if (n0 + kKeys > n_kv) {
      vo += so;
      so = 0;
    }
    if constexpr (C == 2) {
      const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, 0);
      __builtin_memcpy(dst, &x, sizeof(x));
    } else {
#pragma unroll
      for (int i = 0; i < C / 4; ++i) {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rs, vo + i * 16, so, 0);
        __builtin_memcpy(reinterpret_cast<char*>(dst) + i * 16, &x, sizeof(x));
      }
    }
  };

  // A block's K rows go to LDS through registers: loaded (whole rows, so that
  // every line is read once) during the previous block's softmax and PV, and
  // written just before its scores. Only this wave reads them: no barrier.
  float* kl = buf[wave];
  f32x4 kr[LD];
  auto load_k = [&](int n0) {
    if (n0 >= n_kv) return;
#pragma unroll
    for (int i = 0; i < LD; ++i) read(&kr[i], kg, k2, n0, lane / CPR, i * (kWave / CPR), lane % CPR * 4);
  };
  vrow vf[KT][NE];
  auto load_v = [&](int n0) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int e = 0; e < NE; ++e)
        read(&vf[kt][e], vg, v2, n0, Mfma<W>::row(0, slot), kt * W + Mfma<W>::row(e, 0), lw * DT);
  };
  load_k(wave * kKeys);
  for (int n0 = wave * kKeys; n0 < n_kv; n0 += kWaves * kKeys) {
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int f = i * kWave + lane;
      *reinterpret_cast<f32x4*>(&kl[(f / CPR) * P + (f % CPR) * 4]) = kr[i];
    }
    load_v(n0);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the K rows are in LDS
    Acc s[KT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) s[kt] = (Acc){};
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (kQLds && j % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // else every LDS read is hoisted, and spills
      const f32x4 qv = query(j);
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        const f32x4 kf = *reinterpret_cast<const f32x4*>(&kl[(kt * W + lw) * P + j * 4 * SL + slot * 4]);
#pragma unroll
        for (int t = 0; t < 4; ++t) s[kt] = Mfma<W>::mul(kf[t], qv[t], s[kt]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // read before the next block's rows
    load_k(n0 + kWaves * kKeys);

    if (n0 + kKeys > n_kv) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int e = 0; e < NE; ++e)
          if (n0 + kt * W + Mfma<W>::row(e, slot) >= n_kv) s[kt][e] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int e = 0; e < NE; ++e) mx = fmaxf(mx, s[kt][e]);
#pragma unroll
    for (int x = W; x < kWave; x <<= 1) mx = fmaxf(mx, __shfl_xor(mx, x));
    if (__any(mx > m_run)) {
      // raise the running maximum (wave-uniform branch, rare after the first blocks)
      const float m_new = fmaxf(m_run, mx);
      const float alpha = m_run == -INFINITY ? 0.f : expf((m_run - m_new) * scale);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] *= alpha;
      m_run = m_new;
    }
    const float m_use = m_run == -INFINITY ? 0.f : m_run;  // only -inf scores so far: weights 0
    float ls = 0.f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        s[kt][e] = exp_neg((s[kt][e] - m_use) * scale);
        ls += s[kt][e];
      }
    l_run += ls;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[dt] = Mfma<W>::mul(vf[kt][e][dt], s[kt][e], acc[dt]);
  }

  // merge: the waves' softmaxes, each rescaled to the common maximum
  float l_tot = l_run;
#pragma unroll
  for (int x = W; x < kWave; x <<= 1) l_tot += __shfl_xor(l_tot, x);
  if (slot == 0) {
    m_part[wave][lw] = m_run;
    l_part[wave][lw] = l_tot;
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    vrow r;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) r[dt] = acc[dt][e];
    *reinterpret_cast<vrow_lds*>(&kl[lw * P + Mfma<W>::row(e, slot) * DT]) = r;
  }
  __syncthreads();
  for (int f = threadIdx.x; f < W * CPR; f += kThreads) {
    const int r = f / CPR, c = (f - r * CPR) * 4;
    const int qrow = qt * W + r;
    if (qrow >= n_q) continue;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) m = fmaxf(m, m_part[w][r]);
    f32x4 sum = {};
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float mw = m_part[w][r];
      const float wt = mw == -INFINITY ? 0.f : expf((mw - m) * scale);  // 0: no finite score (or no key) in this wave
      l = fmaf(wt, l_part[w][r], l);
      const f32x4 a = *reinterpret_cast<const f32x4*>(&buf[w][r * P + c]);
#pragma unroll
      for (int u = 0; u < 4; ++u) sum[u] = fmaf(wt, a[u], sum[u]);
    }
    const float inv = 1.f / l;
    f32x4u out = {sum[0] * inv, sum[1] * inv, sum[2] * inv, sum[3] * inv};
    *reinterpret_cast<f32x4u*>(o + (long)qrow * d + col0 + c) = out;
  }
}

template <int DH, int W>
void launch_w(const float* q, const float* k, const float* v, float* o, int n_q, int n_kv, int heads,
              float scale, hipStream_t s, const float* k2, const float* v2, int n_split) {
  const int n_qtiles = (n_q + W - 1) / W;
  const dim3 grid((unsigned)((long)n_qtiles * heads));
  const int d = heads * DH;
  if (n_split < n_kv || d > kMaxOffsetRow)
    hipLaunchKernelGGL((attention_f32_kernel<DH, W, true>), grid, dim3(kThreads), 0, s, q, k, v, o, n_q, n_kv,
                       heads, d, scale, n_qtiles, k2, v2, n_split);
  else
    hipLaunchKernelGGL((attention_f32_kernel<DH, W, false>), grid, dim3(kThreads), 0, s, q, k, v, o, n_q, n_kv,
                       heads, d, scale, n_qtiles, k2, v2, n_split);
}

template <int DH>
void launch_dh(const float* q, const float* k, const float* v, float* o, int n_q, int n_kv, int heads,
               float scale, hipStream_t s, const float* k2, const float* v2, int n_split) {
  // 32 queries per workgroup, or 16 where that fills the CUs better: a round of
  // 16-query workgroups takes 0.57 of a round of 32-query ones (each wave loads
  // the same rows for half the products)
  const long cus = compute_units();
  auto rounds = [&](long w) { return (((n_q + w - 1) / w) * heads + cus - 1) / cus; };
  const bool small = 0.57 * rounds(16) < rounds(32);
  if (small)
    launch_w<DH, 16>(q, k, v, o, n_q, n_kv, heads, scale, s, k2, v2, n_split);
  else
    launch_w<DH, 32>(q, k, v, o, n_q, n_kv, heads, scale, s, k2, v2, n_split);
}

}  // namespace

hipError_t launch_attention_f32(const void* q, const void* k, const void* v, void* o, int n_q,
                                int n_kv, int heads, int head_dim, float scale, hipStream_t s,
                                const void* k2, const void* v2, int n_split) {
  if (!k2 || !v2) n_split = n_kv;
  if (n_q <= 0) return hipSuccess;
  const float* qf = static_cast<const float*>(q);
  const float* kf = static_cast<const float*>(k);
  const float* vf = static_cast<const float*>(v);
  float* of = static_cast<float*>(o);
  const float* k2f = static_cast<const float*>(k2);
  const float* v2f = static_cast<const float*>(v2);
  if (head_dim == 64)
    launch_dh<64>(qf, kf, vf, of, n_q, n_kv, heads, scale, s, k2f, v2f, n_split);
  else
    launch_dh<128>(qf, kf, vf, of, n_q, n_kv, heads, scale, s, k2f, v2f, n_split);
  return hipGetLastError();
}

}  // namespace hsa
