// Row-indexed fp32 GEMM: C[crow(m)] = A[arow(m)] B^T, the fp32 variant of the
// projections of the layer step (Section 2.3) for fp32 workloads.
//
// Bound by the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and
// sums at 154 TFLOP/s, twice the rate of unpacked FMAs), one 32 x 32 tile per
// wave, four waves per workgroup, k slabs staged through two LDS buffers with
// the next slab's global loads in flight during the MFMAs. Against 4 x 4 FMA
// blocks per thread with 4-byte loads: Q/K/V of 2499 rows at d = 768 275 ->
// 112 us (79 TFLOP/s), of 682 rows at d = 256 33 -> 10 us.
// Two arrangements of the four waves (template KS):
//   KS = 1  a 64 x 64 output tile, 2 x 2 waves, slabs of 32 k.
//   KS = 4  a 32 x 32 output tile whose k the waves split (slabs of 64, 16 per
//           wave), summed through LDS at the end: for grids that would leave
//           CUs without a workgroup.
// Arbitrary M, Nc and K (ragged edges are masked). The product is formed
// transposed (B rows are the MFMA A operand), so a lane holds runs of four
// columns of one output row. An optional per-row scale multiplies each product
// row, an optional tanh GELU follows, and an optional fp32 residual, indexed
// like the output, is added before the store.
#include "common.h"

namespace hsa {
namespace {

constexpr int kThreads = 256;

// fp32 rows are only 4-byte aligned
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Epilogue of four columns n .. n+3 of product row m (output z).
__device__ __forceinline__ void store4(const RowGemm& g, const RowGemmOut& oz, int z, int m, int n, f32x4 v) {
  if (m >= g.M || n >= g.Nc) return;
  const int crow = oz.c_rows ? oz.c_rows[m] : m;
  if (crow < 0 || crow >= oz.c_limit) return;
  if (g.row_scale) {
    const float rs = g.row_scale[m];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] *= rs;
  }
  if (g.gelu) {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = gelu_tanh(v[u]);
  }
  if (g.rope_cs && ((g.rope_outs >> z) & 1)) {  // pairs (n, n+1), (n+2, n+3) of a 4-aligned run
    const RopeRow rr = rope_row(g, m);
    const int k = (n % g.rope_dh) >> 1;
    const f32x2 r0 = rope_pair(g, rr, k, v[0], v[1]);
    const f32x2 r1 = rope_pair(g, rr, k + 1, v[2], v[3]);
    v = (f32x4){r0[0], r0[1], r1[0], r1[1]};
  }
  float* cb = static_cast<float*>(oz.C);  // may alias the residual
  long orow = crow;
  if (oz.C2 && crow >= oz.c_split) {  // rows past the split go to the second buffer
    cb = static_cast<float*>(oz.C2);
    orow = crow - oz.c_split;
  }
  const long e = orow * g.ldc + n;
  const float* R = static_cast<const float*>(g.residual);
  if (n + 4 <= g.Nc) {
    if (R) {
      const f32x4u r = *reinterpret_cast<const f32x4u*>(R + e);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += r[u];
    }
    *reinterpret_cast<f32x4u*>(cb + e) = v;
  } else {
    for (int u = 0; n + u < g.Nc; ++u) cb[e + u] = R ? v[u] + R[e + u] : v[u];
  }
}

template <int KS>
__global__ __launch_bounds__(kThreads) void row_gemm_f32_kernel(RowGemm g) {
  constexpr int T = KS == 1 ? 64 : 32;   // output tile side
  constexpr int TK = KS == 1 ? 32 : 64;  // k per slab
  constexpr int P = TK + 4;              // padded LDS row: 8 rows' 16-byte reads on distinct banks
  constexpr int LOADS = T * TK / 4 / kThreads;  // 16-byte loads per thread per operand per slab
  constexpr int CPR = TK / 4;                   // 16-byte chunks per slab row
  __shared__ __attribute__((aligned(16))) float As[2][T * P];
  __shared__ __attribute__((aligned(16))) float Bs[2][T * P];

  const int tiles_m = (g.M + T - 1) / T;
  const int tiles_n1 = (g.Nc + T - 1) / T;
  const int per_out = tiles_m * tiles_n1;
  const int item = xcd_contiguous(blockIdx.x, per_out * g.n_out);
  const int z = item / per_out;
  const int rem = item - z * per_out;
  const int tm = rem % tiles_m;
  const int tn = rem / tiles_m;
  const RowGemmOut oz = row_gemm_out(g, z);

  const float* __restrict__ A = static_cast<const float*>(g.A);
  const float* __restrict__ B = static_cast<const float*>(oz.B);
  const int t = threadIdx.x;
  const int lane = t & (kWave - 1), wave = t / kWave;
  const int l32 = lane & 31, hi = lane >> 5;

  // load i of this thread: slab row lr(i), k offset lk
  const int lk = (t % CPR) * 4;
  const float* a_src[LOADS];
  const float* b_src[LOADS];
  bool a_ok[LOADS], b_ok[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int lr = t / CPR + i * (kThreads / CPR);
    const int m = tm * T + lr, n = tn * T + lr;
    int arow = -1;
    if (m < g.M) arow = g.a_rows ? g.a_rows[m] : m;
    a_ok[i] = arow >= 0 && arow < g.a_limit;
    b_ok[i] = n < g.Nc;
    a_src[i] = A + (long)(a_ok[i] ? arow : 0) * g.lda;
    b_src[i] = B + (long)(b_ok[i] ? n : 0) * g.ldb;
  }
  f32x4 ra[LOADS], rb[LOADS];
  auto load = [&](int k0) {
    const int k = k0 + lk;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      if (k + 4 <= g.K) {
        ra[i] = *reinterpret_cast<const f32x4u*>(a_src[i] + k);
        rb[i] = *reinterpret_cast<const f32x4u*>(b_src[i] + k);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          ra[i][u] = k + u < g.K ? a_src[i][k + u] : 0.f;
          rb[i][u] = k + u < g.K ? b_src[i][k + u] : 0.f;
        }
      }
      if (!a_ok[i]) ra[i] = (f32x4){};
      if (!b_ok[i]) rb[i] = (f32x4){};
    }
  };
  auto stage = [&](int b) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int lr = t / CPR + i * (kThreads / CPR);
      *reinterpret_cast<f32x4*>(&As[b][lr * P + lk]) = ra[i];
      *reinterpret_cast<f32x4*>(&Bs[b][lr * P + lk]) = rb[i];
    }
  };

  // this wave's rows of the tile (wm, wn) and its k range of a slab
  const int wm = KS == 1 ? (wave & 1) * 32 : 0, wn = KS == 1 ? (wave >> 1) * 32 : 0;
  constexpr int WK = TK / KS;  // k per wave and slab
  const int wk = KS == 1 ? 0 : wave * WK;
  const int ao = (wm + l32) * P + wk + hi * 4, bo = (wn + l32) * P + wk + hi * 4;

  f32x16 acc = (f32x16){};
  load(0);
  stage(0);
  __syncthreads();
  int b = 0;
  for (int k0 = 0; k0 < g.K; k0 += TK, b ^= 1) {
    const bool more = k0 + TK < g.K;
    if (more) load(k0 + TK);
#pragma unroll
    for (int j = 0; j < WK / 8; ++j) {
      const f32x4 av = *reinterpret_cast<const f32x4*>(&As[b][ao + j * 8]);
      const f32x4 bv = *reinterpret_cast<const f32x4*>(&Bs[b][bo + j * 8]);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[u], av[u], acc, 0, 0, 0);
    }
    if (more) stage(b ^ 1);  // last read one slab ago, before the previous barrier
    __syncthreads();
  }

  // acc[e]: product row wm + l32, column wn + (e/4)*8 + hi*4 + e%4
  if constexpr (KS == 1) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      store4(g, oz, z, tm * T + wm + l32, tn * T + wn + c * 8 + hi * 4,
             (f32x4){acc[4 * c], acc[4 * c + 1], acc[4 * c + 2], acc[4 * c + 3]});
  } else {
    // wave w sums the four waves' columns w*8 .. w*8+7 (the slabs are no longer read)
    f32x4* red = reinterpret_cast<f32x4*>(&As[0][0]);  // [wave][c][lane]
    static_assert(2 * T * P * 4 >= 4 * 4 * kWave * 16, "the partial tiles fit in the A slabs");
#pragma unroll
    for (int c = 0; c < 4; ++c)
      red[(wave * 4 + c) * kWave + lane] = (f32x4){acc[4 * c], acc[4 * c + 1], acc[4 * c + 2], acc[4 * c + 3]};
    __syncthreads();
    f32x4 v = red[wave * kWave + lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f32x4 p = red[(w * 4 + wave) * kWave + lane];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] += p[u];
    }
    store4(g, oz, z, tm * T + l32, tn * T + wave * 8 + hi * 4, v);
  }
}

}  // namespace

hipError_t launch_row_gemm_f32(const RowGemm& g, hipStream_t s) {
  if (g.M <= 0 || g.Nc <= 0 || g.n_out <= 0) return hipSuccess;
  auto tiles = [&](long t) { return ((g.M + t - 1) / t) * ((g.Nc + t - 1) / t) * g.n_out; };
  // 64 x 64 tiles, or split-k 32 x 32 tiles below one and a half of the former
  // per CU: 300 x 1536 x 1536 Q/K/V (360 tiles of 64) 64 us against 76, but
  // 2499 x 768 x 768 (480 tiles) 46 against 44 and 8000 x 1536 x 1536 483
  // against 397 (split-k tiles load twice the bytes per product).
  if (2 * tiles(64) >= 3 * (long)compute_units())
    hipLaunchKernelGGL(row_gemm_f32_kernel<1>, dim3((unsigned)tiles(64)), dim3(kThreads), 0, s, g);
  else
    hipLaunchKernelGGL(row_gemm_f32_kernel<4>, dim3((unsigned)tiles(32)), dim3(kThreads), 0, s, g);
  return hipGetLastError();
}

}  // namespace hsa
