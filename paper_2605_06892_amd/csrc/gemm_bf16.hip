// Row-indexed bf16 GEMM on CDNA4 matrix cores: C[crow(m)] = A[arow(m)] B^T.
//
// This one kernel carries both dense contractions of the layer step:
//   * the fresh Q/K/V projections of the active rows (Section 2.3, step 1),
//     with the gather of x[A_i] fused into the A-tile loads and the cache
//     overwrite K_hat[A_i], V_hat[A_i] (step 2) fused into the K/V epilogues;
//   * the output projection of the active rows with the scatter back to their
//     tokens fused into the epilogue.
// The compact gathered activations are never materialized in HBM.
//
// Tiling (struct Tiling): BM x BN output tile per workgroup of waves in a
// WM x WN grid, K step 64, v_mfma_f32_16x16x32_bf16. Tiles go global -> LDS
// directly (buffer_load_dwordx4 ... lds through one buffer resource over A
// and one over B, or global_load_lds_dwordx4 with 64-bit lane pointers for a
// matrix of 4 GiB or more: one wave instruction fills one contiguous 1 KB
// segment = 8 tile rows of 128 bytes). The 16-byte chunks of tile row r
// sit at slot chunk ^ ((r >> 1) & 7), which keeps the fragment reads (16
// rows, one chunk) on disjoint banks. Each LDS array is a variable of its own
// and the K loops are unrolled by the array count, so the compiler can tell the
// asynchronous loads from reads of another array.
//
// The large tilings (8 waves, 256 rows) run a ping-pong loop: while one of a
// SIMD's two waves issues MFMAs and nothing else, the other reads its next
// fragments and issues loads. With both waves doing both at once, interleaved
// by the compiler around one barrier per step, the matrix pipes were busy 71%
// of the Q/K/V launch at 8190 x 5120; they are now 79-83%. The 32x32x16 MFMA
// then ran at a clock of 1.49 GHz (the card's power limit), 16x16x32 runs at
// 1.61 GHz: it reads and writes half as many accumulators per product. Together
// that launch went from 1045 to 884 us (1.23 -> 1.46 PFLOP/s), the output
// projection of 16380 x 5120 from 667 to 550 us (1.56 PFLOP/s), the FFN's down
// projection of 8190 x 8960 x 1536 from 176 to 148 us, with the same bits.
//
// The small tilings run a ring of four arrays, loaded three steps ahead, with
// one barrier per step: launches of few rows or columns are bound by the
// latency of one workgroup's chain of steps, which a smaller tile shortens, and
// by the CUs left without a workgroup. 400 x 8960 x 1536 products went from 101
// to 41 us, 1000 x 1536 x 1536 from 21.9 to 11.1 us, and those of a block of 500
// rows at d = 256 from 8.5-12 to 5-6 us (kernel alone).
// Every tile row is a contiguous 128-byte run of a token row, so the indexed
// loads stay coalesced; rows outside the problem are read from a valid row and
// their results dropped. The product is formed transposed (B rows drive the
// MFMA A operand), which leaves each lane holding one output row and runs of
// four consecutive columns: one row-index lookup per lane and 8-byte stores.
// Tiles are ordered in groups of 8 tile-rows (4 for wide outputs) and laid
// out contiguously per XCD so the A and B panels a group shares stay in that
// XCD's L2.
#include "common.h"

#include <type_traits>

namespace hsa {
namespace {


typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void global_cvoid;

constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

constexpr int waitcnt_lgkm0() { return 15 | (7 << 4) | (0 << 8) | (3 << 14); }

template <int I>
using Int = std::integral_constant<int, I>;

// f(integral_constant<int, I>) for I = B .. E-1, unrolled at compile time
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Epilogues (after the optional per-row scale): bf16 store, bf16 store of
// (product + bf16 residual) rounded once, fp32 store, bf16 store of the tanh
// GELU of the product.
enum Epilogue { kEpiBf16 = 0, kEpiBf16Residual = 1, kEpiF32 = 2, kEpiBf16Gelu = 3 };

// 16 bytes per lane from base + voff + soff, a buffer resource over the
// nbytes bytes from base, straight into LDS at dst (the wave's 1 KB segment).
// Against 64-bit lane pointers this needs no per-load address arithmetic and
// half the registers; a load past nbytes reads zeros instead of faulting.
__device__ __forceinline__ void buffer_load_lds16(const void* base, unsigned nbytes, bf16* dst, unsigned voff,
                                                  unsigned soff) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)nbytes, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 16, voff, soff, 0, 0);
}

// One tiling of the kernel: BM x BN output tile, K step BK, WAVES waves in a
// WM x (WAVES/WM) grid. STAGES 0: the ping-pong loop of 8 waves (two LDS arrays
// for A tiles, three for B tiles); 4: a ring of four arrays, each an A tile
// followed by a B tile, loaded three steps ahead.
template <int BM_, int BN_, int BK_, int STAGES_, int WAVES_, int WM_>
struct Tiling {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_, WAVES = WAVES_, WM = WM_;
  static constexpr int WN = WAVES / WM, THREADS = WAVES * 64;
  static constexpr int TM = BM / WM, TN = BN / WN;  // wave tile
  static constexpr int MI = TM / 16, NI = TN / 16;  // 16x16 MFMA tiles per wave
  static constexpr int RB = TM / 32;                // 32-row blocks of the wave tile (epilogue)
  static constexpr int CHUNKS = BK / 8;             // 16-byte chunks per tile row
  static constexpr int SEG_ROWS = 64 / CHUNKS;      // tile rows per 1 KB wave load
  static constexpr int SEG_A = BM / SEG_ROWS, SEG_B = BN / SEG_ROWS;
  static constexpr int LOADS = (SEG_A + SEG_B) / WAVES;  // load instructions per lane per stage
  static constexpr bool PING = STAGES == 0;
  static constexpr int ARRAYS = PING ? 5 : STAGES;                        // LDS arrays
  static constexpr int ARRAY = PING ? 256 * BK : (BM + BN) * BK;          // bf16 elements of each
  static_assert(BK == 64, "K step");
  static_assert(LOADS * WAVES == SEG_A + SEG_B && SEG_A % WAVES == 0, "stage load must split evenly over waves");
  static_assert(RB * 32 == TM && NI * 16 == TN, "wave tile");
  static_assert(!PING || (WAVES == 8 && BM <= 256 && BN <= 256), "ping-pong: two halves of four waves");
  static_assert(PING || (STAGES == 4 && LOADS * (STAGES - 2) <= 63), "ring, vmcnt range");
  static_assert(ARRAYS * ARRAY * 2 <= 160 * 1024, "LDS");
  // 16-byte chunk c of tile row r sits at slot c ^ swz(r): any 16 consecutive
  // rows read at one chunk (one fragment read, 256 bytes per 16 lanes) land
  // on 16 distinct 16-byte bank groups
  static __device__ __forceinline__ int swz(int r) { return (r / (16 / CHUNKS)) % CHUNKS; }
};

// Output tile (tm, tn) of output z in tiling TL, staged through the
// workgroup's LDS arrays, separate arrays, so that the compiler can tell the
// asynchronous loads into one from the fragment reads of another.
// BUF: stage loads through buffer resources (A and B each below 4 GiB), else
// through 64-bit lane pointers. ROPE: the RoPE epilogue is compiled in (the
// Q/K/V projection only).
struct LdsArrays {
  bf16* p[5];
};

template <class TL, int EPI, bool BUF, bool ROPE>
__device__ __forceinline__ void row_gemm_tile(const RowGemm& g, int tm, int tn, int z, const LdsArrays& lds) {
  constexpr int BM = TL::BM, BN = TL::BN, BK = TL::BK, WN = TL::WN;
  constexpr int TM = TL::TM, TN = TL::TN, MI = TL::MI, NI = TL::NI, RB = TL::RB, LOADS = TL::LOADS;
  constexpr int SEG_A = TL::SEG_A, CHUNKS = TL::CHUNKS, SEG_ROWS = TL::SEG_ROWS;
  constexpr int RING = TL::PING ? 1 : TL::STAGES;
  // the arrays of step u's A and B tiles (in a ring, those of stage u)
  auto a_tile = [&](int u) -> bf16* { return TL::PING ? lds.p[u % 2] : lds.p[u % RING]; };
  auto b_tile = [&](int u) -> bf16* { return TL::PING ? lds.p[2 + u % 3] : lds.p[u % RING] + BM * BK; };
  const RowGemmOut oz = row_gemm_out(g, z);

  const bf16* __restrict__ A = static_cast<const bf16*>(g.A);
  const bf16* __restrict__ B = static_cast<const bf16*>(oz.B);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l16 = lane & 15, grp = lane >> 4;

  // This lane's rows of the stage loads: segment s = i*WAVES + wave covers
  // tile rows SEG_ROWS*s .. (A tile first, then B tile); the lane fetches
  // row SEG_ROWS*s + lane/CHUNKS, global chunk (lane%CHUNKS) ^ swz(row),
  // into LDS slot lane%CHUNKS.
  const bf16* src[LOADS];  // !BUF: the lane's chunk of its row in A or B
  unsigned voff[LOADS];    // BUF: the same as a byte offset from A or B
  int dst[LOADS];          // element offset of the segment in its tile
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int s = i * TL::WAVES + wave;
    const bool a = s < SEG_A;
    const int trow = (a ? s : s - SEG_A) * SEG_ROWS + lane / CHUNKS;
    const int chunk = (lane % CHUNKS) ^ TL::swz(trow);
    long grow;
    if (a) {
      const int m = tm * BM + trow;
      int row = (m < g.M) ? (g.a_rows ? g.a_rows[m] : m) : 0;
      if (row < 0 || row >= g.a_limit) row = 0;
      grow = (long)row * g.lda;
    } else {
      const int n = min(tn * BN + trow, g.Nc - 1);
      grow = (long)n * g.ldb;
    }
    if constexpr (BUF)
      voff[i] = (unsigned)((grow + chunk * 8) * 2);
    else
      src[i] = (a ? A : B) + grow + chunk * 8;
    dst[i] = (a ? s : s - SEG_A) * 512;
  }
  // segment i of every wave lies in A when i * WAVES < SEG_A (SEG_A is a
  // multiple of WAVES), so the resource of a load is known at compile time
  const unsigned a_bytes = (unsigned)((long)g.a_limit * g.lda * 2), b_bytes = (unsigned)((long)g.Nc * g.ldb * 2);
  constexpr int LOADS_A = SEG_A / TL::WAVES, LOADS_B = LOADS - LOADS_A;
  auto load = [&](bf16* tile, int i, int k0) __attribute__((always_inline)) {
    if constexpr (BUF) {
      if (i < LOADS_A)
        buffer_load_lds16(A, a_bytes, tile + dst[i], voff[i], (unsigned)(k0 * 2));
      else
        buffer_load_lds16(B, b_bytes, tile + dst[i], voff[i], (unsigned)(k0 * 2));
    } else {
      __builtin_amdgcn_global_load_lds((global_cvoid*)(src[i] + k0), (lds_void*)(tile + dst[i]), 16, 0, 0);
    }
  };
  auto issue_a = [&](auto st, int k0) {
#pragma unroll
    for (int i = 0; i < LOADS_A; ++i) load(a_tile(decltype(st)::value), i, k0);
  };
  auto issue_b = [&](auto st, int k0) {
#pragma unroll
    for (int i = LOADS_A; i < LOADS; ++i) load(b_tile(decltype(st)::value), i, k0);
  };

  // fragment read offsets: row (tile-local) l16 + 16*t, chunk half*4 + grp;
  // swz(l16 + 16 t) = swz(l16)
  const int xr = ((grp ^ TL::swz(l16)) * 8);
  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = (f32x4){};

  bf16x8 af[MI], bfr[NI];
  auto barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the fragments of half a K step (32 k) of step u
  auto read = [&](auto uc, int half) __attribute__((always_inline)) {
    const int off = (half * 32) ^ xr;
    const bf16* Ar = a_tile(decltype(uc)::value) + (wm * TM + l16) * BK + off;
    const bf16* Br = b_tile(decltype(uc)::value) + (wn * TN + l16) * BK + off;
#pragma unroll
    for (int j = 0; j < NI; ++j) bfr[j] = *reinterpret_cast<const bf16x8*>(Br + j * 16 * BK);
#pragma unroll
    for (int i = 0; i < MI; ++i) af[i] = *reinterpret_cast<const bf16x8*>(Ar + i * 16 * BK);
    __builtin_amdgcn_sched_barrier(0);
  };
  // the reads are done: the arrays may be rewritten after the next barrier
  auto read_done = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());
  };
  auto mfmas = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
  };

  const int nk = g.K / BK;
  // ring, g.rms: sums of squares of the lane's A rows, eight each, so that their chains of
  // roundings are as short as those of row_rms_scale (the fp32 velocities of a head at
  // d = 5120 are 4.5e-7 off the exact product with either; 4.9e-7 with one sum a row)
  float sq[MI][2][4] = {};
  if constexpr (TL::PING) {
    // Ping-pong K loop. Waves w and w + 4 share a SIMD; the waves of one half
    // read fragments and issue tile loads while the other half's run MFMAs and
    // nothing else, and a barrier swaps the roles. Step k of a wave takes four
    // slots, two of each kind, each over half of the step's k:
    //   M0  read the fragments of the first half; issue the loads of A for step
    //       k+1 (its array was last read in the other half's M1 of step k-1, one
    //       slot ago)
    //   C0  the MFMAs
    //   M1  read the second half; issue the loads of B for step k+2
    //   C1  the MFMAs
    // Waves 4-7 run one slot behind. Step k+1's tiles must have landed before
    // waves 0-3 enter its M0: waves 0-3 wait for their loads at the end of C1,
    // waves 4-7 at the end of M1 (the same slot); the loads of B for step k+2
    // stay in flight. The loads past the last step repeat its own (their lines
    // are in L2 and nobody reads the copies): every step then has the same loads
    // and waits, so that the compiler adds none of its own.
    auto step = [&](auto uc, int k, auto late) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      read(uc, 0);
      issue_a(std::integral_constant<int, u + 1>{}, min(k + 1, nk - 1) * BK);
      read_done();
      barrier();
      mfmas();
      barrier();
      read(uc, 1);
      issue_b(std::integral_constant<int, u + 2>{}, min(k + 2, nk - 1) * BK);
      read_done();
      if constexpr (decltype(late)::value) __builtin_amdgcn_s_waitcnt(waitcnt_vm(LOADS_B));
      barrier();
      mfmas();
      if constexpr (!decltype(late)::value) __builtin_amdgcn_s_waitcnt(waitcnt_vm(LOADS_B));
      barrier();
    };
    // all steps of one half of the waves (a loop of its own for each half),
    // unrolled so that every array is a compile-time choice
    auto steps = [&](auto late) __attribute__((always_inline)) {
      int k = 0;
      while (true) {
        step(Int<0>{}, k, late);
        if (++k == nk) break;
        step(Int<1>{}, k, late);
        if (++k == nk) break;
        step(Int<2>{}, k, late);
        if (++k == nk) break;
        step(Int<3>{}, k, late);
        if (++k == nk) break;
        step(Int<4>{}, k, late);
        if (++k == nk) break;
        step(Int<5>{}, k, late);
        if (++k == nk) break;
      }
    };
    issue_b(Int<0>{}, 0);
    issue_a(Int<0>{}, 0);
    if (nk <= 2) {
      // One or two steps, whose tiles all fit: every wave reads and multiplies as it
      // can. The loop's slots would mostly be spent alone here, and its loads past the
      // last step be more than the others (8190 x 64 -> 5120 30.3 us with the loop, 28.2 so).
      if (nk == 2) {
        issue_b(Int<1>{}, BK);
        issue_a(Int<1>{}, BK);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(LOADS));
      } else {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      }
      barrier();
      read(Int<0>{}, 0);
      mfmas();
      read(Int<0>{}, 1);
      mfmas();
      if (nk == 2) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        barrier();
        read(Int<1>{}, 0);
        mfmas();
        read(Int<1>{}, 1);
        mfmas();
      }
    } else {
      issue_b(Int<1>{}, BK);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(LOADS_B));
      barrier();
      if (__builtin_amdgcn_readfirstlane(wave) >= 4) {
        barrier();
        steps(std::true_type{});
      } else {
        steps(std::false_type{});
        barrier();
      }
    }
  } else {
    // Ring K loop: step k's stage has landed and everyone is done with step
    // k-1's, whose array takes the loads of step k+RING-1 (past the last step,
    // the last step's again).
    // With g.rms a wave also sums the squares of its A rows, 8 channels of
    // row l16 of each row tile per fragment (a launch of few tiles waits for its
    // chain of steps, not for these; a kernel of its own for them costs 4 us:
    // an iteration of three blocks, 500 rows at d = 256, 241 -> 220 us).
    auto squares = [&](int half) __attribute__((always_inline)) {
      if (!g.rms) return;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bf16x2 pair = {af[i][2 * u], af[i][2 * u + 1]};
          sq[i][half][u] = __builtin_amdgcn_fdot2_f32_bf16(pair, pair, sq[i][half][u], false);
        }
    };
    auto step = [&](auto uc, int k) __attribute__((always_inline)) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(LOADS * (RING - 2)));
      barrier();
      read(uc, 0);
      using Next = Int<decltype(uc)::value + RING - 1>;
      issue_a(Next{}, min(k + RING - 1, nk - 1) * BK);
      issue_b(Next{}, min(k + RING - 1, nk - 1) * BK);
      mfmas();
      squares(0);
      read(uc, 1);
      mfmas();
      squares(1);
      read_done();
    };
    static_for<0, RING - 1>([&](auto uc) {
      issue_a(uc, min(decltype(uc)::value, nk - 1) * BK);
      issue_b(uc, min(decltype(uc)::value, nk - 1) * BK);
    });
    int k = 0;
    while (true) {
      step(Int<0>{}, k);
      if (++k == nk) break;
      step(Int<1>{}, k);
      if (++k == nk) break;
      step(Int<2>{}, k);
      if (++k == nk) break;
      step(Int<3>{}, k);
      if (++k == nk) break;
    }
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // the repeated loads, before the epilogue takes the arrays

  // Epilogue through LDS. acc[i][j][e] is output row (tile row + i*16 + l16),
  // column (tile col + j*16 + grp*4 + e): a lane holds 4 columns
  // of one row, so direct stores would write 16-byte pieces of 32 rows per
  // instruction. Instead, for each 32-row block i, every wave writes its
  // fp32 values (row scale, RoPE and GELU applied) to its own LDS region,
  // then reads them back row-contiguous, 4 columns per lane (the residual is
  // added there, then the value rounded once), and stores runs of 4 columns
  // per lane, 128 bytes or more per row. Two or more waves share an
  // LDS array; the scatter target of each row travels through
  // LDS too. Every global load of the epilogue (row indices, row scales,
  // RoPE positions and angles, residuals) precedes its first store: the
  // results of all blocks are held in registers and stored after the last
  // one. A wave waits for a load by counting its outstanding memory
  // accesses, stores included, so a load behind a store would also wait for
  // that store (measured: the output projection 2-9% faster this way).
  // Each lane fills whole entries of the row tables (one lane of the 16-row tiles'
  // four for each row, every row tile by itself, took 63 VALU instructions more) and the
  // staging has no bank conflicts: 8190 x 64 -> 5120 28.2 -> 26.3 us, 8190 x 512 -> 5120
  // 52.0 -> 50.5.
  constexpr int QPR = TN / 4;         // 4-column groups per row
  constexpr int NT = QPR / 2;         // read-back passes of the wave per block
  constexpr int REGION = 32 * TN * 4 + TM * (8 + 4);
  constexpr int PER = TL::PING ? 2 : (TL::WAVES + RING - 1) / RING;  // waves per array
  static_assert(PER * REGION <= TL::ARRAY * 2 && PER * TL::ARRAYS >= TL::WAVES, "epilogue staging must fit");
  static_assert(QPR % 2 == 0, "the wave covers whole rows in each read-back pass");
  __syncthreads();  // every wave is done with the stages
  bf16* staging = lds.p[0];
#pragma unroll
  for (int i = 1; i < TL::ARRAYS; ++i)
    if (wave / PER == i) staging = lds.p[i];
  char* region = reinterpret_cast<char*>(staging) + (wave % PER) * REGION;
  f32x4* blk = reinterpret_cast<f32x4*>(region);
  // 4-column group q of row r sits at q ^ f(r): the writes (16 rows, 4 groups) and
  // the reads (whole rows) that are served together hit disjoint banks
  auto slot = [](int r, int q) { return r * QPR + (q ^ (QPR == 16 ? r & 15 : QPR == 8 ? (r >> 1) & 7 : r & 7)); };
  static_assert(QPR == 8 || QPR == 16 || QPR == 24, "staging rows of 32, 64 or 96 columns");
  // per block i, row r: output element offset and target (0: C, 1: C2, -1: none)
  long* row_off = reinterpret_cast<long*>(region + 32 * TN * 4);
  int* row_buf = reinterpret_cast<int*>(region + 32 * TN * 4 + TM * 8);
  const int32_t* c_rows = oz.c_rows;
  const bool rope = ROPE && g.rope_cs && ((g.rope_outs >> z) & 1);
  const int col0 = tn * BN + wn * TN;  // first output column of the wave tile
  const int m0 = tm * BM + wm * TM + l16;  // the lane's row in row tile 0
  constexpr int RT = (TM + 63) / 64;       // rows of the tables per lane
  int crow[RT];
  float rs[MI];
  RopeRow rr[MI];
  // Loads under a lane condition would each be waited for inside their
  // branch, one after the other: every load here and below reads a valid
  // address unconditionally (row M-1 for the rows past M) and its value is
  // selected afterwards.
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int m = tm * BM + wm * TM + t * 64 + lane;
    const int cr = c_rows ? c_rows[min(m, g.M - 1)] : m;
    crow[t] = m < g.M ? cr : -1;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int mc = min(m0 + i * 16, g.M - 1);
    rs[i] = g.row_scale ? g.row_scale[mc] : 1.f;
    if constexpr (!TL::PING) {
      if (g.rms) {
        float t = ((sq[i][0][0] + sq[i][0][1]) + (sq[i][0][2] + sq[i][0][3])) +
                  ((sq[i][1][0] + sq[i][1][1]) + (sq[i][1][2] + sq[i][1][3]));
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        rs[i] = 1.0f / sqrtf(t / (float)g.K + g.rms_eps);
      }
    }
    rr[i] = RopeRow{0, 0, 0};
    if (rope) rr[i] = rope_row(g, mc);
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    int buf = -1;
    long obase = 0;
    if (crow[t] >= 0 && crow[t] < oz.c_limit) {
      const bool second = oz.C2 && crow[t] >= oz.c_split;  // rows past the split go to C2
      buf = second ? 1 : 0;
      obase = (long)(second ? crow[t] - oz.c_split : crow[t]) * g.ldc;
    }
    if (TM % 64 == 0 || lane < TM) {
      row_off[t * 64 + lane] = obase;
      row_buf[t * 64 + lane] = buf;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the row tables are visible
  typedef typename std::conditional<EPI == kEpiF32, f32x4, bf16x4>::type OutT;
  OutT ov[RB][NT];  // block i, read-back pass t: the lane's 4 output values
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    if constexpr (EPI == kEpiBf16Residual) {  // the residual first takes the output's place
      __builtin_amdgcn_sched_barrier(0);  // one block's residuals at a time (registers)
      bool in[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int f = lane + 64 * t;
        const int r = f / QPR, cq = f - r * QPR;
        const int n = col0 + cq * 4;
        in[t] = row_buf[i * 32 + r] >= 0 && n < g.Nc;
        // element 0 of the residual exists: the launcher runs no residual
        // product without output rows
        ov[i][t] = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(g.residual) +
                                                    (in[t] ? row_off[i * 32 + r] + n : 0));
      }
      // an empty asm that uses every value keeps the loads unconditional (the
      // compiler would otherwise move each into a branch of its own)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        asm volatile("" : "+v"(ov[i][t]));
        if (!in[t]) ov[i][t] = (bf16x4){};
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int it = 2 * i + h;  // row tile
      // its RoPE angles, all loaded before any is used (every index is in the
      // table, so the loads need no condition)
      f32x2 cs[NI][2];
      if (rope) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int k = ((col0 + j * 16 + grp * 4) % g.rope_dh) >> 1;
          cs[j][0] = rope_angle(g, rr[it], k);
          cs[j][1] = rope_angle(g, rr[it], k + 1);
        }
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        f32x4 v = acc[it][j];
        if (g.row_scale || (!TL::PING && g.rms)) v *= rs[it];
        if (rope) {
          const f32x2 r0 = rope_rotate(cs[j][0], v[0], v[1]);
          const f32x2 r1 = rope_rotate(cs[j][1], v[2], v[3]);
          v = (f32x4){r0[0], r0[1], r1[0], r1[1]};
        }
        if constexpr (EPI == kEpiBf16Gelu) {
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = gelu_tanh(v[u]);
        }
        blk[slot(h * 16 + l16, j * 4 + grp)] = v;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // row-contiguous read-back: 4 columns per lane, QPR lanes per row
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int f = lane + 64 * t;
      const int r = f / QPR, cq = f - r * QPR;
      f32x4 v = blk[slot(r, cq)];
      if constexpr (EPI == kEpiF32) {
        ov[i][t] = v;
      } else {
        if constexpr (EPI == kEpiBf16Residual) v += __builtin_convertvector(ov[i][t], f32x4);
        ov[i][t] = to_bf16x4(v);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // reads done before the next block's writes
  }
  // the stores read their targets from the row tables again (a compiler-only
  // barrier): kept from the residual loads, 64-bit offsets would fill 64
  // registers and spill
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < RB; ++i) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int f = lane + 64 * t;
      const int r = f / QPR, cq = f - r * QPR;
      const int rb = row_buf[i * 32 + r];
      const int n = col0 + cq * 4;
      if (rb < 0 || n >= g.Nc) continue;
      const long o = row_off[i * 32 + r] + n;
      *reinterpret_cast<OutT*>(static_cast<typename std::conditional<EPI == kEpiF32, float, bf16>::type*>(
          rb ? oz.C2 : oz.C) + o) = ov[i][t];
    }
  }
}

// The tilings (see launch_best); a 256 x 256 tile splits into two 256 x 128
// halves.
using TBig = Tiling<256, 256, 64, 0, 8, 2>;
using T192 = Tiling<256, 192, 64, 0, 8, 4>;
using TMid = Tiling<256, 128, 64, 0, 8, 4>;
using T128 = Tiling<128, 128, 64, 4, 8, 2>;
using T64x128 = Tiling<64, 128, 64, 4, 8, 2>;
using T64 = Tiling<64, 64, 64, 4, 4, 2>;

// NOUT (1 or 3) is the number of outputs sharing A; it is a template
// parameter so the Q/K/V projection and the output projection are distinct
// kernels in profiles. Workgroup b takes tile item xcd_contiguous(b, tiles):
// tiles are ordered in groups of g.group_m tile-rows that sweep all tile-columns
// (of all outputs) together, and each XCD runs a contiguous range of items.
// With the 256 x 256 tiling, the workgroups from g.split_from on take halves:
// workgroups split_from + 2j and split_from + 2j + 1 compute the two 256 x 128
// halves of the tile workgroup split_from + j would have taken. The launcher
// sets split_from so that a last, partly filled round of big tiles becomes
// one round of halves.
template <class TL, int NOUT, int EPI, bool BUF>
__global__ __launch_bounds__(TL::THREADS) void row_gemm_bf16_kernel(RowGemm g) {
  constexpr bool kSplit = std::is_same<TL, TBig>::value;
  static_assert(!kSplit || TMid::THREADS == TL::THREADS, "halves");
  __shared__ __attribute__((aligned(16))) bf16 L0[TL::ARRAY], L1[TL::ARRAY], L2[TL::ARRAY], L3[TL::ARRAY],
      L4[TL::ARRAYS > 4 ? TL::ARRAY : 1];
  const LdsArrays lds{{L0, L1, L2, L3, L4}};

  const int tiles_m = (g.M + TL::BM - 1) / TL::BM;
  const int tiles_n1 = (g.Nc + TL::BN - 1) / TL::BN;  // per output
  const int tiles_n = tiles_n1 * NOUT;                 // over all outputs side by side
  const int total = tiles_m * tiles_n;
  int b = blockIdx.x, half = -1;
  if constexpr (kSplit) {
    if (b >= g.split_from) {
      half = (b - g.split_from) & 1;
      b = g.split_from + (b - g.split_from) / 2;
    }
  }
  const int item = xcd_contiguous(b, total);
  const int group = item / (g.group_m * tiles_n);
  const int first_m = group * g.group_m;
  const int gm = min(g.group_m, tiles_m - first_m);
  const int r = item - group * g.group_m * tiles_n;
  const int tm = first_m + r % gm;
  const int tnc = r / gm;
  const int z = tnc / tiles_n1;
  const int tn = tnc - z * tiles_n1;
  if constexpr (kSplit) {
    if (half >= 0) {
      row_gemm_tile<TMid, EPI, BUF, NOUT == 3>(g, tm, tn * 2 + half, z, lds);
      return;
    }
  }
  row_gemm_tile<TL, EPI, BUF, NOUT == 3>(g, tm, tn, z, lds);
}

// Cost of a launch: rounds x cost per round, in units of a full round of 256 x
// 256 tiles (waves of 128 x 64: the fastest per FLOP). The finer grids of the
// others fill the last round, or the only one, better. `full` is the cost of a
// round where all CUs work, `first` what the first round costs more than that:
// with few workgroups (or one round) each waits for its own loads and
// barriers, and small tiles lose more to that. Measured (us, K = 8960, one
// round of few workgroups): 131 (256 x 256), 108, 100, 58, 44, 39 (64 x 64);
// 8190 x 5120 x 5120, per full round: 112, 84, 70, 41, 29, and 32 for two
// workgroups of 64 x 64 per CU.
template <class TL>
struct Cost;
template <>
struct Cost<TBig> { static constexpr double full = 1.0, first = 0.0; static constexpr int per_cu = 1; };
template <>
struct Cost<T192> { static constexpr double full = 0.78, first = 0.04; static constexpr int per_cu = 1; };
template <>
struct Cost<TMid> { static constexpr double full = 0.64, first = 0.12; static constexpr int per_cu = 1; };
template <>
struct Cost<T128> { static constexpr double full = 0.38, first = 0.06; static constexpr int per_cu = 1; };
template <>
struct Cost<T64x128> { static constexpr double full = 0.26, first = 0.075; static constexpr int per_cu = 1; };
template <>
struct Cost<T64> { static constexpr double full = 0.30, first = 0.09; static constexpr int per_cu = 2; };

// With the 256 x 256 tiling, a last round at most half full is run as halves
// and costs a round of 256 x 128 tiles.
template <class TL>
bool split_tail(long tiles) {
  const long cus = compute_units(), rem = tiles % cus;
  return std::is_same<TL, TBig>::value && tiles > cus && rem > 0 && 2 * rem <= cus;
}
template <class TL>
double estimate(const RowGemm& g) {
  typedef Cost<TL> C;
  const long tiles = (long)((g.M + TL::BM - 1) / TL::BM) * ((g.Nc + TL::BN - 1) / TL::BN) * g.n_out;
  const long cus = compute_units(), slots = cus * C::per_cu;
  if (split_tail<TL>(tiles)) return (double)(tiles / cus) + Cost<TMid>::full;
  // a CU with one workgroup where two fit: measured as if the round were full,
  // without what the first costs more
  if (C::per_cu > 1 && tiles <= cus) return C::full;
  return (double)((tiles + slots - 1) / slots) * C::full + C::first;
}

// buffer resources address 4 GiB - 1 bytes from their base (32-bit offsets)
bool buffer_sized(const RowGemm& g) {
  const long lim = 0xffffffffL;
  return (long)g.a_limit * g.lda * 2 <= lim && (long)g.Nc * g.ldb * 2 <= lim;
}

template <class TL, int NOUT, int EPI>
hipError_t launch(const RowGemm& g0, hipStream_t s) {
  const long tiles = (long)((g0.M + TL::BM - 1) / TL::BM) * ((g0.Nc + TL::BN - 1) / TL::BN) * NOUT;
  RowGemm g = g0;
  // tile-row groups: 8, or 4 for outputs of 32 or more tile-columns (the FFN
  // up projection at 8960 columns: 7% faster at 32760 rows, neutral at 8190)
  g.group_m = (g0.Nc + TL::BN - 1) / TL::BN >= 32 ? 4 : 8;
  g.split_from = 0x7fffffff;
  long grid = tiles;
  if (split_tail<TL>(tiles)) {
    const long rem = tiles % compute_units();
    g.split_from = (int)(tiles - rem);
    grid = tiles + rem;
  }
  if constexpr (TL::PING) {
    if (!buffer_sized(g)) {
      hipLaunchKernelGGL((row_gemm_bf16_kernel<TL, NOUT, EPI, false>), dim3((unsigned)grid), dim3(TL::THREADS), 0, s, g);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((row_gemm_bf16_kernel<TL, NOUT, EPI, true>), dim3((unsigned)grid), dim3(TL::THREADS), 0, s, g);
  return hipGetLastError();
}

constexpr int kLargeTilings = 3;  // of the six, the first three run the ping-pong loop

// The tiling of least estimated cost; a smaller one must win by 2%. Matrices
// of 4 GiB or more take one of the large three (the others have no 64-bit
// loads: such a product has rows or columns for many large tiles).
int best_tiling(const RowGemm& g) {
  const double cost[] = {estimate<TBig>(g), estimate<T192>(g),    estimate<TMid>(g),
                         estimate<T128>(g), estimate<T64x128>(g), estimate<T64>(g)};
  int best = 0;
  const int n = buffer_sized(g) ? 6 : kLargeTilings;
  for (int i = 1; i < n; ++i)
    if (cost[i] < 0.98 * cost[best]) best = i;
  return best;
}

template <int NOUT, int EPI>
hipError_t launch_best(const RowGemm& g, hipStream_t s) {
  typedef hipError_t (*Launch)(const RowGemm&, hipStream_t);
  static constexpr Launch with[] = {launch<TBig, NOUT, EPI>, launch<T192, NOUT, EPI>,    launch<TMid, NOUT, EPI>,
                                    launch<T128, NOUT, EPI>, launch<T64x128, NOUT, EPI>, launch<T64, NOUT, EPI>};
  return with[best_tiling(g)](g, s);
}

}  // namespace

hipError_t launch_row_gemm_bf16(const RowGemm& g, hipStream_t s) {
  if (g.M <= 0 || g.Nc <= 0 || (g.n_out != 1 && g.n_out != 3)) return hipSuccess;
  if (g.K % TBig::BK) return hipErrorInvalidValue;
  if (g.rope_cs && g.rope_outs && g.n_out != 3) return hipErrorInvalidValue;  // RoPE: Q/K/V only
  if (g.residual && g.out[0].c_limit <= 0) return hipSuccess;  // no output row
  if (g.n_out == 3) return launch_best<3, kEpiBf16>(g, s);
  if (g.c_f32) return launch_best<1, kEpiF32>(g, s);
  if (g.gelu) return launch_best<1, kEpiBf16Gelu>(g, s);
  if (g.residual) return launch_best<1, kEpiBf16Residual>(g, s);
  return launch_best<1, kEpiBf16>(g, s);
}

hipError_t launch_rms_row_gemm_bf16(const RowGemm& g0, float eps, float* scale, hipStream_t s) {
  if (g0.M <= 0 || g0.Nc <= 0) return hipSuccess;
  RowGemm g = g0;
  if (best_tiling(g) >= kLargeTilings) {
    g.rms = 1;
    g.rms_eps = eps;
  } else {
    const hipError_t e = launch_row_rms_scale(g.A, true, g.M, g.K, eps, scale, s);
    if (e != hipSuccess) return e;
    g.row_scale = scale;
  }
  return launch_row_gemm_bf16(g, s);
}

}  // namespace hsa
