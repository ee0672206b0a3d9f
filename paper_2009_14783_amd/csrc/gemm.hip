// GEMM kernels: C[M,N] = sum_k A(m,k) B(n,k) with fused epilogues.
//   bf16: MFMA 32x32x16 tiles, fp32 accumulation, LDS double buffering.  Operands whose
//         contraction index is NOT the contiguous one are staged in their natural layout and read
//         with the LDS transpose read of gfx950, so every global and LDS access is 16/8 bytes wide.
//   fp32: gemm_f32.hip.
#include "gemm_dev.h"

#include <algorithm>
#include <atomic>
#include <vector>

hipError_t gemm_wide_launch_kk(int cfg, const GemmDev& p, int splits, hipStream_t s);
hipError_t gemm_wide_launch_kn(int cfg, const GemmDev& p, int splits, hipStream_t s);
hipError_t gemm_wide_launch_nn(int cfg, const GemmDev& p, int splits, hipStream_t s);
hipError_t gemm_group_launch_nn(int cfg, const GemmGroupDev& g, hipStream_t s);
void gemm_f32_launch(bool a_kmajor, bool b_kmajor, const GemmDev& p, hipStream_t s);
void gemm_f32_group_launch(int tile, const GemmGroupDev& g, hipStream_t s);

namespace {

template <bool KMAJ, int R, int BK, int NT>
struct OperandTile {
  // k-major rows are stored without padding and with their 16-byte chunks permuted: chunk j of row r sits
  // at position j ^ ((r / 4) % 4).  Sixteen rows read at one k-offset then fall into sixteen different
  // 16-byte bank groups, and so do the four 64-byte rows that sixteen lanes write at once.
  static_assert(!KMAJ || BK == 32, "the chunk permutation is written for four chunks per row");
  static constexpr int LD = KMAJ ? BK : (R + MPAD);
  static __device__ __forceinline__ int swz(int row, int chunk) { return (chunk ^ ((row >> 2) & 3)) * 8; }
  static constexpr int ELEMS = KMAJ ? R * LD : BK * LD;
  static constexpr int CPR = KMAJ ? BK / 8 : R / 8;       // 8-element chunks per stored row
  static constexpr int NCH = R * BK / 8 / NT;             // chunks per thread
  static_assert(R * BK / 8 % NT == 0, "tile must split evenly over the threads");

  // Per-thread state of the global side: one 32-bit byte offset per chunk from the start of the matrix
  // (advanced every k-tile; the matrix start is uniform, so a load needs one address register) and whether
  // the chunk's position along the non-contraction index is inside the matrix.
  struct Cursor {
    const char* base;     // start of the matrix: always readable, also the address of masked-out chunks
    unsigned off[NCH];
    unsigned step;        // bytes from one k-tile to the next
    int koff[NCH];        // contraction offset of the chunk inside a k-tile
    bool ok[NCH];
  };
  static __device__ __forceinline__ void init(Cursor& cu, const bf16* __restrict__ base, int64_t ld, int row0, int rext, int kbeg, int tid) {
    cu.base = (const char*)base;
    cu.step = (unsigned)(KMAJ ? (int64_t)BK * 2 : (int64_t)BK * ld * 2);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * NT;
      const int a = c / CPR, b = (c % CPR) * 8;
      if (KMAJ) { cu.ok[i] = row0 + a < rext; cu.koff[i] = b; cu.off[i] = (unsigned)(((int64_t)(row0 + a) * ld + kbeg + b) * 2); }
      else      { cu.ok[i] = row0 + b < rext; cu.koff[i] = a; cu.off[i] = (unsigned)(((int64_t)(kbeg + a) * ld + row0 + b) * 2); }
    }
  }
  // global -> registers for the k-tile that starts at k0, then advance.  The loads are unconditional
  // (no branch, so the hardware load counter can be waited on exactly): a chunk outside the matrix or
  // beyond kend reads the start of the matrix instead and is zeroed when it is written to LDS.
  static __device__ __forceinline__ void load(uint4 (&reg)[NCH], Cursor& cu, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const bool ok = cu.ok[i] && k0 + cu.koff[i] < kend;
      reg[i] = *(const uint4*)(cu.base + (ok ? cu.off[i] : 0u));
      cu.off[i] += cu.step;
    }
  }
  // registers -> LDS for the k-tile that started at k0 (chunks that were masked out become zeros)
  static __device__ __forceinline__ void store(const uint4 (&reg)[NCH], bf16* s, int tid, const Cursor& cu, int k0, int kend) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + i * NT;
      const int a = c / CPR, b = (c % CPR) * 8;
      // branch-free select: an all-ones or all-zeros word per chunk
      const unsigned keep = (cu.ok[i] && k0 + cu.koff[i] < kend) ? 0xffffffffu : 0u;
      uint4 v = reg[i];
      v.x &= keep; v.y &= keep; v.z &= keep; v.w &= keep;
      *(uint4*)(s + a * LD + (KMAJ ? swz(a, b >> 3) : b)) = v;
    }
  }
  // LDS -> MFMA operand: lane gets elements (row = rbase + lane%32, k = ks*16 + 8*(lane/32) + 0..7)
  static __device__ __forceinline__ bf16x8 frag(const bf16* s, int rbase, int ks, int lane) {
    if (KMAJ) {
      const int row = rbase + (lane & 31);
      return *(const bf16x8*)(s + row * LD + swz(row, ks * 2 + (lane >> 5)));
    } else {
      // Transpose read: within each group of 16 lanes, lane i receives, as element e, the (i%4)-th
      // 16-bit value of the 8 bytes addressed by lane 4*e + i/4 of the group.  With lane s of a
      // group pointing at row (kb + s/4), columns nb + 4*(s%4)..+3, lane i ends up with rows
      // kb..kb+3 of column nb + i.
      const int kb = ks * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
      const int nb = rbase + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      typedef s16x4 __attribute__((address_space(3))) * lds_v4;
      s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(s + kb * LD + nb));
      s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(s + (kb + 4) * LD + nb));
      union { struct { s16x4 lo, hi; } p; bf16x8 v; } u;
      u.p.lo = lo; u.p.hi = hi;
      return u.v;
    }
  }
};

// Block tile BM x BN x BK, WGM x WGN waves, each wave (BM/WGM) x (BN/WGN) as 32x32x16 MFMA tiles.
// A block's split index selects a contiguous range of k-tiles (split-K); with more than one split the raw fp32
// sums go to p.partial[z][M][N] and splitk_reduce_kernel applies the epilogue.
// waves per SIMD the register allocator should leave room for: accumulators take
// (BM/WGM)*(BN/WGN)/64 registers per lane out of 512
constexpr int gemm_occupancy(int bm, int bn, int wgm, int wgn) {
  const int acc = (bm / wgm) * (bn / wgn) / 64;
  return acc <= 64 ? 3 : (acc <= 128 ? 2 : 1);
}

// dynamic LDS of a block: the two pipeline stages of both operands, and at least the staging area of
// the epilogue (one 32-row slab of fp32 results per wave) when that is not much larger
template <bool AK, bool BKM, int BM, int BN, int BK, int WGM, int WGN>
constexpr size_t gemm_lds_bytes() {
  constexpr int NT = 64 * WGM * WGN;
  const size_t pipe = 2 * sizeof(bf16) * (size_t)(OperandTile<AK, BM, BK, NT>::ELEMS + OperandTile<BKM, BN, BK, NT>::ELEMS);
  const size_t stage = (size_t)WGM * WGN * 32 * (BN / WGN + 4) * sizeof(float);
  return (stage > pipe && stage <= pipe + pipe / 4) ? stage : pipe;
}

template <bool AK, bool BKM, int BM, int BN, int BK, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(gemm_occupancy(BM, BN, WGM, WGN), 8)))
void gemm_bf16_mfma(GemmDev p) {
  constexpr int NT = 64 * WGM * WGN;
  typedef OperandTile<AK, BM, BK, NT> TA;
  typedef OperandTile<BKM, BN, BK, NT> TB;
  constexpr int WM = BM / WGM, WN = BN / WGN, TI = WM / 32, TJ = WN / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  bf16* const sA0 = (bf16*)lds_raw;                       // two A buffers, then two B buffers
  bf16* const sB0 = (bf16*)lds_raw + 2 * TA::ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  // Tile order.  Workgroups are handed to the 8 XCDs round-robin by linear id, and each XCD has its own
  // L2: give every XCD a contiguous range of tiles, and walk the tiles in groups of 8 tile rows so that
  // the tiles in flight on one XCD share operand panels.
  // The same holds across the k-splits (blockIdx.z): an XCD then works on one or two splits
  // instead of all of them, and fetches only their share of the operands.  Blocks beyond the last
  // multiple of 8 keep their place.
  const int nbx = gridDim.x, nby = gridDim.y, nb = nbx * nby;
  int v = (blockIdx.z * nby + blockIdx.y) * nbx + blockIdx.x;
  const int per_xcd = (nb * (int)gridDim.z) >> 3;
  if (v < 8 * per_xcd) v = (v & 7) * per_xcd + (v >> 3);
  const int split = v / nb;
  const int b = v - split * nb;
  constexpr int GM = 8;
  const int group = b / (GM * nbx), first_m = group * GM;
  const int gm = min(GM, nby - first_m);
  const int in_group = b - group * GM * nbx;
  const int m0 = (first_m + in_group % gm) * BM, n0 = (in_group / gm) * BN;
  const int kbeg = split * p.k_per_split;
  const int kend = min(p.K, kbeg + p.k_per_split);

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  typename TA::Cursor ca;
  typename TB::Cursor cb;
  TA::init(ca, (const bf16*)p.A, p.lda, m0, p.M, kbeg, tid);
  TB::init(cb, (const bf16*)p.B, p.ldb, n0, p.N, kbeg, tid);
  // Software pipeline with a prefetch distance of two k-tiles: tile t is fetched from global memory
  // into register set t%2 during iteration t-2, moved to LDS buffer t%2 during iteration t-1 and
  // consumed during iteration t, so a global load has two iterations of MFMA work to hide behind.
  // The tile count is rounded up to even; a tile beyond the range loads nothing real and is all zeros.
  uint4 ra0[TA::NCH], rb0[TB::NCH], ra1[TA::NCH], rb1[TB::NCH];
  const int nk = ((kend - kbeg + BK - 1) / BK + 1) & ~1;
  TA::load(ra0, ca, kbeg, kend);
  TB::load(rb0, cb, kbeg, kend);
  TA::load(ra1, ca, kbeg + BK, kend);
  TB::load(rb1, cb, kbeg + BK, kend);
  TA::store(ra0, sA0, tid, ca, kbeg, kend);
  TB::store(rb0, sB0, tid, cb, kbeg, kend);
  __syncthreads();

  // One k-tile of work, in the order the hardware queues like it: all fragment reads of the tile, the
  // MFMAs of its first half, then the LDS writes of the next tile (they need the global loads issued one
  // iteration ago and complete behind the second half's MFMAs), then the second half.
  static_assert(BK == 32, "the main loop is written for two 16-deep MFMA steps per k-tile");
  bf16x8 fa[2][TI], fb[2][TJ];
  auto frags = [&](int cur) {
    const bf16* sAc = sA0 + cur * TA::ELEMS;
    const bf16* sBc = sB0 + cur * TB::ELEMS;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < TI; ++i) fa[ks][i] = TA::frag(sAc, wm * WM + i * 32, ks, lane);
#pragma unroll
      for (int j = 0; j < TJ; ++j) fb[ks][j] = TB::frag(sBc, wn * WN + j * 32, ks, lane);
    }
  };
  auto mfmas = [&](int ks) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
  };

  for (int kt = 0; kt < nk; kt += 2) {
    const int k0 = kbeg + kt * BK;
    // even tile kt: in LDS buffer 0; register set 0 is free, set 1 holds tile kt+1
    TA::load(ra0, ca, k0 + 2 * BK, kend);
    TB::load(rb0, cb, k0 + 2 * BK, kend);
    frags(0);
    mfmas(0);
    TA::store(ra1, sA0 + TA::ELEMS, tid, ca, k0 + BK, kend);
    TB::store(rb1, sB0 + TB::ELEMS, tid, cb, k0 + BK, kend);
    mfmas(1);
    __syncthreads();
    // odd tile kt+1: in LDS buffer 1; register set 1 is free, set 0 holds tile kt+2
    TA::load(ra1, ca, k0 + 3 * BK, kend);
    TB::load(rb1, cb, k0 + 3 * BK, kend);
    frags(1);
    mfmas(0);
    if (kt + 2 < nk) {
      TA::store(ra0, sA0, tid, ca, k0 + 2 * BK, kend);
      TB::store(rb0, sB0, tid, cb, k0 + 2 * BK, kend);
    }
    mfmas(1);
    __syncthreads();
  }

  // The epilogue is selected once per block.  When the staging area fits into the LDS the main loop
  // used, results go out through LDS in whole lines; otherwise straight from the registers.
  const int rbase = m0 + wm * WM, cbase = n0 + wn * WN;
  constexpr int STAGE_FLOATS = 32 * (WN + 4);
  constexpr bool kStage = (size_t)WGM * WGN * STAGE_FLOATS * sizeof(float) <= gemm_lds_bytes<AK, BKM, BM, BN, BK, WGM, WGN>();
  if constexpr (kStage) {
    float* stage = (float*)lds_raw + wave * STAGE_FLOATS;     // the last loop iteration ended with a barrier
    if (p.partial) tile_epilogue_lds<EPI_PARTIAL, TI, TJ>(p, acc, rbase, cbase, lane, split, stage);
    else if (p.c_f32) tile_epilogue_lds<EPI_F32, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
    else if (p.epi == 0) tile_epilogue_lds<EPI_ACT, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
    else if (p.epi == 1) tile_epilogue_lds<EPI_ACT_RES, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
    else if (p.epi == 2) tile_epilogue_lds<EPI_ACT_GELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
    else if (p.epi == 3) tile_epilogue_lds<EPI_ACT_DGELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
    else if (p.epi == 4) tile_epilogue_lds<EPI_ACT_RELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
    else tile_epilogue_lds<EPI_ACT_DRELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage);
  } else {
    if (p.partial) tile_epilogue<EPI_PARTIAL, TI, TJ>(p, acc, rbase, cbase, lane, split);
    else if (p.c_f32) tile_epilogue<EPI_F32, TI, TJ>(p, acc, rbase, cbase, lane, 0);
    else if (p.epi == 0) tile_epilogue<EPI_ACT, TI, TJ>(p, acc, rbase, cbase, lane, 0);
    else if (p.epi == 1) tile_epilogue<EPI_ACT_RES, TI, TJ>(p, acc, rbase, cbase, lane, 0);
    else if (p.epi == 2) tile_epilogue<EPI_ACT_GELU, TI, TJ>(p, acc, rbase, cbase, lane, 0);
    else if (p.epi == 3) tile_epilogue<EPI_ACT_DGELU, TI, TJ>(p, acc, rbase, cbase, lane, 0);
    else if (p.epi == 4) tile_epilogue<EPI_ACT_RELU, TI, TJ>(p, acc, rbase, cbase, lane, 0);
    else tile_epilogue<EPI_ACT_DRELU, TI, TJ>(p, acc, rbase, cbase, lane, 0);
  }
}

// sums the split-K partials in split order and applies the epilogue (four columns per thread)
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmDev p, int splits) {
  const int64_t mn = (int64_t)p.M * p.N;
  if ((p.N & 3) == 0) {
    const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (idx >= mn) return;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int z = 0; z < splits; ++z) {
      const float4 t = *(const float4*)(p.partial + z * mn + idx);
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    const int row = (int)(idx / p.N), col = (int)(idx % p.N);
    GemmDev q = p;
    q.partial = nullptr;
    if (p.c_f32) store_quad<EPI_F32>(q, row, col, s, quad_aligned<EPI_F32>(q), 0);
    else if (p.epi == 0) store_quad<EPI_ACT>(q, row, col, s, quad_aligned<EPI_ACT>(q), 0);
    else if (p.epi == 1) store_quad<EPI_ACT_RES>(q, row, col, s, quad_aligned<EPI_ACT_RES>(q), 0);
    else if (p.epi == 2) store_quad<EPI_ACT_GELU>(q, row, col, s, quad_aligned<EPI_ACT_GELU>(q), 0);
    else if (p.epi == 3) store_quad<EPI_ACT_DGELU>(q, row, col, s, quad_aligned<EPI_ACT_DGELU>(q), 0);
    else if (p.epi == 4) store_quad<EPI_ACT_RELU>(q, row, col, s, quad_aligned<EPI_ACT_RELU>(q), 0);
    else store_quad<EPI_ACT_DRELU>(q, row, col, s, quad_aligned<EPI_ACT_DRELU>(q), 0);
  } else {
    for (int t = 0; t < 4; ++t) {
      const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4 + t;
      if (idx >= mn) return;
      float s = 0.f;
      for (int z = 0; z < splits; ++z) s += p.partial[z * mn + idx];
      epilogue_store<bf16>(p, (int)(idx / p.N), (int)(idx % p.N), s);
    }
  }
}

}  // namespace

namespace {

template <bool AK, bool BKM, int BM, int BN, int BK, int WGM, int WGN>
hipError_t launch_one(const GemmDev& p, dim3 grid, hipStream_t s) {
  constexpr int NT = 64 * WGM * WGN;
  constexpr size_t lds = gemm_lds_bytes<AK, BKM, BM, BN, BK, WGM, WGN>();
  auto kern = gemm_bf16_mfma<AK, BKM, BM, BN, BK, WGM, WGN>;
  static bool configured = false;          // per instantiation; the attribute is per process and device-wide
  if (!configured && lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  configured = true;
  hipLaunchKernelGGL(kern, grid, dim3(NT), lds, s, p);
  return hipSuccess;
}

template <int BM, int BN, int BK, int WGM, int WGN>
hipError_t launch_cfg(const GemmArgs& g, const GemmDev& p, int splits, hipStream_t s) {
  dim3 grid((g.N + BN - 1) / BN, (g.M + BM - 1) / BM, splits);
  if (g.a_kmajor && g.b_kmajor) return launch_one<true, true, BM, BN, BK, WGM, WGN>(p, grid, s);
  if (g.a_kmajor) return launch_one<true, false, BM, BN, BK, WGM, WGN>(p, grid, s);
  return launch_one<false, false, BM, BN, BK, WGM, WGN>(p, grid, s);
}

// The two tables of gelu_tab_eval (the normal cdf, then GELU'), computed by the compiler: nothing has to be launched or waited for before
// the first product that reads them, which may be one that a graph captures.
// exp(-y) and the normal cdf for non-negative arguments, by series whose terms are all positive: exp(y) = sum y^n / n!,
// Phi(x) = 1/2 + exp(-x^2/2) / sqrt(2 pi) x sum x^(2n) / (1 3 ... (2n + 1)).
constexpr double series_exp_neg(double y) {
  double term = 1.0, sum = 1.0;
  for (int n = 1; term > 1e-18 * sum; ++n) { term *= y / n; sum += term; }
  return 1.0 / sum;
}
constexpr double series_cdf(double x, double pdf) {
  double term = x, sum = x;
  for (int n = 1; term > 1e-18 * sum; ++n) { term *= x * x / (2 * n + 1); sum += term; }
  return 0.5 + pdf * sum;
}
struct alignas(16) GeluTables { float2 entry[2][kGeluTabN]; };      // read 16 bytes at a time
constexpr GeluTables make_gelu_tables() {
  GeluTables t{};
  double node[2][kGeluTabN + 1] = {};
  for (int k = 0; k <= kGeluTabN / 2; ++k) {
    const double x = 2.0 * (double)kGeluTabR / kGeluTabN * k;
    const double pdf = 0.39894228040143267794 * series_exp_neg(0.5 * x * x), cdf = series_cdf(x, pdf);
    const int hi = kGeluTabN / 2 + k, lo = kGeluTabN / 2 - k;
    node[0][hi] = cdf; node[1][hi] = cdf + x * pdf;
    node[0][lo] = 1.0 - cdf; node[1][lo] = 1.0 - cdf - x * pdf;
  }
  for (int w = 0; w < 2; ++w)
    for (int k = 0; k < kGeluTabN; ++k) {
      t.entry[w][k].x = (float)node[w][k];
      t.entry[w][k].y = (float)(node[w][k + 1] - node[w][k]);
    }
  return t;
}
static __device__ GeluTables gelu_tables = make_gelu_tables();
// the address of a table on the current device
static hipError_t gelu_table(int which, const float2** out) {
  constexpr int kMaxDevices = 64;
  static std::atomic<const float2*> known[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const float2* p = dev < kMaxDevices ? known[dev].load(std::memory_order_relaxed) : nullptr;
  if (!p) {
    void* q = nullptr;
    e = hipGetSymbolAddress(&q, HIP_SYMBOL(gelu_tables));
    if (e != hipSuccess) return e;
    p = (const float2*)q;
    if (dev < kMaxDevices) known[dev].store(p, std::memory_order_relaxed);
  }
  *out = p + which * kGeluTabN;
  return hipSuccess;
}

// Tile configurations.  0: gemm_bf16_mfma (any shape, every epilogue).  5: gemm_bf16_wide (global -> registers -> LDS).  2: gemm_bf16_ksplit
// (the waves of a block share out the contraction).  The others: gemm_bf16_dma (global -> LDS).  What a launch takes is modelled as
//   t0 + k-tiles x (rounds of full CUs x occ w + the last round of r blocks per CU x max(l, r w)) + e x tiles per CU x outputs
// with l the time of a k-tile of 64 when a block has its CU to itself (a chain of load, LDS read and matrix instruction
// latencies), w what it adds to a CU whose blocks cover each other (throughput of the feed from the L2), and e the writing
// of a tile.  The constants (us) are fitted to launches on this chip: rows 264 .. 17472, the forward and activation-gradient products of
// widths 512, 768 and 1024 with their epilogues, weights not in the cache of the launch before (2, 4 and 11, whose launches are shorter than
// the host takes to enqueue them, to a fit over 32 .. 4104 rows, and their t0 raised together until the translation step at 4096 rows per side and BERT-base at 264
// rows agreed).  Over 168 products of 264 to 16384 rows the choice is 1.7 % above the fastest tiling on average and 15 % in the worst case (16384 x 1536 x
// 512), over 408 of up to 17472 rows in another run, with another card and other buffers, 1.1 % and 12 %.  l of 3 and 6 is the one of a nearly full chip:
// 8192 x 768 x 3072 takes 59.6 us as 256 blocks of 128 x 192 and 51.5 as 192 of 256 x 128.  `use`: the automatic choice considers the
// configuration; the others can be selected for timing (8 is the mirror image of 7 and seldom faster).
// w and e of 11 come from launches of two to eight of its tiles per CU over contractions of up to 1024, whose blocks write under each other's
// products (as 0.183 and 0.43 they priced it 10 - 20 % too high there; us by itself, that choice -> 64 x 64 tiles: 2056 x 2048 x 512 GELU 16.2 -> 14.0, 8736 x 512 x 512
// residual 14.2 -> 12.3, 2056 x 1024 x 1024 residual 13.2 -> 12.2, 3072 x 1536 x 512 12.9 -> 12.2; the steps that hold them level or up to 0.9 % faster).  A t0 of 2.9 instead of 3.5 would
// make products of 264 and 320 rows 5 - 8 % faster by themselves, and the translation step slower that holds them beside others (256 rows per side 2.12 -> 2.15 ms, 1024 2.56 -> 2.60).
// What the tiles of more than 128 x 128 brought, us (128 x 128 before; rows x columns x contraction, epilogue): 16384 x 4096 x 1024 GELU 201 -> 163, x 1024 x 4096
// residual 148 -> 122, x 3072 x 1024 124 -> 107; 8192 x 3072 x 768 GELU 71 -> 58, x 768 x 3072 residual 56 -> 50, x 768 x 2304 45 -> 39;
// 8192^3 1044 -> 1339 TFLOP/s.
struct TileCfg { int bm, bn, bk, occ, use; float t0, l, w, e; };
constexpr TileCfg kTileCfg[] = {
    {128, 128, 32, 3, 0, 3.2f, 0.560f, 0.470f, 2.00f}, {256, 256, 64, 1, 1, 2.5f, 1.494f, 1.494f, 6.14f}, {32, 32, 64, 1, 1, 2.5f, 0.011f, 0.104f, 0.90f},
    {128, 192, 64, 2, 1, 2.5f, 1.050f, 0.693f, 2.36f}, {32, 64, 64, 3, 1, 4.0f, 0.146f, 0.120f, 0.33f},   {128, 128, 64, 2, 1, 3.2f, 0.497f, 0.487f, 1.82f},
    {192, 128, 64, 2, 1, 2.5f, 1.050f, 0.705f, 2.00f}, {64, 128, 64, 2, 1, 2.7f, 0.190f, 0.296f, 1.24f},  {128, 64, 64, 2, 0, 2.7f, 0.228f, 0.305f, 1.19f},
    {128, 128, 64, 2, 1, 2.5f, 0.689f, 0.490f, 1.85f}, {256, 128, 64, 1, 1, 2.5f, 0.814f, 0.814f, 3.92f}, {64, 64, 64, 3, 1, 3.5f, 0.229f, 0.187f, 0.30f},
    {128, 128, 64, 1, 1, 1.4f, 0.482f, 0.390f, 2.42f}, {64, 64, 64, 2, 1, 3.6f, 0.196f, 0.197f, 0.46f}};
constexpr int kNumTileCfg = sizeof(kTileCfg) / sizeof(kTileCfg[0]);
constexpr int kCUs = 256;
float tiles_time(const TileCfg& c, int64_t tiles, float steps, float outputs) {
  const int per_cu = (int)((tiles + kCUs - 1) / kCUs), full = per_cu / c.occ, rem = per_cu % c.occ;
  return c.t0 + steps * (full * std::max(c.l, c.occ * c.w) + (rem ? std::max(c.l, rem * c.w) : 0.0f)) + c.e * per_cu * outputs;
}
int gemm_cfg_override = -1;    // >= 0: use this configuration for every bf16 product of some size that it can serve (timing runs)

constexpr int kMaxBK = 64;

}  // namespace

static hs_status check_gemm_args(hs_ctx* ctx, const GemmArgs& g) {
  if (g.K < 0) return hs_fail(ctx, HS_ERR_INVALID_ARG, "gemm: K < 0");
  if (!g.A || !g.B || !g.C) return hs_fail(ctx, HS_ERR_INVALID_ARG, "gemm: NULL operand");
  if ((g.epi == 1 || g.epi == 3 || g.epi == 5) && !g.aux) return hs_fail(ctx, HS_ERR_INVALID_ARG, "gemm: epilogue needs aux");
  if (g.epi == 2 && (!g.C2 || g.c_f32)) return hs_fail(ctx, HS_ERR_INVALID_ARG, "gemm: GELU epilogue needs C2 and an activation-type C");
  if (g.epi < 0 || g.epi > 5) return hs_fail(ctx, HS_ERR_INVALID_ARG, "gemm: bad epilogue");
  if (g.dtype == HS_BF16) {
    if ((g.lda % 8) || (g.ldb % 8) || ((uintptr_t)g.A % 16) || ((uintptr_t)g.B % 16))
      return hs_fail(ctx, HS_ERR_SHAPE, "gemm(bf16): operand rows must be 16-byte aligned");
    if (g.a_kmajor && g.b_kmajor && (g.K % 8))
      return hs_fail(ctx, HS_ERR_SHAPE, "gemm(bf16): K must be a multiple of 8 when both operands are k-major");
    if (!g.a_kmajor && g.b_kmajor) return hs_fail(ctx, HS_ERR_UNIMPLEMENTED, "gemm(bf16): A m-major with B k-major is not built");
    // the kernels address each operand with 32-bit byte offsets from its start (a few k-tiles of slack)
    const int64_t a_rows = g.a_kmajor ? g.M : g.K, b_rows = g.b_kmajor ? g.N : g.K;
    const int64_t lim = ((int64_t)1 << 32) - 1;
    if ((a_rows + 3 * kMaxBK) * g.lda * 2 + 4 * kMaxBK > lim || (b_rows + 3 * kMaxBK) * g.ldb * 2 + 4 * kMaxBK > lim)
      return hs_fail(ctx, HS_ERR_SHAPE, "gemm(bf16): an operand exceeds 4 GiB");
  }
  return HS_OK;
}

static GemmDev gemm_dev_args(const GemmArgs& g) {
  GemmDev p;
  p.A = g.A; p.B = g.B; p.C = g.C; p.C2 = g.C2; p.bias = g.bias; p.aux = g.aux;
  p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc; p.ldaux = g.ldaux;
  p.M = g.M; p.N = g.N; p.K = g.K; p.c_f32 = g.c_f32; p.epi = g.epi; p.beta = g.beta;
  p.partial = nullptr; p.k_per_split = g.K; p.gelu_tab = nullptr;
  p.drop = (g.drop && g.drop->thr && g.epi == 1) ? *g.drop : DropCfg{0u, 1.0f, 0u, 0u, 0u};
  p.drop_site = g.drop_site;
  p.drop_rows = g.drop_rows;
  p.rowsum = nullptr;
  return p;
}

int gemm_variant_count() { return 12; }      // 12 and 13 are left to the automatic choice (gemm_choice says where it takes them)
void gemm_set_variant(int variant) { gemm_cfg_override = variant; }

// whether the kernels other than gemm_bf16_mfma are built with the epilogue this product needs (see wide_epilogues in gemm_wide.h)
static bool wide_supports(const GemmArgs& g) {
  if (g.a_kmajor && g.b_kmajor) return g.c_f32 ? true : (g.epi == 0 || g.epi == 1 || g.epi == 2 || g.epi == 4);
  if (g.a_kmajor) return !g.c_f32 && (g.epi == 0 || g.epi == 1 || g.epi == 3 || g.epi == 5);
  return g.c_f32 != 0;
}

// Configuration and number of k-splits of a product: the fastest by the model above among those that can serve it.
// Configuration 0 where an epilogue is needed that the others are not built with; where rows of a k-major operand end
// inside a k-tile, 0 or (from 256 rows, columns and contraction steps on, where it is faster) 5.
static void choose_cfg(const GemmArgs& g, int* cfg, int* splits) {
  const bool supported = wide_supports(g), whole_k = !g.a_kmajor || g.K % 64 == 0 || g.a_kpad;
  const bool some_size = g.M >= 256 && g.N >= 256 && g.K >= 256;
  int only = -1;
  if (!supported) only = 0;
  else if (gemm_cfg_override >= 0) only = some_size ? gemm_cfg_override : 0;
  // a few k-tiles per tile and several tiles per CU: three blocks per CU hide the writing better than what the model would take (8192 x 3072 x 128:
  // 21.0 against 22.5 us, 16384 x 1536 x 64: 17.2, 18.7, 8736 x 2304 x 192: 20.5, 22.5, 30522 x 768 x 64: 18.4, 18.7; with a residual the two are level, with
  // an fp32 result the others win)
  if (only < 0 && g.a_kmajor && g.b_kmajor && g.epi == 0 && !g.c_f32 && g.K < 256 && (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128) > kCUs) only = 0;
  if (supported && !whole_k && only != 0) only = some_size ? 5 : 0;
  const bool gate = g.epi == 5;      // not in the register-staged kernels
  if (gate && (only == 5)) only = 0;
  const float outputs = (g.c_f32 || g.epi) ? 2.0f : 1.0f;
  const bool forward = g.a_kmajor && g.b_kmajor;
  float best = 3.0e38f;
  *cfg = 0; *splits = 1;
  for (int c = 0; c < kNumTileCfg; ++c) {
    if (only >= 0 ? c != only : !kTileCfg[c].use) continue;
    // 12 and 13 are for long contractions of a product that has the chip: with 12 k-tiles their shorter k-tile does not pay for the ring that has to be filled (as the model
    // prices them they would be taken there too; BERT-base 64 x 128 7.25 -> 7.33 ms per step), and a block that needs a CU's whole LDS keeps the other
    // half of a forward batch off it (K = 3072 in the halves of 64 x 128: 7.14 -> 7.19).  Their constants were fitted to the choice that comes out: over
    // 8 products, three widths and 24 row counts from 264 to 17472 2 % faster, 4 % from 776 to 5200 rows.  Two updates of BERT-base with 32 sequences of 64 to
    // 128 positions 9.03 -> 8.71 ms.  Not with an m-major A: both operands then go through the transposing reads, which those constants do not know, and the
    // products that are not grouped have many tiles per CU (37000 x 512 x 3135 with 12: 166 us, without 140; x 4096 206, 184).
    if (only < 0 && c >= 12 && (g.K < 1536 || g.beside || !g.a_kmajor)) continue;
    // With a scratch buffer the contraction can be split over blocks: partial sums go out as fp32 and are added by a second
    // launch (3 us and their way through memory and back at 3.5 TB/s; for contractions beyond 8192, 5 us at the 10 TB/s that the sums get
    // on their way through the caches: 768 x 768 x 32768, both operands k-major, 81 -> 70 us; 3072 x 768 x 16384 152 -> 111).
    const int64_t most = g.ws ? std::min<int64_t>({32, g.K / (4 * kTileCfg[c].bk), (int64_t)(g.ws_bytes / ((size_t)g.M * g.N * sizeof(float)))}) : 1;
    const int64_t tiles = (int64_t)((g.M + kTileCfg[c].bm - 1) / kTileCfg[c].bm) * ((g.N + kTileCfg[c].bn - 1) / kTileCfg[c].bn);
    for (int sp = 1; sp <= std::max<int64_t>(1, most); sp *= 2) {
      // 5 and 9 are the same tile.  The register-staged pipeline (5) has four k-tiles in flight, the direct one (9) two: a block that has
      // its CU to itself is faster with the first from about 16 whole k-tiles on (us, 5 against 9; A m-major, 3072 x 768 x 8192: 73, 99, at K = 1216 16.9, 18.2;
      // 4096 x 1024 x 4096, A k-major: 38.7, 44.7, both k-major 38.3, 43.8), two blocks that cover each other with the second
      // (30522 x 768 x 1232, A m-major: 111, 88; activation gradients of contractions up to 1024 3 % on average over 60 products), and so is any block whose contraction
      // ends inside a k-tile (3072 x 768 x 520: 15.3, 12.0).  Of split contractions beyond 8192 the second with twice the splits
      // is (1216 x 768 x 32768: 85, 77).  Forward products take the first: with one tile per CU it is 8 - 20 % faster by itself, with more the second is 3 %
      // (contractions up to 1024, 96 products) or the first is (longer ones), and twelve training steps of 3 to 20 ms were level to 0.3 % with either.
      const bool lone = !gate && tiles * sp <= kCUs && g.K > 1024 && g.K % 64 == 0 && (sp == 1 || g.K <= 8192);
      if (only < 0 && (c == 5 || c == 9) && c != (forward || lone ? 5 : 9)) continue;
      float steps = (float)((g.K + 63) / 64) / sp;
      // rows that end inside a k-tile do not start on cache lines either: half as much again per k-tile (768 x 768 x 2008: 0.7 us)
      if (!whole_k) steps *= 1.5f;
      // Many k-tiles in a row cost more each: blocks that share operand panels drift apart and fetch them again (3072 x 768 with one tile
      // per CU: 0.46 us per k-tile at K = 8192, 0.58 at 16384).  Not for the products over a padded vocabulary: the fit has
      // them as they run in the step, beside the embedding gradient (split as if alone, they made it 0.4 % slower).
      const bool alone = !g.a_kpad;
      if (alone) steps *= 1.0f + std::max(0.0f, steps - 128.0f) / 512.0f;
      float t = tiles_time(kTileCfg[c], tiles * sp, steps, sp > 1 ? 2.0f : outputs);
      const float mbytes = 8e-6f * sp * (float)g.M * (float)g.N;
      if (sp > 1) t += alone && g.K > 8192 ? 5.0f + mbytes / 10.0f : 3.0f + mbytes / 3.5f;
      if (t < best) { best = t; *cfg = c; *splits = sp; }
    }
  }
}

void gemm_choice(const GemmArgs& g, int* variant, int* splits) { choose_cfg(g, variant, splits); }

// Weight-gradient products (A m-major, B n-major or null for a column of ones, fp32 C = beta C + product, one type and beta for all) in as
// few launches of the grouped kernel as their number allows: no split-K, no partial sums in memory, one ramp-up and one tail.
hs_status launch_gemm_group(hs_ctx* ctx, const GemmArgs* gs, int n, hipStream_t s) {
  std::vector<GroupProb> probs;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = gs[i];
    if (g.a_kmajor || g.b_kmajor || !g.c_f32 || g.bias || g.epi || g.drop || g.dtype != gs[0].dtype || g.beta != gs[0].beta ||
        std::max({g.lda, g.ldb, g.ldc}) > INT32_MAX)
      return hs_fail(ctx, HS_ERR_INVALID_ARG, "grouped gemm: only m-major x n-major products with fp32 results and one type and beta");
    GemmArgs chk = g;
    if (!g.B) { chk.B = g.A; chk.ldb = 8; chk.N = 1; }
    hs_status st = check_gemm_args(ctx, chk);
    if (st != HS_OK) return st;
    if (g.B || g.dtype == HS_FP32) probs.push_back(GroupProb{g.A, g.B, (float*)g.C, nullptr, (int)g.lda, (int)g.ldb, (int)g.ldc, g.M, g.N, g.K});
  }
  for (int i = 0; i < n && gs[0].dtype != HS_FP32; ++i) {      // bf16 bias gradients: beside the weight gradient of the same operand
    const GemmArgs& g = gs[i];
    if (g.B) continue;
    GroupProb* with = nullptr;
    for (GroupProb& q : probs)
      if (q.A == g.A && q.lda == g.lda && q.M == g.M && q.K == g.K && !q.rowsum) { with = &q; break; }
    if (!with || g.ldc != 1) return hs_fail(ctx, HS_ERR_INVALID_ARG, "grouped gemm: a bias gradient without the weight gradient of the same operand");
    with->rowsum = (float*)g.C;      // (as products with a column of ones they were 10 % of the tiles of a BERT-base layer)
  }
  n = (int)probs.size();
  for (int done = 0; done < n;) {
    GemmGroupDev gd;
    gd.n = std::min(n - done, kGroupMax);
    gd.beta = gs[0].beta;
    const bool f32 = gs[0].dtype == HS_FP32;
    double flops = 0, bytes = 0;
    for (int i = 0; i < gd.n; ++i) {
      const GroupProb& q = gd.prob[i] = probs[done + i];
      flops += 2.0 * q.M * (q.N + (q.rowsum ? 1 : 0)) * (double)q.K;
      bytes += ((double)q.M * q.K + (double)q.N * q.K) * esize(gs[0].dtype) + (double)q.M * q.N * 4;
    }
    auto count = [&](int bm, int bn) {      // fills first_tile, returns the number of tiles
      int tiles = 0;
      for (int i = 0; i < gd.n; ++i) {
        gd.first_tile[i] = tiles;
        tiles += ((gd.prob[i].M + bm - 1) / bm) * ((gd.prob[i].N + bn - 1) / bn);
      }
      return gd.first_tile[gd.n] = tiles;
    };
    int cfg = 9;
    if (f32) {
      // Decided by the mean over the products, not by their sum: the two tilings add in different orders, and the same layers have
      // to give the same bits however many of them go out together.  24 each are 144 for the six products of an encoder layer,
      // where the tilings are within an eighth of each other (see gemm_f32_tile).
      cfg = count(128, 128) >= 24 * gd.n ? 128 : 32;
      count(cfg, cfg);
    } else {
      // The tile by the constants of the time model, over the tiles of all problems.  The launch runs beside the chain of activation
      // gradients, so what counts is the time of the CUs that it takes and not how evenly its last round fills them: rounds are not
      // rounded up, and tiles for half of the CUs are as good as tiles for all of them (fewer would last too long behind the last layer).  Ms per
      // step if all CUs have to be filled -> half of them: BERT-large with 16384 rows 153.3 -> 148.8 (256 x 256 tiles on 192 CUs, and the chain on
      // the others: 480 us against 530, its LayerNorm backward 27 against 54), two updates of 4096 rows 10.7 -> 10.2 (256 x 128), the
      // translation step with 4096 rows per side 4.56 -> 4.47 and 4.74 -> 4.67 (256 x 256); a quarter of them: BERT-base with 8192 rows 7.52 -> 7.69.
      // Over 30 steps of other sizes (264 to 12288 rows; translation, BERT-base, BERT-large) all CUs are level or up to 3 % slower than half (BERT-large 12 x 512 17.39 -> 17.87,
      // BERT-base 33 x 128 4.97 -> 5.06, translation 31 x 256 6.51 -> 6.69), a quarter is 1.1 % faster to 2.6 % slower (BERT-base 16 x 128 3.70 -> 3.66, 33 x 128 4.97 -> 5.10).
      float best = 3.0e38f;
      for (int c : {1, 9, 10, 11}) {
        TileCfg t = kTileCfg[c];
        // the grouped 64 x 64 kernel is another one than 11 (it reads fragments ahead) and has its own w and e: with those of 11 passes of up to 64
        // rows take it instead of 256 x 256 tiles (one row of them) and are slower (32 rows: BERT-base 2.126 -> 2.150 ms per step, BERT-large with 64 5.21 -> 5.32)
        if (c == 11) { t.w = 0.183f; t.e = 0.43f; }
        const int tiles = count(t.bm, t.bn);
        float steps = 0.0f;
        for (int i = 0; i < gd.n; ++i) steps += (float)(gd.first_tile[i + 1] - gd.first_tile[i]) * ((gd.prob[i].K + 63) / 64);
        const float per_tile = (tiles ? steps / tiles : 0.0f) * std::max(t.l / t.occ, t.w) + t.e * 2.0f;
        const float time = t.t0 + per_tile * std::max(0.5f, (float)tiles / kCUs);
        if (time < best) { best = time; cfg = c; }
      }
      count(kTileCfg[cfg].bm, kTileCfg[cfg].bn);
    }
    if (gd.first_tile[gd.n] > 0) {
      KScope scope(ctx ? ctx->prof : nullptr, KC_GEMM_DW, flops, bytes, s);
      hipError_t e = hipSuccess;
      if (f32) gemm_f32_group_launch(cfg, gd, s);
      else e = gemm_group_launch_nn(cfg, gd, s);
      if (e == hipSuccess) e = hipGetLastError();
      if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("grouped gemm launch: ") + hipGetErrorString(e));
    }
    done += gd.n;
  }
  return HS_OK;
}

hs_status launch_gemm(hs_ctx* ctx, const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return HS_OK;  // nothing to write
  {
    hs_status st = check_gemm_args(ctx, g);
    if (st != HS_OK) return st;
  }
  GemmDev p = gemm_dev_args(g);
  const double flops = 2.0 * g.M * g.N * (double)g.K;
  const double bytes = ((double)g.M * g.K + (double)g.N * g.K) * esize(g.dtype) + (double)g.M * g.N * (g.c_f32 ? 4 : esize(g.dtype));
  const int kc = (g.a_kmajor && g.b_kmajor) ? KC_GEMM_FWD : (g.a_kmajor ? KC_GEMM_DX : KC_GEMM_DW);
  KScope scope(ctx ? ctx->prof : nullptr, kc, flops, bytes, s);
  if (g.dtype == HS_FP32) {
    gemm_f32_launch(g.a_kmajor, g.b_kmajor, p, s);
  } else {
    int cfg, splits;
    choose_cfg(g, &cfg, &splits);
    if (splits > 1) {
      const int kBK = kTileCfg[cfg].bk;
      p.partial = (float*)g.ws;
      p.k_per_split = (int)(((g.K + splits - 1) / splits + kBK - 1) / kBK * kBK);
      splits = (g.K + p.k_per_split - 1) / p.k_per_split;
    }
    hipError_t e;
    if (cfg != 0 && (g.epi == 2 || g.epi == 3)) {
      e = gelu_table(g.epi == 2 ? 0 : 1, &p.gelu_tab);
      if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("gemm: GELU table: ") + hipGetErrorString(e));
    }
    if (cfg == 0) e = launch_cfg<128, 128, 32, 2, 2>(g, p, splits, s);
    else if (g.a_kmajor && g.b_kmajor) e = gemm_wide_launch_kk(cfg, p, splits, s);
    else if (g.a_kmajor) e = gemm_wide_launch_kn(cfg, p, splits, s);
    else e = gemm_wide_launch_nn(cfg, p, splits, s);
    if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("gemm launch: ") + hipGetErrorString(e));
    if (splits > 1) {
      const int64_t mn = (int64_t)g.M * g.N;
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((mn + 1023) / 1024)), dim3(256), 0, s, p, splits);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("gemm launch: ") + hipGetErrorString(e));
  return HS_OK;
}
