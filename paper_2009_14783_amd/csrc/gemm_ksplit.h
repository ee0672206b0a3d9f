// bf16 MFMA GEMM kernel for products with few output tiles: the waves of a block split the contraction (template).
#pragma once
#include "gemm_dma.h"

namespace {

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel with the contraction split over the waves
// ------------------------------------------------------------------------------------------
// For products so small that a CU gets one tile at most: what counts there is the chain of latencies through the contraction
// (a k-tile of the shared-ring kernel is load wait, barrier, LDS reads, dependent matrix instructions: 0.25 us for 64 x 64,
// 0.13 us for 32 x 32, whatever the depth of the ring), not any throughput.  Every wave of the block computes the whole
// (32 TI) x (32 TJ) tile over the k-tiles w, w + NW, ..., each with a ring of S k-tiles of its own in LDS that it fills with
// direct loads: no barrier until the end, and NW chains run beside each other.  The waves' fp32 tiles then meet in LDS and are
// added in wave order by all threads, eight columns each, on their way through the epilogue.
// 264 x 768 x 3072 (forward, residual epilogue): 7.8 us; 128 x 128 tiles 24.5, 64 x 64 with a shared ring 14.0, 32 x 32 with a
// shared ring 8.6.  264 x 768 x 768: 4.0 us; 10.6, 5.7 and 4.6.
template <int TI_, int TJ_, int NW_, int BK_, int S_, int OCC_>
struct KsCfg {
  static constexpr int TI = TI_, TJ = TJ_, NW = NW_, BK = BK_, S = S_, OCC = OCC_;
  static constexpr int NT = 64 * NW, BM = 32 * TI, BN = 32 * TJ;
  static constexpr int STAGE = (BM + BN) * BK * 2, RING = S * STAGE;    // bytes: one k-tile of both operands; a wave's ring
  static constexpr int LDW = BN + 4;                                    // row stride of the fp32 tiles of the epilogue
  static constexpr size_t EPI_BYTES = (size_t)NW * BM * LDW * sizeof(float);
  static constexpr size_t LDS = (size_t)NW * RING > EPI_BYTES ? (size_t)NW * RING : EPI_BYTES;
  static constexpr int OCTS = BM * BN / 8, NOCT = (OCTS + NT - 1) / NT;   // 8-column pieces of the result, per thread
  static_assert(LDS * OCC <= 160 * 1024, "rings do not fit the LDS of a CU");
};

template <class C, bool AK, bool BKM, int EPIS>
__device__ __forceinline__ void ks_tile(const GemmDev& p, int m0, int n0, int split, unsigned char* lds_raw) {
  constexpr int TI = C::TI, TJ = C::TJ, S = C::S, NW = C::NW, KS = C::BK / 16;
  typedef DmaTile<AK, C::BK, C::BM, 1> TA;
  typedef DmaTile<BKM, C::BK, C::BN, 1> TB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kbeg = split * p.k_per_split + wave * C::BK;
  const int kend = min(p.K, (split + 1) * p.k_per_split);
  const int nk = kend > kbeg ? (kend - kbeg + NW * C::BK - 1) / (NW * C::BK) : 0;      // this wave's k-tiles
  unsigned char* const ring = lds_raw + wave * C::RING;

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  typename TA::Cursor ca;
  typename TB::Cursor cb;
  TA::init(ca, (const bf16*)p.A, p.lda, m0, p.M, kbeg, p.K, lane, 0);
  TB::init(cb, (const bf16*)p.B, p.ldb, n0, p.N, kbeg, p.K, lane, 0);
  ca.step *= NW; cb.step *= NW;
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nk) { TA::issue(ca, ring + s * C::STAGE, 0); TB::issue(cb, ring + s * C::STAGE + TA::BYTES, 0); }
  for (int t0 = 0; t0 < nk; t0 += S) {
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int t = t0 + u;
      if (t < nk) {
        asm volatile("" ::: "memory");
        wait_tiles<TA::NI + TB::NI, S - 2>(min(S - 2, nk - 1 - t));
        asm volatile("" ::: "memory");
        if (t + S - 1 < nk) {
          unsigned char* const nxt = ring + ((u + S - 1) % S) * C::STAGE;
          TA::issue(ca, nxt, 0);
          TB::issue(cb, nxt + TA::BYTES, 0);
        }
        const bf16* sA = (const bf16*)(ring + u * C::STAGE);
        const bf16* sB = (const bf16*)(ring + u * C::STAGE + TA::BYTES);
        bf16x8 fa[KS][TI], fb[KS][TJ];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
          for (int i = 0; i < TI; ++i) fa[ks][i] = TA::frag(sA, i * 32, ks, lane);
#pragma unroll
          for (int j = 0; j < TJ; ++j) fb[ks][j] = TB::frag(sB, j * 32, ks, lane);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
      }
    }
  }
  asm volatile("" ::: "memory");
  wait_loads<0>();
  __syncthreads();               // the rings become the waves' fp32 tiles
  float* const mine = (float*)lds_raw + wave * C::BM * C::LDW;
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) mine[(i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * C::LDW + j * 32 + (lane & 31)] = acc[i][j][r];
  __syncthreads();
  constexpr auto has = [](int mode) { return (EPIS >> mode) & 1; };
  auto finish = [&](auto mode_tag) __attribute__((always_inline)) {
    constexpr int MODE = decltype(mode_tag)::value;
    const bool vec = octet_aligned<MODE>(p);
#pragma unroll
    for (int it = 0; it < C::NOCT; ++it) {
      const int piece = it * C::NT + tid, lr = piece / (C::BN / 8), lc = piece % (C::BN / 8) * 8;
      if (C::OCTS % C::NT && piece >= C::OCTS) break;
      const float* src = (const float*)lds_raw + lr * C::LDW + lc;
      float4 lo = *(const float4*)src, hi = *(const float4*)(src + 4);
#pragma unroll
      for (int w = 1; w < NW; ++w) {           // in wave order: the same sum whatever the timing
        const float4 a = *(const float4*)(src + w * C::BM * C::LDW), b = *(const float4*)(src + w * C::BM * C::LDW + 4);
        lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
        hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
      }
      const int row = m0 + lr, col = n0 + lc;
      if (row < p.M && col < p.N) store_octet<MODE>(p, row, col, lo, hi, vec && col + 7 < p.N, split);
    }
  };
  if (p.partial) { if constexpr (has(EPI_PARTIAL)) finish(std::integral_constant<int, EPI_PARTIAL>{}); }
  else if (p.c_f32) { if constexpr (has(EPI_F32)) finish(std::integral_constant<int, EPI_F32>{}); }
  else if (p.epi == 0) { if constexpr (has(EPI_ACT)) finish(std::integral_constant<int, EPI_ACT>{}); }
  else if (p.epi == 1) { if constexpr (has(EPI_ACT_RES)) finish(std::integral_constant<int, EPI_ACT_RES>{}); }
  else if (p.epi == 2) { if constexpr (has(EPI_ACT_GELU)) finish(std::integral_constant<int, EPI_ACT_GELU>{}); }
  else if (p.epi == 3) { if constexpr (has(EPI_ACT_DGELU)) finish(std::integral_constant<int, EPI_ACT_DGELU>{}); }
  else if (p.epi == 4) { if constexpr (has(EPI_ACT_RELU)) finish(std::integral_constant<int, EPI_ACT_RELU>{}); }
  else { if constexpr (has(EPI_ACT_DRELU)) finish(std::integral_constant<int, EPI_ACT_DRELU>{}); }
}

template <class C, bool AK, bool BKM>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::OCC * C::NW / 4, C::OCC * C::NW / 4)))
void gemm_bf16_ksplit(GemmDev p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  const int nbx = gridDim.x, nby = gridDim.y, nb = nbx * nby;
  int v = (blockIdx.z * nby + blockIdx.y) * nbx + blockIdx.x;
  const int per_xcd = (nb * (int)gridDim.z) >> 3;
  if (v < 8 * per_xcd) v = (v & 7) * per_xcd + (v >> 3);
  const int split = v / nb;
  int tm, tn;
  tile_of_block<8>(v - split * nb, nbx, nby, tm, tn);
  ks_tile<C, AK, BKM, wide_epilogues<AK, BKM>()>(p, tm * C::BM, tn * C::BN, split, lds_raw);
}

template <class C, bool AK, bool BKM>
hipError_t launch_ks_one(const GemmDev& p, int splits, hipStream_t s) {
  auto kern = gemm_bf16_ksplit<C, AK, BKM>;
  static bool configured = false;
  if (!configured && C::LDS > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
    if (e != hipSuccess) return e;
  }
  configured = true;
  hipLaunchKernelGGL(kern, dim3((p.N + C::BN - 1) / C::BN, (p.M + C::BM - 1) / C::BM, splits), dim3(C::NT), C::LDS, s, p);
  return hipSuccess;
}
typedef KsCfg<1, 1, 4, 64, 3, 1> Ks32x32;                // TI TJ NW BK S OCC

// every configuration but 0 (numbers: kTileCfg in gemm.hip), one operand layout per translation unit
template <bool AK, bool BKM>
hipError_t launch_layout(int cfg, const GemmDev& p, int splits, hipStream_t s) {
  switch (cfg) {
    case 2: return launch_ks_one<Ks32x32, AK, BKM>(p, splits, s);
    case 1: return launch_dma_one<Dma256x256, AK, BKM>(p, splits, s);
    case 3: return launch_dma_one<Dma128x192, AK, BKM>(p, splits, s);
    case 6: return launch_dma_one<Dma192x128, AK, BKM>(p, splits, s);
    case 4: return launch_dma_one<Dma32x64, AK, BKM>(p, splits, s);
    case 7: return launch_dma_one<Dma64x128, AK, BKM>(p, splits, s);
    case 8: return launch_dma_one<Dma128x64, AK, BKM>(p, splits, s);
    case 9: return launch_dma_one<Dma128x128, AK, BKM>(p, splits, s);
    case 10: return launch_dma_one<Dma256x128, AK, BKM>(p, splits, s);
    case 11: return launch_dma_one<Dma64x64, AK, BKM>(p, splits, s);
    case 5: return launch_wide<AK, BKM>(p, splits, s);
    default: break;
  }
  if constexpr (AK) {      // never chosen with an m-major A
    if (cfg == 12) return launch_dma_one<Dma128x128Lone, AK, BKM>(p, splits, s);
    if (cfg == 13) return launch_dma_one<Dma64x64Lone, AK, BKM>(p, splits, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace
