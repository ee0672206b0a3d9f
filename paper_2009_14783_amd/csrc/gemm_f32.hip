// fp32 GEMM on the matrix cores: C = A B^T in fp32 throughout (v_mfma_f32_32x32x2_f32: fp32 products, fp32 accumulation).
//
// The operands go from memory straight to the registers of the lanes that feed them to the matrix cores, without LDS.  A step of
// the contraction covers 8 values of k, four MFMAs: lane l of a wave holds row l%32 of its operand at k = 4 (l/32) .. +3, one
// 16-byte load where the operand is k-major and four loads of 128 contiguous bytes per half wave where it is not.  That is 16
// bytes per lane and operand for 256 matrix-core cycles, so the caches keep up even for a lone 32x32 tile.
//
// Two tilings.  Toy models (a few hundred rows, 128 columns) have too few tiles to fill the chip, and what bounds a product is its
// serial chain: 32x32 tiles, with the contraction dealt out over the block's 4 or 16 waves in batches of 32 values, all loads of a
// batch and of the one after it in flight, and one sum over the waves' tiles in LDS.  Larger products: 128x128 tiles, four waves
// of 64x64 each; bound by the loads (85 of the 157 TFLOP/s of fp32 on the matrix cores at 4096 x 3072 x 768).
// Measured, launched back to back, against 64x64 tiles of vector FMAs with four barriers per 16 values of k: [256, 512, 128]
// (rows, columns, contraction) 20 -> 8.6 us, [256, 128, 512] 69 -> 8.8 us, [1024, 768, 768] 106 -> 26 us, [4096, 3072, 768]
// 468 -> 262 us; weight gradients (both operands m-major) [768, 3072, 1024] 218 -> 103 us.
#include "gemm_dev.h"

namespace {
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // the hardware needs 4-byte alignment only

// four values of one row at k .. k + 3: `p` is wave-uniform (one scalar base and a 32-bit lane offset `off`, in bytes, keep the
// addresses out of the vector registers); KM: k-major
__device__ __forceinline__ const float* lane_ptr(const float* p, uint32_t off) { return (const float*)((const char*)p + off); }
template <bool KM>
__device__ __forceinline__ f32x4u load4(const float* p, int64_t ld, uint32_t off) {
  if (KM) return *(const f32x4u*)lane_ptr(p, off);
  f32x4u v;
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = *lane_ptr(p + c * ld, off);
  return v;
}
// the first n (< 4, possibly <= 0) of them, zeros behind
template <bool KM>
__device__ __forceinline__ f32x4u load4_part(const float* p, int64_t ld, uint32_t off, int n) {
  f32x4u v;
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = c < n ? *lane_ptr(p + (KM ? c : c * ld), off) : 0.0f;
  return v;
}

// the tile (tm, tn) of one product; T x T accumulators of 32x32 per wave, W x W waves side by side, KW waves along k
template <bool AK, bool BKM, int T, int W, int KW>
__device__ __forceinline__ void f32_tile(const GemmDev& p, int tm, int tn) {
  constexpr int NQ = T == 1 ? 4 : 1;      // steps of 8 values per batch
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = wave / (W * W), wm = (wave / W) % W, wn = wave % W;
  const int l31 = lane & 31, half = lane >> 5;
  // first row of the wave; rows beyond the last repeat it: their results are not stored
  const int row0 = min((tm * W + wm) * T * 32, p.M - 1), col0 = min((tn * W + wn) * T * 32, p.N - 1);
  const bool ones = p.B == nullptr;        // a column of ones
  const float* A = (const float*)p.A + (AK ? row0 * p.lda : row0);
  const float* B = (const float*)p.B + (ones ? 0 : BKM ? col0 * p.ldb : col0);
  uint32_t oa[T], ob[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const uint32_t r = min(32 * i + l31, p.M - 1 - row0), c = min(32 * i + l31, p.N - 1 - col0);
    oa[i] = 4 * (AK ? r * (uint32_t)p.lda + 4 * half : r + 4 * half * (uint32_t)p.lda);
    ob[i] = 4 * (BKM ? c * (uint32_t)p.ldb + 4 * half : c + 4 * half * (uint32_t)p.ldb);
  }
  const int64_t stepa = AK ? 8 : 8 * p.lda, stepb = BKM ? 8 : 8 * p.ldb;
  const f32x4u zero = {0.f, 0.f, 0.f, 0.f}, one = {1.f, 1.f, 1.f, 1.f};
  f32x16 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int ng = p.K >> 3, nb = (ng + NQ - 1) / NQ;
  f32x4u a[2][NQ][T], b[2][NQ][T];
  auto load = [&](int s, int batch) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int g = batch * NQ + q;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        if (g < ng) {
          a[s][q][i] = load4<AK>(A + g * stepa, p.lda, oa[i]);
          b[s][q][i] = ones ? one : load4<BKM>(B + g * stepb, p.ldb, ob[i]);
        } else {
          a[s][q][i] = zero; b[s][q][i] = zero;
        }
      }
    }
  };
  auto mac = [&](int s) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s][q][i][c], b[s][q][j][c], acc[i][j], 0, 0, 0);
  };
  load(0, kw);
  for (int batch = kw; batch < nb; batch += 2 * KW) {
    load(1, batch + KW);
    mac(0);
    if (batch + KW >= nb) break;
    load(0, batch + 2 * KW);
    mac(1);
  }
  if ((p.K & 7) && kw == KW - 1) {
    const int n = (p.K & 7) - 4 * half;
#pragma unroll
    for (int i = 0; i < T; ++i) {
      a[0][0][i] = load4_part<AK>(A + ng * stepa, p.lda, oa[i], n);
      b[0][0][i] = ones ? one : load4_part<BKM>(B + ng * stepb, p.ldb, ob[i], n);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][0][i][c], b[0][0][j][c], acc[i][j], 0, 0, 0);
  }

  constexpr int S = 32 * T * W;
  __shared__ float part[KW][S * S];      // 64 KB at most
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[kw][((wm * T + i) * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * S + (wn * T + j) * 32 + l31] = acc[i][j][r];
  __syncthreads();
  for (int e = tid; e < S * S; e += 64 * W * W * KW) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < KW; ++w) v += part[w][e];
    epilogue_store<float>(p, tm * S + e / S, tn * S + e % S, v);
  }
}

template <bool AK, bool BKM, int T, int W, int KW>
__global__ __launch_bounds__(64 * W * W * KW) void gemm_f32(GemmDev p) {
  f32_tile<AK, BKM, T, W, KW>(p, blockIdx.y, blockIdx.x);
}

template <int T, int W, int KW>
__global__ __launch_bounds__(64 * W * W * KW) void gemm_f32_group(GemmGroupDev g) {
  int i = 0;
  while (i + 1 < g.n && (int)blockIdx.x >= g.first_tile[i + 1]) ++i;
  const GroupProb& q = g.prob[i];
  GemmDev p{};
  p.A = q.A; p.B = q.B; p.C = q.C; p.lda = q.lda; p.ldb = q.ldb; p.ldc = q.ldc; p.M = q.M; p.N = q.N; p.K = q.K;
  p.c_f32 = 1; p.beta = g.beta;
  const int tiles_n = (q.N + 32 * T * W - 1) / (32 * T * W), tile = (int)blockIdx.x - g.first_tile[i];
  f32_tile<false, false, T, W, KW>(p, tile / tiles_n, tile % tiles_n);
}

template <bool AK, bool BKM>
void launch(const GemmDev& p, int tile, hipStream_t s) {
  const dim3 grid((p.N + tile - 1) / tile, (p.M + tile - 1) / tile);
  // up to 256 values a wave has at most two batches with 4 waves, whose tiles are the cheaper to add up
  if (tile == 128) hipLaunchKernelGGL((gemm_f32<AK, BKM, 2, 2, 1>), grid, dim3(256), 0, s, p);
  else if (p.K <= 256) hipLaunchKernelGGL((gemm_f32<AK, BKM, 1, 1, 4>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((gemm_f32<AK, BKM, 1, 1, 16>), grid, dim3(1024), 0, s, p);
}
}  // namespace

// Side of the square tiles for products with this many 128x128 tiles in all: 128 once they are enough to give most CUs one.  At
// 192 (1024 x 3072 x 768) the two sides take 87 and 96 us, at 144 (768 x 3072 x 1024) 106 and 94 us.
static int gemm_f32_tile(int64_t tiles128) { return tiles128 >= 192 ? 128 : 32; }

void gemm_f32_launch(bool a_kmajor, bool b_kmajor, const GemmDev& p, hipStream_t s) {
  const int tile = gemm_f32_tile((int64_t)((p.M + 127) / 128) * ((p.N + 127) / 128));
  if (a_kmajor && b_kmajor) launch<true, true>(p, tile, s);
  else if (a_kmajor) launch<true, false>(p, tile, s);
  else if (b_kmajor) launch<false, true>(p, tile, s);
  else launch<false, false>(p, tile, s);
}

void gemm_f32_group_launch(int tile, const GemmGroupDev& g, hipStream_t s) {
  const dim3 grid((unsigned)g.first_tile[g.n]);
  if (tile == 128) hipLaunchKernelGGL((gemm_f32_group<2, 2, 1>), grid, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_f32_group<1, 1, 16>), grid, dim3(1024), 0, s, g);
}
