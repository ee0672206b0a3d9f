// bf16 MFMA self-attention (head dimension 64), fp32 softmax statistics: the backward pass of sequences of at most 128 positions.
// Everything else goes to the streaming kernels of attention_general.hip, where the tile scheme of both (owned rows in registers,
// transposed score tiles) is described.
#include "attention_tiles.h"

namespace {

using namespace attn_tiles;

// ------------------------------------------------------------------------------------------
// backward for sequences of at most 128 positions: one block per (sequence, head), no second launch.  Every
// wave first owns 32 queries (dq) with K and V streamed from two LDS tiles, then 32 keys (dk, dv) with Q and dO
// streamed from the SAME two tiles: owned rows never need LDS (their fragments come straight from global memory,
// or out of the tiles just before they are overwritten), so a block takes 37 KiB of LDS and three of them share a CU -
// one round for the 768 blocks of 64 sequences x 12 heads, and the second staging phase of one block runs under
// the arithmetic of the others.
// Scores start from -8 lse and their gradients from -dO . O, and only cut tiles are masked, as in attention_general.hip (the BERT-base step of 64 x
// 128 with dropout 8.17 -> 8.08 ms, without level).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void stage128(bf16* tile, const bf16* __restrict__ src, int64_t ld, int row_limit, int tid) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + i * 256;
    const int r = c >> 3, col = (c & 7) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < row_limit) v = *(const uint4*)(src + (int64_t)r * ld + col);
    *(uint4*)(tile + r * LDT + col) = v;
  }
}

// Up to this many (sequence, head) pairs, the two halves go to a block each: the chip has room for both, and a block's chain is half as long
// (BERT-base, 5 sequences of 88 positions in two passes: 4.23 -> 4.08 ms per step).  Beyond, the second set of loads costs what the shorter chain
// gives (768 pairs: 7.50 -> 7.54 ms per step; 384: level).
constexpr int kFewHeads = 256;

template <bool DROP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3)))
void attn_bwd_fused128_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ out, const float* __restrict__ lse,
                            const bf16* __restrict__ d_out, const int32_t* __restrict__ lens, const int32_t* __restrict__ first, int L, int A,
                            bf16* __restrict__ dqkv, DropCfg drop, uint32_t site) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  bf16* T0 = (bf16*)lds_raw;               // K, then Q
  bf16* T1 = T0 + 128 * LDT;               // V, then dO
  float* st0_s = (float*)(T1 + 128 * LDT);      // what a query's scores and their gradients start from: -8 lse, -dO . O
  float* dp0_s = st0_s + 128;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y, h = blockIdx.x;
  const int H = A * DH;
  const int64_t ld = 3 * (int64_t)H;
  int len = lens[b];
  len = len < 1 ? 1 : (len > L ? L : len);
  const int64_t row0 = first ? first[b] : (int64_t)b * L;
  const int rows = first ? len : L;              // packed rows: the row behind the last one is the next sequence's
  const bf16* base = qkv + row0 * ld + h * DH;
  const bf16* go = d_out + row0 * H + h * DH;
  const bf16* oo = out + row0 * H + h * DH;
  const int own = wave * 32 + (lane & 31);       // the query, then the key, this lane owns
  const bool wave_active = wave * 32 < len;      // wave-uniform

  const bool queries = blockIdx.z == 0, keys = queries == (gridDim.z == 1);      // the halves this block does
  stage128(T0, queries ? base + H : base, ld, len, tid);
  stage128(T1, queries ? base + 2 * H : go, queries ? ld : H, len, tid);
  // the owned queries' fragments of Q and dO, and the row dot product sum_d dO*O (lanes l and l + 32 hold the two halves of a row)
  bf16x8 qf[4], gf[4];
  float drow = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    qf[ks] = frag_rows_global(base, ld, own, len, ks, lane);
    gf[ks] = frag_rows_global(go, H, own, len, ks, lane);
    const bf16x8 of = frag_rows_global(oo, H, own, len, ks, lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) drow = fmaf((float)gf[ks][e], (float)of[e], drow);
  }
  drow += __shfl_xor(drow, 32);
  const float st0 = (own < len) ? lse[((int64_t)b * A + h) * L + own] * -8.0f : 0.f;      // 8: the scores are not scaled yet
  const bool own_cut = wave * 32 + 32 > len;      // some of the wave's rows are padding (wave-uniform)
  if (lane < 32) { dp0_s[own] = -drow; st0_s[own] = st0; }
  __syncthreads();

  f32x16 acc[2], acc2[2];
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
  // ---- queries owned: dq ----
  if (queries && wave_active) {
    for (int kb = 0; kb < len; kb += 32) {
      f32x16 st, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { st[r] = st0; dp[r] = DROP ? 0.f : -drow; }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows(T0, kb, ks, lane), qf[ks], st, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows(T1, kb, ks, lane), gf[ks], dp, 0, 0, 0);
      }
      if (DROP) {
        f32x16 f;
        drop_tile_keys(drop, site, (((uint64_t)b * A + h) * L + own) * (uint64_t)L, kb, lane, f);
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] = fmaf(dp[r], f[r], -drow);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = fast_exp2(st[r] * SCALE2);
      if (own_cut || kb + 32 > len) {
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = (kb + tile_row(r, lane) < len && own < len) ? st[r] : 0.f;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] *= dp[r];
      const bf16x8 s0 = pack8(st, 0), s1 = pack8(st, 1);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_t(T0, kb, 0, 32 * db, lane), s0, acc[db], 0, 0, 0);
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_t(T0, kb, 1, 32 * db, lane), s1, acc[db], 0, 0, 0);
      }
    }
  }
  // ---- keys owned: dk, dv ----
  bf16x8 kf[4], vf[4];
  bf16* const dst = dqkv + row0 * ld + h * DH;
  if (queries) {
    // The owned key/value fragments are the last thing read from K and V.  After the barrier a wave's own 32 rows of
    // tile 0 stage the whole-row stores of dq; after the next one the tiles are refilled with Q and dO.
    if (keys) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) { kf[ks] = frag_rows(T0, wave * 32, ks, lane); vf[ks] = frag_rows(T1, wave * 32, ks, lane); }
    }
    __syncthreads();
    store_owned_rows_lds(dst, ld, wave * 32, rows, acc, 0.125f, lane, T0 + wave * 32 * LDT);
    if (!keys) return;
    __syncthreads();
    stage128(T0, base, ld, len, tid);
    stage128(T1, go, H, len, tid);
    __syncthreads();
  } else {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kf[ks] = frag_rows_global(base + H, ld, own, len, ks, lane);
      vf[ks] = frag_rows_global(base + 2 * H, ld, own, len, ks, lane);
    }
  }
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[db][r] = 0.f; acc2[db][r] = 0.f; }
  if (wave_active) {
    for (int qb = 0; qb < len; qb += 32) {
      f32x16 st, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        st[r] = st0_s[qb + tile_row(r, lane)];
        dp[r] = DROP ? 0.f : dp0_s[qb + tile_row(r, lane)];
      }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows(T0, qb, ks, lane), kf[ks], st, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows(T1, qb, ks, lane), vf[ks], dp, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = fast_exp2(st[r] * SCALE2);
      if (own_cut || qb + 32 > len) {
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = (qb + tile_row(r, lane) < len && own < len) ? st[r] : 0.f;
      }
      if (DROP) {
        f32x16 f;
        drop_tile_queries(drop, site, ((uint64_t)b * A + h) * L, L, qb, own, lane, f);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          dp[r] = st[r] * fmaf(f[r], dp[r], dp0_s[qb + tile_row(r, lane)]);
          st[r] *= f[r];
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] *= st[r];
      }
      const bf16x8 p0 = pack8(st, 0), p1 = pack8(st, 1), s0 = pack8(dp, 0), s1 = pack8(dp, 1);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        acc2[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_t(T1, qb, 0, 32 * db, lane), p0, acc2[db], 0, 0, 0);
        acc2[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_t(T1, qb, 1, 32 * db, lane), p1, acc2[db], 0, 0, 0);
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_t(T0, qb, 0, 32 * db, lane), s0, acc[db], 0, 0, 0);
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_cols_t(T0, qb, 1, 32 * db, lane), s1, acc[db], 0, 0, 0);
      }
    }
  }
  __syncthreads();     // every wave is done with Q and dO: own rows of the tiles stage the stores of dk and dv
  store_owned_rows_lds(dst + H, ld, wave * 32, rows, acc, 0.125f, lane, T0 + wave * 32 * LDT);
  store_owned_rows_lds(dst + 2 * H, ld, wave * 32, rows, acc2, 1.0f, lane, T1 + wave * 32 * LDT);
}

}  // namespace

void launch_attention_self_fwd(const void* qkv, const int32_t* lens, int B, int L, int A, void* out, float* lse, hipStream_t s, const DropCfg& drop,
                               uint32_t site, const int32_t* first);
void launch_attention_self_bwd(const void* qkv, const void* out, const float* lse, const void* d_out, const int32_t* lens, int B, int L, int A,
                               void* dqkv, float* dvec, hipStream_t s, const DropCfg& drop, uint32_t site, const int32_t* first);

void launch_attention_fwd_mfma(const void* qkv, const int32_t* lens, int B, int L, int A, void* out, float* lse, hipStream_t s,
                               const DropCfg& drop, uint32_t site, const int32_t* first) {
  launch_attention_self_fwd(qkv, lens, B, L, A, out, lse, s, drop, site, first);
}

void launch_attention_bwd_mfma(const void* qkv, const void* out, const float* lse, const void* d_out, const int32_t* lens, int B, int L,
                               int A, void* dqkv, float* dvec, hipStream_t s, const DropCfg& drop, uint32_t site, const int32_t* first) {
  if (L <= 128) {
    constexpr size_t lds = 2 * 128 * LDT * sizeof(bf16) + 2 * 128 * sizeof(float);
    static bool configured = false;
    if (!configured) {
      (void)hipFuncSetAttribute((const void*)attn_bwd_fused128_mfma<false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      (void)hipFuncSetAttribute((const void*)attn_bwd_fused128_mfma<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      configured = true;
    }
    const dim3 grid(A, B, (int64_t)A * B <= kFewHeads ? 2 : 1);
    if (drop.thr) hipLaunchKernelGGL(attn_bwd_fused128_mfma<true>, grid, dim3(256), lds, s, (const bf16*)qkv, (const bf16*)out, lse,
                                     (const bf16*)d_out, lens, first, L, A, (bf16*)dqkv, drop, site);
    else hipLaunchKernelGGL(attn_bwd_fused128_mfma<false>, grid, dim3(256), lds, s, (const bf16*)qkv, (const bf16*)out, lse,
                            (const bf16*)d_out, lens, first, L, A, (bf16*)dqkv, drop, site);
    return;
  }
  launch_attention_self_bwd(qkv, out, lse, d_out, lens, B, L, A, dqkv, dvec, s, drop, site, first);
}
