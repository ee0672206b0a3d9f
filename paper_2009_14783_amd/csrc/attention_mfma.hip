// bf16 MFMA attention backward (head dimension 64), fp32 softmax statistics, for at most 128 queries and 128 keys per sequence: self-attention, causal
// or not, and attention over another sequence.  Everything else goes to the streaming kernels of attention_general.hip, where the tile scheme of both (owned rows in
// registers, transposed score tiles) is described.
#include "attention_tiles.h"

namespace {

using namespace attn_tiles;

// ------------------------------------------------------------------------------------------
// One launch, a block of W waves per (sequence, head) pair for up to 32 W queries and keys.  Every wave first owns 32 queries (dq) with K and V
// streamed from two LDS tiles, then 32 keys (dk, dv) with Q and dO streamed from the SAME two tiles: owned rows never need LDS (their fragments come
// straight from global memory, or out of the tiles just before they are overwritten), so a block of four waves takes 37 KiB of LDS and three of them
// share a CU - one round for the 768 blocks of 64 sequences x 12 heads, and the second staging phase of one block runs under the arithmetic of the
// others.  What bounds it is that chain: load, store, product, softmax, product, store, twice.  Blocks are as small as their pairs: with four waves
// for every pair, three of them idle up to 32 positions and hold the places of others (100 sequences of 56 x 12 heads: 25.7 -> 20.7 us).
// Three waves per SIMD cost the variant with dropout 24 spilled registers; two without a spill are slower (64 x 128 step 7.66 -> 7.69 ms).
// Scores start from -8 lse and their gradients from -dO . O, and only cut tiles are masked, as in attention_general.hip (the BERT-base step of 64 x
// 128 with dropout 8.17 -> 8.08 ms, without level).  For the translation model's 128 x 8 pairs of 32 positions,
// where four waves per pair (self-attention) and two streaming launches (causal, and over the encoder output) took 17 us each, one launch takes 10.7:
// its step 4.22 -> 4.04 ms, the same bits.
// ------------------------------------------------------------------------------------------
struct ShortOperands {
  const bf16 *q, *k, *v, *out, *d_out;      // first row of sequence 0
  bf16 *dq, *dk, *dv;
  int64_t ldq, ldkv, lddq, lddkv;
  const float* lse;
  const int32_t *qlens, *klens, *qfirst, *kfirst;      // first: packed rows, or null
  int Lq, Lk, A;
};

// rows 0 .. 32 W - 1 of one matrix, by the 64 W threads of a pair
template <int W>
__device__ __forceinline__ void stage_rows(bf16* tile, const bf16* __restrict__ src, int64_t ld, int row_limit, int tid) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid + i * 64 * W;
    const int r = c >> 3, col = (c & 7) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < row_limit) v = *(const uint4*)(src + (int64_t)r * ld + col);
    *(uint4*)(tile + r * LDT + col) = v;
  }
}
// between the waves of a pair; one wave's LDS operations execute in order anyway
template <int W>
__device__ __forceinline__ void pair_barrier() {
  if (W > 1) __syncthreads();
  else asm volatile("" ::: "memory");
}

// Up to this many waves in all, about one per SIMD, the two halves of a pair go to a block each: the chip has room for both, and a block's chain is
// half as long (256 pairs of up to 32 positions: 8.5 -> 7.5 us; 480 pairs of up to 64: 13.1 -> 12.7 us; BERT-base, 5 sequences of 88 positions in two
// passes: 4.23 -> 4.08 ms per step).  Beyond, the second set of loads costs more than the shorter chain gives (1024 pairs of 32: 11.1 -> 11.9 us; 384
// pairs of 128, 1536 waves: level).
constexpr int kFewWaves = 960;

template <int W, bool CAUSAL, bool DROP>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(3, 3))) void attn_bwd_short_mfma(ShortOperands x, DropCfg drop, uint32_t site) {
  __shared__ __attribute__((aligned(16))) bf16 T0[32 * W * LDT];      // K, then Q
  __shared__ __attribute__((aligned(16))) bf16 T1[32 * W * LDT];      // V, then dO
  __shared__ float st0_s[32 * W], dp0_s[32 * W];      // what a query's scores and their gradients start from: -8 lse, -dO . O
  const int tid = threadIdx.x, lane = tid & 63, w0 = __builtin_amdgcn_readfirstlane(tid >> 6) * 32;
  const int b = blockIdx.y, h = blockIdx.x;
  const int H = x.A * DH;
  const int qlen = min(max(x.qlens[b], 1), x.Lq), klen = min(max(x.klens[b], 1), x.Lk);
  const int qrows = x.qfirst ? qlen : x.Lq, krows = x.kfirst ? klen : x.Lk;      // packed: the row behind the last is the next sequence's
  const int64_t qbase = x.qfirst ? x.qfirst[b] : (int64_t)b * x.Lq, kbase = x.kfirst ? x.kfirst[b] : (int64_t)b * x.Lk;
  const bf16* const q = x.q + qbase * x.ldq + h * DH;
  const bf16* const k = x.k + kbase * x.ldkv + h * DH;
  const bf16* const v = x.v + kbase * x.ldkv + h * DH;
  const bf16* const go = x.d_out + qbase * H + h * DH;
  const bf16* const oo = x.out + qbase * H + h * DH;
  const int own = w0 + (lane & 31);       // the query, then the key, this lane owns

  const bool queries = blockIdx.z == 0, keys = queries == (gridDim.z == 1);      // the halves this block does
  if (queries) {
    stage_rows<W>(T0, k, x.ldkv, klen, tid);
    stage_rows<W>(T1, v, x.ldkv, klen, tid);
  } else {
    stage_rows<W>(T0, q, x.ldq, qlen, tid);
    stage_rows<W>(T1, go, H, qlen, tid);
  }
  // the owned queries' fragments of Q and dO, and the row dot product sum_d dO*O (lanes l and l + 32 hold the two halves of a row)
  bf16x8 qf[4], gf[4];
  float drow = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    qf[ks] = frag_rows_global(q, x.ldq, own, qlen, ks, lane);
    gf[ks] = frag_rows_global(go, H, own, qlen, ks, lane);
    const bf16x8 of = frag_rows_global(oo, H, own, qlen, ks, lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) drow = fmaf((float)gf[ks][e], (float)of[e], drow);
  }
  drow += __shfl_xor(drow, 32);
  const float st0 = (own < qlen) ? x.lse[((int64_t)b * x.A + h) * x.Lq + own] * -8.0f : 0.f;      // 8: the scores are not scaled yet
  if (lane < 32) { dp0_s[own] = -drow; st0_s[own] = st0; }
  pair_barrier<W>();

  f32x16 acc[2], acc2[2];
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
  // ---- queries owned: dq ----
  if (queries && w0 < qlen) {
    const int kend = CAUSAL ? min(klen, w0 + 32) : klen;
    for (int kb = 0; kb < kend; kb += 32) {
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
        drop_tile_keys(drop, site, (((uint64_t)b * x.A + h) * x.Lq + own) * (uint64_t)x.Lk, kb, lane, f);
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] = fmaf(dp[r], f[r], -drow);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = fast_exp2(st[r] * SCALE2);
      if (w0 + 32 > qlen || kb + 32 > klen || (CAUSAL && kb + 31 > w0)) {      // wave-uniform
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb + tile_row(r, lane);
          st[r] = (key < klen && own < qlen && (!CAUSAL || key <= own)) ? st[r] : 0.f;
        }
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
  if (queries) {
    // The owned key/value fragments are the last thing read from K and V.  After the barrier a wave's own 32 rows of
    // tile 0 stage the whole-row stores of dq; after the next one the tiles are refilled with Q and dO.
    if (keys) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) { kf[ks] = frag_rows(T0, w0, ks, lane); vf[ks] = frag_rows(T1, w0, ks, lane); }
    }
    pair_barrier<W>();
    store_owned_rows_lds(x.dq + qbase * x.lddq + h * DH, x.lddq, w0, qrows, acc, 0.125f, lane, T0 + w0 * LDT);
    if (!keys) return;
    pair_barrier<W>();
    stage_rows<W>(T0, q, x.ldq, qlen, tid);
    stage_rows<W>(T1, go, H, qlen, tid);
    pair_barrier<W>();
  } else {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kf[ks] = frag_rows_global(k, x.ldkv, own, klen, ks, lane);
      vf[ks] = frag_rows_global(v, x.ldkv, own, klen, ks, lane);
    }
  }
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[db][r] = 0.f; acc2[db][r] = 0.f; }
  if (w0 < klen) {
    for (int qb = CAUSAL ? w0 : 0; qb < qlen; qb += 32) {
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
      if (w0 + 32 > klen || qb + 32 > qlen || (CAUSAL && qb < w0 + 31)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int qi = qb + tile_row(r, lane);
          st[r] = (qi < qlen && own < klen && (!CAUSAL || own <= qi)) ? st[r] : 0.f;
        }
      }
      if (DROP) {
        f32x16 f;
        drop_tile_queries(drop, site, ((uint64_t)b * x.A + h) * x.Lq, x.Lk, qb, own, lane, f);
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
  pair_barrier<W>();     // every wave is done with Q and dO: own rows of the tiles stage the stores of dk and dv
  store_owned_rows_lds(x.dk + kbase * x.lddkv + h * DH, x.lddkv, w0, krows, acc, 0.125f, lane, T0 + w0 * LDT);
  store_owned_rows_lds(x.dv + kbase * x.lddkv + h * DH, x.lddkv, w0, krows, acc2, 1.0f, lane, T1 + w0 * LDT);
}

template <int W>
void launch_short(const ShortOperands& x, int B, bool causal, hipStream_t s, const DropCfg& drop, uint32_t site) {
  const dim3 grid(x.A, B, (int64_t)x.A * B * W <= kFewWaves ? 2 : 1);
  if (causal) hipLaunchKernelGGL((attn_bwd_short_mfma<W, true, false>), grid, dim3(64 * W), 0, s, x, drop, site);
  else if (drop.thr) hipLaunchKernelGGL((attn_bwd_short_mfma<W, false, true>), grid, dim3(64 * W), 0, s, x, drop, site);
  else hipLaunchKernelGGL((attn_bwd_short_mfma<W, false, false>), grid, dim3(64 * W), 0, s, x, drop, site);
}

}  // namespace

// Whether a problem has a short form (16-byte rows of the gradients; causal: without dropout), and the launch
bool attention_bwd_is_short(const AttnOperands& x, const void* dq, int64_t lddq, const void* dk, const void* dv, int64_t lddkv) {
  auto wide = [](const void* p, int64_t ld) { return !((uintptr_t)p & 15) && !(ld & 7); };
  return x.Lq <= 128 && x.Lk <= 128 && wide(dq, lddq) && wide(dk, lddkv) && wide(dv, lddkv);
}
void launch_attention_bwd_short(const AttnOperands& x, int B, const void* out, const float* lse, const void* d_out, void* dq, int64_t lddq, void* dk, void* dv,
                                int64_t lddkv, hipStream_t s, const DropCfg& drop, uint32_t site) {
  const ShortOperands o{(const bf16*)x.q, (const bf16*)x.k, (const bf16*)x.v, (const bf16*)out, (const bf16*)d_out, (bf16*)dq, (bf16*)dk, (bf16*)dv,
                        x.ldq, x.ldkv, lddq, lddkv, lse, x.qlens, x.klens, x.qfirst, x.kfirst, x.Lq, x.Lk, x.A};
  const int L = x.Lq > x.Lk ? x.Lq : x.Lk;
  if (L <= 32) launch_short<1>(o, B, x.causal, s, drop, site);
  else if (L <= 64) launch_short<2>(o, B, x.causal, s, drop, site);
  else launch_short<4>(o, B, x.causal, s, drop, site);
}
