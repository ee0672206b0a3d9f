// Softmax attention with separate query and key/value sequences (head dimension 64), forward and backward: self-attention over
// sequences of any length (backward: more than 128 positions), the decoder's causal self-attention and its attention over the
// encoder output.  Queries, keys and values
// are row ranges of token-major matrices with their own row strides (head h = columns h*64 .. h*64+63);
// key j of sequence b takes part iff j < klens[b] and, when causal, j <= query index; queries at or beyond
// qlens[b] get zero gradients.  Dropout of the probabilities: self-attention only (the translation model drops sub-layer
// outputs only).
//
// bf16: the MFMA kernels below.  fp32: attention_f32.hip.
//
// A wave OWNS 32 rows (queries, or keys in the dK/dV kernel) whose vectors stay in registers as MFMA B operands, and the block STREAMS
// the other side through LDS in blocks of 64 rows.  Score tiles are computed transposed,
// tile[streamed row][owned row], so that each lane holds ONE owned row (lane % 32) and 16 streamed
// rows: reductions over the streamed index are then in-lane plus one exchange between the two
// half-waves.  The second product needs the score tile as a B operand and the streamed block
// transposed as the A operand; the transposed fragment comes from the LDS transpose read, with
// the 16 contraction slots ordered exactly as the result registers of the score tile are
// (register r of lane l is streamed row 8*(r/4) + 4*(l/32) + r%4), so no data moves between lanes.
//
// What bounds these kernels at the sizes of the encoder is the vector ALU and the latency of a block's chain of load, product, softmax
// and product.  So the next 64 rows are loaded straight into the other half of LDS while the current ones are worked on (one barrier per
// block, no register holds a streamed byte); scores start from -8 lse and their gradients from the row term, which the matrix cores
// then add for nothing, so that a gradient score costs a multiplication, an exponential and a multiplication; masks are applied only in
// the tiles that an end or the diagonal cuts; the forward pass works out the scores and exponentials of two 32-key softmax steps side by side
// and rescales its sums only when a maximum moved.  The query blocks of one head run on one XCD, whose L2 then holds that head's keys and values.
// 32 sequences of 512 positions, 16 heads, in the BERT-large step, against kernels that staged through registers between two barriers, masked
// every score and took one softmax step after the other: dq 132.5 -> 72.9 us, dk and dv 179.6 -> 90.8 (755 TFLOP/s); forward by itself 80.1 -> 55.9 (615).
// A maximum over 64 keys at once would give 52.9 us there (56 x 256 x 12 heads 24.0 instead of 25.3; up to 32 positions all the same), but fewer probabilities are
// then exactly one when they are rounded to bf16: results 0.4 to 1.4 % further from float64 between 40 and 512 positions.
#include "attention_tiles.h"

// attention_mfma.hip
bool attention_bwd_is_short(const AttnOperands& x, const void* dq, int64_t lddq, const void* dk, const void* dv, int64_t lddkv);
void launch_attention_bwd_short(const AttnOperands& x, int B, const void* out, const float* lse, const void* d_out, void* dq, int64_t lddq, void* dk, void* dv,
                                int64_t lddkv, hipStream_t s, const DropCfg& drop, uint32_t site);

namespace {

using namespace attn_tiles;

struct View {
  const void *q, *k, *v;      // first row of sequence 0
  int64_t ldq, ldkv;          // row strides in elements
  const int32_t *qlens, *klens;
  int Lq, Lk, A;
  const int32_t *qfirst, *kfirst;      // packed rows: first row of each sequence, or null (b Lq, b Lk)
};

__device__ __forceinline__ int clamp_len(int n, int L) { return n < 1 ? 1 : (n > L ? L : n); }
// first row of sequence b, and the rows that a sequence has: with packed rows the row behind its last one is the next sequence's
__device__ __forceinline__ int64_t first_row(const int32_t* first, int b, int L) { return first ? first[b] : (int64_t)b * L; }
__device__ __forceinline__ int row_count(const int32_t* first, int len, int L) { return first ? len : L; }

// ------------------------------------------------------------------------------------------
// bf16 MFMA
// ------------------------------------------------------------------------------------------
constexpr int kTileBytes = 64 * DH * 2;                        // 64 streamed rows of one matrix
constexpr int kStageBytes = 2 * kTileBytes;                    // of both streamed matrices
static_assert(2 * kStageBytes >= 4 * 32 * LDT * (int)sizeof(bf16), "the stages hold the four waves' store areas");

// (sequence, head, block of 128 owned rows) of a thread block.  Blocks go round the XCDs one by one; each XCD gets a contiguous range of
// the order in which the row blocks of a head are neighbours.
__device__ __forceinline__ void block_place(int& b, int& h, int& row0) {
  const int nx = gridDim.x, ny = gridDim.y, per_xcd = (nx * ny * (int)gridDim.z) >> 3;
  int v = ((int)blockIdx.z * ny + blockIdx.y) * nx + blockIdx.x;
  if (v < 8 * per_xcd) v = (v & 7) * per_xcd + (v >> 3);
  row0 = (v % nx) * 128;
  const int bh = v / nx;
  h = bh % ny;
  b = bh / ny;
}

// A streamed block in LDS: 64 rows of 128 bytes, unpadded because one load instruction fills 1 KiB in lane order.  Chunk c (16 bytes) of row r
// sits at c ^ chunk_swizzle(r): 16 consecutive rows put the same chunk into 16 different places of 256 bytes (row fragments), and the two
// 64-byte halves change sides every other row (a transposing read takes one half of each of four rows at once).  Neither has bank conflicts: a wave loses
// 48 cycles to them per matrix that it writes, in the store through LDS, at 128, 256 and 512 positions alike (20, 12 and 7 % of the forward pass's LDS cycles).
__device__ __forceinline__ int chunk_swizzle(int row) { return (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1); }

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Loads of one streamed matrix: wave w fetches rows 16 w .. 16 w + 15 of a block, 8 rows per instruction.
struct Stream {
  const bf16* base;       // of row 16 w of the sequence
  int64_t ld;
  unsigned off[2];
  __device__ __forceinline__ void init(const bf16* first, int64_t ld_, int lane, int wave) {
    ld = ld_;
    base = first + (int64_t)wave * 16 * ld;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = i * 8 + (lane >> 3);
      off[i] = (unsigned)(((int64_t)row * ld + (((lane & 7) ^ chunk_swizzle(row)) << 3)) * 2);
    }
  }
  // rows r0 .. r0 + 63 to dst; rows at or beyond limit lie behind the end of the buffer and read as zero
  __device__ __forceinline__ void issue(int r0, int limit, unsigned char* __restrict__ dst, int wave) const {
    const int n = min(16, limit - r0 - wave * 16);
    const int bytes = n > 0 ? (int)(unsigned)(((n - 1) * ld + DH) * 2) : 0;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(base + (int64_t)r0 * ld), 0, bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + (wave * 2 + i) * 1024), 16, (int)off[i], 0, 0, 0);
  }
};

// every load of this wave has landed, every LDS read of it is done, and so it is with the other waves of the block
__device__ __forceinline__ void stage_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x70);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// frag_rows and frag_cols_t of the swizzled layout (rbase a multiple of 32, c0 of 32)
__device__ __forceinline__ bf16x8 srows(const unsigned char* __restrict__ tile, int rbase, int ks, int lane) {
  return *(const bf16x8*)(tile + (rbase + (lane & 31)) * 128 + (((ks * 2 + (lane >> 5)) ^ chunk_swizzle(lane & 15)) << 4));
}
__device__ __forceinline__ bf16x8 scols_t(const unsigned char* __restrict__ tile, int rbase, int step, int c0, int lane) {
  const int r = 4 * (lane >> 5) + ((lane & 15) >> 2), col = c0 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const unsigned char* const row = tile + (rbase + 16 * step + r) * 128 + (col & 7) * 2;
  typedef s16x4 __attribute__((address_space(3))) * lds_v4;
  union { struct { s16x4 lo, hi; } p; bf16x8 v; } u;
  u.p.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(row + (((col >> 3) ^ chunk_swizzle(r)) << 4)));
  u.p.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(row + 8 * 128 + (((col >> 3) ^ chunk_swizzle(r + 8)) << 4)));
  return u.v;
}

// rows row0 + 0..31 of the wave to dst (the matrix row of sequence row 0): whole rows through the wave's LDS area where 16-byte stores may be used
__device__ __forceinline__ void store_wave_rows(bf16* __restrict__ dst, int64_t ld, int row0, int limit, const f32x16 (&acc)[2], float scale,
                                                int lane, bf16* area, bool wide) {
  if (wide) store_owned_rows_lds(dst, ld, row0, limit, acc, scale, lane, area);
  else if (row0 + (lane & 31) < limit) store_owned_rows(dst + (int64_t)(row0 + (lane & 31)) * ld, acc, scale, lane);
}

__device__ __forceinline__ void clear(f32x16 (&acc)[2]) {
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
}

template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DROP ? 3 : 4, DROP ? 3 : 4))) void stream_fwd_mfma(View a, bf16* __restrict__ out, float* __restrict__ lse,
                                                                                                 bool wide, DropCfg drop, uint32_t site) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kStageBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, h, row0;
  block_place(b, h, row0);
  const int H = a.A * DH;
  const int klen = clamp_len(a.klens[b], a.Lk), qrows = a.qfirst ? clamp_len(a.qlens[b], a.Lq) : a.Lq;
  if (row0 >= qrows) return;      // block-uniform
  const int64_t qbase = first_row(a.qfirst, b, a.Lq), kbase = first_row(a.kfirst, b, a.Lk);
  const int w0 = row0 + wave * 32, q = w0 + (lane & 31);
  const int kend = CAUSAL ? min(klen, row0 + 128) : klen;      // block-uniform
  Stream ks_, vs_;
  ks_.init((const bf16*)a.k + kbase * a.ldkv + h * DH, a.ldkv, lane, wave);
  vs_.init((const bf16*)a.v + kbase * a.ldkv + h * DH, a.ldkv, lane, wave);
  auto request = [&](int k0, unsigned char* __restrict__ st) __attribute__((always_inline)) {
    ks_.issue(k0, klen, st, wave);
    vs_.issue(k0, klen, st + kTileBytes, wave);
  };
  request(0, lds);

  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qf[ks] = frag_rows_global((const bf16*)a.q + qbase * a.ldq + h * DH, a.ldq, q, qrows, ks, lane);
  f32x16 o[2];
  clear(o);
  float m2 = -1.0e30f, lsum = 0.f;

  auto step = [&](int k0, const unsigned char* __restrict__ cur, unsigned char* __restrict__ nxt) __attribute__((always_inline)) {
    stage_barrier();
    if (k0 + 64 < kend) request(k0 + 64, nxt);
    if (w0 >= qrows || (CAUSAL && k0 > w0 + 31)) return;
    const unsigned char* const Ks = cur;
    const unsigned char* const Vs = cur + kTileBytes;
    const bool two = k0 + 32 < kend && (!CAUSAL || k0 + 32 <= w0 + 31);      // wave-uniform
    f32x16 st[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) st[t][r] = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
      if (t == 0 || two) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) st[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(srows(Ks, 32 * t, ks, lane), qf[ks], st[t], 0, 0, 0);
      }
    float mloc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kb = k0 + 32 * t;
      if (kb + 32 > klen || (CAUSAL && kb + 31 > w0)) {      // wave-uniform
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb + tile_row(r, lane);
          st[t][r] = (key < klen && (!CAUSAL || key <= q)) ? st[t][r] : -3.0e38f;      // its exponential is 0: m2 is -1e30 at least
        }
      }
      mloc[t] = st[t][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mloc[t] = fmaxf(mloc[t], st[t][r]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) mloc[t] = fmaxf(mloc[t], __shfl_xor(mloc[t], 32));
    float alpha[2], ps[2];
    bool moved[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float mn = (t == 0 || two) ? fmaxf(m2, mloc[t] * SCALE2) : m2;
      alpha[t] = fast_exp2(m2 - mn);
      moved[t] = __any(mn != m2);      // otherwise every lane's factor is 1
      m2 = mn;
      ps[t] = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        st[t][r] = fast_exp2(fmaf(st[t][r], SCALE2, -mn));
        ps[t] += st[t][r];
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
      if (t == 0 || two) {
        if (moved[t]) {
          lsum *= alpha[t];
#pragma unroll
          for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] *= alpha[t];
        }
        lsum += ps[t];
        if (DROP) {      // the row sum keeps every key, the value sum only the survivors (scaled)
          f32x16 f;
          drop_tile_keys(drop, site, (((uint64_t)b * a.A + h) * a.Lq + q) * (uint64_t)a.Lk, k0 + 32 * t, lane, f);
#pragma unroll
          for (int r = 0; r < 16; ++r) st[t][r] *= f[r];
        }
        const bf16x8 p0 = pack8(st[t], 0), p1 = pack8(st[t], 1);
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Vs, 32 * t, 0, 32 * db, lane), p0, o[db], 0, 0, 0);
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Vs, 32 * t, 1, 32 * db, lane), p1, o[db], 0, 0, 0);
        }
      }
  };
  // (one copy of the step: a second one for the other stage made launches over short sequences 1 us longer, and took more registers)
  for (int k0 = 0, at = 0; k0 < kend; k0 += 64, at = kStageBytes - at) step(k0, lds + at, lds + kStageBytes - at);
  lsum += __shfl_xor(lsum, 32);
  if (q < qrows && lane < 32) lse[((int64_t)b * a.A + h) * a.Lq + q] = (m2 + __log2f(lsum)) * LN2;
  __syncthreads();      // every wave is done with the stages
  store_wave_rows(out + qbase * H + h * DH, H, w0, qrows, o, 1.0f / lsum, lane, (bf16*)lds + wave * 32 * LDT, wide);
}

// dq and dvec[q] = sum_d dO[q,d] O[q,d]
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void stream_bwd_dq_mfma(View a, const bf16* __restrict__ out, const float* __restrict__ lse,
                                                       const bf16* __restrict__ d_out, bf16* __restrict__ dq, int64_t lddq,
                                                       float* __restrict__ dvec, bool wide, DropCfg drop, uint32_t site) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kStageBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, h, row0;
  block_place(b, h, row0);
  const int H = a.A * DH;
  const int klen = clamp_len(a.klens[b], a.Lk), qlen = clamp_len(a.qlens[b], a.Lq), qrows = row_count(a.qfirst, qlen, a.Lq);
  if (row0 >= qrows) return;      // block-uniform
  const int64_t qbase = first_row(a.qfirst, b, a.Lq), kbase = first_row(a.kfirst, b, a.Lk);
  const int w0 = row0 + wave * 32, q = w0 + (lane & 31);
  const int kend = row0 >= qlen ? 0 : (CAUSAL ? min(klen, row0 + 128) : klen);
  Stream ks_, vs_;
  ks_.init((const bf16*)a.k + kbase * a.ldkv + h * DH, a.ldkv, lane, wave);
  vs_.init((const bf16*)a.v + kbase * a.ldkv + h * DH, a.ldkv, lane, wave);
  auto request = [&](int k0, unsigned char* __restrict__ st) __attribute__((always_inline)) {
    ks_.issue(k0, klen, st, wave);
    vs_.issue(k0, klen, st + kTileBytes, wave);
  };
  if (kend > 0) request(0, lds);

  // padded queries (q >= qlen) own all-zero fragments and therefore produce zero rows
  bf16x8 qf[4], gf[4];
  float drow = 0.f;
  const bf16* const go = d_out + qbase * H + h * DH;
  const bf16* const oo = out + qbase * H + h * DH;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    qf[ks] = frag_rows_global((const bf16*)a.q + qbase * a.ldq + h * DH, a.ldq, q, qlen, ks, lane);
    gf[ks] = frag_rows_global(go, H, q, qlen, ks, lane);
    const bf16x8 of = frag_rows_global(oo, H, q, qlen, ks, lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) drow = fmaf((float)gf[ks][e], (float)of[e], drow);
  }
  drow += __shfl_xor(drow, 32);
  const float st0 = (q < qlen) ? lse[((int64_t)b * a.A + h) * a.Lq + q] * -8.0f : 0.f;      // 8: the scores are not scaled yet
  f32x16 acc[2];
  clear(acc);

  auto step = [&](int k0, const unsigned char* __restrict__ cur, unsigned char* __restrict__ nxt) __attribute__((always_inline)) {
    stage_barrier();
    if (k0 + 64 < kend) request(k0 + 64, nxt);
    const unsigned char* const Ks = cur;
    const unsigned char* const Vs = cur + kTileBytes;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kb = k0 + 32 * t;
      if (kb < kend && w0 < qlen && (!CAUSAL || kb <= w0 + 31)) {      // wave-uniform
        f32x16 st, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) { st[r] = st0; dp[r] = DROP ? 0.f : -drow; }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(srows(Ks, 32 * t, ks, lane), qf[ks], st, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(srows(Vs, 32 * t, ks, lane), gf[ks], dp, 0, 0, 0);
        }
        if (DROP) {
          f32x16 f;
          drop_tile_keys(drop, site, (((uint64_t)b * a.A + h) * a.Lq + q) * (uint64_t)a.Lk, kb, lane, f);
#pragma unroll
          for (int r = 0; r < 16; ++r) dp[r] = fmaf(dp[r], f[r], -drow);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = fast_exp2(st[r] * SCALE2);
        if (kb + 32 > klen || w0 + 32 > qlen || (CAUSAL && kb + 31 > w0)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = kb + tile_row(r, lane);
            st[r] = (key < klen && q < qlen && (!CAUSAL || key <= q)) ? st[r] : 0.f;
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] *= dp[r];
        const bf16x8 s0 = pack8(st, 0), s1 = pack8(st, 1);
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Ks, 32 * t, 0, 32 * db, lane), s0, acc[db], 0, 0, 0);
          acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Ks, 32 * t, 1, 32 * db, lane), s1, acc[db], 0, 0, 0);
        }
      }
    }
  };
  for (int k0 = 0, at = 0; k0 < kend; k0 += 64, at = kStageBytes - at) step(k0, lds + at, lds + kStageBytes - at);
  if (q < a.Lq && lane < 32) dvec[((int64_t)b * a.A + h) * a.Lq + q] = drow;
  __syncthreads();      // every wave is done with the stages
  store_wave_rows(dq + qbase * lddq + h * DH, lddq, w0, qrows, acc, 0.125f, lane, (bf16*)lds + wave * 32 * LDT, wide);
}

// wave owns 32 keys, streams queries / output gradients and the two numbers of each query -> dk, dv
template <bool CAUSAL, bool DROP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void stream_bwd_dkv_mfma(View a, const float* __restrict__ lse, const bf16* __restrict__ d_out,
                                                        const float* __restrict__ dvec, bf16* __restrict__ dk_out,
                                                        bf16* __restrict__ dv_out, int64_t lddkv, bool wide, DropCfg drop, uint32_t site) {
  constexpr int kStage = kStageBytes + 2 * 64 * (int)sizeof(float);
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kStage];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, h, row0;
  block_place(b, h, row0);
  const int H = a.A * DH;
  const int klen = clamp_len(a.klens[b], a.Lk), qlen = clamp_len(a.qlens[b], a.Lq), krows = row_count(a.kfirst, klen, a.Lk);
  if (row0 >= krows) return;      // block-uniform
  const int64_t qbase = first_row(a.qfirst, b, a.Lq), kbase = first_row(a.kfirst, b, a.Lk);
  const int w0 = row0 + wave * 32, kj = w0 + (lane & 31);       // the key this lane owns
  const int qend = row0 >= klen ? 0 : qlen;
  Stream qs_, gs_;
  qs_.init((const bf16*)a.q + qbase * a.ldq + h * DH, a.ldq, lane, wave);
  gs_.init(d_out + qbase * H + h * DH, H, lane, wave);
  const float* const row_num = (wave == 0 ? lse : dvec) + ((int64_t)b * a.A + h) * a.Lq;
  auto request = [&](int q0, unsigned char* __restrict__ st) __attribute__((always_inline)) {
    qs_.issue(q0, qlen, st, wave);
    gs_.issue(q0, qlen, st + kTileBytes, wave);
    if (wave < 2) {      // one of the two numbers of 64 queries, zero beyond the last
      const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(row_num + q0), 0, min(64, qlen - q0) * 4, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(st + kStageBytes + wave * 256), 4, lane * 4, 0, 0, 0);
    }
  };
  // queries before the block's first key never see it when causal (block-uniform start)
  const int qbeg = CAUSAL ? row0 : 0;
  if (qbeg < qend) request(qbeg, lds);

  bf16x8 kf[4], vf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    kf[ks] = frag_rows_global((const bf16*)a.k + kbase * a.ldkv + h * DH, a.ldkv, kj, klen, ks, lane);
    vf[ks] = frag_rows_global((const bf16*)a.v + kbase * a.ldkv + h * DH, a.ldkv, kj, klen, ks, lane);
  }
  f32x16 dk[2], dv[2];
  clear(dk);
  clear(dv);

  auto step = [&](int q0, const unsigned char* __restrict__ cur, unsigned char* __restrict__ nxt) __attribute__((always_inline)) {
    stage_barrier();
    if (q0 + 64 < qend) request(q0 + 64, nxt);
    const unsigned char* const Qs = cur;
    const unsigned char* const Gs = cur + kTileBytes;
    const float* const lse_s = (const float*)(cur + kStageBytes);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int qb = q0 + 32 * t;
      if (qb < qend && w0 < klen && (!CAUSAL || qb + 31 >= w0)) {      // wave-uniform
        f32x16 st, dp, dvr;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 lv = *(const f32x4*)(lse_s + 32 * t + 8 * g + 4 * (lane >> 5));
          const f32x4 dvv = *(const f32x4*)(lse_s + 64 + 32 * t + 8 * g + 4 * (lane >> 5));
#pragma unroll
          for (int e = 0; e < 4; ++e) { st[4 * g + e] = -8.0f * lv[e]; dvr[4 * g + e] = -dvv[e]; }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] = DROP ? 0.f : dvr[r];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(srows(Qs, 32 * t, ks, lane), kf[ks], st, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(srows(Gs, 32 * t, ks, lane), vf[ks], dp, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = fast_exp2(st[r] * SCALE2);
        if (qb + 32 > qlen || w0 + 32 > klen || (CAUSAL && qb < w0 + 31)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int qi = qb + tile_row(r, lane);
            st[r] = (qi < qlen && kj < klen && (!CAUSAL || kj <= qi)) ? st[r] : 0.f;
          }
        }
        if (DROP) {
          f32x16 f;
          drop_tile_queries(drop, site, ((uint64_t)b * a.A + h) * a.Lq, a.Lk, qb, kj, lane, f);
#pragma unroll
          for (int r = 0; r < 16; ++r) { dp[r] = st[r] * fmaf(f[r], dp[r], dvr[r]); st[r] *= f[r]; }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) dp[r] *= st[r];
        }
        const bf16x8 p0 = pack8(st, 0), p1 = pack8(st, 1), s0 = pack8(dp, 0), s1 = pack8(dp, 1);
#pragma unroll
        for (int db = 0; db < 2; ++db) {
          dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Gs, 32 * t, 0, 32 * db, lane), p0, dv[db], 0, 0, 0);
          dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Gs, 32 * t, 1, 32 * db, lane), p1, dv[db], 0, 0, 0);
          dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Qs, 32 * t, 0, 32 * db, lane), s0, dk[db], 0, 0, 0);
          dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(scols_t(Qs, 32 * t, 1, 32 * db, lane), s1, dk[db], 0, 0, 0);
        }
      }
    }
  };
  for (int q0 = qbeg, at = 0; q0 < qend; q0 += 64, at = kStage - at) step(q0, lds + at, lds + kStage - at);
  __syncthreads();      // every wave is done with the stages
  bf16* const area = (bf16*)lds + wave * 32 * LDT;
  store_wave_rows(dk_out + kbase * lddkv + h * DH, lddkv, w0, krows, dk, 0.125f, lane, area, wide);
  store_wave_rows(dv_out + kbase * lddkv + h * DH, lddkv, w0, krows, dv, 1.0f, lane, area, wide);
}

View make_view(const AttnOperands& x) {
  View v;
  v.q = x.q; v.k = x.k; v.v = x.v; v.ldq = x.ldq; v.ldkv = x.ldkv; v.qlens = x.qlens; v.klens = x.klens;
  v.Lq = x.Lq; v.Lk = x.Lk; v.A = x.A; v.qfirst = x.qfirst; v.kfirst = x.kfirst;
  return v;
}

const DropCfg kNoDrop{0u, 1.0f, 0u, 0u, 0u};

bool wide_rows(const void* p, int64_t ld) { return !((uintptr_t)p & 15) && !(ld & 7); }

void stream_fwd(const AttnOperands& x, int B, void* out, float* lse, hipStream_t s, const DropCfg& drop, uint32_t site) {
  const View v = make_view(x);
  const bool wide = wide_rows(out, 8);
  const dim3 grid((x.Lq + 127) / 128, x.A, B);
  if (x.causal) hipLaunchKernelGGL((stream_fwd_mfma<true, false>), grid, dim3(256), 0, s, v, (bf16*)out, lse, wide, kNoDrop, 0u);
  else if (drop.thr) hipLaunchKernelGGL((stream_fwd_mfma<false, true>), grid, dim3(256), 0, s, v, (bf16*)out, lse, wide, drop, site);
  else hipLaunchKernelGGL((stream_fwd_mfma<false, false>), grid, dim3(256), 0, s, v, (bf16*)out, lse, wide, kNoDrop, 0u);
}

void stream_bwd(const AttnOperands& x, int B, const void* out, const float* lse, const void* d_out, void* dq, int64_t lddq, void* dk, void* dv,
                int64_t lddkv, float* dvec, hipStream_t s, const DropCfg& drop, uint32_t site) {
  if (attention_bwd_is_short(x, dq, lddq, dk, dv, lddkv)) {
    launch_attention_bwd_short(x, B, out, lse, d_out, dq, lddq, dk, dv, lddkv, s, drop, site);
    return;
  }
  const View v = make_view(x);
  const bool wq = wide_rows(dq, lddq), wkv = wide_rows(dk, lddkv) && wide_rows(dv, lddkv);
  const dim3 gq((x.Lq + 127) / 128, x.A, B), gk((x.Lk + 127) / 128, x.A, B);
#define HS_STREAM_BWD(CAUSAL, DROP, D, SITE)                                                                                                \
  do {                                                                                                                                      \
    hipLaunchKernelGGL((stream_bwd_dq_mfma<CAUSAL, DROP>), gq, dim3(256), 0, s, v, (const bf16*)out, lse, (const bf16*)d_out, (bf16*)dq,    \
                       lddq, dvec, wq, D, SITE);                                                                                            \
    hipLaunchKernelGGL((stream_bwd_dkv_mfma<CAUSAL, DROP>), gk, dim3(256), 0, s, v, lse, (const bf16*)d_out, (const float*)dvec, (bf16*)dk, \
                       (bf16*)dv, lddkv, wkv, D, SITE);                                                                                     \
  } while (0)
  if (x.causal) HS_STREAM_BWD(true, false, kNoDrop, 0u);
  else if (drop.thr) HS_STREAM_BWD(false, true, drop, site);
  else HS_STREAM_BWD(false, false, kNoDrop, 0u);
#undef HS_STREAM_BWD
}

AttnOperands self_operands(const void* qkv, const int32_t* lens, int L, int A, const int32_t* first) {
  const bf16* q = (const bf16*)qkv;
  const int64_t H = (int64_t)A * DH;
  return AttnOperands{q, q + H, q + 2 * H, 3 * H, 3 * H, lens, lens, L, L, A, 0, first, first};
}

AttnF32 f32_problem(const AttnOperands& x) {
  return AttnF32{(const float*)x.q, (const float*)x.k, (const float*)x.v, x.ldq, x.ldkv, x.qlens, x.klens, x.Lq, x.Lk, x.A, x.causal,
                 DropCfg{0u, 1.0f, 0u, 0u, 0u}, 0};
}

hs_status check_operands(hs_ctx* ctx, int dtype, const AttnOperands& x, const char* who) {
  if (x.A < 1 || x.Lq < 1 || x.Lk < 1) return hs_fail(ctx, HS_ERR_INVALID_ARG, std::string(who) + ": bad size");
  if (x.causal && x.Lq != x.Lk) return hs_fail(ctx, HS_ERR_SHAPE, std::string(who) + ": causal attention needs Lq == Lk");
  if (!x.q || !x.k || !x.v || !x.qlens || !x.klens) return hs_fail(ctx, HS_ERR_INVALID_ARG, std::string(who) + ": NULL operand");
  const int64_t H = (int64_t)x.A * 64;
  if (x.ldq < H || x.ldkv < H) return hs_fail(ctx, HS_ERR_SHAPE, std::string(who) + ": row stride smaller than A*64");
  if (dtype != HS_BF16 && (x.qfirst || x.kfirst)) return hs_fail(ctx, HS_ERR_UNIMPLEMENTED, std::string(who) + ": packed rows in bf16 only");
  if (dtype == HS_BF16) {       // 16-byte fragment loads
    if ((x.ldq & 7) || (x.ldkv & 7) || ((uintptr_t)x.q & 15) || ((uintptr_t)x.k & 15) || ((uintptr_t)x.v & 15))
      return hs_fail(ctx, HS_ERR_SHAPE, std::string(who) + ": bf16 operands must be 16-byte aligned with strides that are multiples of 8");
  }
  return HS_OK;
}

}  // namespace

hs_status launch_attention_general_fwd(hs_ctx* ctx, int dtype, const AttnOperands& x, int B, void* out, float* lse, hipStream_t s) {
  if (B <= 0) return HS_OK;
  hs_status st = check_operands(ctx, dtype, x, "attention_general_fwd");
  if (st != HS_OK) return st;
  const double pairs = (double)B * x.A * x.Lq * x.Lk * (x.causal ? 0.5 : 1.0);
  KScope scope(ctx ? ctx->prof : nullptr, KC_ATTN_FWD, 4.0 * pairs * 64, (double)B * x.A * 64 * (2.0 * x.Lq + 2.0 * x.Lk) * esize(dtype), s);
  if (dtype == HS_BF16) {
    stream_fwd(x, B, out, lse, s, kNoDrop, 0);
  } else {
    launch_attention_f32_fwd(f32_problem(x), B, (float*)out, lse, s);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("attention_general_fwd: ") + hipGetErrorString(e));
  return HS_OK;
}

hs_status launch_attention_general_bwd(hs_ctx* ctx, int dtype, const AttnOperands& x, int B, const void* out, const float* lse,
                                       const void* d_out, void* dq, int64_t lddq, void* dk, void* dv, int64_t lddkv, float* dvec,
                                       hipStream_t s) {
  if (B <= 0) return HS_OK;
  hs_status st = check_operands(ctx, dtype, x, "attention_general_bwd");
  if (st != HS_OK) return st;
  if (!out || !lse || !d_out || !dq || !dk || !dv || !dvec) return hs_fail(ctx, HS_ERR_INVALID_ARG, "attention_general_bwd: NULL buffer");
  if (dtype == HS_BF16 && ((lddq & 3) || (lddkv & 3) || ((uintptr_t)dq & 7) || ((uintptr_t)dk & 7) || ((uintptr_t)dv & 7)))
    return hs_fail(ctx, HS_ERR_SHAPE, "attention_general_bwd: bf16 gradients must be 8-byte aligned with strides that are multiples of 4");
  const double pairs = (double)B * x.A * x.Lq * x.Lk * (x.causal ? 0.5 : 1.0);
  KScope scope(ctx ? ctx->prof : nullptr, KC_ATTN_BWD, 8.0 * pairs * 64, (double)B * x.A * 64 * (4.0 * x.Lq + 4.0 * x.Lk) * esize(dtype), s);
  if (dtype == HS_BF16) {
    stream_bwd(x, B, out, lse, d_out, dq, lddq, dk, dv, lddkv, dvec, s, kNoDrop, 0);
  } else {
    launch_attention_f32_bwd(f32_problem(x), B, (const float*)out, lse, (const float*)d_out, (float*)dq, lddq, (float*)dk, (float*)dv, lddkv, s);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("attention_general_bwd: ") + hipGetErrorString(e));
  return HS_OK;
}

// bf16 self-attention over packed q | k | v rows (see attention.hip)
void launch_attention_self_fwd(const void* qkv, const int32_t* lens, int B, int L, int A, void* out, float* lse, hipStream_t s, const DropCfg& drop,
                               uint32_t site, const int32_t* first) {
  stream_fwd(self_operands(qkv, lens, L, A, first), B, out, lse, s, drop, site);
}
void launch_attention_self_bwd(const void* qkv, const void* out, const float* lse, const void* d_out, const int32_t* lens, int B, int L, int A,
                               void* dqkv, float* dvec, hipStream_t s, const DropCfg& drop, uint32_t site, const int32_t* first) {
  const int64_t H = (int64_t)A * DH;
  bf16* const d = (bf16*)dqkv;
  stream_bwd(self_operands(qkv, lens, L, A, first), B, out, lse, d_out, d, 3 * H, d + H, d + 2 * H, 3 * H, dvec, s, drop, site);
}
