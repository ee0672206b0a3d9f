// bf16 MFMA GEMM kernel whose operand tiles go from global memory straight into LDS (template); instantiated per
// operand layout in gemm_wide_*.hip beside the wide kernels, with which it shares fragments' layout and epilogues.
#pragma once
#include "gemm_wide.h"

namespace {

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel with direct global -> LDS operand loads
// ------------------------------------------------------------------------------------------
// Block tile (32 TI WGM) x (32 TJ WGN) x BK; WGM x WGN waves of TI x TJ MFMA tiles, times KW groups of waves that share a
// k-tile's 16-deep slices (group g takes slices g, g + KW, ...; the groups' sums are added in group order through LDS).
// A k-tile is fetched by buffer loads that write LDS themselves (16 bytes per lane, one instruction fills 1 KiB of LDS in
// lane order), so that an operand byte never passes through a register and no LDS store instruction is issued.  S stages
// of LDS form a ring, one barrier per k-tile: the tile for k-step t + S - 1 is requested when step t starts or (AHEAD, see ahead_step)
// the one for step t + S before its last slice.  What orders
// the loads against their readers is the wave's own load counter (the hardware retires these loads in order) followed by
// the barrier; both are written out by hand here, because a fence would make every wave wait for all of its loads.
//
// One instruction's 64 lanes land in consecutive 16-byte slots, so the bank-conflict-free LDS layouts are made on
// the global side: the lane that fills slot p of a row fetches the chunk whose number is p XOR a function of the row.
//   k-major operand ([rows, K], a row of the tile is BK contiguous elements): the layout of WideTile, rows
//     unpadded, chunk ^ ((row >> 1) & 7) for BK = 64 and chunk ^ ((row >> 2) & 3) for BK = 32.
//   m-major operand ([K, rows], a row of the tile is R contiguous elements of one contraction index k): a transposing read
//     takes 64 bytes of each of four k-rows at once.  R = 128, 256: chunk ^ ((k & 3) << 2) puts the four into four different
//     64-byte bank groups; R = 64, 192: two k-rows already lie apart, chunk ^ (((k >> 1) & 1) << 2) parts the others;
//     R = 32: the four k-rows are one 256-byte line as they are.
// Small tiles are for products with few of them, where the rate at which a CU is fed does not matter yet: 2048 x 768 x 768 with
// 64 x 64 tiles 7.5 us (128 x 128: 11.6), 1024 x 768 x 3072 14.4 us (34), 512 x 768 x 3072 with 32 x 64 tiles 10.6 us (33).
// From about two 128 x 128 tiles per CU on the feed from the L2 binds (8192 x 3072 x 3072: 106 us, its loads alone 103 us,
// everything but the loads 82 us; 39 bytes per clock and CU), and only the larger tile helps: 256 x 256 (8 waves of 128 x 64, the whole register
// file and 128 KB of LDS) needs half the bytes per flop of 128 x 128, 256 x 128 and 128 x 192 three quarters.  8192^3: 1339, 1236 and
// 1169 TFLOP/s (128 x 192 at 90 % of its rounds), 128 x 128 1132; at the first of these the chip's clock is what binds.
// Rows beyond the matrix edge are clamped to the last row (their products are never stored).  A k-tile that reaches beyond
// the contraction range reads zeros there: rows of an m-major operand beyond K lie behind the end of the operand, where a
// buffer load returns zero; a k-major operand has to end on a whole k-tile or be zero up to there (the launcher checks).
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// R: rows of the tile; NW: waves of the block, which share the tile's load instructions evenly
template <bool KMAJ, int BK, int R, int NW>
struct DmaTile {
  static_assert(BK == 32 || BK == 64, "k-tile of 32 or 64");
  static_assert(R == 32 || R == 64 || R == 128 || R == 192 || R == 256, "32 to 256 rows");
  static constexpr int BYTES = R * BK * 2;
  static constexpr int NI = BYTES / 1024 / NW;         // load instructions per wave and k-tile
  static_assert(NI >= 1 && NI * NW * 1024 == BYTES, "the tile must split evenly over the waves");
  static constexpr int CPR = BK / 8;                   // k-major: chunks per row
  static constexpr int RPI = 64 / CPR;                 // k-major: rows per instruction
  static constexpr int RPF = KMAJ ? 1 : 2;             // LDS reads per fragment
  static __device__ __forceinline__ int mswz(int k) { return R == 128 || R == 256 ? ((k & 3) << 2) : (R == 64 || R == 192 ? (((k >> 1) & 1) << 2) : 0); }
  struct Cursor {
    __amdgpu_buffer_rsrc_t rsrc;
    unsigned off[NI];
    unsigned soff, step;
  };
  static __device__ __forceinline__ void init(Cursor& cu, const bf16* __restrict__ mat, int64_t ld, int row0, int rext, int kbeg, int K, int lane,
                                              int wave) {
    const int64_t rows = KMAJ ? rext : K, cols = KMAJ ? K : rext;
    const int64_t bytes = ((rows - 1) * ld + ((cols + 7) & ~(int64_t)7)) * 2;
    cu.rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)mat, 0, (int)(unsigned)bytes, 0x00020000);
    cu.step = (unsigned)(KMAJ ? (int64_t)BK * 2 : (int64_t)BK * ld * 2);
    cu.soff = (unsigned)(KMAJ ? (int64_t)kbeg * 2 : (int64_t)kbeg * ld * 2);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int j = wave * NI + i;
      if (KMAJ) {
        const int row = j * RPI + lane / CPR, slot = lane % CPR;
        const int chunk = slot ^ (BK == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3));
        const int r = min(row0 + row, rext - 1);
        cu.off[i] = (unsigned)(((int64_t)r * ld + chunk * 8) * 2);
      } else {
        const int id = j * 64 + lane, k = id / (R / 8), slot = id % (R / 8);
        const int chunk = slot ^ mswz(k);
        const int n = min(row0 + chunk * 8, ((rext - 1) >> 3) << 3);
        cu.off[i] = (unsigned)(((int64_t)k * ld + n) * 2);
      }
    }
  }
  // request the cursor's k-tile into the tile at dst (wave-uniform) and advance
  static __device__ __forceinline__ void issue(Cursor& cu, unsigned char* __restrict__ dst, int wave) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(cu.rsrc, (lds_void_ptr)(dst + (wave * NI + i) * 1024), 16, (int)cu.off[i], (int)cu.soff, 0, 0);
    cu.soff += cu.step;
  }
  // LDS -> MFMA operand: lane gets elements (row = rbase + lane%32, k = ks*16 + 8*(lane/32) + 0..7)
  static __device__ __forceinline__ bf16x8 frag(const bf16* __restrict__ s, int rbase, int ks, int lane) {
    if (KMAJ) {
      const int row = rbase + (lane & 31), chunk = ks * 2 + (lane >> 5);
      return *(const bf16x8*)(s + row * BK + (chunk ^ (BK == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3))) * 8);
    } else {
      const int kb = ks * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
      const int nb = rbase + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      const int pos = kb * R + (((nb >> 3) ^ mswz(kb)) << 3) + (nb & 7);     // kb + 4 has the same swizzle
      typedef s16x4 __attribute__((address_space(3))) * lds_v4;
      union { struct { s16x4 lo, hi; } p; bf16x8 v; } u;
      u.p.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(s + pos));
      u.p.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(s + pos + 4 * R));
      return u.v;
    }
  }
};

// The tile shape and pipeline of one configuration.
template <int TI_, int TJ_, int WGM_, int WGN_, int KW_, int BK_, int S_, int OCC_, bool AHEAD_>
struct DmaCfg {
  static constexpr int TI = TI_, TJ = TJ_, WGM = WGM_, WGN = WGN_, KW = KW_, BK = BK_, S = S_, OCC = OCC_;   // OCC: blocks per CU
  static constexpr int NS = WGM * WGN, NW = NS * KW, NT = 64 * NW, BM = 32 * TI * WGM, BN = 32 * TJ * WGN;
  static constexpr int STAGE = (BM + BN) * BK * 2;                      // bytes of a k-tile of both operands
  static constexpr int EPI_FLOATS = 32 * (32 * TJ + 4);                 // a wave's epilogue staging area
  static constexpr size_t RED = (size_t)(KW - 1) * NS * TI * TJ * 16 * 64 * sizeof(float);
  static constexpr size_t EPI_BYTES = (size_t)NS * EPI_FLOATS * sizeof(float) + kGeluTabN * sizeof(float2);
  static constexpr size_t PIPE = (size_t)S * STAGE;
  static constexpr size_t LDS = PIPE > EPI_BYTES ? (PIPE > RED ? PIPE : RED) : (EPI_BYTES > RED ? EPI_BYTES : RED);
  static constexpr int WPE = OCC * NW / 4;                              // waves per SIMD
  static constexpr bool AHEAD = AHEAD_;                                 // fragments read a slice ahead (see ahead_step)
  static_assert(!AHEAD || KW == 1, "all slices of a k-tile in every wave");
  static_assert(S >= 2 && S <= 16, "two to sixteen stages");
  static_assert(BK / 16 % KW == 0, "the k-slices must split evenly over the wave groups");
  static_assert(LDS * OCC <= 160 * 1024, "stages do not fit the LDS of a CU");
};

// s_waitcnt: the wave's vector-memory loads except the newest VM have completed, and so have all its LDS reads
template <int VM>
__device__ __forceinline__ void wait_loads() {
  static_assert(VM >= 0 && VM < 64, "6-bit counter");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x70);
}
// ... with the number of k-tiles that may still be in flight known at run time only (0 .. MAX)
template <int PER, int MAX>
__device__ __forceinline__ void wait_tiles(int ahead) {
  if constexpr (MAX == 0) wait_loads<0>();
  else { if (ahead >= MAX) wait_loads<MAX * PER>(); else wait_tiles<PER, MAX - 1>(ahead); }
}

__device__ __forceinline__ bf16x8 ones_frag() {
  const bf16 one = (bf16)1.0f;
  return bf16x8{one, one, one, one, one, one, one, one};
}

// One k-step: tile `cur` is read (after the wave's share of it has landed and every wave has arrived), the tile
// S - 1 steps ahead is requested into `nxt`, whose last readers passed the same barrier.
template <class C, class TA, class TB>
__device__ __forceinline__ void dma_step(typename TA::Cursor& ca, typename TB::Cursor& cb, unsigned char* __restrict__ nxt,
                                         const unsigned char* __restrict__ cur, f32x16 (&acc)[C::TI][C::TJ], int ahead, bool request, int wm,
                                         int wn, int kg, int lane, int wave) {
  constexpr int KS = C::BK / 16 / C::KW;
  asm volatile("" ::: "memory");      // no LDS access of the step before moves below the barrier, none of this step above it
  wait_tiles<TA::NI + TB::NI, C::S - 2>(ahead);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (request) {
    TA::issue(ca, nxt, wave);
    TB::issue(cb, nxt + TA::BYTES, wave);
  }
  const bf16* sA = (const bf16*)cur;
  const bf16* sB = (const bf16*)(cur + TA::BYTES);
  bf16x8 fa[KS][C::TI], fb[KS][C::TJ];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
    for (int i = 0; i < C::TI; ++i) fa[ks][i] = TA::frag(sA, (wm * C::TI + i) * 32, ks * C::KW + kg, lane);
#pragma unroll
    for (int j = 0; j < C::TJ; ++j) fb[ks][j] = TB::frag(sB, (wn * C::TJ + j) * 32, ks * C::KW + kg, lane);
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int i = 0; i < C::TI; ++i)
#pragma unroll
      for (int j = 0; j < C::TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
}

// fragments of 16-deep slice ks of the k-tile at st
template <class C, class TA, class TB, bool RS>
__device__ __forceinline__ void read_slice(bf16x8 (&fa)[C::TI], bf16x8 (&fb)[C::TJ], bf16x8& fr, const unsigned char* __restrict__ st, int ks,
                                           int wm, int wn, int lane) {
  const bf16* sA = (const bf16*)st;
  const bf16* sB = (const bf16*)(st + TA::BYTES);
#pragma unroll
  for (int i = 0; i < C::TI; ++i) fa[i] = TA::frag(sA, (wm * C::TI + i) * 32, ks, lane);
#pragma unroll
  for (int j = 0; j < C::TJ; ++j) fb[j] = TB::frag(sB, (wn * C::TJ + j) * 32, ks, lane);
  if (RS) fr = TA::frag(sA, (wm * C::TI + wn % C::TI) * 32, ks, lane);
}

// One k-step of the pipeline that reads fragments one 16-deep slice ahead.  On entry fragment set 0 holds slice 0 of tile `cur`.  The
// barrier sits before the last slice: by then every wave has read all of `cur`, which the tile S steps ahead is requested into, and the
// wave's share of `nxt` has landed; the last slice's MFMAs cover the meeting and the first fragment reads of `nxt`.  The issue order
// per MFMA is prescribed.  RS: fr / accr as described at dma_tile.
template <class C, class TA, class TB, bool RS>
__device__ __forceinline__ void ahead_step(typename TA::Cursor& ca, typename TB::Cursor& cb, unsigned char* __restrict__ cur,
                                           const unsigned char* __restrict__ nxt, bf16x8 (&fa)[2][C::TI], bf16x8 (&fb)[2][C::TJ], bf16x8 (&fr)[2],
                                           f32x16 (&acc)[C::TI][C::TJ], f32x16& accr, int wm, int wn, int lane, int wave) {
  constexpr int KS = C::BK / 16, TI = C::TI, TJ = C::TJ, NM = TI * TJ, NL = TA::NI + TB::NI;
  constexpr int NF = TI + TJ, FPM = (NF + NM - 1) / NM;      // fragments per slice, and per MFMA
  static_assert(KS % 2 == 0, "fragment sets alternate");
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int fc = s & 1, fn = fc ^ 1;
    const bool last = s == KS - 1;
    if (last) {
      asm volatile("" ::: "memory");
      wait_loads<(C::S - 2) * NL>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    read_slice<C, TA, TB, RS>(fa[fn], fb[fn], fr[fn], last ? nxt : (const unsigned char*)cur, last ? 0 : s + 1, wm, wn, lane);
    if (last) {
      TA::issue(ca, cur, wave);
      TB::issue(cb, cur + TA::BYTES, wave);
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[fc][i], fb[fc][j], acc[i][j], 0, 0, 0);
    if (RS) {
      accr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[fc], ones_frag(), accr, 0, 0, 0);
    } else {
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                       // MFMA
#pragma unroll
        for (int f = q * FPM; f < (q + 1) * FPM && f < NF; ++f) {                                // fragment reads of the next slice
          if (f < TI) __builtin_amdgcn_sched_group_barrier(0x100, TA::RPF, 0);
          else __builtin_amdgcn_sched_group_barrier(0x100, TB::RPF, 0);
        }
        if (last) __builtin_amdgcn_sched_group_barrier(0x020, (NL + NM - 1) / NM, 0);            // loads
      }
    }
  }
}

// ROWSUM: where p.rowsum is set, the block also adds up the rows of A (a bias gradient beside the weight gradient of the same
// operand): wave column wn takes the wn-th 32 rows of its waves' TI x 32 with one more MFMA per slice, against a column of ones.  Those blocks run
// without the prescribed issue order.  What the row sums cost, one launch after the other: 2 % of the weight gradients of 8192 x 768 (1.57 ms with, 1.54 without), 6 % of
// those of 16384 x 1024 (39.9, 37.4 over four passes); in the step 0 and 0.3 of 145 ms.  As products with a column of ones they were 10 % of the tiles.
template <class C, bool AK, bool BKM, int EPIS, bool ROWSUM = false>
__device__ __forceinline__ void dma_tile(const GemmDev& p, int m0, int n0, int split, unsigned char* lds_raw) {
  static_assert(!ROWSUM || C::WGN >= C::TI, "a wave column for each 32 of a wave's rows");
  constexpr int TI = C::TI, TJ = C::TJ, S = C::S;
  typedef DmaTile<AK, C::BK, C::BM, C::NW> TA;
  typedef DmaTile<BKM, C::BK, C::BN, C::NW> TB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / C::NS, ws = wave % C::NS, wm = ws / C::WGN, wn = ws % C::WGN;
  const int kbeg = split * p.k_per_split;
  const int kend = min(p.K, kbeg + p.k_per_split);
  const int nk = (kend - kbeg + C::BK - 1) / C::BK;

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  typename TA::Cursor ca;
  typename TB::Cursor cb;
  TA::init(ca, (const bf16*)p.A, p.lda, m0, p.M, kbeg, p.K, lane, wave);
  TB::init(cb, (const bf16*)p.B, p.ldb, n0, p.N, kbeg, p.K, lane, wave);

  f32x16 accr;      // ROWSUM only
  if constexpr (C::AHEAD) {
    const unsigned past = 0x80000000u;      // as in wide_tile: the requests of the last steps go beyond the operand
    bf16x8 fa[2][TI], fb[2][TJ], fr[2];
    auto flow = [&](auto rs) __attribute__((always_inline)) {
      constexpr bool RS = decltype(rs)::value;
      if (RS) {
#pragma unroll
        for (int r = 0; r < 16; ++r) accr[r] = 0.0f;
      }
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (s >= nk) ca.soff = cb.soff = past;
        TA::issue(ca, lds_raw + s * C::STAGE, wave);
        TB::issue(cb, lds_raw + s * C::STAGE + TA::BYTES, wave);
      }
      asm volatile("" ::: "memory");
      wait_loads<(S - 1) * (TA::NI + TB::NI)>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      read_slice<C, TA, TB, RS>(fa[0], fb[0], fr[0], lds_raw, 0, wm, wn, lane);
      for (int t0 = 0; t0 < nk; t0 += S) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
          const int t = t0 + u;
          if (t < nk) {
            if (t + S >= nk) ca.soff = cb.soff = past;
            ahead_step<C, TA, TB, RS>(ca, cb, lds_raw + u * C::STAGE, lds_raw + ((u + 1) % S) * C::STAGE, fa, fb, fr, acc, accr, wm, wn, lane, wave);
          }
        }
      }
    };
    if constexpr (ROWSUM) { if (p.rowsum) flow(std::true_type{}); else flow(std::false_type{}); }
    else flow(std::false_type{});
  } else {
    static_assert(!ROWSUM, "row sums go with fragments read ahead");
    // tiles 0 .. S-2 into stages 0 .. S-2
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
      if (s < nk) {
        TA::issue(ca, lds_raw + s * C::STAGE, wave);
        TB::issue(cb, lds_raw + s * C::STAGE + TA::BYTES, wave);
      }
    // Step t reads stage t % S and requests tile t + S - 1 into stage (t - 1) % S.  At its start the wave has requested
    // tiles up to min(t + S - 2, nk - 1): the counter is waited down to the loads of the tiles behind tile t.
    for (int t0 = 0; t0 < nk; t0 += S) {
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const int t = t0 + u;
        if (t < nk)
          dma_step<C, TA, TB>(ca, cb, lds_raw + ((u + S - 1) % S) * C::STAGE, lds_raw + u * C::STAGE, acc, min(S - 2, nk - 1 - t), t + S - 1 < nk,
                              wm, wn, kg, lane, wave);
      }
    }
  }
  asm volatile("" ::: "memory");
  wait_loads<0>();
  __builtin_amdgcn_s_barrier();   // every wave is done with the operand stages: they become the staging area of the epilogue
  asm volatile("" ::: "memory");

  if constexpr (C::KW > 1) {      // the other groups' sums, in group order; a lane reads the 16 bytes that its counterpart wrote
    float4* const red = (float4*)lds_raw;
    if (kg > 0) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            red[((((kg - 1) * C::NS + ws) * TI + i) * TJ + j) * 256 + q * 64 + lane] =
                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int g = 0; g < C::KW - 1; ++g)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 v = red[(((g * C::NS + ws) * TI + i) * TJ + j) * 256 + q * 64 + lane];
              acc[i][j][4 * q] += v.x; acc[i][j][4 * q + 1] += v.y; acc[i][j][4 * q + 2] += v.z; acc[i][j][4 * q + 3] += v.w;
            }
    }
    __syncthreads();
  }

  const int rbase = m0 + wm * TI * 32, cbase = n0 + wn * TJ * 32;
  if constexpr (ROWSUM) {
    if (p.rowsum && wn < TI && (lane & 31) == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = rbase + wn * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row < p.M) p.rowsum[row] = (p.beta != 0.0f) ? p.beta * p.rowsum[row] + accr[r] : accr[r];
      }
    }
  }
  float* stage = (float*)lds_raw + ws * C::EPI_FLOATS;
  float2* const tab = (float2*)((float*)lds_raw + C::NS * C::EPI_FLOATS);
  if (p.gelu_tab && (((EPIS >> EPI_ACT_GELU) | (EPIS >> EPI_ACT_DGELU)) & 1)) {
    for (int i = tid; i < kGeluTabN / 2; i += C::NT) ((float4*)tab)[i] = ((const float4*)p.gelu_tab)[i];
    __syncthreads();
  }
  if (C::KW > 1 && kg > 0) return;
  constexpr auto has = [](int mode) { return (EPIS >> mode) & 1; };
  if (p.partial) { if constexpr (has(EPI_PARTIAL)) tile_epilogue_pipe<EPI_PARTIAL, TI, TJ>(p, acc, rbase, cbase, lane, split, stage, tab); }
  else if (p.c_f32) { if constexpr (has(EPI_F32)) tile_epilogue_pipe<EPI_F32, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
  else if (p.epi == 0) { if constexpr (has(EPI_ACT)) tile_epilogue_pipe<EPI_ACT, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
  else if (p.epi == 1) { if constexpr (has(EPI_ACT_RES)) tile_epilogue_pipe<EPI_ACT_RES, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
  else if (p.epi == 2) { if constexpr (has(EPI_ACT_GELU)) tile_epilogue_pipe<EPI_ACT_GELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
  else if (p.epi == 3) { if constexpr (has(EPI_ACT_DGELU)) tile_epilogue_pipe<EPI_ACT_DGELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
  else if (p.epi == 4) { if constexpr (has(EPI_ACT_RELU)) tile_epilogue_pipe<EPI_ACT_RELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
  else { if constexpr (has(EPI_ACT_DRELU)) tile_epilogue_pipe<EPI_ACT_DRELU, TI, TJ>(p, acc, rbase, cbase, lane, 0, stage, tab); }
}

template <class C, bool AK, bool BKM>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE, C::WPE)))
void gemm_bf16_dma(GemmDev p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  // tile order as in gemm_bf16_wide
  const int nbx = gridDim.x, nby = gridDim.y, nb = nbx * nby;
  int v = (blockIdx.z * nby + blockIdx.y) * nbx + blockIdx.x;
  const int per_xcd = (nb * (int)gridDim.z) >> 3;
  if (v < 8 * per_xcd) v = (v & 7) * per_xcd + (v >> 3);
  const int split = v / nb;
  int tm, tn;
  tile_of_block<(C::BM >= 256) ? 4 : 8>(v - split * nb, nbx, nby, tm, tn);
  dma_tile<C, AK, BKM, wide_epilogues<AK, BKM>()>(p, tm * C::BM, tn * C::BN, split, lds_raw);
}

template <class C, bool AK, bool BKM>
hipError_t launch_dma_one(const GemmDev& p, int splits, hipStream_t s) {
  auto kern = gemm_bf16_dma<C, AK, BKM>;
  static bool configured = false;
  if (!configured && C::LDS > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
    if (e != hipSuccess) return e;
  }
  configured = true;
  hipLaunchKernelGGL(kern, dim3((p.N + C::BN - 1) / C::BN, (p.M + C::BM - 1) / C::BM, splits), dim3(C::NT), C::LDS, s, p);
  return hipSuccess;
}

// several weight-gradient products in one launch (see group_problem)
template <class C>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE, C::WPE)))
void gemm_bf16_dma_group(GemmGroupDev g) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  int tm, tn;
  const GemmDev p = group_problem<C::BM, C::BN>(g, tm, tn);
  dma_tile<C, false, false, 1 << EPI_F32, true>(p, tm * C::BM, tn * C::BN, 0, lds_raw);
}
template <class C>
hipError_t launch_dma_group(const GemmGroupDev& g, hipStream_t s) {
  auto kern = gemm_bf16_dma_group<C>;
  static bool configured = false;
  if (!configured && C::LDS > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
    if (e != hipSuccess) return e;
  }
  configured = true;
  hipLaunchKernelGGL(kern, dim3(g.first_tile[g.n]), dim3(C::NT), C::LDS, s, g);
  return hipSuccess;
}

// the configurations of gemm_bf16_dma that are built (numbers: kTileCfg in gemm.hip)
typedef DmaCfg<1, 1, 1, 2, 2, 64, 4, 3, false> Dma32x64;       // TI TJ WGM WGN KW BK S OCC AHEAD
typedef DmaCfg<1, 1, 2, 2, 1, 64, 3, 3, false> Dma64x64;
typedef DmaCfg<1, 1, 2, 2, 1, 64, 3, 3, true> Dma64x64Group;
typedef DmaCfg<1, 2, 2, 2, 1, 64, 3, 2, true> Dma64x128;
typedef DmaCfg<2, 1, 2, 2, 1, 64, 3, 2, true> Dma128x64;
typedef DmaCfg<2, 2, 2, 2, 1, 64, 2, 2, true> Dma128x128;
// For products of about one tile per CU and a long contraction: twice the waves of Dma128x128, which cover each other's reads and waits where no second block
// does, and a ring of four; 64 x 64 with fragments read ahead and a ring of four, two blocks per CU.  us against the fastest of the others: 3136 x 768 x 3072
// 29.3 -> 24.6, 3136 x 768 x 2304 (B n-major) 23.4 -> 19.8, 2056 x 1024 x 4096 35.4 -> 30.1; 64 x 64: 1032 x 768 x 3072 16.0 -> 13.3, 520 x 1024 x 4096 19.1 -> 15.9.
// (Measured and not kept: rings of six to nine stages with four waves, level; four waves of 128 x 128, 128 x 64 or 96 x 128, 5 - 30 % slower than eight
// waves of half the size: one wave per SIMD has nothing to run under its waits.)
typedef DmaCfg<2, 1, 2, 4, 1, 64, 4, 1, true> Dma128x128Lone;
typedef DmaCfg<1, 1, 2, 2, 1, 64, 4, 2, true> Dma64x64Lone;
typedef DmaCfg<2, 3, 2, 2, 1, 64, 2, 2, true> Dma128x192;
typedef DmaCfg<3, 2, 2, 2, 1, 64, 2, 2, true> Dma192x128;
typedef DmaCfg<2, 2, 4, 2, 1, 64, 3, 1, true> Dma256x128;
typedef DmaCfg<4, 2, 2, 4, 1, 64, 2, 1, true> Dma256x256;

}  // namespace
