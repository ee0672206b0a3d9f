// fp32 softmax attention on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and sums), head dimension 64: the encoder's
// self-attention (with dropout of the probabilities) and the general form (separate query and key sequences, causal or not).
//
// A wave owns 32 rows of one side, one per lane of a half wave, and walks the other side in blocks of 32 rows, the operands read
// from memory into registers without LDS.  Scores: lane l feeds row l%32 at four head columns 8 t + 4 (l/32) .. +3, one 16-byte load.  The
// 32x32 result leaves lane l with the 16 rows 8 (r/4) + 4 (l/32) + r%4 of column l%32 - which is an operand of the second
// product as it stands, when step r of its contraction is fed the rows 8 (r/4) + r%4 and, in the upper half, +4.
// With one wave per 32 rows the serial chain bounds it at the toy sizes this type is used at: 64 MFMAs of 64 cycles, 1.9 us, per
// 32 streamed rows forward, so the second product's operand is loaded ahead of the scores too.
// Backward: one launch, the first blocks own queries (dq), the others keys (dk, dv); both need the row dot products of dO and O
// and each side computes its own, so neither waits for the other.
// Six attentions of 24 and 32 rows, 6 sequences, 2 heads: 7.0 us forward and 12.4 us backward on average (50 and 107 + 75 us with one
// thread per row at 4 sequences of 64; there 11 and 17 us now).
#include "attention_tiles.h"

namespace {
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // the hardware needs 4-byte alignment only
constexpr int D = 64;

struct Rows { const float* p; int64_t ld; };      // head column 0 of row 0 of one sequence

// 8 x 4 head columns of row r, lane half `half` (zeros from row n on)
__device__ __forceinline__ void load_row(f32x4u (&f)[8], const Rows& x, int r, int n, int half) {
  const float* q = x.p + (int64_t)(r < n ? r : 0) * x.ld + 4 * half;
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = *(const f32x4u*)(q + 8 * t);
  if (r >= n) {
#pragma unroll
    for (int t = 0; t < 8; ++t) f[t] = f32x4u{0.f, 0.f, 0.f, 0.f};
  }
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
// [32 rows of a] x [32 rows of b] over the 64 head columns
__device__ __forceinline__ f32x16 dot_rows(const f32x4u (&a)[8], const f32x4u (&b)[8]) {
  f32x16 s = zero16();
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int c = 0; c < 4; ++c) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t][c], b[t][c], s, 0, 0, 0);
  return s;
}
__device__ __forceinline__ int row_of(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }
// columns 32 db + l%32 of the 32 rows from row0 (zeros from row n on), in the order of row_of: loaded ahead of the scores that weigh them
__device__ __forceinline__ void load_cols(float (&f)[2][16], const Rows& x, int row0, int n, int l31, int half) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float* q = x.p + (int64_t)min(row0 + row_of(r, half), n - 1) * x.ld + l31;
    f[0][r] = q[0]; f[1][r] = q[32];
  }
  if (row0 + 32 > n) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (row0 + row_of(r, half) >= n) { f[0][r] = 0.f; f[1][r] = 0.f; }
  }
}
// acc[db] (head columns 32 db .. +31 by rows, owned row by lane) += sum over the 32 rows of f[row] w[row]
__device__ __forceinline__ void add_rows(f32x16 (&acc)[2], const float (&f)[2][16], const f32x16& w) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int db = 0; db < 2; ++db) acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(f[db][r], w[r], acc[db], 0, 0, 0);
}
// The same where causality leaves pairs of the block out: their weights are zeros, and a zero times an infinity or a NaN would reach
// the owned rows that must not see it.  Where the block holds such a value, its rows are added one at a time, each to the owned rows
// that take part (`takes`: whether the lane's owned row takes the streamed row).
template <class Takes>
__device__ __forceinline__ void add_rows_causal(f32x16 (&acc)[2], const float (&f)[2][16], const f32x16& w, const Rows& x, int row0, int l31,
                                                int half, Takes takes) {
  bool finite = true;
#pragma unroll
  for (int r = 0; r < 16; ++r) finite = finite && fabsf(f[0][r]) <= 3.4028235e38f && fabsf(f[1][r]) <= 3.4028235e38f;
  if (__all(finite)) { add_rows(acc, f, w); return; }
  for (int i = 0; i < 32; ++i) {
    float wi = 0.f;      // the weight of row i lies at register 4 (i/8) + i%4 of the half wave (i/4) % 2
#pragma unroll
    for (int r = 0; r < 16; ++r) wi = r == 4 * (i >> 3) + (i & 3) ? w[r] : wi;
    wi = __shfl(wi, l31 + 32 * ((i >> 2) & 1));
    if (takes(row0 + i)) {
      const float* q = x.p + (int64_t)(row0 + i) * x.ld;
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[db][r] = fmaf(wi, q[32 * db + row_of(r, half)], acc[db][r]);
    }
  }
}
__device__ __forceinline__ void store_row(float* o, const f32x16 (&acc)[2], float scale, int half) {
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4u v;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = scale * acc[db][4 * g + c];
      *(f32x4u*)(o + 32 * db + 8 * g + 4 * half) = v;
    }
}

struct Problem {
  AttnF32 a;
  int b, h, H, klen, qlen;
  Rows q, k, v;
  __device__ Problem(const AttnF32& x, int b_, int h_) : a(x), b(b_), h(h_) {
    H = a.A * D;
    klen = min(max(a.klens[b], 1), a.Lk);
    qlen = min(max(a.qlens[b], 1), a.Lq);
    q = {a.q + (int64_t)b * a.Lq * a.ldq + h * D, a.ldq};
    k = {a.k + (int64_t)b * a.Lk * a.ldkv + h * D, a.ldkv};
    v = {a.v + (int64_t)b * a.Lk * a.ldkv + h * D, a.ldkv};
  }
  __device__ Rows rows_h(const float* p) const { return {p + (int64_t)b * a.Lq * H + h * D, (int64_t)H}; }     // of a [B*Lq, H] matrix
  __device__ int64_t stat(int qi) const { return ((int64_t)b * a.A + h) * a.Lq + qi; }
  // dropout factor of the probability of (query, key)
  __device__ float factor(int qi, int key) const { return drop_factor1(a.drop, a.site, (uint64_t)stat(qi) * a.Lk + key); }
};

__global__ __launch_bounds__(64) void attn_f32_fwd(AttnF32 x, float* __restrict__ out, float* __restrict__ lse) {
  const Problem p(x, blockIdx.z, blockIdx.y);
  const int lane = threadIdx.x, l31 = lane & 31, half = lane >> 5;
  const int qi = blockIdx.x * 32 + l31;
  const int kend = x.causal ? min(p.klen, (int)blockIdx.x * 32 + 32) : p.klen;
  f32x4u qf[8];
  load_row(qf, p.q, qi, x.Lq, half);
  f32x16 o[2] = {zero16(), zero16()};
  float m = -1.0e30f, l = 0.f;
  for (int k0 = 0; k0 < kend; k0 += 32) {
    f32x4u kf[8];
    float vc[2][16];
    load_row(kf, p.k, k0 + l31, p.klen, half);
    load_cols(vc, p.v, k0, p.klen, l31, half);
    f32x16 s = dot_rows(kf, qf);
    float mloc = m;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + row_of(r, half);
      s[r] = (key < p.klen && (!x.causal || key <= qi)) ? 0.125f * s[r] : -INFINITY;
      mloc = fmaxf(mloc, s[r]);
    }
    const float mn = fmaxf(mloc, __shfl_xor(mloc, 32));
    const float alpha = __expf(m - mn);
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float e = __expf(s[r] - mn);      // 0 for the pairs left out (mn is never below the finite start of m); a NaN score stays one
      ps += e;
      // dropout acts on the normalised probabilities: the row sum keeps every key, the value sum the survivors
      s[r] = x.drop.thr ? e * p.factor(qi, k0 + row_of(r, half)) : e;
    }
    l = l * alpha + ps;
    m = mn;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    if (x.causal && k0 == (int)blockIdx.x * 32) add_rows_causal(o, vc, s, p.v, k0, l31, half, [&](int key) { return key < p.klen && key <= qi; });
    else add_rows(o, vc, s);
  }
  l += __shfl_xor(l, 32);
  if (qi < x.Lq) {
    store_row(out + ((int64_t)p.b * x.Lq + qi) * p.H + p.h * D, o, 1.0f / l, half);
    if (half == 0) lse[p.stat(qi)] = m + logf(l);
  }
}

__device__ __forceinline__ float dot_own(const f32x4u (&a)[8], const f32x4u (&b)[8]) {
  float d = 0.f;
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int c = 0; c < 4; ++c) d = fmaf(a[t][c], b[t][c], d);
  return d + __shfl_xor(d, 32);
}

__global__ __launch_bounds__(64) void attn_f32_bwd(AttnF32 x, int q_blocks, const float* __restrict__ out, const float* __restrict__ lse,
                                                   const float* __restrict__ d_out, float* __restrict__ dq, int64_t lddq,
                                                   float* __restrict__ dk, float* __restrict__ dv, int64_t lddkv) {
  const Problem p(x, blockIdx.z, blockIdx.y);
  const int lane = threadIdx.x, l31 = lane & 31, half = lane >> 5;
  const Rows go = p.rows_h(d_out), oo = p.rows_h(out);
  if ((int)blockIdx.x < q_blocks) {
    const int q0 = blockIdx.x * 32, qi = q0 + l31;
    const int kend = q0 >= p.qlen ? 0 : x.causal ? min(p.klen, q0 + 32) : p.klen;     // padded queries get zero gradient
    f32x4u qf[8], gf[8], of[8];
    load_row(qf, p.q, qi, p.qlen, half);
    load_row(gf, go, qi, p.qlen, half);
    load_row(of, oo, qi, p.qlen, half);
    const float row_dot = dot_own(gf, of), row_lse = qi < p.qlen ? lse[p.stat(qi)] : 0.f;
    f32x16 acc[2] = {zero16(), zero16()};
    for (int k0 = 0; k0 < kend; k0 += 32) {
      f32x4u kf[8], vf[8];
      load_row(kf, p.k, k0 + l31, p.klen, half);
      load_row(vf, p.v, k0 + l31, p.klen, half);
      float kc[2][16];
      load_cols(kc, p.k, k0, p.klen, l31, half);
      f32x16 s = dot_rows(kf, qf);
      const f32x16 dp = dot_rows(vf, gf);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + row_of(r, half);
        const bool ok = key < p.klen && qi < p.qlen && (!x.causal || key <= qi);
        const float f = x.drop.thr ? p.factor(qi, key) : 1.0f;
        s[r] = ok ? __expf(0.125f * s[r] - row_lse) * (f * dp[r] - row_dot) : 0.f;
      }
      if (x.causal && k0 == q0)
        add_rows_causal(acc, kc, s, p.k, k0, l31, half, [&](int key) { return key < p.klen && qi < p.qlen && key <= qi; });
      else add_rows(acc, kc, s);
    }
    if (qi >= p.qlen) { acc[0] = zero16(); acc[1] = zero16(); }      // whatever the keys held
    if (qi < x.Lq) store_row(dq + ((int64_t)p.b * x.Lq + qi) * lddq + p.h * D, acc, 0.125f, half);
  } else {
    const int k0 = ((int)blockIdx.x - q_blocks) * 32, kj = k0 + l31;
    f32x4u kf[8], vf[8];
    load_row(kf, p.k, kj, p.klen, half);
    load_row(vf, p.v, kj, p.klen, half);
    f32x16 ak[2] = {zero16(), zero16()}, av[2] = {zero16(), zero16()};
    // padded keys take no part; queries before the first own key never see it when causal
    for (int q0 = k0 >= p.klen ? p.qlen : x.causal ? k0 : 0; q0 < p.qlen; q0 += 32) {
      f32x4u qf[8], gf[8], of[8];
      load_row(qf, p.q, q0 + l31, p.qlen, half);
      load_row(gf, go, q0 + l31, p.qlen, half);
      load_row(of, oo, q0 + l31, p.qlen, half);
      float gc[2][16], qc[2][16];
      load_cols(gc, go, q0, p.qlen, l31, half);
      load_cols(qc, p.q, q0, p.qlen, l31, half);
      const float row_dot = dot_own(gf, of), row_lse = q0 + l31 < p.qlen ? lse[p.stat(q0 + l31)] : 0.f;
      f32x16 s = dot_rows(qf, kf), dp = dot_rows(gf, vf);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = row_of(r, half), qi = q0 + i;
        const bool ok = qi < p.qlen && kj < p.klen && (!x.causal || kj <= qi);
        const float f = x.drop.thr ? p.factor(qi, kj) : 1.0f;
        const float lse_i = __shfl(row_lse, i), dot_i = __shfl(row_dot, i);      // by all lanes: before anything that depends on ok
        const float e = ok ? __expf(0.125f * s[r] - lse_i) : 0.f;
        dp[r] = ok ? e * (f * dp[r] - dot_i) : 0.f;
        s[r] = e * f;
      }
      if (x.causal && q0 == k0) {
        auto takes = [&](int qi) { return qi < p.qlen && kj < p.klen && kj <= qi; };
        add_rows_causal(av, gc, s, go, q0, l31, half, takes);
        add_rows_causal(ak, qc, dp, p.q, q0, l31, half, takes);
      } else {
        add_rows(av, gc, s);
        add_rows(ak, qc, dp);
      }
    }
    if (kj >= p.klen) { ak[0] = ak[1] = zero16(); av[0] = av[1] = zero16(); }
    if (kj < x.Lk) {
      store_row(dk + ((int64_t)p.b * x.Lk + kj) * lddkv + p.h * D, ak, 0.125f, half);
      store_row(dv + ((int64_t)p.b * x.Lk + kj) * lddkv + p.h * D, av, 1.0f, half);
    }
  }
}
}  // namespace

void launch_attention_f32_fwd(const AttnF32& x, int B, float* out, float* lse, hipStream_t s) {
  hipLaunchKernelGGL(attn_f32_fwd, dim3((x.Lq + 31) / 32, x.A, B), dim3(64), 0, s, x, out, lse);
}

void launch_attention_f32_bwd(const AttnF32& x, int B, const float* out, const float* lse, const float* d_out, float* dq, int64_t lddq, float* dk,
                              float* dv, int64_t lddkv, hipStream_t s) {
  const int qb = (x.Lq + 31) / 32, kb = (x.Lk + 31) / 32;
  hipLaunchKernelGGL(attn_f32_bwd, dim3(qb + kb, x.A, B), dim3(64), 0, s, x, qb, out, lse, d_out, dq, lddq, dk, dv, lddkv);
}
