// Softmax attention over the real keys of each sequence, head dimension 64.
// qkv is [B*L, 3H]: per token the query, key and value vectors of all heads; head h occupies
// columns h*64 .. h*64+63 of each third.  Key l' of sequence b takes part iff l' < lens[b].
//
// This file: the dispatch by type.  bf16: attention_general.hip (and attention_mfma.hip); fp32: attention_f32.hip.
#include "common.h"

namespace {
constexpr int D = 64;

AttnF32 f32_problem(const void* qkv, const int32_t* lens, int L, int A, const DropCfg& drop, uint32_t site) {
  const int H = A * D;
  const float* q = (const float*)qkv;
  return AttnF32{q, q + H, q + 2 * H, 3 * (int64_t)H, 3 * (int64_t)H, lens, lens, L, L, A, 0, drop, site};
}
}  // namespace

void launch_attention_self_fwd(const void* qkv, const int32_t* lens, int B, int L, int A, void* out, float* lse, hipStream_t s,
                               const DropCfg& drop, uint32_t site, const int32_t* first);
void launch_attention_self_bwd(const void* qkv, const void* out, const float* lse, const void* d_out, const int32_t* lens, int B, int L,
                               int A, void* dqkv, float* dvec, hipStream_t s, const DropCfg& drop, uint32_t site, const int32_t* first);

hs_status launch_attention_fwd(hs_ctx* ctx, int dtype, const void* qkv, const int32_t* lens, int B, int L, int A, void* out, float* lse,
                               hipStream_t s, const DropCfg* drop_in, uint32_t site, const int32_t* first) {
  if (B <= 0 || L <= 0) return HS_OK;
  if (first && dtype != HS_BF16) return hs_fail(ctx, HS_ERR_UNIMPLEMENTED, "attention: packed rows in bf16 only");
  const DropCfg drop = (drop_in && drop_in->thr) ? *drop_in : DropCfg{0u, 1.0f, 0u, 0u, 0u};
  if (drop.thr && (L & 3)) return hs_fail(ctx, HS_ERR_SHAPE, "attention with dropout: the padded length must be a multiple of 4");
  const double fl = 4.0 * B * A * (double)L * L * D;
  const double by = (double)B * L * A * D * 4.0 * esize(dtype);
  KScope scope(ctx ? ctx->prof : nullptr, KC_ATTN_FWD, fl, by, s);
  if (dtype == HS_BF16) launch_attention_self_fwd(qkv, lens, B, L, A, out, lse, s, drop, site, first);
  else launch_attention_f32_fwd(f32_problem(qkv, lens, L, A, drop, site), B, (float*)out, lse, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("attention_fwd: ") + hipGetErrorString(e));
  return HS_OK;
}

hs_status launch_attention_bwd(hs_ctx* ctx, int dtype, const void* qkv, const void* out, const float* lse, const void* d_out,
                               const int32_t* lens, int B, int L, int A, void* dqkv, float* dvec, hipStream_t s, const DropCfg* drop_in,
                               uint32_t site, const int32_t* first) {
  if (B <= 0 || L <= 0) return HS_OK;
  if (first && dtype != HS_BF16) return hs_fail(ctx, HS_ERR_UNIMPLEMENTED, "attention: packed rows in bf16 only");
  const DropCfg drop = (drop_in && drop_in->thr) ? *drop_in : DropCfg{0u, 1.0f, 0u, 0u, 0u};
  if (drop.thr && (L & 3)) return hs_fail(ctx, HS_ERR_SHAPE, "attention with dropout: the padded length must be a multiple of 4");
  const double fl = 8.0 * B * A * (double)L * L * D;   // dV, dP, dQ, dK (recomputing the scores is not counted)
  const double by = (double)B * L * A * D * 8.0 * esize(dtype);
  KScope scope(ctx ? ctx->prof : nullptr, KC_ATTN_BWD, fl, by, s);
  if (dtype == HS_BF16) {
    launch_attention_self_bwd(qkv, out, lse, d_out, lens, B, L, A, dqkv, dvec, s, drop, site, first);
  } else {
    float* d = (float*)dqkv;
    launch_attention_f32_bwd(f32_problem(qkv, lens, L, A, drop, site), B, (const float*)out, lse, (const float*)d_out, d, 3 * (int64_t)A * D,
                             d + A * D, d + 2 * A * D, 3 * (int64_t)A * D, s);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hs_fail(ctx, HS_ERR_HIP, std::string("attention_bwd: ") + hipGetErrorString(e));
  return HS_OK;
}
