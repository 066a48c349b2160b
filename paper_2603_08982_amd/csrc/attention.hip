// Fused block-sparse exact attention + centroid compensation.
// Paper: Eq. (1) (compensated attention map), Eq. (6) (output), Algorithm 2 (a skipped key
// cluster enters the online softmax as one pseudo-key with logit q.kbar*scale + ln|k_c| and
// value vbar), "Linear Compensation" (cost O((Nq Ck + rho Nk Nq) d)).
//
// Work decomposition: the query rows of one query cluster are cut into tiles of BM rows; a
// tile never straddles two query clusters because the routing mask is per query cluster.
// The routed key clusters of that query cluster are concatenated into one virtual key
// sequence (cluster-contiguous K/V rows make every piece a contiguous row range), consumed
// in tiles of 64 keys regardless of cluster boundaries; the centroids of the skipped
// clusters follow as extra 64-key tiles with a per-key bias log2|k_b| (-inf for routed or
// empty clusters). One online softmax (base-2 exponent domain) runs over both phases.
//
// bf16 kernel (gfx950 MFMA, v_mfma_f32_32x32x16_bf16): each wave owns 32 query rows and
// computes the TRANSPOSED score tile S^T = K Q^T, so that every lane holds scores of a
// single query (lane%32) and row max / row sum need one cross-lane exchange (with lane^32)
// instead of a butterfly; exp2'd scores are then already in B-operand layout for
// O^T += V^T P^T. V stays row-major in LDS and is fetched with the LDS transpose read.
// fp32 kernel: the same decomposition on the fp32 matrix cores (attention_f32.hip).
#include "attention.h"

using namespace svgear;

extern "C" size_t svgear_sparse_attn_comp_workspace(int B, int H, int64_t Nq, int64_t Nk, int d, int Cq, int Ck) {
  if (B <= 0 || H <= 0 || Nq <= 0 || Cq <= 0 || Ck <= 0 || d <= 0) return 0;
  const size_t BH = (size_t)B * H;
  const size_t bf16 = 2 * align_up(BH * Ck * d * 2, 256) + plan_bf16_workspace((int64_t)BH, Cq, Nq, Nk, d);
  const size_t f32 = f32_workspace((int64_t)BH, Nq, Nk, Cq, d);
  return bf16 > f32 ? bf16 : f32;
}

static int attn_run(const void* qp, const void* kp, const void* vp, svgear_dtype dt, const float* kbar,
                    const float* vbar, const int32_t* q_offsets, const int32_t* k_offsets, const uint32_t* mask_bits,
                    const int32_t* row_ptr, const int32_t* col_idx, int B, int H, int64_t Nq, int64_t Nk, int d, int Cq,
                    int Ck, float scale, void* op, float* lse, void* ws, size_t ws_bytes, void* stream, int part,
                    const int32_t* tok_perm = nullptr, const int64_t* qstride = nullptr,
                    const int64_t* ostride = nullptr) {
  if (!qp || !kp || !vp || !kbar || !vbar || !q_offsets || !k_offsets || !mask_bits || !row_ptr || !col_idx || !op ||
      B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || Cq <= 0 || Ck <= 0 || Cq > 8192 || Ck > 8192 ||
      Nq > INT32_MAX / 2 || Nk > INT32_MAX / 2 || (d != 64 && d != 128) || (dt != SVGEAR_F32 && dt != SVGEAR_BF16) ||
      !(scale > 0.f))
    return SVGEAR_ERR_INVALID;
  const void* ptrs[] = {qp, kp, vp, kbar, vbar, op};
  for (const void* q : ptrs)
    if (reinterpret_cast<uintptr_t>(q) % 16) return SVGEAR_ERR_INVALID;
  Strides q_st{0, 0, 0}, out_st{0, 0, 0};
  if (tok_perm) {  // token order at both ends: strides in elements, rows 16-byte aligned
    const int64_t es = dt == SVGEAR_F32 ? 4 : 2;
    if (!qstride || !ostride) return SVGEAR_ERR_INVALID;
    for (int i = 0; i < 3; ++i)
      if (qstride[i] < 0 || (qstride[i] * es) % 16 || ostride[i] < 0 || (ostride[i] * es) % 16)
        return SVGEAR_ERR_INVALID;
    if (qstride[2] < d || ostride[2] < d) return SVGEAR_ERR_INVALID;
    q_st = Strides{qstride[0], qstride[1], qstride[2]};
    out_st = Strides{ostride[0], ostride[1], ostride[2]};
  }
  if (!ws || ws_bytes < svgear_sparse_attn_comp_workspace(B, H, Nq, Nk, d, Cq, Ck)) return SVGEAR_ERR_WORKSPACE;
  const int BH = B * H;
  if ((int64_t)BH * ((int64_t)ceil_div(Nq, 64) + Cq + 1) > INT32_MAX / 2) return SVGEAR_ERR_UNSUPPORTED;
  if (part != 0 && !(dt == SVGEAR_BF16 && d == 128)) return SVGEAR_ERR_UNSUPPORTED;
  if (dt == SVGEAR_BF16 && !attn_bf16_supported(d, Ck)) return SVGEAR_ERR_UNSUPPORTED;
  // the d = 128 bf16 kernel addresses K/V rows of a head by 32-bit byte offsets (256 bytes a row)
  if (dt == SVGEAR_BF16 && d == 128 && Nk > (int64_t)(UINT32_MAX / 256)) return SVGEAR_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);
  AttnArgs a{qp, kp, vp, kbar, vbar, nullptr, nullptr, q_offsets, k_offsets, mask_bits, row_ptr, col_idx,
             nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
             Nq, Nk, BH, Cq, Ck, 0, scale, op, lse, part, tok_perm, q_st, out_st, H, nullptr, nullptr, 1, 0, nullptr};
  if (dt == SVGEAR_F32) return launch_attn_f32(a, d, ws, ws_bytes, s);
  Workspace w(ws, ws_bytes);
  bf16_t* kbar16 = w.take<bf16_t>((size_t)BH * Ck * d);
  bf16_t* vbar16 = w.take<bf16_t>((size_t)BH * Ck * d);
  if (!w.ok()) return SVGEAR_ERR_WORKSPACE;
  a.kbar16 = kbar16;
  a.vbar16 = vbar16;
  const int rc = plan_bf16(a, d, kbar16, vbar16, static_cast<char*>(ws) + w.used, ws_bytes - w.used, s);
  if (rc != SVGEAR_OK) return rc;
  return launch_attn_bf16(a, d, s);
}

extern "C" int svgear_sparse_attn_comp(const void* qp, const void* kp, const void* vp, svgear_dtype dt,
                                       const float* kbar, const float* vbar, const int32_t* q_offsets,
                                       const int32_t* k_offsets, const uint32_t* mask_bits, const int32_t* row_ptr,
                                       const int32_t* col_idx, int B, int H, int64_t Nq, int64_t Nk, int d, int Cq,
                                       int Ck, float scale, void* op, float* lse, void* ws, size_t ws_bytes,
                                       void* stream) {
  return attn_run(qp, kp, vp, dt, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx, B, H, Nq, Nk, d, Cq,
                  Ck, scale, op, lse, ws, ws_bytes, stream, 0);
}

extern "C" int svgear_sparse_attn_comp_token_order(const void* q, const int64_t qstride[3], const void* kp,
                                                   const void* vp, svgear_dtype dt, const float* kbar,
                                                   const float* vbar, const int32_t* q_offsets,
                                                   const int32_t* k_offsets, const uint32_t* mask_bits,
                                                   const int32_t* row_ptr, const int32_t* col_idx,
                                                   const int32_t* q_perm, int B, int H, int64_t Nq, int64_t Nk, int d,
                                                   int Cq, int Ck, float scale, void* o, const int64_t ostride[3],
                                                   float* lse, void* ws, size_t ws_bytes, void* stream) {
  if (!q_perm || !qstride || !ostride) return SVGEAR_ERR_INVALID;
  return attn_run(q, kp, vp, dt, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx, B, H, Nq, Nk, d, Cq,
                  Ck, scale, o, lse, ws, ws_bytes, stream, 0, q_perm, qstride, ostride);
}

extern "C" size_t svgear_sparse_attn_two_stage_workspace(int B, int H, int64_t Nq, int64_t Nk, int d, int Cq,
                                                         int Ck) {
  const size_t base = svgear_sparse_attn_comp_workspace(B, H, Nq, Nk, d, Cq, Ck);
  if (base == 0) return 0;
  const size_t BH = (size_t)B * H;
  return align_up(base, 256) + 2 * align_up(BH * Nq * d * 2, 256) + 2 * align_up(BH * Nq * 4, 256);
}

extern "C" int svgear_sparse_attn_two_stage(const void* qp, const void* kp, const void* vp, svgear_dtype dt,
                                            const float* kbar, const float* vbar, const int32_t* q_offsets,
                                            const int32_t* k_offsets, const uint32_t* mask_bits,
                                            const int32_t* row_ptr, const int32_t* col_idx, int B, int H, int64_t Nq,
                                            int64_t Nk, int d, int Cq, int Ck, float scale, void* op, float* lse,
                                            void* ws, size_t ws_bytes, void* stream) {
  if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || Cq <= 0 || Ck <= 0 || !op) return SVGEAR_ERR_INVALID;
  if (!(dt == SVGEAR_BF16 && d == 128)) return SVGEAR_ERR_UNSUPPORTED;
  if (!ws || ws_bytes < svgear_sparse_attn_two_stage_workspace(B, H, Nq, Nk, d, Cq, Ck)) return SVGEAR_ERR_WORKSPACE;
  const size_t base = align_up(svgear_sparse_attn_comp_workspace(B, H, Nq, Nk, d, Cq, Ck), 256);
  const size_t BH = (size_t)B * H;
  Workspace w(static_cast<char*>(ws) + base, ws_bytes - base);
  bf16_t* o_r = w.take<bf16_t>(BH * Nq * d);
  bf16_t* o_c = w.take<bf16_t>(BH * Nq * d);
  float* lse_r = w.take<float>(BH * Nq);
  float* lse_c = w.take<float>(BH * Nq);
  if (!w.ok()) return SVGEAR_ERR_WORKSPACE;
  int rc = attn_run(qp, kp, vp, dt, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx, B, H, Nq, Nk, d,
                    Cq, Ck, scale, o_r, lse_r, ws, base, stream, 1);
  if (rc != SVGEAR_OK) return rc;
  rc = attn_run(qp, kp, vp, dt, kbar, vbar, q_offsets, k_offsets, mask_bits, row_ptr, col_idx, B, H, Nq, Nk, d, Cq,
                Ck, scale, o_c, lse_c, ws, base, stream, 2);
  if (rc != SVGEAR_OK) return rc;
  return launch_merge(o_r, lse_r, o_c, lse_c, (int64_t)BH * Nq, d, static_cast<bf16_t*>(op), lse,
                      static_cast<hipStream_t>(stream));
}
