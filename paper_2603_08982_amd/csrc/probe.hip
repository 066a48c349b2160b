// Error probe: estimated compensation error of every (query cluster, key cluster) block.
// Paper: Eq. (7) (value-aware estimate), Eq. (5) (plain estimate), Algorithm 1 (row
// stabiliser m_a = max_b Sbar_ab; streaming over the keys of a cluster without writing
// logits to memory), "Error-Aware Routing" (error-to-size ratio).
//
// Logits come from the matrix cores, in tiles of keys x query centroids that leave a lane with 16
// keys of one centroid, so a block's error accumulates in the lane. The squared difference of Eq. (7)
// is expanded around the cluster mean instead of around zero:
//   W vbar - w v_j = (W - w) vbar - w delta_j,   delta_j = v_j - vbar
//   || . ||^2 = (W-w)^2 |vbar|^2 - 2 (W-w) w (vbar.delta_j) + w^2 |delta_j|^2
// so each key contributes O(1) work per query centroid after its logit, and no term
// cancels catastrophically when the cluster is tight. |delta_j|^2 and vbar.delta_j do not
// depend on a and are computed once per key by the whole workgroup.
#include <type_traits>

#include "common.h"

namespace svgear {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr float kMaxExponent = 40.0f;  // e^40 squared still fits fp32

// A one-dimensional launch in two dimensions (2^24 workgroups of 256 threads are too many for one): where a workgroup
// stands in it. Rows are a multiple of 8 long, so that workgroups go round the XCDs as they would in one.
constexpr int64_t kGridRow = 1 << 20;
static inline dim3 long_grid(int64_t blocks) {
  return blocks <= kGridRow ? dim3((unsigned)blocks) : dim3((unsigned)kGridRow, (unsigned)ceil_div(blocks, kGridRow));
}
__device__ __forceinline__ int long_grid_index() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }

// A power of two near the largest component of a cluster's mean value (bf16 inputs): the block errors take their
// weights' differences times it, so that squares summed before they meet |vbar|^2 stay as far from the ends of a
// float's range as the errors themselves do.
__device__ __forceinline__ float value_scale(float largest) {
  const int e = (int)(__float_as_uint(largest) >> 23 & 255u);
  return __uint_as_float((uint32_t)min(max(e, 127 - 60), 127 + 62) << 23);
}
__device__ __forceinline__ float inverse_scale(float s) { return __uint_as_float((254u << 23) - __float_as_uint(s)); }

// |delta_j|^2 and -2 vbar . delta_j / value_scale of every clustered key (delta_j = v_j - vbar of its cluster), bf16
// inputs: what the block errors need of the values. 256 threads per (head, key cluster): 16 key slots x 16 lanes of 8 dims (d = 64: 32 x 8).
// They depend on nothing the centroid logits compute, so both share a launch, the logits' workgroups first: 5 heads,
// 200 x 500 centroids 20 + 29 us apart, 38 together; 8 x 2,000 keys, 30 x 60: the whole call 39 -> 33. (Not with the
// matrix-core form of the logits, whose registers cost the streaming half its waves: 40 heads, 300 x 1,000 centroids
// 85 + 168 apart, 300 together.)
struct ValueStats {
  const float* vbar;
  const bf16_t* vp;
  int64_t Nk, stride;  // of nd and dd
  float* nd;
  float* dd;
  int clusters;  // of all heads; 0: none wanted
};

template <int D>
__device__ __forceinline__ void value_stats(const ValueStats& p, const int32_t* k_offsets, int Ck, int cluster, int tid) {
  constexpr int LPK = D / 8;  // lanes per key
  constexpr int SLOTS = 256 / LPK;
  if (cluster >= p.clusters) return;
  const int b = cluster % Ck, bh = cluster / Ck;
  const int slot = tid / LPK, lane = tid % LPK;
  const int32_t* off = k_offsets + (int64_t)bh * (Ck + 2);
  const int start = off[b], end = off[b + 1];
  const float* vb = p.vbar + ((int64_t)bh * Ck + b) * D + lane * 8;
  float vbl[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) vbl[k] = vb[k];
  float largest = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) largest = fmaxf(largest, fabsf(vbl[k]));
#pragma unroll
  for (int o = LPK / 2; o > 0; o >>= 1) largest = fmaxf(largest, __shfl_xor(largest, o));
  const float dd_scale = -2.0f * inverse_scale(value_scale(largest));
  const bf16_t* vh = p.vp + (int64_t)bh * p.Nk * D + lane * 8;
  constexpr int INFLIGHT = 4;  // independent key fetches per lane group
  for (int j0 = start + slot; j0 < end; j0 += INFLIGHT * SLOTS) {
    uint4 raw[INFLIGHT];
#pragma unroll
    for (int u = 0; u < INFLIGHT; ++u) {
      const int j = j0 + u * SLOTS;
      raw[u] = j < end ? *reinterpret_cast<const uint4*>(vh + (int64_t)j * D) : uint4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < INFLIGHT; ++u) {
      const int j = j0 + u * SLOTS;
      const uint32_t w[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
      float p_nd = 0.f, p_dd = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d0 = __uint_as_float(w[i] << 16) - vbl[2 * i];
        const float d1 = __uint_as_float(w[i] & 0xffff0000u) - vbl[2 * i + 1];
        p_nd = __builtin_fmaf(d0, d0, p_nd);
        p_dd = __builtin_fmaf(d0, vbl[2 * i], p_dd);
        p_nd = __builtin_fmaf(d1, d1, p_nd);
        p_dd = __builtin_fmaf(d1, vbl[2 * i + 1], p_dd);
      }
#pragma unroll
      for (int o = LPK / 2; o > 0; o >>= 1) {
        p_nd += __shfl_xor(p_nd, o);
        p_dd += __shfl_xor(p_dd, o);
      }
      if (lane == 0 && j < end) {
        p.nd[(int64_t)bh * p.stride + j] = p_nd;
        p.dd[(int64_t)bh * p.stride + j] = dd_scale * p_dd;
      }
    }
  }
}

// Sbar[a][b] = qbar_a . kbar_b * scale; mrow[a] = max over non-empty b.
// With q3 != nullptr (grid.x = Cq rounded up to 32) it also writes qbar split into three bf16
// pieces q = hi + mid + lo (exact: 3 x 8 significant bits), laid out as B operands of
// v_mfma_f32_32x32x16_bf16: [a-block][piece][s][lane = a%32 + 32*((k%16)/8)][k%8], zero rows
// for a >= Cq.
constexpr int kSbarRows = 4;  // query centroids per workgroup: each kbar row fetched serves all of them

template <int D>
__global__ void __launch_bounds__(256)
sbar_kernel(const float* __restrict__ qbar, const float* __restrict__ kbar, const int32_t* __restrict__ k_offsets,
            int Cq, int Ck, float scale, float* __restrict__ sbar, float* __restrict__ mrow,
            bf16_t* __restrict__ q3, int groups, int logit_blocks, ValueStats stats) {
  __shared__ float q[kSbarRows][D];
  __shared__ float red[kSbarRows][4];
  const int block = long_grid_index();
  if (block >= logit_blocks) return value_stats<D>(stats, k_offsets, Ck, block - logit_blocks, threadIdx.x);
  const int a0 = block % groups * kSbarRows, bh = block / groups;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < kSbarRows * D; i += 256) {
    const int a = a0 + i / D;
    q[i / D][i % D] = a < Cq ? qbar[((int64_t)bh * Cq + a) * D + i % D] : 0.f;
  }
  __syncthreads();
  if (q3) {
    constexpr int KSN = D / 16;
    for (int i = threadIdx.x; i < kSbarRows * D; i += 256) {
      const int a = a0 + i / D, k = i % D, ab = a >> 5, nab = (Cq + 31) >> 5;
      const float v = q[i / D][k];
      const bf16_t hi = f32_to_bf16(v);
      const float r1 = v - bf16_to_f32(hi);
      const bf16_t mid = f32_to_bf16(r1);
      const bf16_t lo = f32_to_bf16(r1 - bf16_to_f32(mid));
      const int ln = (a & 31) + 32 * ((k & 15) >> 3);
      bf16_t* dst = q3 + ((((int64_t)bh * nab + ab) * 3) * KSN + (k >> 4)) * 512 + ln * 8 + (k & 7);
      dst[0] = hi;
      dst[(int64_t)KSN * 512] = mid;
      dst[(int64_t)2 * KSN * 512] = lo;
    }
  }
  if (a0 >= Cq) return;
  const int32_t* off = k_offsets + (int64_t)bh * (Ck + 2);
  float mx[kSbarRows];
#pragma unroll
  for (int r = 0; r < kSbarRows; ++r) mx[r] = -INFINITY;
  for (int b = threadIdx.x; b < Ck; b += 256) {
    const float4* kb = reinterpret_cast<const float4*>(kbar + ((int64_t)bh * Ck + b) * D);
    float dot[kSbarRows];
#pragma unroll
    for (int r = 0; r < kSbarRows; ++r) dot[r] = 0.f;
#pragma unroll 8
    for (int t = 0; t < D / 4; ++t) {
      const float4 v = kb[t];
#pragma unroll
      for (int r = 0; r < kSbarRows; ++r) {  // one fma chain per (a, b), dims in order
        dot[r] = __builtin_fmaf(q[r][4 * t], v.x, dot[r]);
        dot[r] = __builtin_fmaf(q[r][4 * t + 1], v.y, dot[r]);
        dot[r] = __builtin_fmaf(q[r][4 * t + 2], v.z, dot[r]);
        dot[r] = __builtin_fmaf(q[r][4 * t + 3], v.w, dot[r]);
      }
    }
    const bool live = off[b + 1] > off[b];
#pragma unroll
    for (int r = 0; r < kSbarRows; ++r) {
      if (a0 + r >= Cq) break;
      const float sv = dot[r] * scale;
      sbar[((int64_t)bh * Cq + a0 + r) * Ck + b] = sv;
      if (live) mx[r] = fmaxf(mx[r], sv);
    }
  }
#pragma unroll
  for (int r = 0; r < kSbarRows; ++r) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx[r] = fmaxf(mx[r], __shfl_xor(mx[r], o));
    if (lane == 0) red[r][wave] = mx[r];
  }
  __syncthreads();
  if (threadIdx.x < kSbarRows && a0 + threadIdx.x < Cq) {
    const int r = threadIdx.x;
    mrow[(int64_t)bh * Cq + a0 + r] = fmaxf(fmaxf(red[r][0], red[r][1]), fmaxf(red[r][2], red[r][3]));
  }
}

// The same for many centroids: one workgroup per 32 query centroids, whose waves take the 32-blocks of
// key centroids in turn. The dot products run on fp32 MFMAs, k-step s contracting dims 2s (lanes 0-31) and
// 2s + 1: every product is the fma chain over the dims in order, bit for bit that of the kernel above,
// which fetches every key centroid Cq / 4 times. 40 heads, 300 x 1,000 centroids of 128: 240 -> 113 us, 86 with half
// the fetches of a row (the next block's rows fetched ahead cost half the waves: 119);
// with too few workgroups for the chip the longer chain of each loses (5 heads, 200 x 500: 20 -> 33), so
// run_sbar asks for one a CU.
constexpr int kSbarWaves = 8;

// dims h, 2 + h, 4 + h ... of a row: the operands of steps 0 .. D/2 - 1 for lane half h. The lane halves fetch
// alternate 16-byte pieces of the row, each piece once, and exchange them (v_permlane32_swap: the high lanes of one
// register for the low lanes of another).
template <int D>
__device__ __forceinline__ void row_operands(const float* row, int h, float (&x)[D / 2]) {
  auto swap = [](float a, float b, float& lo, float& hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    lo = __uint_as_float(r[0]);  // a of the low lanes, b of the low lanes
    hi = __uint_as_float(r[1]);  // a of the high lanes, b of the high lanes
  };
#pragma unroll
  for (int u = 0; u < D / 8; ++u) {
    const float4 v = *reinterpret_cast<const float4*>(row + 8 * u + 4 * h);
    swap(v.x, v.y, x[4 * u], x[4 * u + 2]);
    swap(v.z, v.w, x[4 * u + 1], x[4 * u + 3]);
  }
}

template <int D>
__global__ void __launch_bounds__(64 * kSbarWaves)
sbar_mfma_kernel(const float* __restrict__ qbar, const float* __restrict__ kbar, const int32_t* __restrict__ k_offsets,
            int Cq, int Ck, float scale, float* __restrict__ sbar, float* __restrict__ mrow,
            bf16_t* __restrict__ q3) {
  __shared__ float red[kSbarWaves][32];
  const int ab = blockIdx.x, bh = blockIdx.y, a0 = 32 * ab;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (q3) {
    constexpr int KSN = D / 16;
    const int nab = (Cq + 31) >> 5;
    for (int i = tid; i < 32 * D; i += 64 * kSbarWaves) {
      const int a = a0 + i / D, k = i % D;
      const float v = a < Cq ? qbar[((int64_t)bh * Cq + a) * D + k] : 0.f;
      const bf16_t hi = f32_to_bf16(v);
      const float r1 = v - bf16_to_f32(hi);
      const bf16_t mid = f32_to_bf16(r1);
      const bf16_t lo = f32_to_bf16(r1 - bf16_to_f32(mid));
      const int ln = (a & 31) + 32 * ((k & 15) >> 3);
      bf16_t* dst = q3 + ((((int64_t)bh * nab + ab) * 3) * KSN + (k >> 4)) * 512 + ln * 8 + (k & 7);
      dst[0] = hi;
      dst[(int64_t)KSN * 512] = mid;
      dst[(int64_t)2 * KSN * 512] = lo;
    }
  }
  const int32_t* off = k_offsets + (int64_t)bh * (Ck + 2);
  const int a = a0 + li;
  float q[D / 2];
  row_operands<D>(qbar + ((int64_t)bh * Cq + min(a, Cq - 1)) * D, lh, q);
  float* out = sbar + ((int64_t)bh * Cq + min(a, Cq - 1)) * Ck;
  float mx = -INFINITY;
  for (int b0 = 32 * wave; b0 < Ck; b0 += 32 * kSbarWaves) {
    float kf[D / 2];
    row_operands<D>(kbar + ((int64_t)bh * Ck + min(b0 + li, Ck - 1)) * D, lh, kf);
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int s = 0; s < D / 2; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s], q[s], acc, 0, 0, 0);
    // register r is key centroid b0 + 8 (r/4) + 4 lh + r%4, query centroid a
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int b = b0 + 8 * g + 4 * lh;
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[r] = acc[4 * g + r] * scale;
        if (b + r < Ck && off[b + r + 1] > off[b + r]) mx = fmaxf(mx, v[r]);
      }
      if (a >= Cq) continue;
      if (b + 4 <= Ck && (Ck & 3) == 0) {
        *reinterpret_cast<float4*>(out + b) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (b + r < Ck) out[b + r] = v[r];
      }
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (lh == 0) red[wave][li] = mx;
  __syncthreads();
  if (tid < 32 && a0 + tid < Cq) {
    float m = red[0][tid];
#pragma unroll
    for (int w = 1; w < kSbarWaves; ++w) m = fmaxf(m, red[w][tid]);
    mrow[(int64_t)bh * Cq + a0 + tid] = m;
  }
}

// fp32 inputs: block errors with the logits qbar_a . k_j on fp32 matrix cores (bound: those, 157 TFLOP/s
// nominal). One workgroup per (head, key cluster, group of kF32Cents query centroids); its four waves
// take the cluster's 32-key blocks in turn (CW = 4). Clusters of about one block leave three of them idle:
// up to 40 keys a cluster each wave takes a cluster of its own (CW = 1), provided that gives every CU a
// workgroup. us a call with four waves a cluster, with one: 40 heads x 9,000 keys, 400 clusters 518, 338;
// 8 x 6,000, 200 clusters 172, 171; 40 x 4,000, 60 clusters (67 keys) 150, 184; 1 x 4,096, 400 clusters, too
// few for the chip, 72, 75. A wave keeps the keys of its block as A operands of
// v_mfma_f32_32x32x2_f32, works out |delta_j|^2 and vbar . delta_j of those keys once, and passes the
// centroids by, 32 at a time; the error of a centroid accumulates in the lanes that hold its keys.
// Every logit is the fma chain over the dims in order, as the centroid logits are: where all keys of a
// cluster equal its centroid (a cluster of one key) W - w is 0 and so is the score, exactly.
// The kernel before kept one query centroid per lane and did its dot products on the vector ALU:
// 32 centroids x 64 clusters of one head of 4,096 keys, d = 64: 112 -> 12 us.
constexpr int kF32Cents = 128;

// (d = 64 asks for waves: without a bound the logits go to AGPRs, and each through a move: 40 x 4,000 keys of 64, 30 x 60
// clusters 72 -> 61 us. d = 128 does not: 8 x 6,000, 100 x 200 213 -> 208 with two waves, but 8 x 4,640, 156 x 53, too
// few workgroups for the chip, 154 -> 162.)
template <int D, bool VALUE_AWARE, int CW>
__global__ void __launch_bounds__(256, D == 128 ? 1 : VALUE_AWARE ? 2 : 3)
block_error_f32_kernel(const float* __restrict__ qbar, const float* __restrict__ vbar, const float* __restrict__ kp,
                       const float* __restrict__ vp, const int32_t* __restrict__ k_offsets,
                       const float* __restrict__ sbar, const float* __restrict__ mrow, int64_t Nk, int Cq, int Ck,
                       float scale, float* __restrict__ scores) {
  constexpr int QS = D / 2;
  constexpr int NB = kF32Cents / 32;
  constexpr int CLUSTERS = 4 / CW;  // of the workgroup
  __shared__ float part[4][kF32Cents];
  __shared__ __attribute__((aligned(16))) float s_vb[CLUSTERS][D];
  const int bh = blockIdx.y, a0 = blockIdx.z * kF32Cents;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int in_wg = wave / CW, share = wave % CW, b = blockIdx.x * CLUSTERS + in_wg;
  const int32_t* off = k_offsets + (int64_t)bh * (Ck + 2);
  const int start = b < Ck ? off[b] : 0, end = b < Ck ? off[b + 1] : 0;
  const int n_cent = min(kF32Cents, Cq - a0), nb = (n_cent + 31) / 32;
  float* out = scores + ((int64_t)bh * Cq + a0) * Ck + b;
  const float* kh = kp + (int64_t)bh * Nk * D;
  const float* vh = vp + (int64_t)bh * Nk * D;
  if (VALUE_AWARE && b < Ck && share == 0)
    for (int t = lane; t < D; t += 64) s_vb[in_wg][t] = vbar[((int64_t)bh * Ck + b) * D + t];
  __syncthreads();
  const float* vb = s_vb[in_wg] + lh * QS;
  float E[NB], W[NB], m[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int a = a0 + 32 * i + li;
    m[i] = a < Cq ? mrow[(int64_t)bh * Cq + a] : 0.f;
    W[i] = a < Cq && end > start ? __expf(fminf(sbar[((int64_t)bh * Cq + a) * Ck + b] - m[i], kMaxExponent)) : 0.f;
  }
  float nvb = 0.f;
  if (VALUE_AWARE) {  // |vbar_b|^2
#pragma unroll 4
    for (int t = 0; t < QS; ++t) nvb = __builtin_fmaf(vb[t], vb[t], nvb);
    nvb += __shfl_xor(nvb, 32);
  }
  // Blocks k, k + 4, ... of a cluster make the k-th of four partial sums whoever takes them, so that the
  // scores do not depend on the form.
  float both[2][NB] = {};
  for (int quarter = share; quarter < 4 && start + 32 * quarter < end; quarter += CW) {
#pragma unroll
    for (int i = 0; i < NB; ++i) E[i] = 0.f;
    for (int j0 = start + 32 * quarter; j0 < end; j0 += 128) {
      const int j = min(j0 + li, end - 1);  // (rows past the cluster's end are not counted below)
      float kf[QS];
      row_operands<D>(kh + (int64_t)j * D, lh, kf);
      float nd = 0.f, dd = 0.f;
      if (VALUE_AWARE) {
        const float4* vr = reinterpret_cast<const float4*>(vh + (int64_t)j * D + lh * QS);
#pragma unroll 8
        for (int t = 0; t < QS / 4; ++t) {
          const float4 v = vr[t], w = reinterpret_cast<const float4*>(vb)[t];
          const float d0 = v.x - w.x, d1 = v.y - w.y, d2 = v.z - w.z, d3 = v.w - w.w;
          nd = __builtin_fmaf(d0, d0, nd); dd = __builtin_fmaf(d0, w.x, dd);
          nd = __builtin_fmaf(d1, d1, nd); dd = __builtin_fmaf(d1, w.y, dd);
          nd = __builtin_fmaf(d2, d2, nd); dd = __builtin_fmaf(d2, w.z, dd);
          nd = __builtin_fmaf(d3, d3, nd); dd = __builtin_fmaf(d3, w.w, dd);
        }
        nd += __shfl_xor(nd, 32);
        dd += __shfl_xor(dd, 32);
      }
      // register r of a score tile is key j0 + 8 (r/4) + 4 lh + r%4
      float nn[16], dl[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = 8 * (r >> 2) + 4 * lh + (r & 3);
        nn[r] = __shfl(nd, key);
        dl[r] = __shfl(dd, key);
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (i >= nb) break;
        float q[QS];
        row_operands<D>(qbar + ((int64_t)bh * Cq + min(a0 + 32 * i + li, Cq - 1)) * D, lh, q);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < QS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s], q[s], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (j0 + 8 * (r >> 2) + 4 * lh + (r & 3) >= end) continue;
          const float w = __expf(fminf(acc[r] * scale - m[i], kMaxExponent));
          const float g = W[i] - w;
          if (VALUE_AWARE) {
            E[i] = __builtin_fmaf(g * g, nvb, E[i]);
            E[i] = __builtin_fmaf(-2.0f * g * w, dl[r], E[i]);
            E[i] = __builtin_fmaf(w * w, nn[r], E[i]);
          } else {
            E[i] = __builtin_fmaf(g, g, E[i]);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const float e = E[i] + __shfl_xor(E[i], 32);
      both[0][i] += quarter < 2 ? e : 0.f;
      both[1][i] += quarter < 2 ? 0.f : e;
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (lh == 0) part[wave][32 * i + li] = both[0][i] + both[1][i];
  __syncthreads();
  if (b >= Ck) return;
  const float n = end > start ? (float)(end - start) : INFINITY;  // empty: score 0, never routed nor compensated
  for (int t = share * 64 + lane; t < n_cent; t += 64 * CW) {
    float e = part[in_wg * CW][t];
    if constexpr (CW == 4) e = (e + part[1][t]) + (part[2][t] + part[3][t]);
    out[(int64_t)t * Ck] = e / n;
  }
}

// ---- bf16 inputs: the probe on the matrix cores -----------------------------------------
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
  union { uint4 u; bf16x8 b; } c;
  c.u = v;
  return c.b;
}

// Block errors with the logits qbar_a . k_j on bf16 MFMAs (qbar in three exact bf16 pieces,
// so the logits carry fp32-level accuracy). One workgroup per (head, `clusters` consecutive
// key clusters, group of 128 query centroids); wave w owns query centroids 32w..32w+31 of the
// group and keeps their operand fragments in registers across those key clusters. The score
// tile is keys x centroids: a lane holds 16 keys of ONE query centroid per 32-key block, so
// the block error accumulates lane-locally.
// The 32-key blocks of the workgroup's key clusters form one sequence, worked at in pairs. Each block is copied
// once by the whole workgroup, straight from global memory into a ring of kProbeStages LDS buffers, two pairs
// ahead of the one being computed, together with its per-key value statistics; the 16-byte chunks of a row are
// XOR-swizzled with the row index so that the operand reads of 32 rows do not collide. One barrier per pair.
// Nothing else is fetched in the loop: a load the compiler waits for would drain the copies.
// A block of a wave is 24 MFMAs (d = 128, 768 cycles of its SIMD) and as long on the vector ALU for the errors
// of its 512 pairs, and a SIMD holds two waves (96 registers of centroid fragments; three waves spill): the errors
// of block k - 1 are written between the MFMAs of block k. At 40 heads, 300 x 1,000 centroids vector issue is busy 54 % of
// the launch, the matrix cores 41 %, with 233 vector and 105 scalar instructions a block of a wave. The whole call: 1,870 us
// with the weights and bounds of a cluster fetched when it begins, 1,660 with all of a workgroup's fetched at its start,
// 1,605 with a barrier per pair of blocks, some 1,500 with no branch per register in a cluster's last block and the groups
// of query centroids side by side on an XCD. Two waves a workgroup, no wave without centroids at 300 of them, took the same.
// d = 64 has half the MFMAs and fragments and is bound by the vector ALU and latencies: three waves a SIMD,
// for which the statistics are read group by group (240 heads x 2,000 keys, 60 clusters, 30 centroids: the
// whole call 127 us with two waves, 103 with three).
constexpr int kProbeClusters = 8;  // most key clusters per workgroup
constexpr int kProbeWaves = 4;     // per workgroup, 32 query centroids each
constexpr int kProbeStages = 6;    // LDS ring buffers: the pair of blocks at work and two pairs in flight

template <int D, bool VALUE_AWARE>
__global__ void __launch_bounds__(64 * kProbeWaves, D == 64 ? 3 : 2)
block_error_mfma_kernel(const bf16_t* __restrict__ q3, const float* __restrict__ vbar, const bf16_t* __restrict__ kp,
                        const int32_t* __restrict__ k_offsets, const float* __restrict__ sbar,
                        const float* __restrict__ mrow, const float* __restrict__ nd, const float* __restrict__ dd,
                        int64_t Nk, int64_t stat_stride, int Cq, int Ck, float scale, int clusters, int cgroups, int heads,
                        float* __restrict__ scores) {
  constexpr int KSN = D / 16;
  constexpr int CPR = D / 8;             // 16-byte chunks per key row
  constexpr int RPI = 64 / CPR;          // key rows per copy instruction of a wave
  constexpr int NCH = 32 / RPI / kProbeWaves;      // copy instructions per wave per block
  constexpr int TILE_B = 32 * D * 2;     // bytes of a block in LDS
  constexpr int LPB = NCH + (VALUE_AWARE ? 1 : 0);  // loads per wave per block
  constexpr int PF = kProbeStages - 2;   // blocks copied ahead when a pair starts, besides the pair
  static_assert(32 % (RPI * kProbeWaves) == 0 && (CPR == 16 || CPR == 8), "tile split / swizzle assume d = 64 or 128");
  __shared__ __attribute__((aligned(1024))) unsigned char ktile[kProbeStages][TILE_B];
  // [|delta|^2 x 32, vbar.delta x 32]; read one block later than the keys, so one buffer more
  __shared__ __attribute__((aligned(256))) float stat[kProbeStages + 1][64];
  // scores of the workgroup's key clusters, per wave [query centroid][key cluster]: they leave together at the
  // end, 16 bytes at a time, instead of each by itself a score row apart
  __shared__ __attribute__((aligned(16))) float sc[kProbeWaves][32][kProbeClusters];
  // centroid weights W of the wave's query centroids; value_scale and |vbar|^2 over its square of the key clusters
  __shared__ float s_w[kProbeWaves][kProbeClusters][32], s_scale[kProbeClusters], s_nvb[kProbeClusters];
  // The groups of query centroids that read the same keys run side by side on one XCD (workgroups go round-robin
  // over the eight): every eight workgroups take eight sets of clusters, the next eight the same sets again.
  const int sets = (Ck + clusters - 1) / clusters * heads;
  const int wg = long_grid_index(), set = wg / (8 * cgroups) * 8 + (wg & 7), cgroup = wg / 8 % cgroups;
  if (set >= sets) return;
  const int per_head = (Ck + clusters - 1) / clusters;
  const int bh = set / per_head, tid = threadIdx.x;
  const int lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ab = cgroup * kProbeWaves + wave, nab = (Cq + 31) >> 5;
  const bool wave_on = ab < nab;  // waves past the last centroid block still help copying
  const int a = 32 * ab + li;
  const bool live = wave_on && a < Cq;
  const int32_t* off = k_offsets + (int64_t)bh * (Ck + 2);
  const int b_lo = set % per_head * clusters, b_end = min(b_lo + clusters, Ck);
  // empty key clusters score 0 (each wave reads and writes its own part of sc only)
  if (lh == 0) {
#pragma unroll
    for (int i = 0; i < kProbeClusters; ++i) sc[wave][li][i] = 0.f;
  }
  auto flush = [&]() {  // the wave's scores to global memory
    if (!live || lh != 0) return;
    float* dst = scores + ((int64_t)bh * Cq + a) * Ck + b_lo;
    if ((b_end - b_lo) % 4 == 0 && clusters % 4 == 0 && (Ck % 4) == 0) {
      for (int i = 0; i < b_end - b_lo; i += 4)
        *reinterpret_cast<float4*>(dst + i) = *reinterpret_cast<const float4*>(&sc[wave][li][i]);
    } else {
      for (int i = 0; i < b_end - b_lo; ++i) dst[i] = sc[wave][li][i];
    }
  };
  bf16x8 bq[3][KSN];
  if (wave_on) {
    const bf16_t* src = q3 + (((int64_t)bh * nab + ab) * 3 * KSN) * 512 + lane * 8;
#pragma unroll
    for (int pc = 0; pc < 3; ++pc)
#pragma unroll
      for (int s = 0; s < KSN; ++s)
        bq[pc][s] = as_bf16x8(*reinterpret_cast<const uint4*>(src + (pc * KSN + s) * 512));
  }
  const float m_a = live ? mrow[(int64_t)bh * Cq + a] : 0.f;
  // exponentials as exp2 with the constants folded: e^(x scale - m) = 2^(x scale2 - m2)
  constexpr float kLog2e = 1.4426950408889634f;
  const float scale2 = scale * kLog2e, neg_m2 = -m_a * kLog2e, cap2 = kMaxExponent * kLog2e;
  // what the loop needs to know about the workgroup's clusters: a fetch in the loop would have to wait for the
  // block copies in flight before it
  const int bounds = off[min(b_lo + lane, Ck)];  // lane i: first key of cluster b_lo + i
  {
    float w[kProbeClusters];
#pragma unroll
    for (int i = 0; i < kProbeClusters; ++i)
      w[i] = live && i < clusters ? sbar[((int64_t)bh * Cq + a) * Ck + min(b_lo + i, Ck - 1)] : 0.f;
#pragma unroll
    for (int i = 0; i < kProbeClusters; ++i)
      if (lh == 0) s_w[wave][i][li] = live ? __expf(fminf(w[i] - m_a, kMaxExponent)) : 0.f;
  }
  if (VALUE_AWARE) {  // |vbar_b|^2 and value_scale: D/64 dims per lane, then across the wave, its clusters side by side
    constexpr int PER = kProbeClusters / kProbeWaves;
    float nvb[PER], largest[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const float* vb = vbar + ((int64_t)bh * Ck + min(b_lo + wave + u * kProbeWaves, Ck - 1)) * D;
      nvb[u] = largest[u] = 0.f;
#pragma unroll
      for (int t = 0; t < D / 64; ++t) {
        const float v = vb[lane + 64 * t];
        nvb[u] = __builtin_fmaf(v, v, nvb[u]);
        largest[u] = fmaxf(largest[u], fabsf(v));
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        nvb[u] += __shfl_xor(nvb[u], o);
        largest[u] = fmaxf(largest[u], __shfl_xor(largest[u], o));
      }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const float scale_b = value_scale(largest[u]), inv = inverse_scale(scale_b);
      if (lane == 0) {
        s_scale[wave + u * kProbeWaves] = scale_b;
        s_nvb[wave + u * kProbeWaves] = nvb[u] * inv * inv;
      }
    }
  }
  SVGEAR_WAIT_VMCNT(0);  // from here on vmcnt counts the block copies only
  const bf16_t* kh = kp + (int64_t)bh * Nk * D;
  const float* ndh = nd + (int64_t)bh * stat_stride;
  const float* ddh = dd + (int64_t)bh * stat_stride;
  const uint32_t lds_k = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)&ktile[0][0];
  const uint32_t lds_s = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)&stat[0][0];

  // position in the sequence of blocks: cluster b, keys j0 .. of [start, end)
  struct Cursor { int b, start, end, j0; };
  auto seek = [&](Cursor& c) {  // first non-empty cluster at or after c.b
    while (c.b < b_end) {
      c.start = __builtin_amdgcn_readlane(bounds, c.b - b_lo);
      c.end = __builtin_amdgcn_readlane(bounds, c.b + 1 - b_lo);
      if (c.end > c.start) break;
      ++c.b;
    }
    c.j0 = c.start;
  };
  auto advance = [&](Cursor& c) {
    c.j0 += 32;
    if (c.j0 >= c.end) {
      ++c.b;
      seek(c);
    }
  };
  // row r of a block keeps its 16-byte chunk c at position c ^ swz(r)
  auto swz = [](int r) { return CPR == 16 ? (r & 15) : ((r >> 1) & 7); };
  auto issue = [&](const Cursor& c, int k) {  // block k of the sequence; rows past the cluster's end repeat its last key
    const int buf = k % kProbeStages;
    const bf16_t* base = kh + (int64_t)c.j0 * D;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int inst = wave * NCH + i;
      const int row = inst * RPI + lane / CPR;
      const int chunk = (lane % CPR) ^ swz(row);
      const uint32_t at = (uint32_t)min(row, c.end - 1 - c.j0) * (D * 2) + chunk * 16;
      async_copy_16B(base, at, __builtin_amdgcn_readfirstlane(lds_k + buf * TILE_B + inst * 1024));
    }
    if (VALUE_AWARE) {  // every wave copies the 64 statistics (same values to the same words)
      const int j = min(c.j0 + li, c.end - 1);
      async_copy_4B((lh ? ddh : ndh) + j, __builtin_amdgcn_readfirstlane(lds_s + (k % (kProbeStages + 1)) * 256));
    }
  };

  Cursor fc{b_lo, 0, 0, 0};  // next block to copy
  seek(fc);
  if (fc.b >= b_end) {  // nothing but empty clusters (uniform over the workgroup)
    flush();
    return;
  }
  Cursor pc = fc;             // block whose errors are being added up
  int issued = 0;
  for (; issued < PF && fc.b < b_end; ++issued) {
    issue(fc, issued);
    advance(fc);
  }
  float E = 0.f, U = 0.f, W = 0.f, vs = 1.f, nvb = 0.f;
  f32x16 acc_even, acc_odd;  // logits of the even and odd blocks
  // logits of block k (MF) and errors of block k - 1 (RANK: 0 none, 1 a full block, 2 a cluster's last one,
  // whose unused rows do not count)
  auto block = [&](int k, f32x16& acc_new, const f32x16& acc, auto mf_tag, auto rank_tag) __attribute__((always_inline)) {
    constexpr bool MF = decltype(mf_tag)::value;
    constexpr int RANK = decltype(rank_tag)::value;
    constexpr int RPS = 16 / KSN;  // registers ranked per k-step
    const unsigned char* kr = &ktile[k % kProbeStages][li * (D * 2)];
    const float* st = stat[(k + kProbeStages) % (kProbeStages + 1)];  // block k - 1
    const int key = swz(li);
    bf16x8 ak[KSN];
    auto rd = [&](int s) { ak[s] = as_bf16x8(*reinterpret_cast<const uint4*>(kr + (((2 * s + lh) ^ key) << 4))); };
    float nn[16], dl[16];
    if constexpr (MF) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc_new[r] = 0.f;
      rd(0);
      rd(1);
    }
    auto rd_stats = [&](int g) {  // of the keys that registers 4g .. 4g + 3 hold
      if constexpr (RANK != 0 && VALUE_AWARE) {
        const float4 n4 = *reinterpret_cast<const float4*>(st + 8 * g + 4 * lh);
        const float4 d4 = *reinterpret_cast<const float4*>(st + 32 + 8 * g + 4 * lh);
        nn[4 * g] = n4.x; nn[4 * g + 1] = n4.y; nn[4 * g + 2] = n4.z; nn[4 * g + 3] = n4.w;
        dl[4 * g] = d4.x; dl[4 * g + 1] = d4.y; dl[4 * g + 2] = d4.z; dl[4 * g + 3] = d4.w;
      }
    };
#pragma unroll
    for (int g = 0; g < (D == 64 ? 1 : 4); ++g) rd_stats(g);
#pragma unroll
    for (int s = 0; s < KSN; ++s) {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (MF) {
        if (s + 2 < KSN) rd(s + 2);
#pragma unroll
        for (int pc3 = 0; pc3 < 3; ++pc3)
          acc_new = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak[s], bq[pc3][s], acc_new, 0, 0, 0);
      }
      if (D == 64 && s + 1 < KSN) rd_stats(s + 1);
      if constexpr (RANK != 0) {
        // register r is key j0 + 8(r/4) + 4lh + r%4, query centroid a. Per key, with u = W - w:
        //   |W vbar - w v_j|^2 = u^2 |vbar|^2 + w (-2 u vbar.delta_j + w |delta_j|^2),
        // the u^2 in a sum of their own, which takes its factor at the end of the cluster; u comes times value_scale,
        // its other factors over it (unscaled, 6,200 keys at the cap overflowed the sum whatever the values were, and
        // weights below e^-44 lost digits; with |vbar|^2 in the term instead, a multiplication more a pair: 2 % of
        // the call above)
#pragma unroll
        for (int r = s * RPS; r < (s + 1) * RPS; ++r) {
          const float w = __builtin_amdgcn_exp2f(fminf(__builtin_fmaf(acc[r], scale2, neg_m2), cap2));
          const float u = VALUE_AWARE ? __builtin_fmaf(-vs, w, W) : W - w;
          float uu = __builtin_fmaf(u, u, U), e = E;
          if (VALUE_AWARE) e = __builtin_fmaf(w, __builtin_fmaf(u, dl[r], w * nn[r]), E);
          // (an unused row, which repeats the cluster's last key, does not count: a select of the sums, no
          // product of 0 with a value that has overflowed, and no branch per register: the compiler would
          // rather make one)
          if constexpr (RANK == 2) {
            asm volatile("" : "+v"(uu), "+v"(e));
            const bool used = pc.j0 + 8 * (r >> 2) + 4 * lh + (r & 3) < pc.end;
            uu = used ? uu : U;
            e = used ? e : E;
          }
          U = uu;
          E = e;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  using No = std::integral_constant<int, 0>;
  using Full = std::integral_constant<int, 1>;
  using Last = std::integral_constant<int, 2>;
  auto iteration = [&](int k, f32x16& acc_new, f32x16& acc) __attribute__((always_inline)) {
    const bool mf = k < issued;  // block k exists
    if (mf && (k & 1) == 0) {  // blocks k and k + 1 have landed once at most the copies of later ones are outstanding
      const int ahead = issued - k - 2;
      if (ahead >= 2) SVGEAR_WAIT_VMCNT(2 * LPB);
      else if (ahead == 1) SVGEAR_WAIT_VMCNT(LPB);
      else SVGEAR_WAIT_VMCNT(0);
      __syncthreads();  // everyone's part of them is in LDS; everyone is done with the pair before
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (fc.b < b_end) {
          issue(fc, issued);
          advance(fc);
          ++issued;
        }
    }
    if (k == 0) {
      if (wave_on) block(k, acc_new, acc, std::true_type{}, No{});
      return true;
    }
    if (pc.j0 == pc.start) {  // first block of key cluster pc.b
      E = U = 0.f;
      W = s_w[wave][pc.b - b_lo][li];
      if (VALUE_AWARE) {
        vs = s_scale[pc.b - b_lo];
        nvb = s_nvb[pc.b - b_lo];
        W *= vs;
      }
    }
    if (wave_on) {
      const bool full = pc.j0 + 32 <= pc.end;
      if (mf && full) block(k, acc_new, acc, std::true_type{}, Full{});
      else if (mf) block(k, acc_new, acc, std::true_type{}, Last{});
      else if (full) block(k, acc_new, acc, std::false_type{}, Full{});
      else block(k, acc_new, acc, std::false_type{}, Last{});
      if (pc.j0 + 32 >= pc.end) {  // last block of the cluster
        // (both lanes' sums first: a lane without a key would multiply 0 by a norm that may have overflowed)
        float Et = U + __shfl_xor(U, 32);
        if (VALUE_AWARE) Et = __builtin_fmaf(Et, nvb, E + __shfl_xor(E, 32));
        if (lh == 0) sc[wave][li][pc.b - b_lo] = Et / (float)(pc.end - pc.start);
      }
    }
    advance(pc);
    return mf;
  };
  for (int k = 0;; k += 2) {  // (two at a time: the accumulators swap their parts without a move)
    if (!iteration(k, acc_even, acc_odd)) break;
    if (!iteration(k + 1, acc_odd, acc_even)) break;
  }
  flush();
}

}  // namespace

// Centroid logits and their row maxima (q3: see sbar_kernel), and beside them the statistics of the values.
static int run_logits(const float* qbar, const float* kbar, const int32_t* k_offsets, int BH, int d, int Cq, int Ck,
                      float scale, float* sbar, float* mrow, bf16_t* q3, const ValueStats& stats, hipStream_t s) {
  int groups = 1, blocks = 0;
  if (ceil_div(Cq, 32) * BH >= 256) {
    auto kern = d == 64 ? sbar_mfma_kernel<64> : sbar_mfma_kernel<128>;
    kern<<<dim3((unsigned)ceil_div(Cq, 32), BH), 64 * kSbarWaves, 0, s>>>(qbar, kbar, k_offsets, Cq, Ck, scale, sbar, mrow, q3);
    SVGEAR_LAUNCH_CHECK();
  } else {
    groups = (int)ceil_div(q3 ? align_up(Cq, 32) : Cq, kSbarRows);
    blocks = groups * BH;
  }
  if (blocks + stats.clusters > 0) {
    auto kern = d == 64 ? sbar_kernel<64> : sbar_kernel<128>;
    kern<<<long_grid((int64_t)blocks + stats.clusters), 256, 0, s>>>(qbar, kbar, k_offsets, Cq, Ck, scale, sbar, mrow, q3, groups, blocks, stats);
    SVGEAR_LAUNCH_CHECK();
  }
  return SVGEAR_OK;
}

int run_sbar(const float* qbar, const float* kbar, const int32_t* k_offsets, int BH, int d, int Cq, int Ck,
             float scale, float* sbar, float* mrow, bf16_t* q3, hipStream_t s) {
  return run_logits(qbar, kbar, k_offsets, BH, d, Cq, Ck, scale, sbar, mrow, q3, ValueStats{}, s);
}

int run_probe(const float* qbar, const float* kbar, const float* vbar, const void* kp, const void* vp,
              svgear_dtype dt, const int32_t* k_offsets, int BH, int64_t Nk, int d, int Cq, int Ck, float scale,
              bool value_aware, float* scores, float* sbar, float* mrow, bf16_t* q3, float* nd, float* dd,
              hipStream_t s) {
  const bool mfma = dt == SVGEAR_BF16;
  const int64_t stat_stride = probe_stat_stride(Nk);
  ValueStats stats{};
  if (mfma && value_aware) stats = ValueStats{vbar, static_cast<const bf16_t*>(vp), Nk, stat_stride, nd, dd, BH * Ck};
  const int rc = run_logits(qbar, kbar, k_offsets, BH, d, Cq, Ck, scale, sbar, mrow, mfma ? q3 : nullptr, stats, s);
  if (rc != SVGEAR_OK) return rc;
  if (mfma) {
    const bf16_t* k16 = static_cast<const bf16_t*>(kp);
    const int groups = (int)ceil_div(ceil_div(Cq, 32), kProbeWaves);
    // key clusters a workgroup: its start (fragments, weights, the first copies) is worth some three clusters of
    // 75 keys, but a launch wants two rounds of the 512 workgroups that are resident at once. us a call with 1, 2, 4, 8:
    // 40 heads, 300 x 1,000 centroids 2205, 1840, 1561, 1493; 5 x 200 x 500 247, 231, 225, 234; 8 x 30 x 60 38, 40, 44, 50
    const int64_t units = (int64_t)BH * Ck * groups;
    const int clusters = units >= 8192 ? kProbeClusters : units >= 2048 ? 4 : units >= 1024 ? 2 : 1;
    const dim3 gb = long_grid((int64_t)align_up(ceil_div(Ck, clusters) * BH, 8) * groups);
#define SVGEAR_PM(D, VA)                                                                                     \
  block_error_mfma_kernel<D, VA><<<gb, 64 * kProbeWaves, 0, s>>>(q3, vbar, k16, k_offsets, sbar, mrow, nd, dd, Nk, stat_stride, \
                                                    Cq, Ck, scale, clusters, groups, BH, scores)
    if (d == 64) { if (value_aware) SVGEAR_PM(64, true); else SVGEAR_PM(64, false); }
    else { if (value_aware) SVGEAR_PM(128, true); else SVGEAR_PM(128, false); }
#undef SVGEAR_PM
    SVGEAR_LAUNCH_CHECK();
    return SVGEAR_OK;
  }
  const unsigned groups = (unsigned)ceil_div(Cq, kF32Cents);
  const bool wave_each = Nk <= (int64_t)40 * Ck && (int64_t)BH * Ck * groups >= 1024;
  const dim3 grid((unsigned)(wave_each ? ceil_div(Ck, 4) : Ck), BH, groups);
  using Kernel = decltype(&block_error_f32_kernel<64, true, 4>);
  static const Kernel kernels[2][2][2] = {
      {{block_error_f32_kernel<64, false, 4>, block_error_f32_kernel<64, false, 1>},
       {block_error_f32_kernel<64, true, 4>, block_error_f32_kernel<64, true, 1>}},
      {{block_error_f32_kernel<128, false, 4>, block_error_f32_kernel<128, false, 1>},
       {block_error_f32_kernel<128, true, 4>, block_error_f32_kernel<128, true, 1>}}};
  kernels[d == 128][value_aware][wave_each]<<<grid, 256, 0, s>>>(qbar, vbar, static_cast<const float*>(kp),
                                                                 static_cast<const float*>(vp), k_offsets, sbar, mrow,
                                                                 Nk, Cq, Ck, scale, scores);
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}

}  // namespace svgear
