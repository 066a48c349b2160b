// fp32 kernel of the fused block-sparse attention + centroid compensation.
// Paper: Eq. (1), Eq. (6), Algorithm 2 (see attention.hip for the decomposition).
//
// What bounds it: fp32 matrix cores (157 TFLOP/s nominal; a library fp32 product reaches 153 here).
// Every product runs on v_mfma_f32_32x32x2_f32, whose accumulation is a chain of fp32 fmas, so
// nothing is narrower than fp32 anywhere; a 32x32x2 step takes 64 cycles for 64 lanes x 2 operand
// words, so operands, softmax and barriers all hide behind the matrix work.
//   * A workgroup owns a block of 32 query rows of one cluster; its waves take the 32-key tiles in
//     turn and meet once, at the end. S^T = K Q^T: a lane owns one query (lane % 32) and the 16 keys
//     8 (r / 4) + 4 (lane / 32) + r % 4 of a tile.
//   * Those registers are B operands of O^T += V^T P^T as they stand: step r contracts the two keys
//     that register r holds in the two lane halves. The rows of O^T are dealt to the D / 32
//     accumulators so that a lane reads its D / 32 values of V with one LDS read.
//   * The contraction index of S is dealt to the lane halves as dims 0 .. D/2-1 and D/2 .. D-1, so
//     one 16-byte LDS read feeds four steps; 16-byte chunks of a K row are XOR-swizzled.
//   * A wave copies its tiles from global memory straight into LDS of its own: the next K tile while
//     it contracts V, the next V tile while it contracts K (4,096 cycles each at d = 128), so one
//     buffer of each suffices and the loop has no barrier. (The first version shared the tiles
//     among four waves of 32 rows: clusters of 124 rows fill 2.7 waves of a tile, and a barrier a
//     step made the others wait for the SIMD that had two: 0.67 ms where this one takes 0.51.)
//     Unused keys of a tile come from a row of zeros, so no value of a masked row meets the sums.
//   * Short problems have fewer query blocks than the chip has CUs (one head of 4,096 rows: 160), so
//     the keys of a block are dealt to several workgroups there and their (O, max, sum) merged in a
//     fixed order (f32_splits).
// Measured (d = 128, 8 heads x 5,957 rows, 48 / 160 clusters, a quarter routed): 8.7 -> 0.51 ms, 76 TFLOP/s
// of 153; of the rest a fifth is rows and keys that fill no block, a fifth a workgroup's start and end.
// The kernel before kept one query row per lane on the vector ALU. Error against 64 bits: 7.3e-7 -> 2.0e-7.
#include "attention.h"

#include <type_traits>

namespace svgear {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kF32Keys = 32;  // keys per tile
constexpr int kF32Rows = 32;  // query rows per workgroup
constexpr int kF32Target = 512;  // workgroups wanted (256 to 1024: the same; 3,000: 0.51 -> 0.58 ms for the merge)

static inline size_t f32_lds_bytes(int d, int waves, int Ck) {
  return (size_t)waves * (2 * kF32Keys * d * 4 + 2 * kF32Keys * 8 + kF32Keys * 4 + 2 * kF32Rows * 4) + (2 * (size_t)(Ck + 3) + 1) * 4;
}

// ------------------------------------------------------------------------------ plan
// Tile list of every head: tile -> (query cluster, first row). One workgroup per head. With at most
// kPlanSort clusters the tiles of the clusters that route the most keys come first: lists differ
// by two orders of magnitude, and a long one that starts last has the chip to itself (measured at
// 8 heads x 5,957 rows: 0.58 -> 0.51 ms).
constexpr int kZeros = 128;  // floats in the row of zeros
constexpr int kPlanThreads = 1024, kPlanSort = 1024;
__global__ void __launch_bounds__(kPlanThreads)
plan_kernel(const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ k_offsets,
            const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int Cq, int Ck, int BM,
            int max_tiles, int32_t* __restrict__ tile_a, int32_t* __restrict__ tile_row0, int32_t* __restrict__ n_tiles,
            float* __restrict__ zeros) {
  extern __shared__ int32_t first[];  // Cq+2: tiles of the clusters, then their first tile, in list order
  __shared__ int32_t len[kPlanSort], order[kPlanSort];
  const int bh = blockIdx.x, R = Cq + 1, Cc = Ck + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const int32_t* rp = row_ptr + (int64_t)bh * (R + 1);
  const bool sorted = R <= kPlanSort;
  if (bh == 0 && threadIdx.x < kZeros) zeros[threadIdx.x] = 0.f;
  if (sorted) {
    for (int a = wave; a < R; a += kPlanThreads / 64) {  // a wave per cluster, its lanes over the routed key clusters
      const int32_t* ci = col_idx + (int64_t)bh * R * Cc + rp[a];
      const int ne = rp[a + 1] - rp[a];
      int n = 0;
      for (int e = lane; e < ne; e += 64) n += max(ko[ci[e] + 1] - ko[ci[e]], 0);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
      if (lane == 0) len[a] = n;
    }
    __syncthreads();
    for (int a = threadIdx.x; a < R; a += kPlanThreads) {
      int rank = 0;
      for (int b = 0; b < R; ++b) rank += len[b] > len[a] || (len[b] == len[a] && b < a);
      order[rank] = a;
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < R; i += kPlanThreads) {
    const int a = sorted ? order[i] : i;
    first[i] = (qo[a + 1] - qo[a] + BM - 1) / BM;
  }
  __syncthreads();
  if (wave == 0) {
    int carry = 0;
    for (int i0 = 0; i0 < R; i0 += 64) {
      const int i = i0 + lane, c = i < R ? first[i] : 0;
      int incl = c;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      if (i < R) first[i] = carry + incl - c;
      carry += __shfl(incl, 63);
    }
    if (lane == 0) {
      first[R] = carry;
      n_tiles[bh] = carry < max_tiles ? carry : max_tiles;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < R; i += kPlanThreads) {
    const int a = sorted ? order[i] : i;
    const int lo = first[i], hi = first[i + 1];
    for (int t = lo; t < hi && t < max_tiles; ++t) {
      tile_a[(int64_t)bh * max_tiles + t] = a;
      tile_row0[(int64_t)bh * max_tiles + t] = qo[a] + (t - lo) * BM;
    }
  }
}

// (two waves a SIMD asked for at d = 64: without a bound the accumulators go to AGPRs, and every score through a move;
// 8 heads x 5,957 rows 244 -> 235 us. d = 128 needs more registers than two waves have.)
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, D == 64 ? 2 : 1)
attn_f32_kernel(AttnArgs p) {
  constexpr int CPR = D / 4;                // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;             // rows per copy instruction
  constexpr int COPIES = kF32Keys / RPI;    // copy instructions per tensor and tile
  constexpr int TILE = kF32Keys * D * 4;
  constexpr int DB = D / 32;                // accumulators of O^T
  constexpr int QS = D / 2;                 // steps of S
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];  // per wave: K tile, V tile
  const float** ptr_s = reinterpret_cast<const float**>(smem + NW * 2 * TILE);  // per wave [keys] K rows, [keys] V rows
  float* bias_s = reinterpret_cast<float*>(ptr_s + NW * 2 * kF32Keys);          // per wave [keys]
  float* ml_s = bias_s + NW * kF32Keys;                                   // per wave [rows] maximum, [rows] sum
  // routed clusters e < ne: first virtual position, first row; then, from ne + 1 on, the
  // compensated clusters: index, bias bits
  int32_t* ent0 = reinterpret_cast<int32_t*>(ml_s + NW * 2 * kF32Rows);
  int32_t* ent1 = ent0 + (p.Ck + 3);
  int32_t* n_comp = ent1 + (p.Ck + 3);

  // XCD-aware order: workgroups go round-robin over the 8 XCDs; each gets one contiguous range of
  // blocks, so that blocks that share routed K/V share an L2
  const int total = gridDim.x, wg = blockIdx.x;
  const int logical = (wg & 7) * (total >> 3) + (wg >> 3);
  const int bh = logical / p.max_tiles, tile = logical % p.max_tiles;
  if (bh >= p.BH || tile >= p.n_tiles[bh]) return;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Cq = p.Cq, Ck = p.Ck, R = Cq + 1, Cc = Ck + 1, W = (Cc + 31) / 32;
  const int a = p.tile_a[(int64_t)bh * p.max_tiles + tile];
  const int row0 = p.tile_row0[(int64_t)bh * p.max_tiles + tile];
  const int32_t* qo = p.q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = p.k_offsets + (int64_t)bh * (Ck + 2);
  const int n_rows = min(qo[a + 1] - row0, kF32Rows);
  const int32_t* rp = p.row_ptr + (int64_t)bh * (R + 1);
  const int32_t* ci = p.col_idx + (int64_t)bh * R * Cc + rp[a];
  const int ne = min(rp[a + 1] - rp[a], Cc);

  // ---- virtual key sequence of the routed clusters (wave 0), list of the compensated ones (wave 1)
  if (wave == 0) {
    int carry = 0;
    for (int e0 = 0; e0 < ne; e0 += 64) {
      const int e = e0 + lane;
      int sz = 0;
      if (e < ne) {
        const int b = ci[e];
        const int ps = ko[b];
        sz = max(ko[b + 1] - ps, 0);
        ent1[e] = ps;
      }
      int incl = sz;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      if (e < ne) ent0[e] = carry + incl - sz;
      carry += __shfl(incl, 63);
    }
    if (lane == 0) ent0[ne] = carry;
  } else if (wave == 1) {
    int at = ne + 1;
    if (a < Cq) {
      const uint32_t* mrow = p.mask_bits + ((int64_t)bh * R + a) * W;
      for (int b0 = 0; b0 < Ck; b0 += 64) {
        const int b = b0 + lane;
        const int sz = b < Ck ? ko[b + 1] - ko[b] : 0;
        const bool on = sz > 0 && !mask_bit(mrow, b);
        const unsigned long long votes = __ballot(on);
        const int slot = at + __popcll(votes & ((1ull << lane) - 1ull));
        if (on && slot < Ck + 3) {
          ent0[slot] = b;
          ent1[slot] = __float_as_int(log2f((float)sz));
        }
        at += __popcll(votes);
      }
    }
    if (lane == 0) *n_comp = min(at, Ck + 3) - (ne + 1);
  }
  // ---- query rows (B operand of S^T): the lane's half of row li
  float q[QS];
  {
    const float4* qr = reinterpret_cast<const float4*>(static_cast<const float*>(p.qp) +
                                                       q_row_offset(p, bh, row0 + min(li, n_rows - 1), D) + lh * QS);
#pragma unroll
    for (int t = 0; t < QS / 4; ++t) {
      const float4 v = qr[t];
      q[4 * t] = v.x; q[4 * t + 1] = v.y; q[4 * t + 2] = v.z; q[4 * t + 3] = v.w;
    }
  }
  SVGEAR_WAIT_VMCNT(0);  // from here on vmcnt counts the tile copies only
  __syncthreads();
  const int n_r = __builtin_amdgcn_readfirstlane(ent0[ne]);
  const int n_c = __builtin_amdgcn_readfirstlane(*n_comp);
  const int nt_r = (n_r + kF32Keys - 1) / kF32Keys;
  const int T = nt_r + (n_c + kF32Keys - 1) / kF32Keys;
  const int split = blockIdx.y, splits = gridDim.y;
  const int t_lo = (int)((int64_t)T * split / splits), t_hi = (int)((int64_t)T * (split + 1) / splits);

  const float* kh = static_cast<const float*>(p.kp) + (int64_t)bh * p.Nk * D;
  const float* vh = static_cast<const float*>(p.vp) + (int64_t)bh * p.Nk * D;
  const float* kc = p.kbar + (int64_t)bh * Ck * D;
  const float* vc = p.vbar + (int64_t)bh * Ck * D;
  unsigned char* Kw = smem + wave * 2 * TILE;
  unsigned char* Vw = Kw + TILE;
  float* bias = bias_s + wave * kF32Keys;
  const uint32_t lds_k = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)Kw;
  const uint32_t lds_v = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)Vw;

  // the cluster that this lane's first virtual position lies in: the last e with ent0[e] <= it
  int t = t_lo + wave, cur = 0;
  for (int hi = ne; hi - cur > 1;) {
    const int mid = (cur + hi) >> 1;
    if (ent0[mid] <= t * kF32Keys + li) cur = mid;
    else hi = mid;
  }
  // rows and bias of key li of a tile (both lane halves alike) to the wave's tables
  const float** kptr = ptr_s + wave * 2 * kF32Keys;
  const float** vptr = kptr + kF32Keys;
  auto map_tile = [&](int tt) __attribute__((always_inline)) {
    const float* kr = p.zeros;
    const float* vr = p.zeros;
    float b = -INFINITY;
    if (tt < nt_r) {
      const int pos = tt * kF32Keys + li;
      if (pos < n_r) {
        while (pos >= ent0[cur + 1]) ++cur;
        const int64_t at = (int64_t)(ent1[cur] + (pos - ent0[cur])) * D;
        kr = kh + at;
        vr = vh + at;
        b = 0.f;
      }
    } else {
      const int e = (tt - nt_r) * kF32Keys + li;
      if (e < n_c) {
        const int64_t at = (int64_t)ent0[ne + 1 + e] * D;
        kr = kc + at;
        vr = vc + at;
        b = __int_as_float(ent1[ne + 1 + e]);
      }
    }
    kptr[li] = kr;
    vptr[li] = vr;
    bias[li] = b;
  };
  // copy i of a tile: rows i RPI .. of it, `row` read from the table beforehand. The 16-byte chunks
  // of a K row are swizzled on the global side of the copy.
  const int slot = lane % CPR, sub = lane / CPR;
  auto copy_k = [&](int i, const float* row) __attribute__((always_inline)) {
    async_copy_16B(row + 4 * (slot ^ ((i * RPI + sub) & (CPR - 1))),
                   __builtin_amdgcn_readfirstlane(lds_k + i * 1024));
  };
  auto copy_v = [&](int i, const float* row) __attribute__((always_inline)) {
    async_copy_16B(row + 4 * slot, __builtin_amdgcn_readfirstlane(lds_v + i * 1024));
  };

  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m = -INFINITY, l = 0.f;
  const float c = p.scale * kLog2e;

  // The copies of V(t) are issued between the first MFMAs of S(t), those of K(t + 1) between the first
  // of PV(t): each lands under the second half of the product it is issued in. Operand reads run
  // AHEAD fragments before the MFMAs that consume them (the order is pinned: left alone,
  // the compiler sinks each read to its use).
  constexpr int AHEAD = 4;
  constexpr int CPI = COPIES / 8;  // copies per fragment, over the first 8 fragments
  if (t < t_hi) {
    map_tile(t);
#pragma unroll
    for (int i = 0; i < COPIES; ++i) copy_k(i, kptr[i * RPI + sub]);
  }
  for (; t < t_hi; t += NW) {
    SVGEAR_WAIT_VMCNT(0);  // the K tile has landed
    asm volatile("" ::: "memory");
    const unsigned char* kr = Kw + li * (D * 4);
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; ++r) s0[r] = s1[r] = 0.f;
    {
      constexpr int NF = QS / 4;
      float4 kf[NF];
      const float* vrow[COPIES];
      auto read_k = [&](int u) {  // dims lh D/2 + 4u ..: chunk lh CPR/2 + u of row li
        kf[u] = *reinterpret_cast<const float4*>(kr + (((lh * (CPR / 2) + u) ^ (li & (CPR - 1))) << 4));
      };
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) read_k(u);
#pragma unroll
      for (int i = 0; i < COPIES; ++i) vrow[i] = vptr[i * RPI + sub];
#pragma unroll
      for (int u = 0; u < NF; ++u) {
        __builtin_amdgcn_sched_barrier(0);
        if (u + AHEAD < NF) read_k(u + AHEAD);
        s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u].x, q[4 * u], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u].y, q[4 * u + 1], s1, 0, 0, 0);
        if (u < 8) {
#pragma unroll
          for (int i = 0; i < CPI; ++i) copy_v(CPI * u + i, vrow[CPI * u + i]);
        }
        s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u].z, q[4 * u + 2], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[u].w, q[4 * u + 3], s1, 0, 0, 0);
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b4 = *reinterpret_cast<const float4*>(bias + 8 * g + 4 * lh);
      const float bb[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s0[4 * g + r] = __builtin_fmaf(s0[4 * g + r] + s1[4 * g + r], c, bb[r]);
        mx = fmaxf(mx, s0[4 * g + r]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (__any(mx > m)) {
      const float m_new = fmaxf(m, mx);
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m = m_new;
    }
    const float m_use = m == -INFINITY ? 0.f : m;
    float ls = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s0[r] = __builtin_amdgcn_exp2f(s0[r] - m_use);
      ls += s0[r];
    }
    l += ls;
    const bool more = t + NW < t_hi;
    if (more) map_tile(t + NW);
    SVGEAR_WAIT_VMCNT(0);  // the V tile has landed
    asm volatile("" ::: "memory");
    const unsigned char* vt = Vw + li * (DB * 4);
    auto contract = [&](auto more_tag) __attribute__((always_inline)) {
      constexpr bool MORE = decltype(more_tag)::value;
      float4 vf[16];
      const float* krow[COPIES];
      auto read_v = [&](int r) {  // keys 8 (r/4) + r%4 (low lanes) and + 4 (high lanes)
        const unsigned char* vr = vt + (8 * (r >> 2) + 4 * lh + (r & 3)) * (D * 4);
        if constexpr (DB == 4) {
          vf[r] = *reinterpret_cast<const float4*>(vr);
        } else {
          const float2 v2 = *reinterpret_cast<const float2*>(vr);
          vf[r].x = v2.x;
          vf[r].y = v2.y;
        }
      };
#pragma unroll
      for (int r = 0; r < AHEAD; ++r) read_v(r);
      if (MORE) {
#pragma unroll
        for (int i = 0; i < COPIES; ++i) krow[i] = kptr[i * RPI + sub];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        __builtin_amdgcn_sched_barrier(0);
        if (r + AHEAD < 16) read_v(r + AHEAD);
        o[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r].x, s0[r], o[0], 0, 0, 0);
        o[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r].y, s0[r], o[1], 0, 0, 0);
        if (MORE && r < 8) {
#pragma unroll
          for (int i = 0; i < CPI; ++i) copy_k(CPI * r + i, krow[CPI * r + i]);
        }
        if constexpr (DB == 4) {
          o[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r].z, s0[r], o[2], 0, 0, 0);
          o[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r].w, s0[r], o[3], 0, 0, 0);
        }
      }
    };
    if (more) contract(std::true_type{});
    else contract(std::false_type{});
    // every read of the V tile has returned before the next tile's copies overwrite it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }

  // ---- the waves' parts meet in LDS (each in its own K tile), added in wave order
  l += __shfl_xor(l, 32);
  if (lh == 0) {
    ml_s[wave * 2 * kF32Rows + li] = m;
    ml_s[wave * 2 * kF32Rows + kF32Rows + li] = l;
  }
  // lane holds rows i = 8 (r/4) + 4 lh + r%4 of every accumulator: dims DB i .. DB i + DB - 1;
  // 16-byte chunks are rotated by the row so that the 32 rows of a store fall on different banks
  float* part = reinterpret_cast<float*>(Kw) + li * D;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int dim = DB * (8 * (r >> 2) + 4 * lh + (r & 3));
    float* d = part + (((dim >> 2) + li) % CPR) * 4 + (dim & 3);
    if constexpr (DB == 4) *reinterpret_cast<float4*>(d) = make_float4(o[0][r], o[1][r], o[2][r], o[3][r]);
    else *reinterpret_cast<float2*>(d) = make_float2(o[0][r], o[1][r]);
  }
  __syncthreads();
  const int64_t rows_all = (int64_t)p.BH * p.Nq;
  for (int u = tid; u < n_rows * CPR; u += 64 * NW) {
    const int i = u / CPR, ch = u % CPR;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, ml_s[w * 2 * kF32Rows + i]);
    const float m_use = M == -INFINITY ? 0.f : M;
    float lt = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(ml_s[w * 2 * kF32Rows + i] - m_use);
      const float4 v = *reinterpret_cast<const float4*>(smem + w * 2 * TILE + (i * D + ((ch + i) % CPR) * 4) * 4);
      lt = __builtin_fmaf(f, ml_s[w * 2 * kF32Rows + kF32Rows + i], lt);
      acc.x = __builtin_fmaf(f, v.x, acc.x);
      acc.y = __builtin_fmaf(f, v.y, acc.y);
      acc.z = __builtin_fmaf(f, v.z, acc.z);
      acc.w = __builtin_fmaf(f, v.w, acc.w);
    }
    if (splits == 1) {
      int64_t lse_idx;
      float* d = static_cast<float*>(p.op) + out_row_offset(p, bh, row0 + i, D, lse_idx) + 4 * ch;
      float f = lt > 0.f ? 1.0f / lt : 0.f;
      if (!(lt >= 0.f)) f = lt;  // NaN stays NaN
      *reinterpret_cast<float4*>(d) = make_float4(acc.x * f, acc.y * f, acc.z * f, acc.w * f);
      if (p.lse && ch == 0) p.lse[lse_idx] = (M + log2f(lt)) * kLn2;
    } else {
      const int64_t at = split * rows_all + (int64_t)bh * p.Nq + row0 + i;
      if (ch == 0) p.part_ml[at] = make_float2(M, lt);
      *reinterpret_cast<float4*>(p.part_o + at * D + 4 * ch) = acc;
    }
  }
}

// Adds the splits of every row, in split order: one thread per 4 dims.
template <int D>
__global__ void __launch_bounds__(256)
merge_f32_kernel(AttnArgs p, int splits) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t rows = (int64_t)p.BH * p.Nq, row = u / (D / 4);
  if (row >= rows) return;
  const int dim = 4 * (int)(u % (D / 4));
  float M = -INFINITY;
  for (int s = 0; s < splits; ++s) M = fmaxf(M, p.part_ml[s * rows + row].x);
  float l = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < splits; ++s) {
    const float2 ml = p.part_ml[s * rows + row];
    if (ml.x == -INFINITY && ml.y == 0.f) continue;  // no key there
    const float w = __builtin_amdgcn_exp2f(ml.x - M);
    const float4 v = *reinterpret_cast<const float4*>(p.part_o + (s * rows + row) * D + dim);
    l = __builtin_fmaf(w, ml.y, l);
    acc.x = __builtin_fmaf(w, v.x, acc.x);
    acc.y = __builtin_fmaf(w, v.y, acc.y);
    acc.z = __builtin_fmaf(w, v.z, acc.z);
    acc.w = __builtin_fmaf(w, v.w, acc.w);
  }
  float f = l > 0.f ? 1.0f / l : 0.f;
  if (!(l >= 0.f)) f = l;
  int64_t lse_idx;
  const int bh = (int)(row / p.Nq);
  float* d = static_cast<float*>(p.op) + out_row_offset(p, bh, row - (int64_t)bh * p.Nq, D, lse_idx) + dim;
  *reinterpret_cast<float4*>(d) = make_float4(acc.x * f, acc.y * f, acc.z * f, acc.w * f);
  if (p.lse && dim == 0) p.lse[lse_idx] = (M + log2f(l)) * kLn2;
}

template <int D, int NW>
int launch(const AttnArgs& a, int splits, hipStream_t s) {
  const unsigned total = (unsigned)align_up((size_t)a.BH * a.max_tiles, 8);
  const size_t lds = f32_lds_bytes(D, NW, a.Ck);
  auto kern = attn_f32_kernel<D, NW>;
  SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
  kern<<<dim3(total, splits), 64 * NW, lds, s>>>(a);
  SVGEAR_LAUNCH_CHECK();
  if (splits > 1) {
    merge_f32_kernel<D><<<(unsigned)ceil_div((int64_t)a.BH * a.Nq * (D / 4), 256), 256, 0, s>>>(a, splits);
    SVGEAR_LAUNCH_CHECK();
  }
  return SVGEAR_OK;
}

// Workgroups the keys of a query block are dealt to: as many as give the chip two rounds of
// workgroups (one of d = 128, two of d = 64 fit a CU); a split costs a pass over its partial rows,
// so a problem that fills the chip by itself is not split.
static int f32_splits(int64_t BH, int64_t Nq, int64_t Nk, int Cq) {
  const int64_t tiles = BH * (ceil_div(Nq, kF32Rows) + Cq / 2);  // a cluster's last block is half full
  const int64_t want = ceil_div((int64_t)kF32Target, tiles), most = Nk / (16 * kF32Keys);
  const int64_t n = want < most ? want : most;
  return (int)(n < 1 ? 1 : (n > 8 ? 8 : n));
}

}  // namespace

size_t f32_workspace(int64_t BH, int64_t Nq, int64_t Nk, int Cq, int d) {
  const int n = f32_splits(BH, Nq, Nk, Cq);
  const size_t rows = (size_t)BH * Nq, tiles = (size_t)BH * (ceil_div(Nq, kF32Rows) + Cq + 1);
  return 2 * align_up(tiles * 4, 256) + align_up(BH * 4, 256) + align_up(kZeros * 4, 256) +
         (n > 1 ? align_up(n * rows * d * 4, 256) + align_up(n * rows * sizeof(float2), 256) : 0);
}

int launch_attn_f32(AttnArgs& a, int d, void* ws, size_t ws_bytes, hipStream_t s) {
  Workspace w(ws, ws_bytes);
  const int splits = f32_splits(a.BH, a.Nq, a.Nk, a.Cq);
  const size_t rows = (size_t)a.BH * a.Nq;
  a.max_tiles = (int)(ceil_div(a.Nq, kF32Rows) + a.Cq + 1);
  int32_t* tile_a = w.take<int32_t>((size_t)a.BH * a.max_tiles);
  int32_t* tile_row0 = w.take<int32_t>((size_t)a.BH * a.max_tiles);
  int32_t* n_tiles = w.take<int32_t>(a.BH);
  a.zeros = w.take<float>(kZeros);
  if (splits > 1) {
    a.part_o = w.take<float>(splits * rows * d);
    a.part_ml = w.take<float2>(splits * rows);
  }
  if (!w.ok()) return SVGEAR_ERR_WORKSPACE;
  a.tile_a = tile_a;
  a.tile_row0 = tile_row0;
  a.n_tiles = n_tiles;
  plan_kernel<<<a.BH, kPlanThreads, (a.Cq + 2) * sizeof(int32_t), s>>>(a.q_offsets, a.k_offsets, a.row_ptr, a.col_idx,
                                                                      a.Cq, a.Ck, kF32Rows, a.max_tiles, tile_a,
                                                                      tile_row0, n_tiles, a.zeros);
  SVGEAR_LAUNCH_CHECK();
  // four waves fill a CU's LDS with their tiles at d = 128; lists of thousands of key clusters
  // leave room for two
  constexpr size_t kLds = 160 * 1024;
  if (d == 64) return launch<64, 4>(a, splits, s);
  if (f32_lds_bytes(d, 4, a.Ck) <= kLds) return launch<128, 4>(a, splits, s);
  return launch<128, 2>(a, splits, s);
}

}  // namespace svgear
