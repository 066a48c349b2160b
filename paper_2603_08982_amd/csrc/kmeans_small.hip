// k-means of small calls: every iteration of every head in one launch (definitions: kmeans.hip).
//
// A small call is bound by its chain of short dependent launches, three an iteration (assign, sort, means), not by
// its work: a head of 4,096 fp32 rows of 64 with 64 centroids took 19 us an iteration, of which the matrix cores need
// one. Here an iteration is two phases of tasks: tiles (rows against every centroid, the exact scores of
// assign_mfma_kernel) and groups (the means of a few clusters, summed slot by slot in the order of means_kernel: the
// results of the two paths are the same bits). A group finds its members in the labels itself, in row order, so nothing
// is sorted. What a phase costs is latency: about 1 us until the last task of a phase is seen, 2.5 for a tile,
// 5 for a group (labels 2, rows 2, the mean, its norm and tables 1).
//
// Order and progress: a workgroup claims the next task of its head, in order, when it is done with the one it has,
// and a task waits only for tasks before it, which resident workgroups hold. Whichever workgroups are resident, the
// first unfinished task is being worked on, so every wait ends, without all workgroups being there at once.
#include "kmeans.h"

#include <algorithm>
#include <type_traits>

namespace svgear {
namespace {

// Data that workgroups hand to each other inside a launch (labels, centroids and their tables) is stored and loaded
// past the XCDs' own L2 caches, as relaxed atomics of agent scope are (sc1). Fences of that scope would write back
// and invalidate a whole L2, the rows in it too: 26 us an iteration of the call above instead of 12.
__device__ __forceinline__ void store_shared(int32_t* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_shared(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int load_shared(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t shared_table(void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ float4 load_shared(__amdgpu_buffer_rsrc_t t, int byte) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(t, byte, 0, 16);  // sc1: agent scope
  return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ void store_shared(__amdgpu_buffer_rsrc_t t, int byte, float4 v) {
  const u32x4 u = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
  __builtin_amdgcn_raw_buffer_store_b128(u, t, byte, 0, 16);
}

// Eight waves a workgroup, one workgroup a CU (some 220 to 250 registers a lane: the row operands, two sets of
// centroid fragments, 16 rows in flight).
constexpr int kWaves = 8;
constexpr int kMaxParts = 8;      // most parts a cluster is summed in (means_parts)
constexpr int kLongCluster = 256;  // rows from which a cluster is summed by four waves wherever it lies
__host__ __device__ static inline int small_share(int n) { return ((n + kWaves - 1) / kWaves + 255) & ~255; }
// |c|^2 of eight centroids to a cache line
__device__ __forceinline__ int norm_at(int c) { return (c >> 3) * 32 + (c & 7); }

template <typename T, int D, int kShareWaves>
__global__ void __launch_bounds__(64 * kWaves, 2)
kmeans_small_kernel(SmallKmeans p) {
  using Share = std::integral_constant<int, kShareWaves>;
  constexpr int kUnits = kWaves / kShareWaves;  // clusters (or parts of one) at work at the same time
  constexpr int VEC = 16 / sizeof(T);   // elements per 16 bytes
  constexpr int LPR = D / VEC;          // lanes per row
  constexpr int SLOTS = 256 / LPR;      // member slots of a cluster's sum
  constexpr int RPL = 64 / LPR;         // rows a wave fetches at once, for slots RPL j + lane / LPR of its 4 / waves j
  constexpr int HALVES = D / 64;        // a 32-centroid block's operands come in pieces of 64 dims
  static_assert(SLOTS == 4 * RPL, "slots");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_task, s_cnt[kWaves][kWaves], s_live[kUnits], s_moved[kWaves];
  __shared__ float s_norm[kUnits];
  __shared__ float s_best[4][256];
  __shared__ int s_arg[4][256];
  __shared__ __attribute__((aligned(16))) float s_red[kUnits][SLOTS][D], s_mean[kUnits][D];
  __shared__ __attribute__((aligned(16))) float s_part[kMaxParts][D];
  const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = p.n, C = p.C;
  const int share = small_share(n);                    // labels a wave looks through
  uint16_t* near = reinterpret_cast<uint16_t*>(smem);  // [8][share]: row in the wave's share << 3 | cluster of the group
  uint16_t* members = near + kWaves * share;           // [n], the group's clusters one after the other
  int32_t* claim = p.state + (int64_t)bh * kSmallState;
  int32_t* tiles_done = claim + kSmallLine;
  int32_t* groups_done = tiles_done + kSmallLine * kSmallSpread;
  const T* xh = static_cast<const T*>(p.x) + head_base(p.st, bh, p.H);
  const T* x2h = p.x2 ? static_cast<const T*>(p.x2) + head_base(p.st, bh, p.H) : nullptr;
  // labels of iteration it: the two buffers in turn, the last iteration's in the caller's
  auto label_rows = [&](int it) { return ((p.iters - 1 - it) & 1 ? p.labels2 : p.labels) + (int64_t)bh * n; };
  const __amdgpu_buffer_rsrc_t tab = shared_table(p.cperm + (int64_t)bh * p.Cpad * D, (int64_t)p.Cpad * D * 4);
  float* cnb = p.norms + (int64_t)bh * p.Cpad * 4;
  const __amdgpu_buffer_rsrc_t norms = shared_table(cnb, (int64_t)p.Cpad * 16);
  const uint64_t below = (1ull << lane) - 1ull;

  auto wait_for = [&](const int32_t* counters, int target) {
    if (wave == 0) {
      for (;;) {
        int v = lane < kSmallSpread ? load_shared(counters + kSmallLine * lane) : 0;
#pragma unroll
        for (int o = 1; o < kSmallSpread; o <<= 1) v += __shfl_xor(v, o);
        if (__builtin_amdgcn_readfirstlane(v) >= target) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __syncthreads();
  };

  // ---- nearest centroid of the rows of one tile: row_waves x 32 rows, their centroid blocks dealt to col_waves
  auto assign_tile = [&](int it, int tile) {
    const int RW = p.row_waves, CW = p.col_waves, rw = wave / CW, cw = wave % CW;
    const bool on = rw < RW;
    const int pos = (tile * RW + rw) * 32 + li, row = pos < n ? pos : n - 1;
    float xb[D / 2];
    load_row_operands<D>(xh + (int64_t)row * p.st.n, lh, xb);
    if (it > 0) wait_for(groups_done, it * p.groups);
    const int nblk = on ? (C + 31) / 32 : 0;
    float best = INFINITY;
    int arg = 0;
    float4 f[8];
    auto fetch = [&](int blk, int half) {
#pragma unroll
      for (int q = 0; q < 8; ++q) f[q] = load_shared(tab, (blk * 32 * D + half * 2048 + q * 256 + lane * 4) * 4);
    };
    if (cw < nblk) fetch(cw, 0);
    for (int blk = cw; blk < nblk; blk += CW) {
      float nn[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 v = load_shared(norms, norm_at(32 * blk + 8 * g + 4 * lh) * 4);
        nn[4 * g] = v.x; nn[4 * g + 1] = v.y; nn[4 * g + 2] = v.z; nn[4 * g + 3] = v.w;
      }
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int half = 0; half < HALVES; ++half) {
        float4 now[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) now[q] = f[q];
        if (half + 1 < HALVES) fetch(blk, half + 1);
        else if (blk + CW < nblk) fetch(blk + CW, 0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int s = 32 * half + 4 * q;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(now[q].x, xb[s + 0], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(now[q].y, xb[s + 1], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(now[q].z, xb[s + 2], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(now[q].w, xb[s + 3], acc, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float score = __builtin_fmaf(-2.0f, acc[r], nn[r]);
        if (score < best) { best = score; arg = 32 * blk + 8 * (r >> 2) + 4 * lh + (r & 3); }
      }
    }
    const float ob = __shfl_xor(best, 32);
    const int oa = __shfl_xor(arg, 32);
    if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
    if (on && lh == 0) {
      s_best[cw][32 * rw + li] = best;
      s_arg[cw][32 * rw + li] = arg;
    }
    __syncthreads();
    const int at = tile * RW * 32 + tid;
    if (tid < 32 * RW && at < n) {
      float b = s_best[0][tid];
      int a = s_arg[0][tid];
      for (int w = 1; w < CW; ++w) {
        const float b2 = s_best[w][tid];
        const int a2 = s_arg[w][tid];
        if (b2 < b || (b2 == b && a2 < a)) { b = b2; a = a2; }
      }
      store_shared(label_rows(it) + at, a);
    }
  };

  // the rows members[from, to) added up by a team of WAVES waves: a lane's 16 bytes of its slots, to s_red[u]
  const int unit = wave / kShareWaves;
  auto sum_rows = [&](auto waves_tag, const T* src, int from, int to, int u) {
    constexpr int WAVES = decltype(waves_tag)::value, J = 4 / WAVES;
    const int j0 = (wave % WAVES) * J;
    float acc[J][VEC];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[j][e] = 0.f;
    const int slot0 = RPL * j0 + lane / LPR;
    const T* base = src + (lane % LPR) * VEC;
    auto add = [&](float (&a)[VEC], uint4 v) {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (sizeof(T) == 4) {
          a[i] += __uint_as_float(w[i]);
        } else {
          a[2 * i] += __uint_as_float(w[i] << 16);
          a[2 * i + 1] += __uint_as_float(w[i] & 0xffff0000u);
        }
      }
    };
    constexpr int B = 16;  // rows in flight a lane; those past the end count as rows of zeros
    for (int k = from + slot0; k < to; k += B / J * SLOTS) {
      uint4 v[B];
      int row[B];
      auto member = [&](int i) { return k + i / J * SLOTS + RPL * (i % J); };
#pragma unroll
      for (int i = 0; i < B; ++i) row[i] = members[min(member(i), to - 1)];
#pragma unroll
      for (int i = 0; i < B; ++i) v[i] = *reinterpret_cast<const uint4*>(base + (int64_t)row[i] * p.st.n);
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const bool in = member(i) < to;
        add(acc[i % J], make_uint4(in ? v[i].x : 0u, in ? v[i].y : 0u, in ? v[i].z : 0u, in ? v[i].w : 0u));
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int e = 0; e < VEC; e += 4)
        *reinterpret_cast<float4*>(&s_red[u][slot0 + RPL * j][(lane % LPR) * VEC + e]) =
            make_float4(acc[j][e], acc[j][e + 1], acc[j][e + 2], acc[j][e + 3]);
  };
  // dims lane and lane + 64 of unit u's sum: its slots in order
  auto unit_sum = [&](int u, float (&out)[HALVES]) {
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
      float s = s_red[u][0][lane + 64 * h];
#pragma unroll
      for (int k = 1; k < SLOTS; ++k) s += s_red[u][k][lane + 64 * h];
      out[h] = s;
    }
  };

  // The means of the group's clusters (row j: cluster c0 + j, in s_mean[j]) to dst and, with tables, to what the
  // next iteration reads, by the whole workgroup: neighbouring threads fill a line (stored cluster by cluster,
  // 16 bytes here and there, the stores took 1 to 8 us instead of 0.4).
  auto publish = [&](float* dst, int c0, int rows, bool tables) {
    const __amdgpu_buffer_rsrc_t out = shared_table(dst + (int64_t)bh * C * D, (int64_t)C * D * 4);
    for (int u = tid; u < rows * (D / 4); u += 64 * kWaves) {
      const int j = u / (D / 4), d = 4 * (u % (D / 4));
      if (s_live[j])  // (a cluster without members keeps its centroid)
        store_shared(out, ((c0 + j) * D + d) * 4, *reinterpret_cast<const float4*>(&s_mean[j][d]));
    }
    if (!tables) return;
    for (int u = tid; u < rows * (D / 4); u += 64 * kWaves) {
      const int j = u % rows, q = u / rows >> 1, h = u / rows & 1, c = c0 + j;
      const float4 v0 = *reinterpret_cast<const float4*>(&s_mean[j][8 * q]);
      const float4 v1 = *reinterpret_cast<const float4*>(&s_mean[j][8 * q + 4]);
      if (s_live[j])
        store_shared(tab, (((c >> 5) * (D / 8) + q) * 64 + (c & 31) + 32 * h) * 16,
                     h ? make_float4(v0.y, v0.w, v1.y, v1.w) : make_float4(v0.x, v0.z, v1.x, v1.z));
    }
    if (tid < rows && s_live[tid]) store_shared(cnb + norm_at(c0 + tid), s_norm[tid]);
  };
  // one cluster's mean by one wave into s_mean[u], and |mean|^2, one chain over the dims in order
  auto finish = [&](int u, const float (&sum)[HALVES], int cnt) {
    float* row = s_mean[u];
#pragma unroll
    for (int h = 0; h < HALVES; ++h) row[lane + 64 * h] = sum[h] / (float)cnt;
    __builtin_amdgcn_wave_barrier();
    float acc = 0.f;
#pragma unroll 8
    for (int k = 0; k < D / 4; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(row + 4 * k);
      acc = __builtin_fmaf(v.x, v.x, acc);
      acc = __builtin_fmaf(v.y, v.y, acc);
      acc = __builtin_fmaf(v.z, v.z, acc);
      acc = __builtin_fmaf(v.w, v.w, acc);
    }
    if (lane == 0) s_norm[u] = acc;
  };

  // ---- means of one group of clusters: one to every kShareWaves waves, or one in all, whose parts they share
  auto update = [&](int it, int group) {
    const int P = p.parts, G = P == 1 ? kUnits : 1, c0 = group * G;
    wait_for(tiles_done, (it + 1) * p.tiles);
    // the rows of the group's clusters among this wave's share of all rows, in order
    const int lo = wave * share, hi = min(lo + share, n);
    uint16_t* mine = near + lo;
    int kept = 0;
    // a bit per cluster of the group that rows came to or left in this iteration: the others keep their means, which
    // would be the same sums again (9,600 bf16 rows of 128, 200 centroids, one with nine rows in ten, 10 iterations:
    // 706 -> 326 us). From the third iteration on: in the second nearly every cluster has moved, and to look costs 1 us.
    const bool compare = it >= 2;
    uint32_t moved = compare ? 0u : ~0u;
    const __amdgpu_buffer_rsrc_t labels = shared_table(label_rows(it), (int64_t)n * 4);
    const __amdgpu_buffer_rsrc_t labels_before = shared_table(label_rows(compare ? it - 1 : it), (int64_t)n * 4);
    constexpr int U = 4;
    for (int i0 = lo; i0 < hi; i0 += 256 * U) {
      u32x4 l[U];  // (rows past the end read as label 0)
#pragma unroll
      for (int u = 0; u < U; ++u) l[u] = __builtin_amdgcn_raw_buffer_load_b128(labels, (i0 + 256 * u + 4 * lane) * 4, 0, 16);
      if (compare) {
        u32x4 b[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          b[u] = __builtin_amdgcn_raw_buffer_load_b128(labels_before, (i0 + 256 * u + 4 * lane) * 4, 0, 16);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e)  // (a label of another group sets bit 31; equal ones cancel. Without comparisons,
                                       // whose lane masks spilled scalar registers: 12 x 2,400 fp32 rows of 64 in 60
                                       // clusters, 4 iterations 68.0 -> 66.1 us)
            moved |= 1u << min(l[u][e] - (unsigned)c0, 31u) ^ 1u << min(b[u][e] - (unsigned)c0, 31u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + 256 * u + 4 * lane;
        uint64_t votes[4];
        int to = kept;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          votes[e] = __ballot(l[u][e] - (unsigned)c0 < (unsigned)G && i + e < hi);
          to += __popcll(votes[e] & below);
          kept += __popcll(votes[e]);
        }
        if (votes[0] | votes[1] | votes[2] | votes[3]) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (votes[e] >> lane & 1) mine[to++] = (uint16_t)(((i + e - lo) << 3) | (l[u][e] - c0));
        }
      }
    }
    if (compare) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) moved |= __shfl_xor(moved, o);
      if (lane == 0) s_moved[wave] = (int)moved;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < kWaves) s_cnt[wave][lane] = 0;
    for (int e = lane; e < kept; e += 64) atomicAdd(&s_cnt[wave][mine[e] & 7], 1);
    __syncthreads();
    const bool last = it + 1 == p.iters;
    if (compare) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) moved |= (uint32_t)s_moved[w];
      moved &= (1u << kWaves) - 1u;
    }
    if (moved == 0 && !last) return;
    // lane 8 k + w: where wave w's members of cluster k begin
    const int here = s_cnt[lane & 7][lane >> 3];
    int upto = here;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(upto, o);
      if (lane >= o) upto += t;
    }
    int next = upto - here;
    const int own = P == 1 ? unit : 0, begin = __shfl(next, 8 * own), count = __shfl(upto, 8 * own + 7) - begin;
    const bool lead = wave % kShareWaves == 0;
    int longest = upto - __shfl_up(upto, 8);  // (lanes 8 k + 7 hold a cluster's rows)
    if (lane < 8) longest = upto;
    longest = lane % 8 == 7 ? longest : 0;
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) longest = max(longest, __shfl_xor(longest, o));
    longest = __shfl(longest, 7);
    for (int e = 0; e < kept; e += 64) {
      const int v = e + lane < kept ? mine[e + lane] : -1, c = v < 0 ? -1 : v & 7;
      int to = __shfl(next, 8 * (c & 7) + wave);
#pragma unroll
      for (int k = 0; k < kWaves; ++k) {
        const uint64_t votes = __ballot(c == k);
        if (c == k) to += __popcll(votes & below);
        if (lane >> 3 == k) next += __popcll(votes);
      }
      if (c >= 0) members[to] = (uint16_t)(lo + (v >> 3));
    }
    __syncthreads();
    if (last && lane == 0 && lead && c0 + unit < C && unit < G) p.counts[(int64_t)bh * C + c0 + unit] = count;
    const int len = (((count + P - 1) / P) + SLOTS - 1) / SLOTS * SLOTS;
    for (int t = 0; t < (last && x2h ? 2 : 1); ++t) {
      const T* src = t ? x2h : xh;
      const bool live = count > 0 && (t == 1 || (moved >> own & 1u));
      if (lane == 0 && lead) s_live[unit] = live;
      float s[HALVES];
      if (P == 1) {
        // (a long cluster would keep its one or two waves busy for all the others: four take it)
        const bool alone = kShareWaves == 4 || count <= kLongCluster;
        if (live && alone) sum_rows(Share{}, src, begin, begin + count, unit);
        __syncthreads();
        if (lead && live && alone) {
          unit_sum(unit, s);
          finish(unit, s, count);
        }
        if (kShareWaves < 4 && longest > kLongCluster) {
          for (int k = 0; k < kUnits; k += 2) {
            const int c = k + wave / 4, from = __shfl(upto - here, 8 * c), n_c = __shfl(upto, 8 * c + 7) - from;
            const bool on = n_c > kLongCluster && (t == 1 || (moved >> c & 1u));
            if (on) sum_rows(std::integral_constant<int, 4>{}, src, from, from + n_c, c);
            __syncthreads();
            if (on && wave % 4 == 0) {
              unit_sum(c, s);
              finish(c, s, n_c);
            }
          }
        }
      } else if constexpr (kShareWaves == 4) {
        for (int p0 = 0; live && p0 < P; p0 += kUnits) {  // (P parts of the members; an empty one adds a zero)
          const int from = min((p0 + unit) * len, count), to = min(from + len, count);
          sum_rows(Share{}, src, from, to, unit);
          __syncthreads();
          if (lead && p0 + unit < P) {
            unit_sum(unit, s);
#pragma unroll
            for (int h = 0; h < HALVES; ++h) s_part[p0 + unit][lane + 64 * h] = s[h];
          }
          __syncthreads();
        }
        if (wave == 0 && live) {
#pragma unroll
          for (int h = 0; h < HALVES; ++h) {
            s[h] = s_part[0][lane + 64 * h];
            for (int part = 1; part < P; ++part) s[h] += s_part[part][lane + 64 * h];
          }
          finish(0, s, count);
        }
      }
      __syncthreads();
      publish(t ? p.cent2 : p.cent, c0, G, !last);
      __syncthreads();
    }
  };

  const int per_iteration = p.tiles + p.groups, all = p.iters * per_iteration;
  if (tid == 0) s_task = __hip_atomic_fetch_add(claim, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  int task = __builtin_amdgcn_readfirstlane(s_task);
  while (task < all) {
    const int it = task / per_iteration, r = task - it * per_iteration;
    const bool tile = r < p.tiles;
    if (tile) assign_tile(it, r);
    else update(it, r - p.tiles);
    int next = 0;  // (claimed while the task's stores are on their way)
    if (tid == 0) next = __hip_atomic_fetch_add(claim, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    SVGEAR_WAIT_VMCNT(0);
    __syncthreads();
    if (tid == 0) {
      int32_t* counters = tile ? tiles_done : groups_done;
      __hip_atomic_fetch_add(counters + kSmallLine * (r % kSmallSpread), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_task = next;
    }
    __syncthreads();
    task = __builtin_amdgcn_readfirstlane(s_task);
  }
}

template <typename T, int D, int SHARE>
int launch_share(const SmallKmeans& a, hipStream_t s) {
  const size_t lds = (kWaves * (size_t)small_share(a.n) + align_up(a.n, 8)) * 2;
  auto kern = kmeans_small_kernel<T, D, SHARE>;
  SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
  // at most a workgroup a CU: with more, the first heads' workgroups fill the chip and the last heads run after them
  // (5 x 600 rows, 100 centroids: 110 us with 512, 68 with 256)
  kern<<<dim3(std::min(a.tiles + a.groups, 256 / a.BH), a.BH), 64 * kWaves, lds, s>>>(a);
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}
template <typename T, int D>
int launch_shape(const SmallKmeans& a, int share, hipStream_t s) {
  return share == 1 ? launch_share<T, D, 1>(a, s) : share == 2 ? launch_share<T, D, 2>(a, s) : launch_share<T, D, 4>(a, s);
}

// The shape of a call's work (waves a cluster as the result).
int set_shape(SmallKmeans& a) {
  // four waves, one a SIMD, share a tile's rows and centroid blocks; all eight where the tiles outnumber the CUs
  const int nblk = (a.C + 31) / 32;
  a.col_waves = nblk >= 4 ? 4 : nblk >= 2 ? 2 : 1;
  a.row_waves = 4 / a.col_waves;
  if (a.BH * ceil_div(a.n, 32 * a.row_waves) > 256) a.row_waves *= 2;
  a.tiles = (int)ceil_div(a.n, 32 * a.row_waves);
  a.parts = means_parts(a.n, a.C);
  // waves a cluster: as many as leave the groups within one round (4,096 rows, 64 centroids, 10 iterations: 151 us
  // with one, 128 with two, 124 with four; 12 x 1,200 rows, 100 centroids: 317, 309, 408)
  int share = 4;
  if (a.parts == 1 && a.BH * ceil_div(a.C, 2) > 256) share = a.BH * ceil_div(a.C, 4) > 256 ? 1 : 2;
  a.groups = a.parts == 1 ? (int)ceil_div(a.C, kWaves / share) : a.C;
  return share;
}

}  // namespace

// Two lines, since which way is faster depends on the rows. Measured against the launches of their own, which give every
// part of a cluster a workgroup but wait for the longest one and assign undecided rows again; 2, 4 and 10 iterations.
//  * One round: groups within a round of the CUs, tiles within one or (four waves a cluster, one block of centroids a
//    wave) two, no cluster many workgroups' work. Faster whatever the rows: over 1 to 300 heads of 130 to 16,384 rows in
//    1 to 2,000 clusters, spread evenly over 128 components or nine in ten in one cluster, 1.46 times on average, 0.93 to 1
//    in the least favourable variants (two iterations of a few hundred rows 36 -> 38 us; bf16, 10 iterations, a dominant
//    cluster: 2 x 4,800, 300 centroids 282 -> 302, 16 x 4,800, 10 centroids 270 -> 292).
//  * Some rounds more: faster for rows as a video model has them (32 to 256 components that follow the position, a fifth of
//    the rows strayed, centroids started at rows, so that some clusters hold several components).
//    Of 149 calls and layers of such rows between the lines, single calls, us step by step and here: bf16 5 x 13,230, 31
//    centroids 153 -> 73; 24 x 3,528, 24 151 -> 76; 40 x 2,592, 31 420 -> 212; 8 x 2,376, 226 82 -> 66; fp32 2 x 11,200, 31
//    302 -> 174; 12 x 8,316, 31 610 -> 392; layers of 1 x 13,300, 20 / 28 622 -> 316, 5 x 7,000, 13 / 33 780 -> 598. With the
//    wider line none of them is more than 1.2 % slower than by sizes alone (200,000 rows, 64 centroids), 15 are over 5 % faster.
//    Rows spread evenly over 128 components, 2 and 10 iterations, step by step and here: bf16 24 x 4,800, 48 centroids
//    158 -> 128 and 617 -> 521; 5 x 4,800, 200 97 -> 84 and 418 -> 341; fp32 12 x 8,316, 31 136 -> 98 and 641 -> 382; slower with
//    2 and 4 iterations of one head's long clusters, 1 x 16,384 in 16 67 -> 73 (fp32 78 -> 90), or of many short ones,
//    bf16 12 x 2,400, 100 61 -> 67; 40 x 300, 64 49 -> 53 (10: 214 -> 161).
//    Past it: 40 x 4,180 bf16 rows, 43 centroids (1,320 tiles) 278 -> 292; fp32 layers, whose tiles take longer, 40 x
//    1,650, 56 key clusters 947 -> 1,189, 12 x 12,720, 11 / 34 2,166 -> 2,270; more than 64 centroids of many heads, 24 x
//    1,680 to 3,400 rows 1.1 times as long.
bool kmeans_small_takes(int64_t BH, int64_t nv, int C, int iters, bool bf16) {
  if (BH > 64 || nv > kSmallRows || iters > kSmallIterations) return false;
  SmallKmeans a{};
  a.BH = (int)BH;
  a.n = (int)nv;
  a.C = C;
  const int share = set_shape(a);
  const int64_t tiles = BH * a.tiles, groups = BH * a.groups;
  const bool long_clusters = a.parts > 2 && (a.parts > 4 || (BH < 8 && nv > 5000));
  if (groups <= 256 && (tiles <= 256 || (tiles <= 512 && share == 4 && C <= 128)) && !long_clusters) return true;
  if (BH * nv > 200000 || groups > (bf16 ? 576 : 400) || tiles > (bf16 ? 1024 : 448)) return false;
  return C <= 64 || (BH <= 12 && BH * ceil_div(nv, 64) <= 640 && BH * ceil_div(C, 8) <= 256);
}

int launch_kmeans_small(SmallKmeans a, int d, bool bf16, hipStream_t s) {
  const int share = set_shape(a);
  if (bf16) return d == 64 ? launch_shape<bf16_t, 64>(a, share, s) : launch_shape<bf16_t, 128>(a, share, s);
  return d == 64 ? launch_shape<float, 64>(a, share, s) : launch_shape<float, 128>(a, share, s);
}

}  // namespace svgear
