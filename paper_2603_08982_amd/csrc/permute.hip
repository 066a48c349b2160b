// Cluster permutation: stable counting sort of token indices by cluster label, row
// gather into cluster-contiguous order, and the inverse row scatter.
// Paper: Motivation, "Structured Redundancy in Attention Computation" (tokens of a cluster
// are laid out contiguously so the attention map becomes a grid of blocks).
//
// The sort is integer-only and deterministic: per-chunk histograms (LDS integer atomics),
// an exclusive scan over (cluster, chunk), then a stable in-chunk ranking without atomics.
#include "common.h"

#include <mutex>

namespace svgear {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxLabels = 8192;  // most labels the entry points accept
constexpr int kManyLabels = 3700;  // labels from which scatter_kernel keeps neither positions nor an order in LDS

__device__ __forceinline__ int token_label(const int32_t* labels, int64_t i, int64_t nv, int C) {
  if (i >= nv) return C;  // tail pseudo-cluster
  int l = labels[i];
  return l < 0 ? 0 : (l >= C ? C - 1 : l);  // out-of-range labels are clamped
}

__global__ void __launch_bounds__(kThreads)
hist_kernel(const int32_t* __restrict__ labels, int64_t N, int64_t nv, int C, int nchunks,
            int32_t* __restrict__ chunk_hist) {
  extern __shared__ int32_t h[];
  const int bh = blockIdx.y, chunk = blockIdx.x;
  for (int c = threadIdx.x; c <= C; c += kThreads) h[c] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)chunk * kSortChunk;
  const int64_t hi = min(N, lo + kSortChunk);
  const int32_t* lab = labels + (int64_t)bh * nv;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) atomicAdd(&h[token_label(lab, i, nv, C)], 1);
  __syncthreads();
  int32_t* out = chunk_hist + ((int64_t)bh * nchunks + chunk) * (C + 1);
  for (int c = threadIdx.x; c <= C; c += kThreads) out[c] = h[c];
}

// Tiles of cluster c, n positions from `off` on (see sort_labels in common.h); the next cluster's
// tiles start at index `next`.
__device__ __forceinline__ void write_tiles(int4* tiles, int c, int off, int n, int next, int tile_len) {
  const int start = off / tile_len + c, nt = (n + tile_len - 1) / tile_len, end = off + n;
  for (int j = 0; j < nt; ++j) {
    const int p0 = off + j * tile_len;
    tiles[start + j] = make_int4(c, p0, p0 + tile_len < end ? p0 + tile_len : end, 0);
  }
  for (int j = start + nt; j < next; ++j) tiles[j] = make_int4(-1, 0, 0, 0);
}

// Turns per-chunk histograms into per-chunk start positions and writes the offsets. One workgroup a head, as wide as
// they come: a thread walks the chunks of a label (40 heads, 37 chunks, 1,000 labels: 22 us with 256 threads).
constexpr int kScanThreads = 1024;
__global__ void __launch_bounds__(kScanThreads)
scan_kernel(int32_t* __restrict__ chunk_hist, int64_t N, int C, int nchunks,
            int32_t* __restrict__ offsets, int4* __restrict__ tiles, int tile_cap, int tile_len) {
  extern __shared__ int32_t tot[];  // C+1 totals, then C+1 exclusive offsets
  int32_t* offs = tot + (C + 1);
  const int bh = blockIdx.x;
  int32_t* hist = chunk_hist + (int64_t)bh * nchunks * (C + 1);
  // label totals: loads only, eight in flight per thread
  for (int c = threadIdx.x; c <= C; c += kScanThreads) {
    int32_t run = 0;
    int k = 0;
    for (; k + 8 <= nchunks; k += 8) {
      int32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = hist[(int64_t)(k + u) * (C + 1) + c];
#pragma unroll
      for (int u = 0; u < 8; ++u) run += v[u];
    }
    for (; k < nchunks; ++k) run += hist[(int64_t)k * (C + 1) + c];
    tot[c] = run;
  }
  __syncthreads();
  // exclusive scan of the C+1 totals: each thread takes a contiguous run of labels
  {
    const int per = (C + 1 + kScanThreads - 1) / kScanThreads;
    const int lo = threadIdx.x * per, hi = lo + per < C + 1 ? lo + per : C + 1;
    int32_t sum = 0;
    for (int c = lo; c < hi; ++c) sum += tot[c];
    __shared__ int32_t part[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t run = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t t = __shfl_up(run, o);
      if (lane >= o) run += t;
    }
    if (lane == 63) part[wave] = run;
    __syncthreads();
    run -= sum;
    for (int w = 0; w < wave; ++w) run += part[w];
    for (int c = lo; c < hi; ++c) {
      offs[c] = run;
      run += tot[c];
    }
  }
  __syncthreads();
  // start of every (chunk, label) segment: offset of the label plus the label's count in the
  // earlier chunks; eight chunks per round (loads first, then the stores)
  int32_t* o = offsets + (int64_t)bh * (C + 2);
  for (int c = threadIdx.x; c <= C; c += kScanThreads) {
    int32_t run = offs[c];
    o[c] = run;
    int k = 0;
    for (; k + 8 <= nchunks; k += 8) {
      int32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = hist[(int64_t)(k + u) * (C + 1) + c];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        hist[(int64_t)(k + u) * (C + 1) + c] = run;
        run += v[u];
      }
    }
    for (; k < nchunks; ++k) {
      const int32_t v = hist[(int64_t)k * (C + 1) + c];
      hist[(int64_t)k * (C + 1) + c] = run;
      run += v;
    }
  }
  if (threadIdx.x == 0) o[C + 1] = (int32_t)N;
  if (tiles) {  // tiles of the clusters (see sort_labels in common.h)
    int4* ta = tiles + (int64_t)bh * tile_cap;
    for (int c = threadIdx.x; c < C; c += kScanThreads) {
      write_tiles(ta, c, offs[c], tot[c], c + 1 < C ? offs[c + 1] / tile_len + c + 1 : tile_cap, tile_len);
    }
  }
}

// Stable placement without atomics: each of the four waves takes a contiguous quarter of the chunk, 64 tokens at a
// time. The rank of a token among the lanes with the same label comes from ballots over the label bits, the last lane
// of a label adds their number to the wave's own counter of it (16 bits: a quarter has 512 tokens), and once the
// counters of all four waves are there every token knows its position: equal labels keep ascending token order.
// What bounds it is latency and, with many heads, stores: all labels are fetched at once, the ballots of all steps run
// side by side, and the chunk's tokens are put in order in LDS first, so that a store writes runs of positions. 40 heads
// of 75,600 random labels of 1,000 / 100: 38 / 16 us with waves that claimed their positions one after the other and
// stored from there, 25 / 19 stored from the tokens' own order, 23 / 15 now; one head 8.5 -> 6.7.
// MANY labels leave a chunk no runs to store, and the table of positions and the order leave two workgroups a CU from
// 3,700 labels on, one from 6,000: there tokens are stored from their own order, each by its label's first position
// from global memory. The whole sort of 100 heads of 75,600, us (positions claimed wave by wave, in order, this): 3,000
// labels 186, 136, 145; 4,000 212, 245, 151; 8,192 329, 419, 207; 8 heads of 20,000: 40, 29, 24; 49, 36, 26; 77, 48, 37.
template <bool MANY>
__global__ void __launch_bounds__(kThreads)
scatter_kernel(const int32_t* __restrict__ labels, int64_t N, int64_t nv, int C, int nchunks,
               const int32_t* __restrict__ chunk_hist, int32_t* __restrict__ perm) {
  constexpr int WAVES = kThreads / 64, ITERS = kSortChunk / kThreads;
  extern __shared__ int32_t base[];  // C + 1 first positions of the chunk's labels (MANY: only what follows)
  uint16_t* cnt = reinterpret_cast<uint16_t*>(base + (MANY ? 0 : C + 1));  // [wave][C + 1]: counts, then of the waves before
  const int bh = blockIdx.y, chunk = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t* hist = chunk_hist + ((int64_t)bh * nchunks + chunk) * (C + 1);
  const int32_t* lab = labels + (int64_t)bh * nv;
  int32_t* out = perm + (int64_t)bh * N;
  const int64_t first = (int64_t)chunk * kSortChunk + wave * (64 * ITERS) + lane;
  const int nbits = 32 - __clz(C + 1);
  const uint64_t below = (1ull << lane) - 1ull;
  int my[ITERS], rank[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int64_t i = first + 64 * it;
    my[it] = i < N ? token_label(lab, i, nv, C) : C + 1;
  }
  int at[ITERS];  // MANY: first position of the token's label
#pragma unroll
  for (int it = 0; it < ITERS; ++it) at[it] = MANY && my[it] <= C ? hist[my[it]] : 0;
  for (int c = threadIdx.x; c <= C; c += kThreads) {
    if constexpr (!MANY) base[c] = hist[c];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) cnt[w * (C + 1) + c] = 0;
  }
  __syncthreads();
  uint16_t* mine = cnt + wave * (C + 1);
  uint64_t same[ITERS];  // lanes with the label of this one (all steps side by side: a ballot waits for a comparison)
#pragma unroll
  for (int it = 0; it < ITERS; ++it) same[it] = ~0ull;
  for (int bit = 0; bit < nbits; ++bit) {
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int on = __builtin_amdgcn_sbfe(my[it], bit, 1);  // 0 or -1
      same[it] &= ~(__ballot(on != 0) ^ (uint64_t)(int64_t)on);
    }
  }
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int before = my[it] <= C ? mine[my[it]] : 0, total = __popcll(same[it]);
    rank[it] = __popcll(same[it] & below);
    if (my[it] <= C && rank[it] == total - 1) mine[my[it]] = (uint16_t)(before + total);  // after every lane's read
    rank[it] += before;
    __builtin_amdgcn_wave_barrier();  // the next step reads what other lanes wrote
  }
  __syncthreads();
  if constexpr (MANY) {
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      if (my[it] > C) continue;
      for (int w = 0; w < wave; ++w) rank[it] += cnt[w * (C + 1) + my[it]];
      out[at[it] + rank[it]] = (int32_t)(first + 64 * it);
    }
    return;
  }
  // first place of every (label, wave) in the chunk's order: each thread takes a contiguous run of labels
  __shared__ int wave_sum[WAVES];
  const int per = (C + kThreads) / kThreads, c_lo = threadIdx.x * per, c_hi = min(C + 1, c_lo + per);
  int sum = 0;
  for (int c = c_lo; c < c_hi; ++c)
#pragma unroll
    for (int w = 0; w < WAVES; ++w) sum += cnt[w * (C + 1) + c];
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wave; ++w) run += wave_sum[w];
  for (int c = c_lo; c < c_hi; ++c) {
    base[c] -= run;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const int v = cnt[w * (C + 1) + c];
      cnt[w * (C + 1) + c] = (uint16_t)run;
      run += v;
    }
  }
  __syncthreads();
  __shared__ uint32_t order[kSortChunk];  // token of the chunk | label << 16
#pragma unroll
  for (int it = 0; it < ITERS; ++it)
    if (my[it] <= C) order[mine[my[it]] + rank[it]] = (uint32_t)(wave * (64 * ITERS) + 64 * it + lane) | (uint32_t)my[it] << 16;
  __syncthreads();
  const int64_t lo = (int64_t)chunk * kSortChunk;
  const int n = (int)min((int64_t)kSortChunk, N - lo);
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int p = it * kThreads + threadIdx.x;
    if (p < n) out[base[order[p] >> 16] + p] = (int32_t)lo + (int32_t)(order[p] & 0xffffu);
  }
}

// The whole sort of a head by one workgroup, for heads of up to 8,192 tokens: each of the 16 waves
// takes a contiguous run of tokens, counts its labels in a histogram of its own (the lanes with the
// same label found by ballots, one of them adds: no atomics), the columns of the histograms are
// scanned over waves and labels, and the tokens are placed in wave order, which is token order.
// A short sort is bound by the number of launches and their latencies, not by its few hundred
// kilobytes: at 667 tokens 4.2 us instead of 10 in three launches, at 4,096 8.1 instead of 15 (the
// whole layers of those sizes, 10 and 22 sorts, 0.58 -> 0.47 and 0.75 -> 0.63 ms). Longer heads keep
// the three kernels above, whose chunks spread over the chip: 18,135 tokens took 18 us with them and
// 33 in one workgroup, about 2 us more per 1,024 tokens.
constexpr int kSmallWaves = 16, kSmallStep = 64 * kSmallWaves, kSmallIters = 8, kSmallLabels = 2048;

template <int ITERS>
__global__ void __launch_bounds__(64 * kSmallWaves)
sort_small_kernel(const int32_t* __restrict__ labels, int N, int nv, int C, int32_t* __restrict__ perm,
                  int32_t* __restrict__ offsets, int4* __restrict__ tiles, int tile_cap, int tile_len) {
  extern __shared__ int32_t cnt[];  // [wave][C + 1]
  __shared__ int32_t wave_sum[kSmallWaves];
  const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_it = (N + kSmallStep - 1) / kSmallStep;
  const int first = wave * 64 * n_it + lane;
  const int32_t* lab = labels + (int64_t)bh * nv;
  int32_t* out = perm + (int64_t)bh * N;
  int32_t* mine = cnt + wave * (C + 1);
  const int nbits = 32 - __clz(C + 1);
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t tok[ITERS];  // label, then | rank among the wave's equal labels << 14 | (their number - 1) << 20
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int i = first + 64 * it;
    tok[it] = it < n_it && i < N ? (uint32_t)token_label(lab, i, nv, C) : (uint32_t)(C + 1);
  }
  for (int c = tid; c < kSmallWaves * (C + 1); c += kSmallStep) cnt[c] = 0;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    if (it < n_it) {
      const int my = (int)tok[it];
      uint64_t same = ~0ull;
      for (int bit = 0; bit < nbits; ++bit) {
        const uint64_t vote = __ballot((my >> bit) & 1);
        same &= ((my >> bit) & 1) ? vote : ~vote;
      }
      const int rank = __popcll(same & below), total = __popcll(same);
      tok[it] |= ((uint32_t)rank << 14) | ((uint32_t)(total - 1) << 20);
      if (my <= C && rank == total - 1) mine[my] += total;
    }
  }
  __syncthreads();
  int carry = 0;
  for (int c0 = 0; c0 <= C; c0 += kSmallStep) {  // start of every (label, wave) segment
    const int c = c0 + tid;
    int tot = 0;
    if (c <= C)
      for (int w = 0; w < kSmallWaves; ++w) tot += cnt[w * (C + 1) + c];
    int incl = tot;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int start = carry + incl - tot, all = 0;
    for (int w = 0; w < kSmallWaves; ++w) {
      if (w < wave) start += wave_sum[w];
      all += wave_sum[w];
    }
    carry += all;
    if (c <= C) {
      offsets[(int64_t)bh * (C + 2) + c] = start;
      int run = start;
      for (int w = 0; w < kSmallWaves; ++w) {
        const int v = cnt[w * (C + 1) + c];
        cnt[w * (C + 1) + c] = run;
        run += v;
      }
      if (tiles && c < C)
        write_tiles(tiles + (int64_t)bh * tile_cap, c, start, tot, c + 1 < C ? (start + tot) / tile_len + c + 1 : tile_cap,
                    tile_len);
    }
    __syncthreads();
  }
  if (tid == 0) offsets[(int64_t)bh * (C + 2) + C + 1] = N;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int my = (int)(tok[it] & 0x3fffu);
    if (it < n_it && my <= C) {
      const int i = first + 64 * it, rank = (int)((tok[it] >> 14) & 63u), total = (int)((tok[it] >> 20) & 63u) + 1;
      const int b = mine[my];
      out[b + rank] = i;
      if (rank == total - 1) mine[my] = b + total;  // issued after every lane's read
    }
  }
}

// dst[k][bh][p][:] = src[k][b,h,perm[p],:] in 16-byte units, tensor k = blockIdx.z.
struct GatherArgs {
  const uint4* src[4];
  uint4* dst[4];
  Strides st[4];  // in 16-byte units
};
__global__ void __launch_bounds__(kThreads)
gather_rows_kernel(GatherArgs g, int H, const int32_t* __restrict__ perm, int64_t N, int row_units) {
  const int bh = blockIdx.y, k = blockIdx.z;
  const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (u >= N * row_units) return;
  const int64_t p = u / row_units;
  const int v = (int)(u % row_units);
  const int64_t row = perm[(int64_t)bh * N + p];
  g.dst[k][((int64_t)bh * N + p) * row_units + v] = g.src[k][head_base(g.st[k], bh, H) + row * g.st[k].n + v];
}

// dst[b,h,perm[p],:] = src[bh][p][:]
__global__ void __launch_bounds__(kThreads)
scatter_rows_kernel(const uint4* __restrict__ src, const int32_t* __restrict__ perm, int64_t N,
                    int row_units, uint4* __restrict__ dst, Strides st_units, int H) {
  const int bh = blockIdx.y;
  const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (u >= N * row_units) return;
  const int64_t p = u / row_units;
  const int v = (int)(u % row_units);
  const int64_t row = perm[(int64_t)bh * N + p];
  dst[head_base(st_units, bh, H) + row * st_units.n + v] = src[((int64_t)bh * N + p) * row_units + v];
}

bool strides_ok(const int64_t st[3], size_t es, const void* p) {
  if (!st) return false;
  for (int i = 0; i < 3; ++i)
    if (st[i] < 0 || (st[i] * (int64_t)es) % 16 != 0) return false;
  return (reinterpret_cast<uintptr_t>(p) % 16) == 0;
}

}  // namespace

int sort_labels(const int32_t* labels, int BH, int64_t N, int64_t n_tail, int C, int32_t* perm,
                int32_t* offsets, int32_t* chunk_hist, hipStream_t s, int4* tiles, int tile_cap, int tile_len) {
  const int nchunks = (int)sort_chunks(N);
  const int64_t nv = N - n_tail;
  if (tiles && (tile_len < 1 || tile_cap < (int)(N / tile_len) + C + 1)) return SVGEAR_ERR_INVALID;
  if (N <= kSmallIters * kSmallStep && C <= kSmallLabels) {
    const size_t lds = (size_t)kSmallWaves * (C + 1) * sizeof(int32_t);
    auto kern = N <= kSmallStep ? sort_small_kernel<1>
                : N <= 4 * kSmallStep ? sort_small_kernel<4> : sort_small_kernel<kSmallIters>;
    SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds));
    kern<<<BH, kSmallStep, lds, s>>>(labels, (int)N, (int)nv, C, perm, offsets, tiles, tile_cap, tile_len);
    SVGEAR_LAUNCH_CHECK();
    return SVGEAR_OK;
  }
  dim3 grid(nchunks, BH);
  hist_kernel<<<grid, kThreads, (C + 1) * sizeof(int32_t), s>>>(labels, N, nv, C, nchunks, chunk_hist);
  SVGEAR_LAUNCH_CHECK();
  // two tables of C+1 counters: a few bytes over the default 64 KB at the largest C
  SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(scan_kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)(2 * (C + 1) * sizeof(int32_t))));
  scan_kernel<<<BH, kScanThreads, 2 * (C + 1) * sizeof(int32_t), s>>>(chunk_hist, N, C, nchunks, offsets, tiles, tile_cap,
                                                                  tile_len);
  SVGEAR_LAUNCH_CHECK();
  // four counters of 16 bits a label and, below kManyLabels, C + 1 positions. (The limit is raised in every call and to
  // what the most labels take: static LDS counts too, and a call of another thread never finds it below its own need.)
  const bool many = C >= kManyLabels;
  const auto scatter_lds = [=](int labels) {
    return (size_t)(labels + 1) * ((many ? 0 : sizeof(int32_t)) + kThreads / 64 * sizeof(uint16_t));
  };
  auto scatter = many ? scatter_kernel<true> : scatter_kernel<false>;
  SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(scatter), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)scatter_lds(many ? kMaxLabels : kManyLabels)));
  scatter<<<grid, kThreads, scatter_lds(C), s>>>(labels, N, nv, C, nchunks, chunk_hist, perm);
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}

}  // namespace svgear

using namespace svgear;

extern "C" size_t svgear_permute_workspace(int B, int H, int64_t N, int C) {
  if (B <= 0 || H <= 0 || N <= 0 || C <= 0) return 0;
  return align_up((size_t)B * H * sort_chunks(N) * (C + 1) * sizeof(int32_t), 256);
}

namespace svgear {
namespace {

// dst[k][bh][p][:] = src[k][b,h,perm[p],:] for every tensor k, as if one were moved after the other
int gather_tensors(const int32_t* perm, int BH, int H, int64_t N, int n_tensors, const void* const* src,
                   const int64_t (*sstride)[3], void* const* dst, svgear_dtype dt, int d, hipStream_t s) {
  const int row_units = (int)(d * esize(dt) / 16);
  const int upe = (int)(16 / esize(dt));  // elements per 16-byte unit
  GatherArgs g{};
  for (int k = 0; k < n_tensors; ++k) {
    g.src[k] = static_cast<const uint4*>(src[k]);
    g.dst[k] = static_cast<uint4*>(dst[k]);
    g.st[k] = Strides{sstride[k][0] / upe, sstride[k][1] / upe, sstride[k][2] / upe};
  }
  // One launch moves them all (two tensors of 600 rows a head 33 -> 25 us with the sort), unless the
  // destination of one meets the rows of another: a caller may send V's rows to where K's were.
  struct Span { uintptr_t lo, hi; };
  Span from[4], to[4];
  for (int k = 0; k < n_tensors; ++k) {
    from[k].lo = reinterpret_cast<uintptr_t>(src[k]);
    from[k].hi = from[k].lo + 16 * (uintptr_t)((BH / H - 1) * g.st[k].b + (H - 1) * g.st[k].h + (N - 1) * g.st[k].n + row_units);
    to[k].lo = reinterpret_cast<uintptr_t>(dst[k]);
    to[k].hi = to[k].lo + 16 * (uintptr_t)BH * N * row_units;
  }
  auto meet = [](const Span& x, const Span& y) { return x.lo < y.hi && y.lo < x.hi; };
  bool apart = true;
  for (int j = 0; j < n_tensors; ++j)
    for (int k = 0; k < n_tensors; ++k)
      if (j != k && (meet(to[j], from[k]) || meet(to[j], to[k]))) apart = false;
  const int step = apart ? n_tensors : 1;
  for (int k = 0; k < n_tensors; k += step) {
    GatherArgs part{};
    for (int i = 0; i < step; ++i) {
      part.src[i] = g.src[k + i];
      part.dst[i] = g.dst[k + i];
      part.st[i] = g.st[k + i];
    }
    gather_rows_kernel<<<dim3((unsigned)ceil_div(N * row_units, kThreads), BH, step), kThreads, 0, s>>>(part, H, perm, N,
                                                                                                        row_units);
    SVGEAR_LAUNCH_CHECK();
  }
  return SVGEAR_OK;
}

}  // namespace
}  // namespace svgear

extern "C" int svgear_permute(const int32_t* labels, int B, int H, int64_t N, int64_t n_tail, int C,
                              int32_t* perm, int32_t* offsets, int n_tensors, const void* const* src,
                              const int64_t (*sstride)[3], void* const* dst, svgear_dtype dt, int d,
                              void* ws, size_t ws_bytes, void* stream) {
  if (!labels || !perm || !offsets || B <= 0 || H <= 0 || N <= 0 || n_tail < 0 || n_tail >= N || C <= 0 ||
      C > N - n_tail || N > INT32_MAX / 2 || n_tensors < 0 || n_tensors > 4 || C > kMaxLabels)
    return SVGEAR_ERR_INVALID;
  if (dt != SVGEAR_F32 && dt != SVGEAR_BF16) return SVGEAR_ERR_INVALID;
  if (n_tensors > 0) {
    if (!src || !dst || !sstride || (d != 64 && d != 128)) return SVGEAR_ERR_INVALID;
    for (int k = 0; k < n_tensors; ++k)
      if (!src[k] || !dst[k] || !strides_ok(sstride[k], esize(dt), src[k]) ||
          reinterpret_cast<uintptr_t>(dst[k]) % 16)
        return SVGEAR_ERR_INVALID;
  }
  if (!ws || ws_bytes < svgear_permute_workspace(B, H, N, C)) return SVGEAR_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int BH = B * H;
  int rc = sort_labels(labels, BH, N, n_tail, C, perm, offsets, static_cast<int32_t*>(ws), s);
  if (rc != SVGEAR_OK) return rc;
  return gather_tensors(perm, BH, H, N, n_tensors, src, sstride, dst, dt, d, s);
}

// ---- the same call for callers that cannot allocate -----------------------------------------
// The sort's chunk histograms live in a file-scope device array instead of a caller workspace.
// In host code the array's NAME is only a stand-in for the symbol; its device address is taken
// once per device with hipGetSymbolAddress and that address is what the kernels receive.
namespace svgear {
namespace {

constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call there).
int static_scratch(void** out) {
  int dev = -1;
  SVGEAR_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SVGEAR_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    SVGEAR_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return SVGEAR_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return SVGEAR_OK;
}

}  // namespace
}  // namespace svgear

extern "C" size_t svgear_permute_static_capacity(void) { return kStaticScratchBytes; }

extern "C" int svgear_permute_static(const int32_t* labels, int B, int H, int64_t N, int64_t n_tail, int C,
                                     int32_t* perm, int32_t* offsets, int n_tensors, const void* const* src,
                                     const int64_t (*sstride)[3], void* const* dst, svgear_dtype dt, int d,
                                     void* stream) {
  if (B <= 0 || H <= 0 || N <= 0 || C <= 0) return SVGEAR_ERR_INVALID;
  if (svgear_permute_workspace(B, H, N, C) > kStaticScratchBytes) return SVGEAR_ERR_WORKSPACE;
  void* ptr = nullptr;
  const int rc = static_scratch(&ptr);
  if (rc != SVGEAR_OK) return rc;
  // every counter of the histogram area in use is written by hist_kernel before it is read,
  // so what an earlier call left in the array does not matter
  return svgear_permute(labels, B, H, N, n_tail, C, perm, offsets, n_tensors, src, sstride, dst, dt, d, ptr,
                        kStaticScratchBytes, stream);
}

extern "C" int svgear_permute_rows(const int32_t* perm, int B, int H, int64_t N, int n_tensors,
                                   const void* const* src, const int64_t (*sstride)[3], void* const* dst,
                                   svgear_dtype dt, int d, void* stream) {
  if (!perm || B <= 0 || H <= 0 || N <= 0 || N > INT32_MAX / 2 || n_tensors < 1 || n_tensors > 4 || !src || !dst ||
      !sstride || (d != 64 && d != 128) || (dt != SVGEAR_F32 && dt != SVGEAR_BF16))
    return SVGEAR_ERR_INVALID;
  for (int k = 0; k < n_tensors; ++k)
    if (!src[k] || !dst[k] || !strides_ok(sstride[k], esize(dt), src[k]) || reinterpret_cast<uintptr_t>(dst[k]) % 16)
      return SVGEAR_ERR_INVALID;
  return gather_tensors(perm, B * H, H, N, n_tensors, src, sstride, dst, dt, d, static_cast<hipStream_t>(stream));
}

extern "C" int svgear_unpermute(const void* op, const int32_t* perm, svgear_dtype dt, int B, int H, int64_t N,
                                int d, void* o, const int64_t ostride[3], void* stream) {
  if (!op || !perm || !o || B <= 0 || H <= 0 || N <= 0 || N > INT32_MAX / 2 || (d != 64 && d != 128))
    return SVGEAR_ERR_INVALID;
  if (dt != SVGEAR_F32 && dt != SVGEAR_BF16) return SVGEAR_ERR_INVALID;
  if (!strides_ok(ostride, esize(dt), o) || reinterpret_cast<uintptr_t>(op) % 16) return SVGEAR_ERR_INVALID;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int row_units = (int)(d * esize(dt) / 16);
  const int upe = (int)(16 / esize(dt));
  Strides st{ostride[0] / upe, ostride[1] / upe, ostride[2] / upe};
  dim3 grid((unsigned)ceil_div(N * row_units, kThreads), B * H);
  scatter_rows_kernel<<<grid, kThreads, 0, s>>>(static_cast<const uint4*>(op), perm, N, row_units,
                                                static_cast<uint4*>(o), st, H);
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}
