// Greedy error-to-cost routing under a cost budget, and the svgear_probe_route entry point.
// Paper: "Error-Aware Routing" (blocks are taken in descending order of error-to-size ratio
// until the budget is exhausted; the rest go to linear compensation); Experiments,
// "Implementation" (per-query-cluster budgets).
//
// "Sort, prefix-sum the costs, cut at the budget" is done without a sort: the cut is the
// first block, in (score desc, index asc) order, whose inclusive cumulative cost exceeds
// the budget. Each block gets a unique 64-bit key that is monotone in that order; a
// most-significant-digit-first radix descent over cost histograms finds the key K* of the cut
// exactly (integer arithmetic only), and block (a,b) is routed iff key > K*. A head with many
// blocks is cut by many workgroups: they build one 12-bit histogram of it, collect the blocks of
// the digit that crosses the budget, and one workgroup descends through those few alone.
//
// The adaptive per-query-cluster budgets (a reading of the top-p allocation the paper
// inherits and does not define) use the same descent over integer mass weights.
#include "common.h"

namespace svgear {

int run_probe(const float* qbar, const float* kbar, const float* vbar, const void* kp, const void* vp,
              svgear_dtype dt, const int32_t* k_offsets, int BH, int64_t Nk, int d, int Cq, int Ck, float scale,
              bool value_aware, float* scores, float* sbar, float* mrow, bf16_t* q3, float* nd, float* dd,
              hipStream_t s);

int run_sbar(const float* qbar, const float* kbar, const int32_t* k_offsets, int BH, int d, int Cq, int Ck,
             float scale, float* sbar, float* mrow, bf16_t* q3, hipStream_t s);

namespace {

constexpr int kSelThreads = 1024;
constexpr int kRowThreads = 256, kLongRowThreads = 512;
constexpr int kLongRow = 4000;  // key clusters from which a row with a budget of its own takes the latter
constexpr int kTopPWeightBits = 20;  // masses are counted in units of 2^-20
constexpr int kTopPIndexBits = 13;   // Ck <= 8192

// Larger score -> larger key; among equal scores lower linear index -> larger key.
__device__ __forceinline__ uint64_t block_key(float score, uint32_t idx) {
  if (score != score) score = INFINITY;  // NaN ranks first
  if (score == 0.f) score = 0.f;         // -0 and +0 tie
  uint32_t u = __float_as_uint(score);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)u << 32) | (uint64_t)(0xFFFFFFFFu - idx);
}

struct CutState {
  unsigned long long hist[256];
  unsigned long long prefix;
  long long remaining;
  long long wave_total[4];
  unsigned int count[256];  // items per digit
  int crossed[2];           // per pass parity: some digit's cumulative weight exceeded what is left
  int single;               // the digit that crossed holds one item: that item is the cut
};

// Walks n_items items in descending key order (keys unique) and returns the key of the first
// one whose inclusive cumulative weight exceeds rem, or 0 if every item fits. visit(it, key,
// weight) returns false for items that do not take part. Called by all threads of the block
// (THREADS >= 256, a multiple of 64). With open_bits < 64 the items share the key bits above
// those, `prefix`.
// Items are visited four at a time per thread, all their loads issued before the first
// histogram update; the digit of the cut is found by a 256-wide scan of the histogram from
// the top digit down (four waves, shuffles), not by one thread walking it. As soon as the
// digit that crosses holds a single item, that item is the cut and one more walk fetches its
// key (scores are mostly distinct, so this happens after three or four of the eight digits).
template <int THREADS, class Visit>
__device__ __forceinline__ unsigned long long radix_cut(CutState& st, long long rem, int n_items, Visit visit,
                                                        int open_bits = 64, unsigned long long prefix0 = 0ull) {
  constexpr int U = 4;
  static_assert(THREADS >= 256 && THREADS % 64 == 0, "the histogram scan uses the first four waves");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) {
    st.remaining = rem > 0 ? rem : 0;
    st.prefix = prefix0;
  }
  for (int pass = 0; open_bits > 0; ++pass) {
    const int width = open_bits < 8 ? open_bits : 8, above = open_bits;
    const int shift = open_bits - width;
    open_bits = shift;
    for (int i = threadIdx.x; i < 256; i += THREADS) {
      st.hist[i] = 0ull;
      st.count[i] = 0u;
    }
    if (threadIdx.x == 0) {
      st.crossed[pass & 1] = 0;
      st.single = 0;
    }
    __syncthreads();
    const unsigned long long prefix = st.prefix;
    const long long left = st.remaining;
    for (int base = 0; base < n_items; base += U * THREADS) {  // same trip count for every thread
      uint64_t key[U];
      unsigned long long weight[U];
      bool on[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int it = base + u * THREADS + (int)threadIdx.x;
        on[u] = it < n_items && visit(it, key[u], weight[u]);
        on[u] = on[u] && (above == 64 || (key[u] >> above) == prefix);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!on[u]) continue;
        const int digit = (int)((key[u] >> shift) & ((1u << width) - 1u));
        atomicAdd(&st.hist[digit], weight[u]);
        atomicAdd(&st.count[digit], 1u);
      }
    }
    __syncthreads();
    // thread i < 256 owns digit 255 - i: inclusive sums in descending digit order
    long long h = 0, incl = 0;
    if (threadIdx.x < 256) {
      h = (long long)st.hist[255 - threadIdx.x];
      incl = h;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const long long t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      if (lane == 63) st.wave_total[wave] = incl;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
      for (int w = 0; w < wave; ++w) incl += st.wave_total[w];
      if (incl > left && incl - h <= left) {  // the first digit that does not fit: one thread at most
        st.remaining = left - (incl - h);
        st.prefix = (prefix << width) | (unsigned long long)(255 - threadIdx.x);
        st.crossed[pass & 1] = 1;
        st.single = st.count[255 - threadIdx.x] == 1u;
      }
    }
    __syncthreads();
    if (!st.crossed[pass & 1]) return 0ull;  // everything fits (can only happen on the first pass)
    if (st.single && shift > 0) {
      const unsigned long long found = st.prefix;  // the leading bits of the cut
      __syncthreads();
      for (int base = 0; base < n_items; base += THREADS) {
        const int it = base + (int)threadIdx.x;
        uint64_t key;
        unsigned long long weight;
        if (it < n_items && visit(it, key, weight) && (key >> shift) == found) st.prefix = key;
      }
      __syncthreads();
      return st.prefix;
    }
  }
  return st.prefix;
}

// Cost of block i of a head (0: one side is empty).
__device__ __forceinline__ unsigned long long block_cost(const int32_t* qo, const int32_t* ko, int i, int Ck) {
  const int a = (int)((unsigned)i / (unsigned)Ck), b = i - a * Ck;
  const int64_t qa = qo[a + 1] - qo[a], kb = ko[b + 1] - ko[b];
  return qa > 0 && kb > 0 ? (unsigned long long)(qa * kb) : 0ull;
}

// What a head's budget leaves for its clustered blocks: the text row and the text column come first.
__device__ __forceinline__ long long head_budget(const int32_t* qo, const int32_t* ko, int Cq, int Ck, int64_t budget) {
  const int64_t Nq = qo[Cq + 1], Nk = ko[Ck + 1];
  const int64_t tq = qo[Cq + 1] - qo[Cq], tk = ko[Ck + 1] - ko[Ck];
  return budget - (tq * Nk + (Nq - tq) * tk);
}

// Adaptive budget of query cluster a: the non-empty key clusters carry the
// centroid attention mass |k_b| exp(Sbar_ab - m_a), counted in integer units of 2^-20 so that
// sums are exact in any order; ordered by weight descending (ties: lower b first), the
// shortest prefix whose weight reaches ceil(top_p * total) is kept, and the budget is the
// cost |q_a| * sum |k_b| of exact attention over it. Called by all kRowThreads threads; wgt: Ck entries of LDS.
template <int THREADS>
__device__ __forceinline__ int64_t top_p_budget(const float* sbar_row, float m, const int32_t* ko, int64_t qa, int Ck,
                                                float top_p, unsigned long long* wgt, CutState& st) {
  __shared__ unsigned long long sh_total, sh_keys;
  if (qa <= 0) return 0;
  if (threadIdx.x == 0) {
    sh_total = 0ull;
    sh_keys = 0ull;
  }
  __syncthreads();
  unsigned long long part = 0ull;
  for (int b = threadIdx.x; b < Ck; b += THREADS) {
    const int32_t kb = ko[b + 1] - ko[b];
    unsigned long long w = 0ull;
    if (kb > 0) {
      const float mass = (float)kb * expf(sbar_row[b] - m) * (float)(1 << kTopPWeightBits);
      if (mass >= 1.f) w = (unsigned long long)mass;  // also drops NaN
    }
    wgt[b] = w;
    part += w;
  }
  if (part) atomicAdd(&sh_total, part);
  __syncthreads();
  const unsigned long long total = sh_total;
  const double want = ceil((double)top_p * (double)total);
  const long long need = want >= 1.0 ? (long long)want : 1ll;
  auto key_of = [&](int b) { return (wgt[b] << kTopPIndexBits) | (unsigned long long)((1 << kTopPIndexBits) - 1 - b); };
  const unsigned long long cut = radix_cut<THREADS>(st, need - 1, Ck, [&](int it, uint64_t& key,
                                                                              unsigned long long& weight) {
    const int b = it;
    if (ko[b + 1] <= ko[b]) return false;
    key = key_of(b);
    weight = wgt[b];
    return true;
  });
  unsigned long long keys = 0ull;
  for (int b = threadIdx.x; b < Ck; b += THREADS) {
    const int32_t kb = ko[b + 1] - ko[b];
    if (kb > 0 && key_of(b) >= cut) keys += (unsigned long long)kb;
  }
  if (keys) atomicAdd(&sh_keys, keys);
  __syncthreads();
  return qa * (int64_t)sh_keys;
}

// Mask words and routed blocks of row a of a head (a whole wave): returns the count and adds the
// lane's share of the cost. 64 consecutive key clusters per step (coalesced score loads), two mask
// words per ballot, four steps at a time; share s of `shares` waves takes every shares-th four.
__device__ __forceinline__ int mask_row(const float* sc, const int32_t* qo, const int32_t* ko, int Cq, int Ck, int a,
                                        uint64_t ks, uint32_t* words, long long& cost, int share = 0, int shares = 1) {
  const int Cc = Ck + 1, W = (Cc + 31) / 32, lane = threadIdx.x & 63;
  const int64_t qa = qo[a + 1] - qo[a];
  int cnt = 0;
  constexpr int U = 4;  // steps whose loads are in flight together
  for (int b00 = 64 * U * share; b00 < W * 32; b00 += 64 * U * shares) {
    int32_t size[U];
    float score[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = min(b00 + 64 * u + lane, Ck);
      size[u] = ko[b + 1] - ko[b];
      score[u] = a < Cq && b < Ck ? sc[(int64_t)a * Ck + b] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b0 = b00 + 64 * u, b = b0 + lane;
      if (b0 >= W * 32) break;
      bool on = false;
      if (qa > 0 && b < Cc && size[u] > 0) {
        on = a == Cq || b == Ck || block_key(score[u], (uint32_t)(a * Ck + b)) > ks;
        if (on) cost += qa * (int64_t)size[u];
      }
      const unsigned long long bits = __ballot(on);
      cnt += __popcll(bits);
      if (lane == 0) {
        words[b0 >> 5] = (uint32_t)bits;
        if ((b0 >> 5) + 1 < W) words[(b0 >> 5) + 1] = (uint32_t)(bits >> 32);
      }
    }
  }
  return cnt;
}

// The set bits of a row, ascending, to ci[pos ...] (a whole wave, a lane per bit).
__device__ __forceinline__ void list_row(const uint32_t* words, int W, int32_t pos, int32_t* ci) {
  const int lane = threadIdx.x & 63;
  for (int w0 = 0; w0 < W; w0 += 2) {
    unsigned long long bits = words[w0];
    if (w0 + 1 < W) bits |= (unsigned long long)words[w0 + 1] << 32;
    if ((bits >> lane) & 1ull) ci[pos + __popcll(bits & ((1ull << lane) - 1ull))] = w0 * 32 + lane;
    pos += __popcll(bits);
  }
}

// Bit mask, CSR lists and routed cost of one head (all threads of a workgroup of kSelThreads), a wave
// per row of blocks. rowcnt: Cq + 2 ints of LDS.
__device__ __forceinline__ void build_head(const float* sc, const int32_t* qo, const int32_t* ko, int Cq, int Ck, int bh,
                                           uint64_t cut, int32_t* rowcnt, unsigned long long* cost_sum,
                                           uint32_t* mask_bits, int32_t* row_ptr, int32_t* col_idx,
                                           int64_t* routed_cost) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int NWAVES = kSelThreads / 64;
  const int R = Cq + 1, Cc = Ck + 1, W = (Cc + 31) / 32;
  uint32_t* mb = mask_bits + (int64_t)bh * R * W;
  if (threadIdx.x == 0) *cost_sum = 0ull;
  __syncthreads();
  long long my_cost = 0;
  for (int a = wave; a < R; a += NWAVES) {
    const int cnt = mask_row(sc, qo, ko, Cq, Ck, a, a < Cq ? cut : 0ull, mb + (int64_t)a * W, my_cost);
    if (lane == 0) rowcnt[a] = cnt;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) my_cost += __shfl_xor(my_cost, o);
  if (lane == 0 && my_cost) atomicAdd(cost_sum, (unsigned long long)my_cost);
  __threadfence_block();
  __syncthreads();
  int32_t* rp = row_ptr + (int64_t)bh * (R + 1);
  if (threadIdx.x == 0) {
    int32_t run = 0;
    for (int a = 0; a < R; ++a) {
      const int32_t c = rowcnt[a];
      rowcnt[a] = run;
      rp[a] = run;
      run += c;
    }
    rp[R] = run;
    routed_cost[bh] = (int64_t)*cost_sum;
  }
  __syncthreads();
  // routed key clusters of every row, ascending
  int32_t* ci = col_idx + (int64_t)bh * R * Cc;
  for (int a = wave; a < R; a += NWAVES) list_row(mb + (int64_t)a * W, W, rowcnt[a], ci);
}

// grid (Cq + 1, BH): rows with budgets of their own: the row's budget (its share of the head's, or with top_p >= 0 the
// adaptive one, for its clustered blocks, the tail column on top), its cut, mask words, routed blocks and cost. One
// launch instead of three or four dependent ones: 5 heads, 200 x 500 centroids 28 + 16 + 8 us, and 5 to clear a counter,
// in 39. A row of thousands of blocks takes twice the threads: its adaptive weights fill so much LDS that two
// workgroups a CU are left of it (24 heads, 400 x 6,000: 3,404 us with 256 threads, 2,581 with 512, 3,205 with 1,024; three
// launches as before 3,070; fixed budgets 795, 752, 1,029, 802), while shorter rows wait for one another in wider ones
// (8 heads, 1,000 x 3,000: 304 with 256, 326 with 512, 486 with 1,024; 2 heads, 1,000 x 4,000: 174, 161, 211).
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
route_rows_kernel(const float* __restrict__ scores, const float* __restrict__ sbar, const float* __restrict__ mrow,
                  const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ k_offsets, int Cq, int Ck,
                  int64_t budget, float top_p, int64_t* __restrict__ row_budget, uint32_t* __restrict__ mask_bits,
                  int32_t* __restrict__ row_count, int64_t* __restrict__ row_cost) {
  extern __shared__ unsigned long long wgt[];  // Ck, with top_p
  __shared__ CutState st;
  __shared__ int s_cnt[THREADS / 64];
  __shared__ long long s_cost[THREADS / 64];
  const int a = blockIdx.x, bh = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int R = Cq + 1, W = (Ck + 1 + 31) / 32;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const float* sc = scores + (int64_t)bh * Cq * Ck;
  unsigned long long cut = 0ull;
  if (a < Cq) {
    const int64_t Nq = qo[Cq + 1], qa = qo[a + 1] - qo[a], at = (int64_t)bh * Cq + a;
    long long rem;
    if (top_p >= 0.f) {
      rem = top_p_budget<THREADS>(sbar + at * Ck, mrow[at], ko, qa, Ck, top_p, wgt, st);
      if (threadIdx.x == 0) row_budget[at] = rem;
      __syncthreads();
    } else {
      rem = (budget * qa) / (Nq > 0 ? Nq : 1) - qa * (ko[Ck + 1] - ko[Ck]);
    }
    cut = radix_cut<THREADS>(st, rem, Ck, [&](int b, uint64_t& key, unsigned long long& weight) {
      weight = block_cost(qo, ko, a * Ck + b, Ck);
      if (weight == 0ull) return false;
      key = block_key(sc[(int64_t)a * Ck + b], (uint32_t)(a * Ck + b));
      return true;
    });
  }
  long long cost = 0;
  const int cnt = mask_row(sc, qo, ko, Cq, Ck, a, cut, mask_bits + ((int64_t)bh * R + a) * W, cost, wave, THREADS / 64);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cost += __shfl_xor(cost, o);
  if (lane == 0) {
    s_cnt[wave] = cnt;
    s_cost[wave] = cost;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int n = 0;
    long long sum = 0;
    for (int w = 0; w < THREADS / 64; ++w) {
      n += s_cnt[w];
      sum += s_cost[w];
    }
    row_count[(int64_t)bh * R + a] = n;
    row_cost[(int64_t)bh * R + a] = sum;
  }
}

// grid (BH): cut, mask, lists and cost of heads of fewer than kWideItems blocks with one budget: a
// small layer is bound by launches, so the two steps share one (they took 8 and 4 us)
__global__ void __launch_bounds__(kSelThreads)
route_small_kernel(const float* __restrict__ scores, const int32_t* __restrict__ q_offsets,
                   const int32_t* __restrict__ k_offsets, int Cq, int Ck, int64_t budget,
                   uint32_t* __restrict__ mask_bits, int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx,
                   int64_t* __restrict__ routed_cost) {
  extern __shared__ int32_t rowcnt[];  // Cq+2
  __shared__ CutState st;
  __shared__ unsigned long long cost_sum;
  const int bh = blockIdx.x;
  const float* sc = scores + (int64_t)bh * Cq * Ck;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const unsigned long long cut = radix_cut<kSelThreads>(st, head_budget(qo, ko, Cq, Ck, budget), Cq * Ck,
                                                       [&](int it, uint64_t& key, unsigned long long& weight) {
    weight = block_cost(qo, ko, it, Ck);
    if (weight == 0ull) return false;
    key = block_key(sc[it], (uint32_t)it);
    return true;
  });
  build_head(sc, qo, ko, Cq, Ck, bh, cut, rowcnt, &cost_sum, mask_bits, row_ptr, col_idx, routed_cost);
}

// ---- one budget over many blocks ---------------------------------------------------------
// What bounds the cut of a head is reading its scores and, with one workgroup per head, the one
// CU that does it: 300 x 1000 blocks of 40 heads took such a cut 1.69 ms (four to five walks
// over 1.2 MB, LDS atomics on the dozen exponents that an 8-bit digit tells apart) and
// the mask and lists 0.35 ms on 40 of 256 CUs. From kWideItems blocks a head on the work is spread:
// two streaming passes over all CUs, after which a single workgroup sees only the blocks of one
// 12-bit digit (an eighth of an octave of scores, a few thousand blocks). Measured at 300 x 1000
// x 40 heads: cut, mask and lists 2.04 -> 0.15 ms (of a whole call of 3.74 before and 1.36 now). Small
// heads stay with one workgroup, three launches fewer (1,800 blocks 19 us a call from given scores); at
// the line one head takes 65 us below it and 39 above.
constexpr int kWideItems = 16384;
constexpr int kHistBits = 12, kHistBins = 1 << kHistBits;
constexpr int kHistThreads = 512;
constexpr int kHistItems = 16 * kHistThreads;  // blocks per workgroup of the streaming passes

struct HeadCut {
  unsigned long long hist[kHistBins];  // summed cost by leading digit
  long long remaining;                 // budget left for the digit that crosses
  int digit;                           // that digit, -1: everything fits
  unsigned int n_cand;                 // blocks collected of it
};

// Clears what the passes below add to (kernels, not memory sets: the call may be captured).
__global__ void __launch_bounds__(256)
route_clear_kernel(HeadCut* __restrict__ cuts, int64_t* __restrict__ routed_cost) {
  HeadCut& hc = cuts[blockIdx.y];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < kHistBins) hc.hist[i] = 0ull;
  if (i == 0) {
    hc.n_cand = 0u;
    routed_cost[blockIdx.y] = 0;
  }
}

// grid (ceil(Cq Ck / kHistItems), BH)
__global__ void __launch_bounds__(kHistThreads)
route_hist_kernel(const float* __restrict__ scores, const int32_t* __restrict__ q_offsets,
                  const int32_t* __restrict__ k_offsets, int Cq, int Ck, HeadCut* __restrict__ cuts) {
  __shared__ unsigned long long h[kHistBins];
  const int bh = blockIdx.y, n_items = Cq * Ck;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const float* sc = scores + (int64_t)bh * Cq * Ck;
  for (int i = threadIdx.x; i < kHistBins; i += kHistThreads) h[i] = 0ull;
  __syncthreads();
  const int lo = blockIdx.x * kHistItems + threadIdx.x;
  float v[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) v[u] = lo + u * kHistThreads < n_items ? sc[lo + u * kHistThreads] : 0.f;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int i = lo + u * kHistThreads;
    if (i >= n_items) break;
    const unsigned long long cost = block_cost(qo, ko, i, Ck);
    if (cost) atomicAdd(&h[(int)(block_key(v[u], (uint32_t)i) >> (64 - kHistBits))], cost);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kHistBins; i += kHistThreads)
    if (h[i]) atomicAdd(&cuts[bh].hist[i], h[i]);
}

// Finds the digit that crosses the budget (every workgroup for itself: 32 KB of L2) and collects
// the indices of its blocks, in any order: keys are unique, so the order does not matter.
__global__ void __launch_bounds__(kHistThreads)
route_collect_kernel(const float* __restrict__ scores, const int32_t* __restrict__ q_offsets,
                     const int32_t* __restrict__ k_offsets, int Cq, int Ck, int64_t budget, HeadCut* __restrict__ cuts,
                     uint32_t* __restrict__ cand) {
  constexpr int PER = kHistBins / kHistThreads;
  __shared__ long long wave_total[kHistThreads / 64];
  __shared__ int digit_s;
  const int bh = blockIdx.y, n_items = Cq * Ck, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const float* sc = scores + (int64_t)bh * Cq * Ck;
  HeadCut& hc = cuts[bh];
  const long long rem = head_budget(qo, ko, Cq, Ck, budget), left = rem > 0 ? rem : 0;
  const int top = kHistBins - 1 - PER * (int)threadIdx.x;  // this thread's digits: top, top - 1, ...
  long long h[PER], sum = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    h[u] = (long long)hc.hist[top - u];
    sum += h[u];
  }
  long long incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wave_total[wave] = incl;
  if (threadIdx.x == 0) digit_s = -1;
  __syncthreads();
  for (int w = 0; w < wave; ++w) incl += wave_total[w];
  if (incl > left && incl - sum <= left) {  // one thread at most
    long long run = incl - sum;
    int u = 0;
    while (run + h[u] <= left) run += h[u++];
    digit_s = top - u;
    if (blockIdx.x == 0) hc.remaining = left - run;
  }
  __syncthreads();
  const int digit = digit_s;
  if (blockIdx.x == 0 && threadIdx.x == 0) hc.digit = digit;
  if (digit < 0) return;
  const int lo = blockIdx.x * kHistItems + threadIdx.x;
  float v[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) v[u] = lo + u * kHistThreads < n_items ? sc[lo + u * kHistThreads] : 0.f;
  unsigned int mine = 0;  // a bit per block of this thread
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int i = lo + u * kHistThreads;
    if (i < n_items && (int)(block_key(v[u], (uint32_t)i) >> (64 - kHistBits)) == digit && block_cost(qo, ko, i, Ck) != 0ull)
      mine |= 1u << u;
  }
  // one addition to the head's counter per workgroup (one per 64 blocks with a hit: 75 us at 300 x 1000 x 40 heads,
  // additions to a line follow each other at some 57 ns; this way 28)
  __shared__ int wave_cand[kHistThreads / 64], base_s;
  const int n_mine = __popc(mine);
  int upto = n_mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(upto, o);
    if (lane >= o) upto += t;
  }
  if (lane == 63) wave_cand[wave] = upto;
  __syncthreads();
  if (threadIdx.x == 0) {
    int all = 0;
    for (int w = 0; w < kHistThreads / 64; ++w) all += wave_cand[w];
    base_s = all ? (int)atomicAdd(&hc.n_cand, (unsigned int)all) : 0;
  }
  __syncthreads();
  int at = base_s + upto - n_mine;
  for (int w = 0; w < wave; ++w) at += wave_cand[w];
#pragma unroll
  for (int u = 0; u < 16; ++u)
    if (mine & (1u << u)) cand[(int64_t)bh * n_items + at++] = (uint32_t)(lo + u * kHistThreads);
}

// grid (BH): the cut among the collected blocks
__global__ void __launch_bounds__(kSelThreads)
route_cut_kernel(const float* __restrict__ scores, const int32_t* __restrict__ q_offsets,
                 const int32_t* __restrict__ k_offsets, int Cq, int Ck, const HeadCut* __restrict__ cuts,
                 const uint32_t* __restrict__ cand, uint64_t* __restrict__ kstar) {
  __shared__ CutState st;
  const int bh = blockIdx.x, n_items = Cq * Ck;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const float* sc = scores + (int64_t)bh * n_items;
  const uint32_t* list = cand + (int64_t)bh * n_items;
  const HeadCut& hc = cuts[bh];
  unsigned long long cut = 0ull;
  if (hc.digit >= 0)
    cut = radix_cut<kSelThreads>(st, hc.remaining, (int)hc.n_cand, [&](int it, uint64_t& key, unsigned long long& weight) {
      const uint32_t i = list[it];
      key = block_key(sc[i], i);
      weight = block_cost(qo, ko, (int)i, Ck);
      return true;
    }, 64 - kHistBits, (unsigned long long)hc.digit);
  if (threadIdx.x == 0) kstar[bh] = cut;
}

// grid (ceil((Cq + 1) / 4), BH): mask words, routed blocks and routed cost, a wave per row of blocks
__global__ void __launch_bounds__(256)
route_mask_kernel(const float* __restrict__ scores, const int32_t* __restrict__ q_offsets,
                  const int32_t* __restrict__ k_offsets, int Cq, int Ck, const uint64_t* __restrict__ kstar,
                  uint32_t* __restrict__ mask_bits, int32_t* __restrict__ row_count,
                  int64_t* __restrict__ routed_cost) {
  const int bh = blockIdx.y, lane = threadIdx.x & 63, a = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int R = Cq + 1, W = (Ck + 1 + 31) / 32;
  __shared__ long long part[4];
  long long cost = 0;
  if (a < R) {
    const int cnt = mask_row(scores + (int64_t)bh * Cq * Ck, q_offsets + (int64_t)bh * (Cq + 2),
                             k_offsets + (int64_t)bh * (Ck + 2), Cq, Ck, a,
                             a < Cq ? kstar[bh] : 0ull,
                             mask_bits + ((int64_t)bh * R + a) * W, cost);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cost += __shfl_xor(cost, o);
    if (lane == 0) row_count[(int64_t)bh * R + a] = cnt;
  }
  if (lane == 0) part[threadIdx.x >> 6] = cost;
  __syncthreads();
  if (threadIdx.x == 0) {
    cost = part[0] + part[1] + part[2] + part[3];
    if (cost) atomicAdd(reinterpret_cast<unsigned long long*>(routed_cost + bh), (unsigned long long)cost);
  }
}

// grid (ceil((Cq + 1) / kListRows), BH): row_ptr and col_idx of kListRows rows; the routed blocks of
// the rows before them are summed by the workgroup itself, and with row_cost the head's cost by its first one
constexpr int kListRows = 16;
__global__ void __launch_bounds__(256)
route_lists_kernel(int Cq, int Ck, const uint32_t* __restrict__ mask_bits, const int32_t* __restrict__ row_count,
                   const int64_t* __restrict__ row_cost, int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx,
                   int64_t* __restrict__ routed_cost) {
  __shared__ long long cost_part[4];
  __shared__ int32_t part[4], start[kListRows + 1];
  const int bh = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int R = Cq + 1, Cc = Ck + 1, W = (Cc + 31) / 32;
  const int a0 = blockIdx.x * kListRows, n = min(kListRows, R - a0);
  const int32_t* rc = row_count + (int64_t)bh * R;
  int32_t before = 0;
  for (int a = threadIdx.x; a < a0; a += 256) before += rc[a];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if (lane == 0) part[wave] = before;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t run = part[0] + part[1] + part[2] + part[3];
    for (int u = 0; u < n; ++u) {
      start[u] = run;
      run += rc[a0 + u];
    }
    start[n] = run;
  }
  __syncthreads();
  if (row_cost && blockIdx.x == 0) {
    long long cost = 0;
    for (int a = threadIdx.x; a < R; a += 256) cost += row_cost[(int64_t)bh * R + a];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cost += __shfl_xor(cost, o);
    if (lane == 0) cost_part[wave] = cost;
    __syncthreads();
    if (threadIdx.x == 0) routed_cost[bh] = cost_part[0] + cost_part[1] + cost_part[2] + cost_part[3];
  }
  if ((int)threadIdx.x < n || ((int)threadIdx.x == n && a0 + n == R))
    row_ptr[(int64_t)bh * (R + 1) + a0 + threadIdx.x] = start[threadIdx.x];
  int32_t* ci = col_idx + (int64_t)bh * R * Cc;
  for (int u = wave; u < n; u += 4)
    list_row(mask_bits + ((int64_t)bh * R + a0 + u) * W, W, start[u], ci);
}

}  // namespace
}  // namespace svgear

using namespace svgear;

extern "C" size_t svgear_probe_route_workspace(int B, int H, int64_t Nk, int d, int Cq, int Ck) {
  if (B <= 0 || H <= 0 || Cq <= 0 || Ck <= 0 || Nk <= 0 || d <= 0) return 0;
  const size_t BH = (size_t)B * H;
  return align_up(BH * Cq * Ck * 4, 256) + align_up(BH * Cq * 4, 256) + align_up(BH * (Cq + 1) * 8, 256) +
         // bf16 probe: qbar in three bf16 pieces (operand order), per-key value statistics
         align_up(BH * align_up(Cq, 32) * d * 3 * 2, 256) + 2 * align_up(BH * probe_stat_stride(Nk) * 4, 256) +
         // many blocks: cost histograms, routed blocks per row (the candidates reuse the centroid logits' place)
         align_up(BH * sizeof(HeadCut), 256) + align_up(BH * (Cq + 1) * 4, 256);
}

namespace {

// top_p < 0: budget_cost rules (per head or per query cluster); otherwise adaptive row budgets.
int probe_route_impl(const float* qbar, const float* kbar, const float* vbar, const void* kp, const void* vp,
                     svgear_dtype dt, const int32_t* q_offsets, const int32_t* k_offsets, int B, int H, int64_t Nq,
                     int64_t Nk, int d, int Cq, int Ck, int64_t budget_cost, float top_p, float scale, unsigned flags,
                     float* scores, uint32_t* mask_bits, int32_t* row_ptr, int32_t* col_idx, int64_t* routed_cost,
                     int64_t* row_budget, void* ws, size_t ws_bytes, void* stream) {
  const bool given = flags & SVGEAR_USE_GIVEN_SCORES;
  const bool adaptive = top_p >= 0.f;
  if (!q_offsets || !k_offsets || !scores || !mask_bits || !row_ptr || !col_idx || !routed_cost || B <= 0 ||
      H <= 0 || Nq <= 0 || Nk <= 0 || Cq <= 0 || Ck <= 0 || Cq > 8192 || Ck > 8192 || budget_cost < 0 ||
      Nq > INT32_MAX / 2 || Nk > INT32_MAX / 2 || (flags & ~7u) || (int64_t)(Cq + 1) * (Ck + 1) > INT32_MAX / 2)
    return SVGEAR_ERR_INVALID;
  if (adaptive && (!row_budget || !(top_p > 0.f && top_p <= 1.f))) return SVGEAR_ERR_INVALID;
  if (!given || adaptive) {
    if (!qbar || !kbar || (d != 64 && d != 128) || reinterpret_cast<uintptr_t>(qbar) % 16 ||
        reinterpret_cast<uintptr_t>(kbar) % 16)
      return SVGEAR_ERR_INVALID;
  }
  if (!given) {
    if (!vbar || !kp || !vp || (dt != SVGEAR_F32 && dt != SVGEAR_BF16) || reinterpret_cast<uintptr_t>(kp) % 16 ||
        reinterpret_cast<uintptr_t>(vp) % 16)
      return SVGEAR_ERR_INVALID;
  }
  if (!ws || ws_bytes < svgear_probe_route_workspace(B, H, Nk, d, Cq, Ck)) return SVGEAR_ERR_WORKSPACE;
  const int BH = B * H;
  Workspace w(ws, ws_bytes);
  float* sbar = w.take<float>((size_t)BH * Cq * Ck);
  float* mrow = w.take<float>((size_t)BH * Cq);
  uint64_t* kstar = w.take<uint64_t>((size_t)BH * (Cq + 1));
  bf16_t* q3 = w.take<bf16_t>((size_t)BH * align_up(Cq, 32) * (d > 0 ? d : 1) * 3);
  float* nd = w.take<float>((size_t)BH * probe_stat_stride(Nk));
  float* dd = w.take<float>((size_t)BH * probe_stat_stride(Nk));
  HeadCut* cuts = w.take<HeadCut>(BH);
  int32_t* row_count = w.take<int32_t>((size_t)BH * (Cq + 1));
  if (!w.ok()) return SVGEAR_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!given) {
    int rc = run_probe(qbar, kbar, vbar, kp, vp, dt, k_offsets, BH, Nk, d, Cq, Ck, scale,
                       !(flags & SVGEAR_PROBE_PLAIN), scores, sbar, mrow, q3, nd, dd, s);
    if (rc != SVGEAR_OK) return rc;
  } else if (adaptive) {
    int rc = run_sbar(qbar, kbar, k_offsets, BH, d, Cq, Ck, scale, sbar, mrow, nullptr, s);
    if (rc != SVGEAR_OK) return rc;
  }
  const int64_t n_items = (int64_t)Cq * Ck;
  const dim3 list_grid((unsigned)ceil_div(Cq + 1, kListRows), BH);
  if (adaptive || (flags & SVGEAR_ROUTE_PER_ROW)) {
    // up to 64 KB of weights for the largest Ck, beside the kernel's static LDS
    const size_t lds = adaptive ? (size_t)Ck * sizeof(unsigned long long) : 0;
    const bool long_row = Ck >= kLongRow;
    auto rows = long_row ? route_rows_kernel<kLongRowThreads> : route_rows_kernel<kRowThreads>;
    SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(rows),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int64_t* row_cost = reinterpret_cast<int64_t*>(kstar);  // (no cut leaves that kernel)
    rows<<<dim3(Cq + 1, BH), long_row ? kLongRowThreads : kRowThreads, lds, s>>>(
        scores, sbar, mrow, q_offsets, k_offsets, Cq, Ck, budget_cost, adaptive ? top_p : -1.f, row_budget, mask_bits,
        row_count, row_cost);
    SVGEAR_LAUNCH_CHECK();
    route_lists_kernel<<<list_grid, 256, 0, s>>>(Cq, Ck, mask_bits, row_count, row_cost, row_ptr, col_idx, routed_cost);
  } else if (n_items >= kWideItems) {
    route_clear_kernel<<<dim3(kHistBins / 256, BH), 256, 0, s>>>(cuts, routed_cost);
    SVGEAR_LAUNCH_CHECK();
    const dim3 grid((unsigned)ceil_div(n_items, kHistItems), BH);
    uint32_t* cand = reinterpret_cast<uint32_t*>(sbar);  // the probe is done with the centroid logits
    route_hist_kernel<<<grid, kHistThreads, 0, s>>>(scores, q_offsets, k_offsets, Cq, Ck, cuts);
    SVGEAR_LAUNCH_CHECK();
    route_collect_kernel<<<grid, kHistThreads, 0, s>>>(scores, q_offsets, k_offsets, Cq, Ck, budget_cost, cuts, cand);
    SVGEAR_LAUNCH_CHECK();
    route_cut_kernel<<<BH, kSelThreads, 0, s>>>(scores, q_offsets, k_offsets, Cq, Ck, cuts, cand, kstar);
    SVGEAR_LAUNCH_CHECK();
    route_mask_kernel<<<dim3((unsigned)ceil_div(Cq + 1, 4), BH), 256, 0, s>>>(scores, q_offsets, k_offsets, Cq, Ck, kstar,
                                                                             mask_bits, row_count, routed_cost);
    SVGEAR_LAUNCH_CHECK();
    route_lists_kernel<<<list_grid, 256, 0, s>>>(Cq, Ck, mask_bits, row_count, nullptr, row_ptr, col_idx, routed_cost);
  } else {
    route_small_kernel<<<BH, kSelThreads, (Cq + 2) * sizeof(int32_t), s>>>(scores, q_offsets, k_offsets, Cq, Ck,
                                                                          budget_cost, mask_bits, row_ptr, col_idx,
                                                                          routed_cost);
  }
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}

}  // namespace

extern "C" int svgear_probe_route(const float* qbar, const float* kbar, const float* vbar, const void* kp,
                                  const void* vp, svgear_dtype dt, const int32_t* q_offsets,
                                  const int32_t* k_offsets, int B, int H, int64_t Nq, int64_t Nk, int d, int Cq,
                                  int Ck, int64_t budget_cost, float scale, unsigned flags, float* scores,
                                  uint32_t* mask_bits, int32_t* row_ptr, int32_t* col_idx, int64_t* routed_cost,
                                  void* ws, size_t ws_bytes, void* stream) {
  return probe_route_impl(qbar, kbar, vbar, kp, vp, dt, q_offsets, k_offsets, B, H, Nq, Nk, d, Cq, Ck, budget_cost,
                          -1.f, scale, flags, scores, mask_bits, row_ptr, col_idx, routed_cost, nullptr, ws, ws_bytes,
                          stream);
}

extern "C" int svgear_probe_route_top_p(const float* qbar, const float* kbar, const float* vbar, const void* kp,
                                        const void* vp, svgear_dtype dt, const int32_t* q_offsets,
                                        const int32_t* k_offsets, int B, int H, int64_t Nq, int64_t Nk, int d,
                                        int Cq, int Ck, float top_p, float scale, unsigned flags, float* scores,
                                        uint32_t* mask_bits, int32_t* row_ptr, int32_t* col_idx,
                                        int64_t* routed_cost, int64_t* row_budget, void* ws, size_t ws_bytes,
                                        void* stream) {
  if (!(top_p > 0.f && top_p <= 1.f) || (flags & SVGEAR_ROUTE_PER_ROW)) return SVGEAR_ERR_INVALID;
  return probe_route_impl(qbar, kbar, vbar, kp, vp, dt, q_offsets, k_offsets, B, H, Nq, Nk, d, Cq, Ck, 0, top_p,
                          scale, flags, scores, mask_bits, row_ptr, col_idx, routed_cost, row_budget, ws, ws_bytes,
                          stream);
}
