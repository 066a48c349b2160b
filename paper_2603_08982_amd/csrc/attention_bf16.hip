// bf16 MFMA kernels of the fused block-sparse attention + centroid compensation.
// Paper: Eq. (1), Eq. (6), Algorithm 2 (see attention.hip for the decomposition).
#include "attention.h"

#include <algorithm>
#include <type_traits>

namespace svgear {
namespace {

// ------------------------------------------------------------------------------ bf16 MFMA
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
  union { uint4 u; bf16x8 b; } c;
  c.u = v;
  return c.b;
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 f = {lo, hi};
  bf16x2 b = __builtin_convertvector(f, bf16x2);
  union { bf16x2 b; uint32_t u; } c;
  c.b = b;
  return c.u;
}

// Data path built on two gfx950 features:
//  * K and V tiles go from global memory straight into LDS (global_load_lds, 16 bytes per
//    lane, a wave fills 1 KB = 4 rows of 256 B (d = 128) or 8 of 128 B contiguously), so no VGPRs
//    stage the tiles and the loads of later tiles fly while tile t is computed;
//  * V stays row-major [key][dim] in LDS and the A operand of O^T += V^T P^T is fetched
//    with the LDS transpose read (ds_read_b64_tr_b16): within a group of 16 lanes, lane j
//    receives element j%4 of the four 8-byte rows addressed by lanes j/4, j/4+4, j/4+8,
//    j/4+12 of the group. Lanes r of a group address V[key0 + r/4][dim0 + 4*(r%4) ..+3],
//    so lane j gets dims dim0+j of keys key0..key0+3.
// Bank conflicts are avoided by XOR-swizzling the 16-byte chunk index inside each row (256 B rows:
// K chunk ^ (row % 16), V chunk ^ 4 (row % 4); 128 B rows, of which two share the 64 banks:
// K chunk ^ (row/2 % 8), V chunk ^ 4 (row/2 % 2)); the swizzle is applied on the global side of the
// copy (a lane picks which global chunk lands in its LDS slot).
// d = 64 is bound by the vector ALU rather than the matrix cores: a 64-key step of a wave has 16
// MFMAs (512 cycles of its SIMD) against some 150 vector instructions and 32 exponentials (about 800).
// It runs the same pipeline; the kernel before staged its tiles through registers, transposed V with
// vector instructions and kept 4 waves a workgroup (24 heads x 32,477 rows, 64 / 300 clusters, a
// quarter routed: 5.21 -> 2.08 ms, 318 -> 797 TFLOP/s).
// log2 headroom before the running maximum is refreshed. None at d = 64: the weight of a row's largest logit
// is then exactly 1 in bf16, and the output's error against 64 bits a few percent smaller (24 heads x 32,477
// rows: 2.28e-3 instead of 2.32e-3; 2.01 -> 2.08 ms).
template <int D>
constexpr float kLazyRescale = D == 64 ? 0.0f : 8.0f;

// The row sums (softmax denominators, log-sum-exp): at d = 128 over the bf16-rounded probabilities that the
// PV product uses, at d = 64 over the probabilities as computed in fp32: the log-sum-exp is within 2e-5 of
// 64 bits (the sum of rounded ones is up to 4e-3 off at a few keys) for 32 additions a step instead of 16
// packed ones (24 heads x 32,477 rows: 1.98 -> 2.00 ms).
template <int D>
constexpr bool kSumRounded = D == 128;

typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
// acc + lo(p) + hi(p) for a packed bf16 pair (v_dot2c_f32_bf16 against (1, 1))
__device__ __forceinline__ float dot2_ones(uint32_t pair, float acc) {
  union { uint32_t u; bf16x2v b; } x, one;
  x.u = pair;
  one.u = 0x3f803f80u;
  return __builtin_amdgcn_fdot2_f32_bf16(x.b, one.b, acc, false);
}

// value held by lane ^ 32 (v_permlane32_swap: a VALU exchange of the two wave halves, no LDS)
__device__ __forceinline__ float swap32(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16* lds_v4i16_ptr;

template <int ROW_BYTES>
__device__ __forceinline__ bf16x8 tr_pair(const unsigned char* lds_base, int off_bytes) {
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(lds_base + off_bytes));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(lds_base + off_bytes + 8 * ROW_BYTES));
  union { struct { v4i16 a, b; } s; bf16x8 v; } c;
  c.s.a = lo;
  c.s.b = hi;
  return c.v;
}

// A wave-uniform pointer the compiler could not prove uniform, moved to scalar registers.
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)(p);
}

// Entries of each of the two key-cluster tables: routed clusters and a sentinel, then, 16-byte
// aligned, the compensated ones, filled up to a whole tile.
__host__ __device__ static inline int list_entries(int Ck) { return (Ck + 72) & ~3; }

// The list counters lie in cache lines of their own: every workgroup adds to one, and additions to one
// line from all XCDs follow each other at some 57 ns (24 heads x 1,200 rows, 4,800 tiles of d = 64: 305 -> 180 us).
__host__ __device__ static constexpr int sched_counter(int list) { return 64 * (1 + list); }
constexpr int kSchedInts = 64 * 9;

static inline size_t lds_bytes(int d, int Ck, int stages) {
  const size_t kv = (size_t)stages * 2 * BN * d * 2;  // K and V, `stages` buffers each
  return kv + (size_t)(stages + 3) * BN * 4 + 2 * (size_t)list_entries(Ck) * 4 + 16;
}

// ---- what the two kernels below share

// Every workgroup claims one tile: the next of the work list of the XCD it runs on (tiles
// of one query cluster are neighbours in a list, so the CUs of an XCD work on the same
// routed K/V at the same time and share it in their L2), or, once that list is used up, of
// the other XCDs' lists. Lists are sorted longest tile first and workgroups start in
// order, so the long tiles start early and the short ones fill the end of the launch. The
// grid covers the tile-count bound; workgroups that find every list used up exit.
// With keys split, a tile is `splits` slots of its list. One thread: slot_s[0] = tile or -1, slot_s[2] = split.
__device__ __forceinline__ void claim_tile(const AttnArgs& p, int splits, int32_t* slot_s) {
  const int my_xcd = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 7;  // XCC_ID
  int found = -1, part = 0;
  for (int xk = 0; xk < 8 && found < 0; ++xk) {
    const int xl = (my_xcd + xk) & 7, slots = p.sched_x[8 + xl] * splits;
    if (p.sched_x[sched_counter(xl)] >= slots) continue;  // used up (the counter only grows)
    const int slot = atomicAdd(p.sched_x + sched_counter(xl), 1);
    if (slot < slots) {
      found = p.sched_x[xl] + slot / splits;
      part = slot % splits;
    }
  }
  slot_s[0] = found;
  slot_s[2] = part;
}

// The key-cluster tables of a tile of query cluster a, by waves 0 and 1: of the routed clusters e < ne the
// first virtual position and the first row, then the end position; from comp0 on, of the compensated ones the
// index and the bias, filled up to a whole tile. slot_s[1] = number of the latter.
__device__ __forceinline__ void cluster_tables(const AttnArgs& p, int bh, int a, int ne, int comp0, int wave, int lane,
                                               int32_t* ent0, int32_t* ent1, int32_t* slot_s) {
  const int Ck = p.Ck, R = p.Cq + 1, Cc = Ck + 1, W = (Cc + 31) / 32;
  const int32_t* ko = p.k_offsets + (int64_t)bh * (Ck + 2);
  if (wave == 0) {
    const int32_t* ci = p.col_idx + (int64_t)bh * R * Cc + p.row_ptr[(int64_t)bh * (R + 1) + a];
    int carry = 0;
    for (int e0 = 0; e0 < ne; e0 += 64) {
      const int e = e0 + lane;
      int sz = 0;
      if (e < ne) {
        const int b = ci[e];
        const int ps = ko[b];
        sz = ko[b + 1] - ps;
        sz = sz > 0 ? sz : 0;
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
    // skipped, non-empty clusters only: a quarter routed leaves a quarter fewer centroid tiles
    int at = comp0;
    if (a < p.Cq) {
      const uint32_t* mrow = p.mask_bits + ((int64_t)bh * R + a) * W;
      for (int b0 = 0; b0 < Ck; b0 += 64) {
        const int b = b0 + lane;
        const int sz = b < Ck ? ko[b + 1] - ko[b] : 0;
        const bool on = sz > 0 && !mask_bit(mrow, b);
        const unsigned long long votes = __ballot(on);
        const int slot = at + __popcll(votes & ((1ull << lane) - 1ull));
        if (on && slot < list_entries(Ck) - (BN - 1)) {
          ent0[slot] = b;
          ent1[slot] = __float_as_int(log2f((float)sz));
        }
        at += __popcll(votes);
      }
    }
    at = min(at, list_entries(Ck) - (BN - 1));
    if (lane < BN - 1) ent1[at + lane] = __float_as_int(-INFINITY);  // the rest of the last tile
    if (lane == 0) slot_s[1] = at - comp0;
  }
}

// Row of K / V, or of the centroid tables, at position `at` of tile t; cur: the thread's segment cursor.
// Positions past the last key or centroid repeat it (their bias is -inf).
__device__ __forceinline__ int key_row(const int32_t* ent0, const int32_t* ent1, int comp0, int nt_r, int n_r, int n_c,
                                       int t, int at, int& cur) {
  if (t >= nt_r) return ent0[comp0 + min((t - nt_r) * BN + at, n_c - 1)];
  const int pos = min(t * BN + at, n_r - 1);
  while (pos >= ent0[cur + 1]) ++cur;
  return ent1[cur] + (pos - ent0[cur]);
}

// 16-byte chunk of a tile row r in LDS: chunk ^ swizzle
template <int D>
__device__ __forceinline__ int k_swz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D>
__device__ __forceinline__ int v_swz(int r) { return D == 128 ? ((r & 3) << 2) : ((r & 2) << 1); }

// Per-lane LDS byte offsets of the first MFMA operands. K row li of a 32-row block, dims 16s + 8lh .. +7:
// chunk (2s + lh) ^ swizzle
template <int D>
__device__ __forceinline__ int k_operand_offset(int li, int lh) { return li * (D * 2) + ((lh ^ k_swz<D>(li)) << 4); }
// V, transpose read: group = lane/16 -> (dim half, key half); r = lane%16
template <int D>
__device__ __forceinline__ int v_operand_offset(int lane) {
  const int r = lane & 15, g = lane >> 4, ddhalf = g & 1, khalf = g >> 1, row = 4 * khalf + (r >> 2);
  return row * (D * 2) + (((2 * ddhalf + ((r & 3) >> 1)) ^ v_swz<D>(row)) << 4) + (r & 1) * 8;
}

template <int D>
__device__ __forceinline__ void rescale_to(float m_new, float& m, float& l, f32x16 (&oacc)[D / 32]) {
  const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - m_new);
  l *= alpha;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
  m = m_new;
}

// One query row's output and log-sum-exp: the lane holds dims 32db + 8g + 4lh + 0..3
template <int D>
__device__ __forceinline__ void store_row(const AttnArgs& p, int bh, int qrow, int lh, const f32x16 (&oacc)[D / 32],
                                          float m, float lt) {
  const float inv = lt > 0.f ? 1.0f / lt : 0.f;
  int64_t lse_idx;
  bf16_t* o = static_cast<bf16_t*>(p.op) + out_row_offset(p, bh, qrow, D, lse_idx);
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint2 w;
      w.x = pack_bf16(oacc[db][4 * g] * inv, oacc[db][4 * g + 1] * inv);
      w.y = pack_bf16(oacc[db][4 * g + 2] * inv, oacc[db][4 * g + 3] * inv);
      *reinterpret_cast<uint2*>(o + 32 * db + 8 * g + 4 * lh) = w;
    }
  if (p.lse && lh == 0) p.lse[lse_idx] = (m + log2f(lt)) * kLn2;
}

// NW waves of 32 query rows (three per SIMD); NSTAGE K/V tile buffers. The first CW waves of
// the workgroup (the oldest wave of every SIMD, which finishes its step first) issue the tile
// copies, after their compute of the step (just before the tile barrier): measured faster
// than issuing them behind the score MFMAs or from more waves.
// WIDE: rows by 64-bit addresses instead of 32-bit byte offsets from the head's first one.
template <int D, int NW, int NSTAGE, int CW, bool WIDE>
__global__ void __launch_bounds__(64 * NW, 1)
attn_bf16_kernel(AttnArgs p) {
  static_assert(D == 64 || D == 128, "swizzles");
  constexpr int ROWB = D * 2;                       // bytes per K/V row
  constexpr int CPR = ROWB / 16;                    // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                     // rows per copy instruction
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int TILE_BYTES = BN * ROWB;
  constexpr int INST_PER_TILE = TILE_BYTES / 1024;  // wave-wide 1 KB copies per tensor tile
  constexpr int LOADS_PER_TILE = 2 * INST_PER_TILE / CW;  // copy instructions per copying wave per tile
  constexpr int RS = NSTAGE + 1;                    // row-map ring
  static_assert(INST_PER_TILE % CW == 0 && CW <= NW, "copies must split evenly over the copying waves");

  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  unsigned char* Ks = smem;                        // [NSTAGE][64 rows][ROWB], chunk-swizzled
  unsigned char* Vs = smem + NSTAGE * TILE_BYTES;  // [NSTAGE][64 rows][ROWB], chunk-swizzled
  int32_t* rowmap = reinterpret_cast<int32_t*>(smem + 2 * NSTAGE * TILE_BYTES);  // [RS][BN]
  float* rag_bias = reinterpret_cast<float*>(rowmap + RS * BN);  // [BN] bias of the ragged routed tile
  // the two tables of cluster_tables
  int32_t* ent0 = reinterpret_cast<int32_t*>(rag_bias + BN);
  int32_t* ent1 = ent0 + list_entries(p.Ck);
  int32_t* slot_s = ent1 + list_entries(p.Ck);  // claimed tile, number of compensated clusters

  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  if (tid == 0) claim_tile(p, 1, slot_s);
  __syncthreads();
  const int claimed = __builtin_amdgcn_readfirstlane(slot_s[0]);
  if (claimed < 0) return;
  const int bh = p.sched_bh[claimed], a = p.sched_a[claimed], row0 = p.sched_row0[claimed];
  const int Ck = p.Ck;
  const int row_end = p.sched_rend[claimed];  // the tile's rows are [row0, row_end), all of query cluster a
  const int32_t* rp = p.row_ptr + (int64_t)bh * (p.Cq + 2);
  const int ne = min(rp[a + 1] - rp[a], Ck + 1);
  const int comp0 = (ne + 1 + 3) & ~3;

  cluster_tables(p, bh, a, ne, comp0, wave, lane, ent0, ent1, slot_s);
  __syncthreads();
  // (part 2 leaves the routed keys out, part 1 the centroid tiles: the two-stage form)
  const int n_r = p.part == 2 ? 0 : __builtin_amdgcn_readfirstlane(ent0[ne]);  // wave-uniform
  const int n_c = p.part == 1 ? 0 : __builtin_amdgcn_readfirstlane(slot_s[1]);
  const int nt_r = (n_r + BN - 1) / BN;
  const int T = nt_r + (n_c + BN - 1) / BN;
  const int nt_full = n_r / BN;  // routed tiles with all 64 keys valid
  if (tid < BN) rag_bias[tid] = (nt_full * BN + tid < n_r) ? 0.f : -INFINITY;

  const bf16_t* kh = static_cast<const bf16_t*>(p.kp) + (int64_t)bh * p.Nk * D;
  const bf16_t* vh = static_cast<const bf16_t*>(p.vp) + (int64_t)bh * p.Nk * D;
  const bf16_t* kc = p.kbar16 + (int64_t)bh * Ck * D;
  const bf16_t* vc = p.vbar16 + (int64_t)bh * Ck * D;

  int cur = 0;  // segment cursor of threads 0..63 (virtual key position -> permuted row)
  auto map_tile = [&](int t) __attribute__((always_inline)) {
    if (tid < BN) rowmap[(t % RS) * BN + tid] = key_row(ent0, ent1, comp0, nt_r, n_r, n_c, t, tid, cur);
  };

  // one wave-wide copy moves rows RPI*inst .. of a tile; lane -> (row, LDS chunk slot).
  // Copy i of this wave is instruction inst = wave + i*CW of the tile: tile row cp_rr + RPI*i*CW,
  // a multiple of 16 rows further on, so the row's swizzle phases, and with them the 16-byte chunk
  // a lane fetches, are the same for every i.
  static_assert((RPI * CW) % 16 == 0, "copy rows of one lane must share their swizzle phase");
  constexpr int CPW = INST_PER_TILE / CW;  // copies per tensor per wave per tile
  const uint32_t lds_k0 = lds_address(Ks), lds_v0 = lds_address(Vs);
  const int cp_rr = RPI * (wave % CW) + lane / CPR;
  const uint32_t cp_koff = (uint32_t)(((lane % CPR) ^ k_swz<D>(cp_rr)) << 4);
  const uint32_t cp_voff = (uint32_t)(((lane % CPR) ^ v_swz<D>(cp_rr)) << 4);
  // permuted rows (of K/V or of the centroid tables) this lane copies for tile t
  auto fetch_rows = [&](int t, int (&rows)[CPW]) __attribute__((always_inline)) {
    const int32_t* rm = rowmap + (t % RS) * BN + cp_rr;
#pragma unroll
    for (int i = 0; i < CPW; ++i) rows[i] = rm[RPI * i * CW];
  };
  auto issue_copies = [&](int t) __attribute__((always_inline)) {
    if (CW < NW && wave >= CW) return;
    int rows[CPW];
    fetch_rows(t, rows);
    const void* kb = uniform_ptr(t < nt_r ? kh : kc);
    const void* vb = uniform_ptr(t < nt_r ? vh : vc);
    const uint32_t kdst = lds_k0 + (t % NSTAGE) * TILE_BYTES + wave * 1024;
    const uint32_t vdst = lds_v0 + (t % NSTAGE) * TILE_BYTES + wave * 1024;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const uint32_t k_lds = __builtin_amdgcn_readfirstlane(kdst + i * CW * 1024);
      const uint32_t v_lds = __builtin_amdgcn_readfirstlane(vdst + i * CW * 1024);
      if constexpr (WIDE) {
        const int64_t rowoff = (int64_t)rows[i] * ROWB;
        async_copy_16B(static_cast<const unsigned char*>(kb) + rowoff + cp_koff, k_lds);
        async_copy_16B(static_cast<const unsigned char*>(vb) + rowoff + cp_voff, v_lds);
      } else {
        const uint32_t rowoff = (uint32_t)rows[i] * ROWB;
        async_copy_16B(kb, rowoff + cp_koff, k_lds);
        async_copy_16B(vb, rowoff + cp_voff, v_lds);
      }
    }
  };

  // (the swizzles are XORs of disjoint bit fields, so operand s / block db is the offset of
  // operand 0 with s << 5 / db << 6 XORed in: one register each instead of a table)
  const int koff0 = k_operand_offset<D>(li, lh), voff0 = v_operand_offset<D>(lane);
  auto koff = [&](int s) { return koff0 ^ (s << 5); };
  auto voff = [&](int db) { return voff0 ^ (db << 6); };

  const bool wave_active = (row0 + 32 * wave) < row_end;
  bf16x8 bq[KS];
  {
    const int qrow = row0 + 32 * wave + li;
    const bf16_t* qr = static_cast<const bf16_t*>(p.qp) + q_row_offset(p, bh, qrow < row_end ? qrow : row_end - 1, D);
#pragma unroll
    for (int s = 0; s < KS; ++s) bq[s] = as_bf16x8(*reinterpret_cast<const uint4*>(qr + 16 * s + 8 * lh));
  }
  // Q must be in registers before the asynchronous tile copies start: the compiler does not
  // see those copies and would otherwise wait for "its" loads inside the main loop
  SVGEAR_WAIT_VMCNT(0);

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m = -INFINITY, l = 0.f;
  const float c = p.scale * kLog2e;

  auto rescale = [&](float m_new) __attribute__((always_inline)) { rescale_to<D>(m_new, m, l, oacc); };

  // ---- S^T = K Q^T of tile t: 64 keys x 32 queries; register r of block kb is key
  // 32kb + 8(r/4) + 4lh + r%4, query li. The scores of tile t+1 are computed at the end of
  // pipeline step t (see below), so they live in registers across the tile barrier.
  f32x16 sacc[2];
  auto scores = [&](int t) __attribute__((always_inline)) {
    const unsigned char* Kb = Ks + (t % NSTAGE) * TILE_BYTES;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[kb][r] = 0.f;
    // the two 32-key blocks alternate so that consecutive MFMAs are independent; operand
    // reads run four fragments ahead of the MFMAs that consume them
    bf16x8 ak[2 * KS];
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i)
      ak[i] = as_bf16x8(*reinterpret_cast<const uint4*>(Kb + (i & 1) * 32 * ROWB + koff(i >> 1)));
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i)
      sacc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak[i], bq[i >> 1], sacc[i & 1], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < 2 * KS - 4; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  };

  // ---- online softmax of tile t in the base-2 domain, from its scores in sacc to the packed
  // bf16 probabilities pk; the running maximum m is refreshed lazily (only when a score
  // exceeds it by more than kLazyRescale), so O is rarely rescaled. BIASED = false: a full
  // routed tile. BIASED = true: per-key additive bias (ragged routed tile: 0 / -inf;
  // compensation tile: log2|k_b| or -inf).
  uint32_t pk[2][8];
  auto softmax = [&](int t, auto biased_tag) __attribute__((always_inline)) {
    constexpr bool BIASED = decltype(biased_tag)::value;
    float ls[4] = {0.f, 0.f, 0.f, 0.f};  // row sums, four independent parts (see kSumRounded)
    if constexpr (!BIASED) {
      // four independent max chains (a single chain of 16 dependent ops stalls the wave)
      float mxa = fmaxf(sacc[0][0], sacc[1][0]), mxb = fmaxf(sacc[0][1], sacc[1][1]);
      float mxc = fmaxf(sacc[0][2], sacc[1][2]), mxd = fmaxf(sacc[0][3], sacc[1][3]);
#pragma unroll
      for (int r = 4; r < 16; r += 4) {
        mxa = fmaxf(fmaxf(mxa, sacc[0][r]), sacc[1][r]);
        mxb = fmaxf(fmaxf(mxb, sacc[0][r + 1]), sacc[1][r + 1]);
        mxc = fmaxf(fmaxf(mxc, sacc[0][r + 2]), sacc[1][r + 2]);
        mxd = fmaxf(fmaxf(mxd, sacc[0][r + 3]), sacc[1][r + 3]);
      }
      float mx = fmaxf(fmaxf(mxa, mxb), fmaxf(mxc, mxd));
      mx = fmaxf(mx, swap32(mx));
      const float ms = mx * c;
      if (__any(ms > m + kLazyRescale<D>)) rescale(fmaxf(m, ms));
      const float neg_m = m == -INFINITY ? 0.f : -m;  // (every score so far -inf: weights of 0, not NaN)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][r], c, neg_m));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][r + 1], c, neg_m));
          if constexpr (!kSumRounded<D>) ls[(r >> 1) & 3] += p0 + p1;
          pk[kb][r >> 1] = pack_bf16(p0, p1);
        }
    } else {
      const float* lwt = t < nt_r ? rag_bias : reinterpret_cast<const float*>(ent1) + comp0 + (t - nt_r) * BN;
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 bias = *reinterpret_cast<const float4*>(lwt + 32 * kb + 8 * g + 4 * lh);
          sacc[kb][4 * g + 0] = __builtin_fmaf(sacc[kb][4 * g + 0], c, bias.x);
          sacc[kb][4 * g + 1] = __builtin_fmaf(sacc[kb][4 * g + 1], c, bias.y);
          sacc[kb][4 * g + 2] = __builtin_fmaf(sacc[kb][4 * g + 2], c, bias.z);
          sacc[kb][4 * g + 3] = __builtin_fmaf(sacc[kb][4 * g + 3], c, bias.w);
#pragma unroll
          for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sacc[kb][4 * g + r]);
        }
      mx = fmaxf(mx, swap32(mx));
      if (__any(mx > m + kLazyRescale<D>)) rescale(fmaxf(m, mx));
      const float m_use = (m == -INFINITY) ? 0.f : m;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const float p0 = __builtin_amdgcn_exp2f(sacc[kb][r] - m_use);
          const float p1 = __builtin_amdgcn_exp2f(sacc[kb][r + 1] - m_use);
          if constexpr (!kSumRounded<D>) ls[(r >> 1) & 3] += p0 + p1;
          pk[kb][r >> 1] = pack_bf16(p0, p1);
        }
    }
    if constexpr (kSumRounded<D>) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int u = 0; u < 8; ++u) ls[u & 3] = dot2_ones(pk[kb][u], ls[u & 3]);
    }
    l += (ls[0] + ls[1]) + (ls[2] + ls[3]);
  };
  // ---- O^T += V^T P^T of tile t: k-step ks covers keys 16ks .. 16ks+15; the transpose reads
  // of k-step ks+1 are issued before the MFMAs of k-step ks
  auto pv = [&](int t) __attribute__((always_inline)) {
    const unsigned char* Vb = Vs + (t % NSTAGE) * TILE_BYTES;
    {
      bf16x8 av[4][DB];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int db = 0; db < DB; ++db) av[ks][db] = tr_pair<ROWB>(Vb, ks * 16 * ROWB + voff(db));
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int kb = ks >> 1, u4 = (ks & 1) * 4;
        const bf16x8 bp = as_bf16x8(make_uint4(pk[kb][u4], pk[kb][u4 + 1], pk[kb][u4 + 2], pk[kb][u4 + 3]));
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[ks][db], bp, oacc[db], 0, 0, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, 2 * DB, 1);  // reads of k-step 0
#pragma unroll
      for (int ks = 0; ks < 3; ++ks)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);  // MFMA (ks, db)
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);  // the two reads of operand (ks+1, db)
        }
      __builtin_amdgcn_sched_group_barrier(0x008, DB, 1);
    }
  };

  // Pipeline step t (between two workgroup barriers). The three waves of a SIMD (wave / 4 =
  // phase group) run the same three phases per step - scores, softmax, PV - but each group
  // starts at a different one, so that while one wave is in its softmax (vector ALU) the other
  // two have matrix work queued:
  //   group 0:  S(t)   softmax(t)  PV(t)
  //   group 1:  softmax(t)  PV(t)  S(t+1)            (prologue: S(0))
  //   group 2:  PV(t)  S(t+1)  softmax(t+1)          (prologue: S(0), softmax(0))
  // (of the six ways to give the three orders to the oldest, middle and youngest wave of a
  // SIMD this one measured fastest, the others 3-6 % slower)
  // Step t therefore reads K(t), K(t+1) and V(t): both must have landed before it starts, and
  // the buffers of tile t are free after its barrier; the copies of tile t+NSTAGE-1 are
  // issued during step t.
  static_assert(NW == 12, "three phase groups of four waves");
  const int group = wave >> 2;
  auto run_step = [&](int t, auto group_tag, auto biased_tag) __attribute__((always_inline)) {
    constexpr int G = decltype(group_tag)::value;
    const bool more = t + NSTAGE - 1 < T;
    if (wave_active) {
      if constexpr (G == 0) {
        scores(t);
        softmax(t, biased_tag);
        pv(t);
      } else if constexpr (G == 1) {
        softmax(t, biased_tag);
        pv(t);
        __builtin_amdgcn_sched_barrier(0);  // keep the two MFMA pipelines in separate scheduling regions
        // (unconditional, so the old and the new scores never have to be live together: the
        // last step recomputes its own tile's scores, which nobody reads)
        scores(t + 1 < T ? t + 1 : t);
      } else {
        pv(t);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < T) {
          scores(t + 1);
          softmax(t + 1, biased_tag);
        } else {
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int u = 0; u < 8; ++u) pk[kb][u] = 0u;
        }
      }
    }
    if (more) issue_copies(t + NSTAGE - 1);
    if (t + NSTAGE < T) map_tile(t + NSTAGE);
    // this wave's copies of tile t+2 must have landed (step t+1 reads K(t+2)); one younger
    // tile may stay in flight
    if (more) SVGEAR_WAIT_VMCNT((NSTAGE - 3) * LOADS_PER_TILE);
    else SVGEAR_WAIT_VMCNT(0);
    __syncthreads();
  };

  // prologue: tiles 0 .. NSTAGE-2 in flight, tiles 0 and 1 landed
#pragma unroll
  for (int t = 0; t < NSTAGE; ++t)
    if (t < T) map_tile(t);
  __syncthreads();
#pragma unroll
  for (int t = 0; t < NSTAGE - 1; ++t)
    if (t < T) issue_copies(t);
  if (T >= NSTAGE - 1) SVGEAR_WAIT_VMCNT((NSTAGE - 3) * LOADS_PER_TILE);
  else SVGEAR_WAIT_VMCNT(0);
  __syncthreads();

  // Every group runs T steps (T barriers). The bias tag belongs to the tile whose softmax the
  // step contains: tile t for groups 0 and 1, tile t+1 for group 2.
  if (group == 0) {
    for (int t = 0; t < nt_full; ++t) run_step(t, std::integral_constant<int, 0>{}, std::false_type{});
    for (int t = nt_full; t < T; ++t) run_step(t, std::integral_constant<int, 0>{}, std::true_type{});
  } else if (group == 1) {
    if (wave_active && T > 0) scores(0);
    for (int t = 0; t < nt_full; ++t) run_step(t, std::integral_constant<int, 1>{}, std::false_type{});
    for (int t = nt_full; t < T; ++t) run_step(t, std::integral_constant<int, 1>{}, std::true_type{});
  } else {
    if (wave_active && T > 0) {
      scores(0);
      if (nt_full > 0) softmax(0, std::false_type{});
      else softmax(0, std::true_type{});
    }
    int t = 0;
    for (; t + 1 < nt_full; ++t) run_step(t, std::integral_constant<int, 2>{}, std::false_type{});
    for (; t < T; ++t) run_step(t, std::integral_constant<int, 2>{}, std::true_type{});
  }

  // ---- epilogue: lane holds query li, dims 32db + 8g + 4lh + 0..3
  if (wave_active) {
    const float lt = l + swap32(l);
    const int qrow = row0 + 32 * wave + li;
    if (qrow < row_end) {
      store_row<D>(p, bh, qrow, lh, oacc, m, lt);
    }
  }
}

// ---- 128-row tiles, two workgroups per CU
// The 12-wave kernel keeps a CU to itself: a tile pays its start (a chain of a dozen fetches, some 20 us
// with the first copies) and its end alone, a cluster of a few dozen rows leaves most of its waves
// idle, and a head or two of a few thousand rows have fewer tiles of 384 rows than the chip has CUs.
// Here a workgroup is four waves (one per SIMD) over 128 rows with two K and two V buffers (64 KB at
// d = 128), so that two of them share a CU and one's start overlaps the other's steps; a wave overlaps
// its own phases (the exponentials of tile t between the MFMAs of S(t + 1), the maximum of tile t + 1
// between those of PV(t)), and where even these tiles are few the keys of a tile are dealt to several
// workgroups (partial rows in fp32, merged in a fixed order). The choice between the two kernels is
// made in bf16_form.
constexpr int kQuadWaves = 4;

template <int D, bool WIDE>
__global__ void __launch_bounds__(64 * kQuadWaves, 2)
attn_bf16_quad_kernel(AttnArgs p) {
  constexpr int NW = kQuadWaves, NSTAGE = 2, CW = kQuadWaves;
  static_assert(D == 64 || D == 128, "swizzles");
  constexpr int ROWB = D * 2;                       // bytes per K/V row
  constexpr int CPR = ROWB / 16;                    // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                     // rows per copy instruction
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int TILE_BYTES = BN * ROWB;
  constexpr int INST_PER_TILE = TILE_BYTES / 1024;  // wave-wide 1 KB copies per tensor tile
  constexpr int RS = 4;                             // row-map ring
  static_assert(INST_PER_TILE % CW == 0 && CW <= NW, "copies must split evenly over the copying waves");

  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
  unsigned char* Ks = smem;                        // [NSTAGE][64 rows][ROWB], chunk-swizzled
  unsigned char* Vs = smem + NSTAGE * TILE_BYTES;  // [NSTAGE][64 rows][ROWB], chunk-swizzled
  int32_t* rowmap = reinterpret_cast<int32_t*>(smem + 2 * NSTAGE * TILE_BYTES);  // [RS][BN]
  float* rag_bias = reinterpret_cast<float*>(rowmap + RS * BN);  // [BN] bias of the ragged routed tile
  // the two tables of cluster_tables
  int32_t* ent0 = reinterpret_cast<int32_t*>(rag_bias + BN);
  int32_t* ent1 = ent0 + list_entries(p.Ck);
  int32_t* slot_s = ent1 + list_entries(p.Ck);  // claimed tile, number of compensated clusters

  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int splits = p.splits;
  if (tid == 0) claim_tile(p, splits, slot_s);
  __syncthreads();
  const int claimed = __builtin_amdgcn_readfirstlane(slot_s[0]);
  if (claimed < 0) return;
  const int split = __builtin_amdgcn_readfirstlane(slot_s[2]);
  const int bh = p.sched_bh[claimed], a = p.sched_a[claimed], row0 = p.sched_row0[claimed];
  const int Ck = p.Ck;
  const int row_end = p.sched_rend[claimed];  // the tile's rows are [row0, row_end), all of query cluster a
  const int32_t* rp = p.row_ptr + (int64_t)bh * (p.Cq + 2);
  const int ne = min(rp[a + 1] - rp[a], Ck + 1);
  const int comp0 = (ne + 1 + 3) & ~3;

  cluster_tables(p, bh, a, ne, comp0, wave, lane, ent0, ent1, slot_s);
  __syncthreads();
  // (part 2 leaves the routed keys out, part 1 the centroid tiles: the two-stage form)
  const int n_r = p.part == 2 ? 0 : __builtin_amdgcn_readfirstlane(ent0[ne]);  // wave-uniform
  const int n_c = p.part == 1 ? 0 : __builtin_amdgcn_readfirstlane(slot_s[1]);
  const int nt_r = (n_r + BN - 1) / BN;
  const int T_all = nt_r + (n_c + BN - 1) / BN;
  // this workgroup's tiles: [t_lo, T)
  const int t_lo = (int)((int64_t)T_all * split / splits), T = (int)((int64_t)T_all * (split + 1) / splits);
  const int nt_full = n_r / BN;  // routed tiles with all 64 keys valid
  if (tid < BN) rag_bias[tid] = (nt_full * BN + tid < n_r) ? 0.f : -INFINITY;

  const bf16_t* kh = static_cast<const bf16_t*>(p.kp) + (int64_t)bh * p.Nk * D;
  const bf16_t* vh = static_cast<const bf16_t*>(p.vp) + (int64_t)bh * p.Nk * D;
  const bf16_t* kc = p.kbar16 + (int64_t)bh * Ck * D;
  const bf16_t* vc = p.vbar16 + (int64_t)bh * Ck * D;

  // segment cursor of threads 0..63 (virtual key position -> permuted row): the last cluster that starts
  // at or before the thread's first position
  int cur = 0;
  for (int hi = ne, pos = min(t_lo * BN + (tid & 63), n_r - 1); hi - cur > 1;) {
    const int mid = (cur + hi) >> 1;
    if (ent0[mid] <= pos) cur = mid;
    else hi = mid;
  }
  auto map_tile = [&](int t) __attribute__((always_inline)) {
    if (tid < BN) rowmap[(t % RS) * BN + tid] = key_row(ent0, ent1, comp0, nt_r, n_r, n_c, t, tid, cur);
  };

  // one wave-wide copy moves rows RPI*inst .. of a tile; lane -> (row, LDS chunk slot).
  // Copy i of this wave is instruction inst = wave + i*CW of the tile: tile row cp_rr + RPI*i*CW,
  // a multiple of 16 rows further on, so the row's swizzle phases, and with them the 16-byte chunk
  // a lane fetches, are the same for every i.
  static_assert((RPI * CW) % 16 == 0, "copy rows of one lane must share their swizzle phase");
  constexpr int CPW = INST_PER_TILE / CW;  // copies per tensor per wave per tile
  const uint32_t lds_k0 = lds_address(Ks), lds_v0 = lds_address(Vs);
  const int cp_rr = RPI * (wave % CW) + lane / CPR;
  const uint32_t cp_koff = (uint32_t)(((lane % CPR) ^ k_swz<D>(cp_rr)) << 4);
  const uint32_t cp_voff = (uint32_t)(((lane % CPR) ^ v_swz<D>(cp_rr)) << 4);
  // permuted rows (of K/V or of the centroid tables) this lane copies for tile t
  auto fetch_rows = [&](int t, int (&rows)[CPW]) __attribute__((always_inline)) {
    const int32_t* rm = rowmap + (t % RS) * BN + cp_rr;
#pragma unroll
    for (int i = 0; i < CPW; ++i) rows[i] = rm[RPI * i * CW];
  };
  auto issue = [&](int t, bool is_k) __attribute__((always_inline)) {
    int rows[CPW];
    fetch_rows(t, rows);
    const void* base = uniform_ptr(is_k ? (t < nt_r ? kh : kc) : (t < nt_r ? vh : vc));
    const uint32_t dst = (is_k ? lds_k0 : lds_v0) + (t % NSTAGE) * TILE_BYTES + wave * 1024;
    const uint32_t off = is_k ? cp_koff : cp_voff;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
      const uint32_t l = __builtin_amdgcn_readfirstlane(dst + i * CW * 1024);
      if constexpr (WIDE) async_copy_16B(static_cast<const unsigned char*>(base) + (int64_t)rows[i] * ROWB + off, l);
      else async_copy_16B(base, (uint32_t)rows[i] * ROWB + off, l);
    }
  };

  // (the swizzles are XORs of disjoint bit fields, so operand s / block db is the offset of
  // operand 0 with s << 5 / db << 6 XORed in: one register each instead of a table)
  const int koff0 = k_operand_offset<D>(li, lh), voff0 = v_operand_offset<D>(lane);
  auto koff = [&](int s) { return koff0 ^ (s << 5); };
  auto voff = [&](int db) { return voff0 ^ (db << 6); };

  // (the blocks of a partly filled tile rotate over the SIMDs with the tile)
  const int my_row0 = row0 + 32 * ((wave + claimed) & (NW - 1));
  const bool wave_active = my_row0 < row_end;
  bf16x8 bq[KS];
  {
    const int qrow = my_row0 + li;
    const bf16_t* qr = static_cast<const bf16_t*>(p.qp) + q_row_offset(p, bh, qrow < row_end ? qrow : row_end - 1, D);
#pragma unroll
    for (int s = 0; s < KS; ++s) bq[s] = as_bf16x8(*reinterpret_cast<const uint4*>(qr + 16 * s + 8 * lh));
  }
  // Q must be in registers before the asynchronous tile copies start: the compiler does not
  // see those copies and would otherwise wait for "its" loads inside the main loop
  SVGEAR_WAIT_VMCNT(0);

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m = -INFINITY, l = 0.f;
  const float c = p.scale * kLog2e;

  auto rescale = [&](float m_new) __attribute__((always_inline)) { rescale_to<D>(m_new, m, l, oacc); };

  f32x16 sA[2], sB[2];
  uint32_t pk[2][8];
  float cc = c;  // factor still to be applied to the scores whose maximum is known
  constexpr int AHEAD = 4;
  // S^T = K Q^T of tile t into sn (registers as above); with EXPS, between its MFMAs, the
  // probabilities of the tile whose scores are sc (running maximum m) into pk
  auto scores = [&](int t, f32x16 (&sn)[2], const f32x16 (&sc)[2], auto exps_tag) __attribute__((always_inline)) {
    constexpr bool EXPS = decltype(exps_tag)::value;
    const unsigned char* Kb = Ks + (t % NSTAGE) * TILE_BYTES;
    bf16x8 kf[2 * KS];
    auto rd = [&](int i) { kf[i] = as_bf16x8(*reinterpret_cast<const uint4*>(Kb + (i & 1) * 32 * ROWB + koff(i >> 1))); };
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sn[kb][r] = 0.f;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) rd(i);
    const float neg_m = m == -INFINITY ? 0.f : -m;
    float ls[4] = {0.f, 0.f, 0.f, 0.f};
    constexpr int E = 16 / (2 * KS);  // pairs of scores per MFMA
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + AHEAD < 2 * KS) rd(i + AHEAD);
      sn[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], bq[i >> 1], sn[i & 1], 0, 0, 0);
      if constexpr (EXPS) {
#pragma unroll
        for (int e = i * E; e < (i + 1) * E; ++e) {
          const int kb = e >> 3, r = 2 * (e & 7);
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kb][r], cc, neg_m));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kb][r + 1], cc, neg_m));
          pk[kb][r >> 1] = pack_bf16(p0, p1);
          if constexpr (kSumRounded<D>) ls[e & 3] = dot2_ones(pk[kb][r >> 1], ls[e & 3]);
          else ls[e & 3] += p0 + p1;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EXPS) l += (ls[0] + ls[1]) + (ls[2] + ls[3]);
  };
  auto max_pair = [&](const f32x16 (&sn)[2], float& mx, int e) __attribute__((always_inline)) {
    const int kb = e >> 3, r = 2 * (e & 7);
    mx = fmaxf(fmaxf(mx, sn[kb][r]), sn[kb][r + 1]);
  };
  // the running maximum covers tile t's scores sn afterwards; a ragged or centroid tile gets its biases
  auto settle = [&](int t, f32x16 (&sn)[2], float mx) __attribute__((always_inline)) {
    cc = c;
    if (t >= nt_full) {
      const float* lwt = t < nt_r ? rag_bias : reinterpret_cast<const float*>(ent1) + comp0 + (t - nt_r) * BN;
      mx = -INFINITY;
      cc = 1.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 bias = *reinterpret_cast<const float4*>(lwt + 32 * kb + 8 * g + 4 * lh);
          sn[kb][4 * g + 0] = __builtin_fmaf(sn[kb][4 * g + 0], c, bias.x);
          sn[kb][4 * g + 1] = __builtin_fmaf(sn[kb][4 * g + 1], c, bias.y);
          sn[kb][4 * g + 2] = __builtin_fmaf(sn[kb][4 * g + 2], c, bias.z);
          sn[kb][4 * g + 3] = __builtin_fmaf(sn[kb][4 * g + 3], c, bias.w);
#pragma unroll
          for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sn[kb][4 * g + r]);
        }
    }
    mx = fmaxf(mx, swap32(mx));
    const float ms = mx * cc;
    if (__any(ms > m + kLazyRescale<D>)) rescale(fmaxf(m, ms));
  };
  // O^T += V^T P^T of tile t, and between its MFMAs the maximum of the scores sn of tile t + 1
  auto values = [&](int t, f32x16 (&sn)[2]) __attribute__((always_inline)) {
    const unsigned char* Vb = Vs + (t % NSTAGE) * TILE_BYTES;
    constexpr int N = 4 * DB;
    bf16x8 vf[N];
    auto rd = [&](int i) { vf[i] = tr_pair<ROWB>(Vb, (i / DB) * 16 * ROWB + voff(i % DB)); };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) rd(i);
    float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int i = 0; i < N; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + AHEAD < N) rd(i + AHEAD);
      const int ks = i / DB, kb = ks >> 1, u4 = (ks & 1) * 4;
      const bf16x8 bp = as_bf16x8(make_uint4(pk[kb][u4], pk[kb][u4 + 1], pk[kb][u4 + 2], pk[kb][u4 + 3]));
      oacc[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i], bp, oacc[i % DB], 0, 0, 0);
      if (i >= N / 4) {
#pragma unroll
        for (int e = (i - N / 4) * 16 / (3 * N / 4); e < (i + 1 - N / 4) * 16 / (3 * N / 4); ++e)
          max_pair(sn, mx[e & 3], e);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (t + 1 < T) settle(t + 1, sn, fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])));
  };

  // Step t reads K(t + 1) and V(t) and copies K(t + 2) and V(t + 1), over K(t) and V(t - 1), which step
  // t - 1 was the last to read.
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (t_lo + u < T) map_tile(t_lo + u);
  __syncthreads();
  if (t_lo < T) {
    issue(t_lo, true);
    issue(t_lo, false);
    if (t_lo + 1 < T) issue(t_lo + 1, true);
  }
  SVGEAR_WAIT_VMCNT(0);
  __syncthreads();
  if (wave_active && t_lo < T) {
    scores(t_lo, sA, sB, std::false_type{});
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) max_pair(sA, mx, e);
    settle(t_lo, sA, mx);
  }
  __syncthreads();  // everyone is done with the first K tile before it is copied over
  auto step = [&](int t, f32x16 (&now)[2], f32x16 (&next)[2]) __attribute__((always_inline)) {
    if (t + 2 < T) issue(t + 2, true);
    if (t + 1 < T) issue(t + 1, false);
    if (wave_active) {
      scores(t + 1 < T ? t + 1 : t, next, now, std::true_type{});  // (the last step's scores are not used)
      values(t, next);
    }
    if (t + 3 < T) map_tile(t + 3);
    SVGEAR_WAIT_VMCNT(0);
    __syncthreads();
  };
  for (int t = t_lo; t < T; t += 2) {
    step(t, sA, sB);
    if (t + 1 < T) step(t + 1, sB, sA);
  }

  // ---- epilogue: lane holds query li, dims 32db + 8g + 4lh + 0..3
  if (wave_active) {
    const float lt = l + swap32(l);
    const int qrow = my_row0 + li;
    if (qrow < row_end && splits > 1) {
      const int64_t rows = (int64_t)p.BH * p.Nq, at = split * rows + (int64_t)bh * p.Nq + qrow;
      if (lh == 0) p.part_ml[at] = make_float2(m, lt);
      float* o = p.part_o + at * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4*>(o + 32 * db + 8 * g + 4 * lh) =
              make_float4(oacc[db][4 * g], oacc[db][4 * g + 1], oacc[db][4 * g + 2], oacc[db][4 * g + 3]);
    } else if (qrow < row_end) {
      store_row<D>(p, bh, qrow, lh, oacc, m, lt);
    }
  }
}

// Adds the splits of every row, in split order: one thread per 8 dims.
template <int D>
__global__ void __launch_bounds__(256)
merge_splits_kernel(AttnArgs p) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t rows = (int64_t)p.BH * p.Nq, row = u / (D / 8);
  if (row >= rows) return;
  const int dim = 8 * (int)(u % (D / 8));
  float M = -INFINITY;
  for (int s = 0; s < p.splits; ++s) M = fmaxf(M, p.part_ml[s * rows + row].x);
  float l = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < p.splits; ++s) {
    const float2 ml = p.part_ml[s * rows + row];
    if (ml.x == -INFINITY && ml.y == 0.f) continue;  // no key there
    const float w = __builtin_amdgcn_exp2f(ml.x - M);
    const float* o = p.part_o + (s * rows + row) * D + dim;
    const float4 v0 = *reinterpret_cast<const float4*>(o), v1 = *reinterpret_cast<const float4*>(o + 4);
    const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    l = __builtin_fmaf(w, ml.y, l);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = __builtin_fmaf(w, v[i], acc[i]);
  }
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  int64_t lse_idx;
  const int bh = (int)(row / p.Nq);
  bf16_t* o = static_cast<bf16_t*>(p.op) + out_row_offset(p, bh, row - (int64_t)bh * p.Nq, D, lse_idx) + dim;
  uint4 w;
  w.x = pack_bf16(acc[0] * inv, acc[1] * inv);
  w.y = pack_bf16(acc[2] * inv, acc[3] * inv);
  w.z = pack_bf16(acc[4] * inv, acc[5] * inv);
  w.w = pack_bf16(acc[6] * inv, acc[7] * inv);
  *reinterpret_cast<uint4*>(o) = w;
  if (p.lse && dim == 0) p.lse[lse_idx] = (M + log2f(l)) * kLn2;
}

// ------------------------------------------------------------------------ work lists
// Item = (head, query cluster); its tiles all run T = #routed key tiles + #centroid tiles
// pipeline steps (the latter counted here as if no cluster were routed: the order alone depends on it). Items are ranked by T, longest first (ties by index), and dealt to the 8
// lists in boustrophedon order, which keeps the lists' totals close; inside a list the
// longest come first, so a list's tail consists of its shortest tiles.
// Steps and tiles of item (bh, a), by a whole wave, its lanes over the routed key clusters.
__device__ __forceinline__ void plan_item(const int32_t* q_offsets, const int32_t* k_offsets, const int32_t* row_ptr,
                                          const int32_t* col_idx, int bh, int a, int Cq, int Ck, int BM, int32_t& T,
                                          int32_t& nt) {
  const int R = Cq + 1, Cc = Ck + 1, lane = threadIdx.x & 63;
  const int32_t* qo = q_offsets + (int64_t)bh * (Cq + 2);
  const int32_t* ko = k_offsets + (int64_t)bh * (Ck + 2);
  const int32_t* rp = row_ptr + (int64_t)bh * (R + 1);
  const int n = qo[a + 1] - qo[a];
  const int32_t* ci = col_idx + (int64_t)bh * R * Cc + rp[a];
  const int ne = rp[a + 1] - rp[a];
  int64_t nr = 0;
  for (int e = lane; e < ne; e += 64) {
    const int b = ci[e];
    const int sz = ko[b + 1] - ko[b];
    nr += sz > 0 ? sz : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) nr += __shfl_xor(nr, o);
  if (lane == 0) {
    const int tiles = n > 0 ? (n + BM - 1) / BM : 0;
    nt = tiles;
    T = tiles > 0 ? (int)((nr + BN - 1) / BN) + (a < Cq ? (Ck + BN - 1) / BN : 0) : 0;
  }
}

// The centroid tables in bf16: a block of a planning kernel per blockDim.x elements of each.
__device__ __forceinline__ void centroids_to_bf16(unsigned block, const float* kbar, const float* vbar, int64_t n,
                                                  bf16_t* kbar16, bf16_t* vbar16) {
  const int64_t i = (int64_t)block * blockDim.x + threadIdx.x;
  if (i >= n) return;
  kbar16[i] = f32_to_bf16(kbar[i]);
  vbar16[i] = f32_to_bf16(vbar[i]);
}

// A wave per item over the whole grid (one workgroup per head took 173 us for 5 heads of 300 clusters,
// this grid 10); the blocks after the item_blocks first ones convert the centroids, a launch less.
__global__ void __launch_bounds__(256)
plan_items_kernel(const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ k_offsets,
                  const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int M, int Cq, int Ck, int BM,
                  int32_t* __restrict__ item_T, int32_t* __restrict__ item_nt, const float* __restrict__ kbar,
                  const float* __restrict__ vbar, int64_t n, bf16_t* __restrict__ kbar16, bf16_t* __restrict__ vbar16) {
  const unsigned item_blocks = (unsigned)(M + 3) / 4;
  if (blockIdx.x >= item_blocks) return centroids_to_bf16(blockIdx.x - item_blocks, kbar, vbar, n, kbar16, vbar16);
  const int i = 4 * blockIdx.x + (threadIdx.x >> 6), R = Cq + 1;
  if (i < M) plan_item(q_offsets, k_offsets, row_ptr, col_idx, i / R, i % R, Cq, Ck, BM, item_T[i], item_nt[i]);
}

// Rank of every item by (T descending, index ascending), by counting: a workgroup ranks 64 items,
// each of its four waves counting over a quarter of all items.
constexpr int kRankItems = 64;
__global__ void __launch_bounds__(256)
plan_rank_kernel(const int32_t* __restrict__ item_T, int M, int32_t* __restrict__ by_rank) {
  __shared__ uint64_t keys[4][64];
  __shared__ int rank_sum[kRankItems];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * kRankItems + lane;
  // larger key = earlier: T descending, then index ascending
  auto key_of = [&](int j) {
    return j < M ? ((uint64_t)(uint32_t)item_T[j] << 32) | (uint32_t)(0x7fffffff - j) : (uint64_t)0;
  };
  const uint64_t mine = key_of(i);
  if (threadIdx.x < kRankItems) rank_sum[threadIdx.x] = 0;
  __syncthreads();
  const int quarter = (M + 3) / 4;
  const int j_lo = wave * quarter, j_hi = min(j_lo + quarter, M);
  int rank = 0;
  for (int j0 = j_lo; j0 < j_hi; j0 += 64) {  // the wave's own tile of keys: no workgroup barrier needed
    keys[wave][lane] = j0 + lane < j_hi ? key_of(j0 + lane) : (uint64_t)0;
    __builtin_amdgcn_wave_barrier();
    const int lim = min(64, j_hi - j0);
    for (int u = 0; u < lim; ++u) rank += keys[wave][u] > mine;
    __builtin_amdgcn_wave_barrier();
  }
  atomicAdd(&rank_sum[lane], rank);
  __syncthreads();
  if (wave == 0 && i < M) by_rank[rank_sum[lane]] = i;
}

// rank r -> (list, position): round r/8 deals one item to every list, odd rounds in reverse
__device__ __forceinline__ int list_of_rank(int r) { return ((r >> 3) & 1) ? 7 - (r & 7) : (r & 7); }

// The lists from the ranked items (one workgroup of 1024).
__device__ __forceinline__ void write_lists(const int32_t* q_offsets, const int32_t* item_nt, const int32_t* by_rank,
                                            int M, int Cq, int32_t* rank_off, int32_t* sched_bh,
                                            int32_t* sched_a, int32_t* sched_row0, int32_t* sched_rend,
                                            int32_t* sched_x) {
  __shared__ int32_t total[8], first[8];
  const int tid = threadIdx.x, R = Cq + 1, lane = tid & 63, wave = tid >> 6;
  const int rounds = (M + 7) / 8;
  // exclusive offsets of every item inside its list (list xl = ranks 8k + pos(k, xl)): a wave per
  // list, four items per lane and step (one list after the other with the whole workgroup and its
  // barriers took 17 us at 22 items and 76 us at 9,624; this way 4 and 56,
  // most of it the expansion below)
  if (wave < 8) {
    const int xl = wave;
    int carry = 0;
    for (int k0 = 0; k0 < rounds; k0 += 256) {
      int r[4], v[4], sum = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + 4 * lane + u;
        r[u] = 8 * k + ((k & 1) ? 7 - xl : xl);
        v[u] = (k < rounds && r[u] < M) ? by_rank[r[u]] : -1;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = v[u] >= 0 ? item_nt[v[u]] : 0;
        sum += v[u];
      }
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      int at = carry + incl - sum;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k0 + 4 * lane + u < rounds && r[u] < M) rank_off[r[u]] = at;
        at += v[u];
      }
      carry += __shfl(incl, 63);
    }
    if (lane == 0) total[xl] = carry;
  }
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int xl = 0; xl < 8; ++xl) {
      first[xl] = run;
      run += total[xl];
    }
  }
  __syncthreads();
  if (tid < 8) {
    sched_x[tid] = first[tid];
    sched_x[8 + tid] = total[tid];
    sched_x[sched_counter(tid)] = 0;
  }
  for (int r = tid; r < M; r += 1024) {
    const int i = by_rank[r], bh = i / R, a = i % R;
    const int nt = item_nt[i];
    const int base = first[list_of_rank(r)] + rank_off[r];
    const int q0 = q_offsets[(int64_t)bh * (Cq + 2) + a], q1 = q_offsets[(int64_t)bh * (Cq + 2) + a + 1];
    // The cluster's 32-row wave blocks are dealt evenly to its nt tiles (sizes differ by at most
    // one block): a cluster of 500 rows becomes two tiles of 8 waves rather than one of 12 and
    // one of 4, whose lone wave per SIMD would leave the matrix cores idle most of the time.
    const int blocks = (q1 - q0 + 31) / 32;
    for (int j = 0; j < nt; ++j) {
      sched_bh[base + j] = bh;
      sched_a[base + j] = a;
      sched_row0[base + j] = q0 + 32 * (int)((int64_t)j * blocks / nt);
      sched_rend[base + j] = min(q1, q0 + 32 * (int)((int64_t)(j + 1) * blocks / nt));
    }
  }
}

__global__ void __launch_bounds__(1024)
plan_lists_kernel(const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ item_nt,
                  const int32_t* __restrict__ by_rank, int M, int Cq, int32_t* __restrict__ rank_off,
                  int32_t* __restrict__ sched_bh, int32_t* __restrict__ sched_a, int32_t* __restrict__ sched_row0,
                  int32_t* __restrict__ sched_rend, int32_t* __restrict__ sched_x) {
  write_lists(q_offsets, item_nt, by_rank, M, Cq, rank_off, sched_bh, sched_a, sched_row0, sched_rend, sched_x);
}

// Ranks and lists of up to kRankListItems items in one workgroup: the counting is M^2 / 1024 LDS reads a
// thread, less than the launch it saves (132 items: 76.5 -> 74.2 us a call; 336 items cost 1.7 us more).
constexpr int kRankListItems = 256;
__global__ void __launch_bounds__(1024)
plan_rank_lists_kernel(const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ item_T,
                       const int32_t* __restrict__ item_nt, int M, int Cq, int32_t* __restrict__ sched_bh,
                       int32_t* __restrict__ sched_a, int32_t* __restrict__ sched_row0,
                       int32_t* __restrict__ sched_rend, int32_t* __restrict__ sched_x) {
  __shared__ int32_t T[kRankListItems], nt[kRankListItems], rank[kRankListItems], by_rank[kRankListItems],
      rank_off[kRankListItems];
  const int tid = threadIdx.x;
  if (tid < M) {
    T[tid] = item_T[tid];
    nt[tid] = item_nt[tid];
    rank[tid] = 0;
  }
  __syncthreads();
  const int width = (M + 63) & ~63, parts = 1024 / width;  // waves of one part rank the items over a stretch of them
  const int part = tid / width, i = tid % width;
  if (part < parts && i < M) {
    const int mine = T[i], lo = (int)((int64_t)M * part / parts), hi = (int)((int64_t)M * (part + 1) / parts);
    int before = 0;
#pragma unroll 8
    for (int j = lo; j < hi; ++j) before += T[j] > mine || (T[j] == mine && j < i);
    atomicAdd(&rank[i], before);
  }
  __syncthreads();
  if (tid < M) by_rank[rank[tid]] = tid;
  __syncthreads();
  write_lists(q_offsets, nt, by_rank, M, Cq, rank_off, sched_bh, sched_a, sched_row0, sched_rend, sched_x);
}

// The whole plan of a call with up to kPlanItems items in one workgroup (block 0: a small layer is
// bound by launches, and the three kernels took 9 us of it; 256 items take 16 waves longer than that),
// and beside it the centroid tables in bf16 (the other blocks).
constexpr int kPlanItems = 64;
__global__ void __launch_bounds__(1024)
plan_small_kernel(const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ k_offsets,
                  const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int M, int Cq, int Ck, int BM,
                  int32_t* __restrict__ sched_bh, int32_t* __restrict__ sched_a, int32_t* __restrict__ sched_row0,
                  int32_t* __restrict__ sched_rend, int32_t* __restrict__ sched_x, const float* __restrict__ kbar,
                  const float* __restrict__ vbar, int64_t n, bf16_t* __restrict__ kbar16, bf16_t* __restrict__ vbar16) {
  if (blockIdx.x > 0) return centroids_to_bf16(blockIdx.x - 1, kbar, vbar, n, kbar16, vbar16);
  __shared__ int32_t item_T[kPlanItems], item_nt[kPlanItems], by_rank[kPlanItems], rank_off[kPlanItems];
  const int wave = threadIdx.x >> 6, R = Cq + 1;
  for (int i = wave; i < M; i += 16)
    plan_item(q_offsets, k_offsets, row_ptr, col_idx, i / R, i % R, Cq, Ck, BM, item_T[i], item_nt[i]);
  __syncthreads();
  for (int i = threadIdx.x; i < M; i += 1024) {  // T descending, then index ascending
    int rank = 0;
    for (int j = 0; j < M; ++j) rank += item_T[j] > item_T[i] || (item_T[j] == item_T[i] && j < i);
    by_rank[rank] = i;
  }
  __syncthreads();
  write_lists(q_offsets, item_nt, by_rank, M, Cq, rank_off, sched_bh, sched_a, sched_row0, sched_rend, sched_x);
}

}  // namespace

// Tile shape: 12 waves x 32 query rows per workgroup (one workgroup per CU, 3 waves per SIMD at 168
// VGPRs), 4 K/V tile buffers.
constexpr int kWaves = 12;
constexpr int kStages = 4;
constexpr int kCopyWaves = 4;

// Tile height and splits of a call, from its sizes alone.
struct Bf16Form {
  int rows;    // per tile: 384 (12-wave kernel) or 128 (four waves, two workgroups per CU)
  int splits;  // workgroups that share the keys of a 128-row tile
};
// Measured at d = 128 unless stated, us a call with a quarter routed (5 % in brackets):
//  * keys split, for the longest tiles: a cluster may have anything from a dozen keys to all of them routed,
//    and a launch ends no sooner than its longest tile. As many splits as the largest of three rules:
//    - fill: workgroups for the 512 that are resident at once, 1,024 keys each or more (fewer, and the
//      merge costs what it saves). 1 head x 11,970 rows, 8 / 942 clusters in one split 176 (84), in five 82
//      (56); 1 x 4,096, 32 / 64 in one 48 (27), in four 32 (28). Rounded to the nearest, since a few
//      workgroups beyond 512 wait for a whole tile: 12 x 2,376, 348 tiles in one 61 (33), in two 55 (47);
//    - fine: two rounds of workgroups at 4,096 keys or more a split: 1 x 37,800, 346 tiles in one split 980
//      (296), in two 543 (181), in three 389 (140); 4 x 10,000, 436 tiles in one 195 (61), in two 137 (69);
//    - spread: up to 1,536 tiles, four rounds at 8,192 keys or more: 1 x 75,600, 641 tiles in one split 1655
//      (487), in two 1010 (285), in four 918 (276); 1 x 118,800, 1,079 tiles in one 2885 (696), in two 2323
//      (534); d = 64, 2 x 75,600, 1,482 tiles in one 1586 (654), in two 1282 (373). Not where the keys are few
//      for so many tiles (8 x 20,000, 1,456 tiles of 128 rows in two 568 (230), the 384-row tile 542 (176)) nor
//      with more tiles, which even out by themselves (3 x 75,600, 1,923 tiles 2406 (631) against 2204 (532));
//  * clusters of at most 160 rows, which fill at most five of twelve waves, 384-row against 128-row tiles:
//    12 x 16,200, 81 rows 1091 -> 804 (427 -> 305); 24 x 10,800, 108 rows 795 -> 627; 24 x 4,000, 20 rows 734 ->
//    437; d = 64, 8 x 32,400, 162 rows 1014 -> 947, 24 x 1,200, 6 rows 386 -> 234 (277 -> 188); larger ones want
//    the larger tile (5 x 75,600, 252 rows 4022 -> 4449; d = 64, 24 x 32,400, 506 rows 2152 -> 2370);
//  * at most four 128-row tiles a CU, d = 128: 3 x 2,000, 1,000 rows 51 -> 41 (36 -> 29); 4 x 18,900 550 -> 529.
//    d = 64 at most 64 of them: 1 x 2,000, 666 rows 35 -> 30; 12 x 7,000 is the same either way (124).
static Bf16Form bf16_form(int64_t BH, int64_t Nq, int64_t Nk, int Cq, int d) {
  const int64_t quads = BH * (ceil_div(Nq, 32 * kQuadWaves) + Cq / 2);  // a cluster's last tile is half full
  const int64_t fill = std::min((512 + quads / 2) / quads, Nk / 1024);
  const int64_t fine = std::min({ceil_div(1024, quads), Nk / 4096, (int64_t)4});
  const int64_t spread =
      quads <= 1536 && Nk >= 16 * quads ? std::min({ceil_div(2048, quads), Nk / 8192, (int64_t)4}) : 1;
  const int64_t n = std::max({fill, fine, spread});
  if (n >= 2) return {32 * kQuadWaves, (int)(n < 8 ? n : 8)};
  if (Nq <= (int64_t)160 * Cq || quads <= (d == 128 ? 1024 : 64)) return {32 * kQuadWaves, 1};
  return {32 * kWaves, 1};
}

// d = 128: 12 bytes per key cluster beside the tile buffers is what the entry point promises.
bool attn_bf16_supported(int d, int Ck) {
  return d == 64 || (size_t)kStages * 2 * BN * 256 + (kStages + 2) * BN * 4 + align_up(Ck, 64) * 4 +
                        align_up((size_t)(2 * (Ck + 2) + 1) * 4, 16) <= 160 * 1024;
}

size_t plan_bf16_workspace(int64_t BH, int Cq, int64_t Nq, int64_t Nk, int d) {
  const Bf16Form f = bf16_form(BH, Nq, Nk, Cq, d);
  const size_t M = (size_t)BH * (Cq + 1), rows = (size_t)BH * Nq;
  const size_t tiles = (size_t)BH * ((size_t)ceil_div(Nq, f.rows) + Cq + 1);
  return 4 * align_up(M * 4, 256) + 4 * align_up(tiles * 4, 256) + align_up(kSchedInts * 4, 256) +
         (f.splits > 1 ? align_up(f.splits * rows * d * 4, 256) + align_up(f.splits * rows * sizeof(float2), 256) : 0);
}

int plan_bf16(AttnArgs& a, int d, bf16_t* kbar16, bf16_t* vbar16, void* ws, size_t ws_bytes, hipStream_t s) {
  Workspace w(ws, ws_bytes);
  Bf16Form f = bf16_form(a.BH, a.Nq, a.Nk, a.Cq, d);
  if (a.part == 2) f.splits = 1;  // the centroids alone are few (two-stage form, 4 x 20,000: 204 -> 173 us)
  const int M = a.BH * (a.Cq + 1), BM = f.rows;
  const size_t tiles = (size_t)a.BH * ((size_t)ceil_div(a.Nq, BM) + a.Cq + 1);
  int32_t* item_T = w.take<int32_t>(M);
  int32_t* item_nt = w.take<int32_t>(M);
  int32_t* by_rank = w.take<int32_t>(M);
  int32_t* rank_off = w.take<int32_t>(M);
  int32_t* sched_bh = w.take<int32_t>(tiles);
  int32_t* sched_a = w.take<int32_t>(tiles);
  int32_t* sched_row0 = w.take<int32_t>(tiles);
  int32_t* sched_rend = w.take<int32_t>(tiles);
  int32_t* sched_x = w.take<int32_t>(kSchedInts);
  a.tile_rows = f.rows;
  a.splits = f.splits;
  if (f.splits > 1) {
    a.part_o = w.take<float>((size_t)f.splits * a.BH * a.Nq * d);
    a.part_ml = w.take<float2>((size_t)f.splits * a.BH * a.Nq);
  }
  if (!w.ok()) return SVGEAR_ERR_WORKSPACE;
  a.sched_bh = sched_bh;
  a.sched_a = sched_a;
  a.sched_row0 = sched_row0;
  a.sched_rend = sched_rend;
  a.sched_x = sched_x;
  const int64_t n = (int64_t)a.BH * a.Ck * d;
  if (M <= kPlanItems) {
    plan_small_kernel<<<(unsigned)(1 + ceil_div(n, 1024)), 1024, 0, s>>>(
        a.q_offsets, a.k_offsets, a.row_ptr, a.col_idx, M, a.Cq, a.Ck, BM, sched_bh, sched_a, sched_row0, sched_rend,
        sched_x, a.kbar, a.vbar, n, kbar16, vbar16);
    SVGEAR_LAUNCH_CHECK();
    return SVGEAR_OK;
  }
  plan_items_kernel<<<(unsigned)(ceil_div(M, 4) + ceil_div(n, 256)), 256, 0, s>>>(
      a.q_offsets, a.k_offsets, a.row_ptr, a.col_idx, M, a.Cq, a.Ck, BM, item_T, item_nt, a.kbar, a.vbar, n, kbar16, vbar16);
  SVGEAR_LAUNCH_CHECK();
  if (M <= kRankListItems) {
    plan_rank_lists_kernel<<<1, 1024, 0, s>>>(a.q_offsets, item_T, item_nt, M, a.Cq, sched_bh, sched_a, sched_row0,
                                              sched_rend, sched_x);
    SVGEAR_LAUNCH_CHECK();
    return SVGEAR_OK;
  }
  plan_rank_kernel<<<(unsigned)ceil_div(M, kRankItems), 256, 0, s>>>(item_T, M, by_rank);
  SVGEAR_LAUNCH_CHECK();
  plan_lists_kernel<<<1, 1024, 0, s>>>(a.q_offsets, item_nt, by_rank, M, a.Cq, rank_off, sched_bh, sched_a, sched_row0,
                                      sched_rend, sched_x);
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}

// Merge of two partial softmax results over disjoint key sets (Algorithm 2's merge step):
// one thread per 8 output elements.
__global__ void __launch_bounds__(256)
merge_kernel(const bf16_t* __restrict__ o1, const float* __restrict__ lse1, const bf16_t* __restrict__ o2,
             const float* __restrict__ lse2, int64_t rows, int d, bf16_t* __restrict__ out,
             float* __restrict__ lse) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (row, group of 8 dims)
  const int per_row = d / 8;
  if (i >= rows * per_row) return;
  const int64_t row = i / per_row;
  const float a = lse1[row], b = lse2[row];
  const float m = fmaxf(a, b);
  float w1 = 0.f, w2 = 0.f;
  if (m > -INFINITY) {
    w1 = expf(a - m);
    w2 = expf(b - m);
  }
  const float den = w1 + w2;
  const float s1 = den > 0.f ? w1 / den : 0.f, s2 = den > 0.f ? w2 / den : 0.f;
  const uint4 x = *reinterpret_cast<const uint4*>(o1 + i * 8), y = *reinterpret_cast<const uint4*>(o2 + i * 8);
  const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
  uint32_t r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float lo = s1 * __uint_as_float(xs[k] << 16) + s2 * __uint_as_float(ys[k] << 16);
    const float hi = s1 * __uint_as_float(xs[k] & 0xffff0000u) + s2 * __uint_as_float(ys[k] & 0xffff0000u);
    r[k] = (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
  }
  *reinterpret_cast<uint4*>(out + i * 8) = make_uint4(r[0], r[1], r[2], r[3]);
  if (lse && (i % per_row) == 0) lse[row] = den > 0.f ? m + logf(den) : -INFINITY;
}

int launch_merge(const bf16_t* o1, const float* lse1, const bf16_t* o2, const float* lse2, int64_t rows, int d,
                 bf16_t* out, float* lse, hipStream_t s) {
  merge_kernel<<<(unsigned)ceil_div(rows * (d / 8), 256), 256, 0, s>>>(o1, lse1, o2, lse2, rows, d, out, lse);
  SVGEAR_LAUNCH_CHECK();
  return SVGEAR_OK;
}

// Grids cover the bound on the number of tiles (one workgroup per tile and split; the rest exit).
template <int D, bool WIDE>
static int launch(const AttnArgs& a, hipStream_t s) {
  const unsigned total = (unsigned)((size_t)a.BH * (ceil_div(a.Nq, a.tile_rows) + a.Cq + 1) * a.splits);
  const bool quad = a.tile_rows == 32 * kQuadWaves;
  const size_t lds = lds_bytes(D, a.Ck, quad ? 2 : kStages);
  auto kern = quad ? attn_bf16_quad_kernel<D, WIDE> : attn_bf16_kernel<D, kWaves, kStages, kCopyWaves, WIDE>;
  SVGEAR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
  kern<<<total, quad ? 64 * kQuadWaves : 64 * kWaves, lds, s>>>(a);
  SVGEAR_LAUNCH_CHECK();
  if (a.splits > 1) {
    merge_splits_kernel<D><<<(unsigned)ceil_div((int64_t)a.BH * a.Nq * (D / 8), 256), 256, 0, s>>>(a);
    SVGEAR_LAUNCH_CHECK();
  }
  return SVGEAR_OK;
}

int launch_attn_bf16(const AttnArgs& a, int d, hipStream_t s) {
  if (!a.sched_x) return SVGEAR_ERR_INVALID;
  if (d == 128) return launch<128, false>(a, s);  // (the entry point takes no more keys)
  return a.Nk > (int64_t)(UINT32_MAX / 128) ? launch<64, true>(a, s) : launch<64, false>(a, s);
}

}  // namespace svgear
