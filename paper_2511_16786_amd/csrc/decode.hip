// Decode-step attention over the compacted, per-layer-ragged cache (Preliminary section, Eq. 2-4,
// for one new token per sequence):  out = softmax(q K^T * scale) V  over the b_l rows each
// (layer, KV head) kept.  Grouped-query attention: query head g reads KV head g / G.
//
// HBM-bound by design: every kept K and V row is read exactly once (2*b_l*d*e bytes per unit),
// so the traffic - and the time - shrinks with the retention ratio.  Work is split over rows
// (flash-decoding style): a workgroup streams a chunk of one unit's rows, keeps online-softmax
// states, merges them through LDS and writes (max, sum, weighted V) for its chunk; a second kernel
// merges the chunks.
//
// Two realisations of the chunk kernel:
//  * bf16 caches: the matrix cores (v_mfma_f32_16x16x32_bf16).  With G query heads per KV head the
//    vector ALUs would have to do G dot products and G weighted sums per row and cap the row rate
//    well below HBM speed; as a 16-wide tile of query heads (G <= 16, padded with zeros) the same
//    work is 0.75 matrix instructions per row.  Scores S^T = K Q^T (bf16 x bf16 products are exact
//    in fp32), probabilities in fp32, then P V with P split into two bf16 terms (hi + lo, 16
//    significant bits) so that the weighted sum keeps fp32-grade accuracy.
//  * fp32 caches: vector ALUs, d/8 lanes per row, one online-softmax state per lane group.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "fc_common.h"
#include "rules.h"

namespace fc {

namespace {

// Scratch of the allocation-free entry point (flashcache_decode_attention_static): the per-chunk
// partial results live in this array instead of a caller workspace.  Every GPU the library runs on
// holds its own copy until the process ends.  In host code the array's name is only a handle: its
// device address is looked up once per device (static_scratch below) and that pointer is what the
// kernels receive.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kDecThreads = 256;
constexpr int kDecUnroll = 4;          // rows per lane group and step
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowHalfMirror = 0x141, kRowMirror = 0x140;

template <int CTRL> __device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// sum over the LPR (8 or 16) adjacent lanes that share a row; every lane gets the sum
template <int LPR> __device__ __forceinline__ float row_sum(float v) {
  v = dpp_add<kQuadXor1>(v);
  v = dpp_add<kQuadXor2>(v);
  v = dpp_add<kRowHalfMirror>(v);
  if (LPR == 16) v = dpp_add<kRowMirror>(v);
  return v;
}

typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// KEEP: with a claim on the last-level cache (see keep_rows), else past it.
template <bool KEEP, typename V> __device__ __forceinline__ V load_vec(const void* p) {
  if constexpr (KEEP) return *static_cast<const V*>(p);
  return __builtin_nontemporal_load(static_cast<const V*>(p));
}
// A lane's 8 of the D floats at p: 4 of the first half and 4 of the second, so that either load takes whole lines.
template <int D, bool KEEP> __device__ __forceinline__ void load8(const float* p, float (&o)[8]) {
  const float4v a = load_vec<KEEP, float4v>(p), b = load_vec<KEEP, float4v>(p + D / 2);
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}

// partial record of one (unit, split): m[G], l[G], o[G][d]  (floats)
__host__ __device__ inline size_t partial_floats(int G, int d) { return (size_t)G * (d + 2); }

// Pieces that a unit's k rows make of the `splits` that a launch has for every unit: none shorter than 128 rows, a step
// for each wave.  Budgets are on the device and differ from layer to layer, so that the cut is made there; workgroups
// beyond it end at once.  28 layers of 4 heads, 7 query heads each, one layer with 2048 rows and 27 with 57: 12.7 us,
// and 12.7 with 128 rows in every layer (cut on the host by the mean budget, which makes one workgroup of each unit: 26.8
// and 12.5; every unit in 10 pieces: 20.1 and 20.0).
__device__ __forceinline__ int pieces_of(int k, int splits) {
  return min(splits, k > 0 ? (k - 1) / 128 + 1 : 1);
}

// Paged source: row j of unit (b,l,h) sits in slot j % page_size of page
// block_table[unit][j / page_size] of caches laid out [num_pages][page_size][d].  table == nullptr
// means the packed layout.  Rows of a page entry that is missing or out of range are not read.
struct PagedSrc {
  const int* table;
  int page_size, max_pages;
  long long num_pages;
};
// cache row index of row `row` of this unit; ok = false (and a readable row) if it has no page
template <bool PAGED>
__device__ __forceinline__ long long cache_row(const PagedSrc& pg, long long packed_base, int unit, int row,
                                               bool& ok) {
  ok = true;
  if (!PAGED) return packed_base + row;
  const int p = row / pg.page_size;
  long long page = -1;
  if (p < pg.max_pages) page = pg.table[(size_t)unit * pg.max_pages + p];
  ok = page >= 0 && page < pg.num_pages;
  return ok ? page * pg.page_size + (row - p * pg.page_size) : 0;
}

// The sum of every lane's value, in a scalar register.
template <int CTRL> __device__ __forceinline__ int dpp_add_int(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
__device__ __forceinline__ int wave_total(int v) {
  v = dpp_add_int<kRowMirror>(dpp_add_int<kRowHalfMirror>(dpp_add_int<kQuadXor2>(dpp_add_int<kQuadXor1>(v))));
  int sum = 0;
#pragma unroll
  for (int row = 0; row < 64; row += 16) sum += __builtin_amdgcn_readlane(v, row);
  return sum;
}

constexpr int kMostRows = (1 << 25) - 1;                   // (64 of them, and 64 times one, are 31 bits)
__device__ __forceinline__ int rows_in(int budget) { return min(max(budget, 0), kMostRows); }

// Which unit a workgroup works on, its budget and (packed) first row.  `may_rank`: the launch's order is layer by layer, of
// each all sequences and heads, and where a sequence's pieces are long (ranks_by_budget) its layers come by falling budget, ties
// by layer; else units as they are numbered.  Every wave sums up and ranks the layers by itself, a lane each, from the
// loads that it would wait for anyway.
struct Place {
  int unit, b, l, h, k;
  long long off;
  long long rows;                                          // of the sequence; paged: its budgets' sum, or (no may_rank) a lane's part of it
};
template <bool PAGED, bool FITS>
__device__ __forceinline__ Place place_of(int at, const int* __restrict__ budgets, const long long* __restrict__ layer_offsets,
                                          int B, int L, int H, int splits, bool may_rank, int row_bytes) {
  Place p;
  p.h = at % H;
  const int lane = threadIdx.x & 63;
  if (!may_rank) {
    p.unit = at;
    p.l = at / H % L;
    p.b = at / H / L;
    p.k = budgets[(size_t)p.b * L + p.l];
    p.off = PAGED ? 0 : layer_offsets[(size_t)p.b * (L + 1) + p.l] + (long long)p.h * p.k;
    int rows = lane ? 0 : rows_in(p.k);
    if (PAGED && !FITS && L > 1) {
      rows = 0;
      for (int l = lane; l < L; l += 64) rows = min(rows + rows_in(budgets[(size_t)p.b * L + l]), kMostRows);
    }
    p.rows = PAGED ? rows : (FITS ? 0 : layer_offsets[(size_t)p.b * (L + 1) + L]);
    return p;
  }
  const int mine = min(lane, L - 1), rank = at / H / B;
  p.b = at / H % B;
  const int k = budgets[(size_t)p.b * L + mine];
  const long long off = PAGED ? 0 : layer_offsets[(size_t)p.b * (L + 1) + mine];
  const int rows = rows_in(k), total = wave_total(lane < L ? rows : 0);
  p.rows = PAGED ? total : (FITS ? 0 : layer_offsets[(size_t)p.b * (L + 1) + L]);
  p.l = rank;
  if (ranks_by_budget(total, L, splits, row_bytes)) {
    const int key = rows * 64 + 63 - mine;                 // (no two alike)
    int above = 0;
#pragma unroll 4
    for (int j = 0; j < L; ++j) above += __builtin_amdgcn_readlane(key, j) > key ? 1 : 0;
    p.l = __builtin_ctzll(__ballot(lane < L && above == rank));
  }
  p.k = __builtin_amdgcn_readlane(k, p.l);
  const unsigned lo = __builtin_amdgcn_readlane((int)off, p.l), hi = __builtin_amdgcn_readlane((int)(off >> 32), p.l);
  p.off = PAGED ? 0 : (long long)((unsigned long long)hi << 32 | lo) + (long long)p.h * p.k;
  p.unit = (p.b * L + p.l) * H + p.h;
  return p;
}

// Whether rows claim the last-level cache (keeps_rows), by what the launch reads if all sequences keep as many as this one.
// What a table or a buffer has room for does not tell.  By the room / by the budgets, us: through tables that reach 32768 rows four
// sequences of 28 layers of 4 heads that keep 300 rows 32.9 / 28.3, one that keeps 1638 30.2 / 27.9, 80 layers of 8 heads
// that keep 400 42.0 / 36.5; packed, a buffer for eight times the 1638 rows 27.5 / 25.4; where rows exceed the cache the same (137.2 /
// 137.8, 108.3 / 109.5, packed 68.0 / 67.7).  Two loops, since a branch at each step's loads costs 3 %.
template <bool PAGED>
__device__ __forceinline__ bool keep_rows(const Place& p, bool may_rank, int B, int H, int row_bytes) {
  return keeps_rows((PAGED ? (long long)(may_rank ? (int)p.rows : wave_total((int)p.rows)) * H : p.rows) * B, row_bytes);
}

// Rows `first`, `first` + NG, ... below r1: the lane group's online softmax.  (A function of its own: the same loop in a lambda of the
// kernel's is scheduled differently and 1 to 9 % slower, 8 sequences of one layer, 8410 rows, four query heads 26.0 / 23.7 us.)
template <typename T, int G, int LPR, bool PAGED, bool KEEP>
__device__ __forceinline__ void walk_rows(const T* __restrict__ kbase, const T* __restrict__ vbase, const PagedSrc& pg,
                                          long long packed_base, int unit, int first, int r1, const float (&q)[G][8],
                                          float (&m)[G], float (&ls)[G], float (&o)[G][8]) {
  constexpr int D = LPR * 8, NG = kDecThreads / LPR;
  for (int row = first; row < r1; row += NG * kDecUnroll) {
    float kv[kDecUnroll][8], vv[kDecUnroll][8];
    bool valid[kDecUnroll];
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const int rr = row + u * NG;
      valid[u] = rr < r1;
      const int rc = valid[u] ? rr : row;               // row itself is always in range
      bool ok;
      const long long ci = cache_row<PAGED>(pg, packed_base, unit, rc, ok);
      valid[u] = valid[u] && ok;
      load8<D, KEEP>(kbase + (size_t)ci * D, kv[u]);
      load8<D, KEEP>(vbase + (size_t)ci * D, vv[u]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float s[kDecUnroll];
      float mx = m[g];
#pragma unroll
      for (int u = 0; u < kDecUnroll; ++u) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = fmaf(q[g][i], kv[u][i], acc);
        acc = row_sum<LPR>(acc);
        s[u] = valid[u] ? acc : -INFINITY;
        mx = fmaxf(mx, s[u]);
      }
      // mx is finite as soon as one row was valid (packed layout: row `row` always is); while no
      // row has been seen the state stays empty
      if (mx == -INFINITY) continue;
      const float alpha = exp2f(m[g] - mx);             // exp2(-inf) = 0 on the first step
      float psum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) o[g][i] *= alpha;
#pragma unroll
      for (int u = 0; u < kDecUnroll; ++u) {
        const float p = exp2f(s[u] - mx);
        psum += p;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[g][i] = fmaf(p, vv[u][i], o[g][i]);
      }
      ls[g] = fmaf(ls[g], alpha, psum);
      m[g] = mx;
    }
  }
}

template <typename T, int G, int LPR, bool PAGED, bool FITS, bool WHOLE>
__global__ __launch_bounds__(kDecThreads) void decode_partial_kernel(
    const T* __restrict__ Q, const T* __restrict__ Kc, const T* __restrict__ Vc,
    const int* __restrict__ budgets, const long long* __restrict__ layer_offsets, int B, int L, int H,
    long long rows_per_seq, float scale_log2e, int splits, bool spread, bool may_rank, float* __restrict__ partial,
    float* __restrict__ whole, PagedSrc pg) {
  constexpr int D = LPR * 8;
  constexpr int NG = kDecThreads / LPR;                 // lane groups (rows in flight per step / unroll)
  constexpr int NW = kDecThreads / 64;                  // waves; their lane groups merge in registers
  __shared__ float sm_m[NW][G], sm_l[NW][G];
  __shared__ float sm_o[NW][G][D];
  const int split = spread ? blockIdx.y : blockIdx.x;
  const Place at = place_of<PAGED, FITS>(spread ? blockIdx.x : blockIdx.y, budgets, layer_offsets, B, L, H, splits, may_rank,
                                   D * (int)sizeof(*Kc));
  const int unit = at.unit, h = at.h, l = at.l, b = at.b, k = at.k;
  const long long off = at.off;
  float* rec = partial + ((size_t)unit * splits + split) * partial_floats(G, D);
  const int tid = threadIdx.x, grp = tid / LPR, sub = tid % LPR;
  const bool bad = k < 0 || (!PAGED && (off < 0 || off + k > rows_per_seq));
  const int pieces = pieces_of(k, splits), chunk = bad ? 0 : (k + pieces - 1) / pieces;
  if (split >= pieces) return;
  const int r0 = min(k, split * chunk), r1 = bad ? 0 : min(k, r0 + chunk);

  // this lane's 8 dims of the G query vectors, pre-multiplied by scale*log2(e)
  float q[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    load8<D, true>(Q + (((size_t)b * L + l) * (H * G) + (size_t)h * G + g) * D + sub * 4, q[g]);
#pragma unroll
    for (int i = 0; i < 8; ++i) q[g][i] *= scale_log2e;
  }
  float m[G], ls[G], o[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY; ls[g] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[g][i] = 0.f;
  }

  const long long packed_base = PAGED ? 0 : (long long)b * rows_per_seq + off;
  const T* kbase = Kc + sub * 4;
  const T* vbase = Vc + sub * 4;
  if (FITS || keep_rows<PAGED>(at, may_rank, B, H, D * (int)sizeof(*Kc)))
    walk_rows<T, G, LPR, PAGED, true>(kbase, vbase, pg, packed_base, unit, r0 + grp, r1, q, m, ls, o);
  else
    walk_rows<T, G, LPR, PAGED, false>(kbase, vbase, pg, packed_base, unit, r0 + grp, r1, q, m, ls, o);

  // merge the lane groups of a wave (lanes that hold the same dims of different rows), then the
  // waves through LDS; the order of the merges is fixed
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float m2 = __shfl_xor(m[g], off, 64), l2 = __shfl_xor(ls[g], off, 64);
      const float M = fmaxf(m[g], m2);
      const float w1 = M > -INFINITY ? exp2f(m[g] - M) : 0.f, w2 = M > -INFINITY ? exp2f(m2 - M) : 0.f;
      ls[g] = ls[g] * w1 + l2 * w2;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float o2 = __shfl_xor(o[g][i], off, 64);
        o[g][i] = o[g][i] * w1 + o2 * w2;
      }
      m[g] = M;
    }
  }
  const int wave = tid >> 6;
  if ((tid & 63) < LPR) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (sub == 0) { sm_m[wave][g] = m[g]; sm_l[wave][g] = ls[g]; }
#pragma unroll
      for (int i = 0; i < 8; ++i) sm_o[wave][g][sub * 4 + (i & 3) + (i >> 2) * (D / 2)] = o[g][i];
    }
  }
  __syncthreads();
  for (int item = tid; item < G * D; item += kDecThreads) {
    const int g = item / D, dim = item % D;
    float M = -INFINITY;
    for (int s2 = 0; s2 < NW; ++s2) M = fmaxf(M, sm_m[s2][g]);
    float acc = 0.f, lt = 0.f;
    if (M > -INFINITY) {
      for (int s2 = 0; s2 < NW; ++s2) {
        const float w = exp2f(sm_m[s2][g] - M);
        acc = fmaf(sm_o[s2][g][dim], w, acc);
        lt = fmaf(sm_l[s2][g], w, lt);
      }
    }
    if constexpr (WHOLE) {                                  // (what the merge makes of a single record)
      whole[((size_t)unit * G + g) * D + dim] = lt > 0.f ? acc / lt : 0.f;
    } else {
      rec[2 * G + (size_t)g * D + dim] = acc;
      if (dim == 0) { rec[g] = M; rec[G + g] = lt; }
    }
  }
}


// ------------------------------------------------------------------ bf16: matrix-core chunk kernel
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr int kTilesPerStep = 2;       // 16-row tiles between two rescales of the accumulators

__device__ __forceinline__ bf16x8 as_bf16x8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_bit_cast(bf16x8, (u32x4{a, b, c, d}));
}

// Operand layouts of v_mfma_f32_16x16x32_bf16 (D = A B + C, wave of 64 lanes, c16 = lane % 16,
// g4 = lane / 16): A holds row c16, k = 8*g4..8*g4+7; B holds column c16, same k; C/D hold column
// c16, rows 4*g4..4*g4+3.  The order of k inside a product is free as long as A and B agree, which
// lets a lane take its k-values from what its loads deliver:
//   scores:  A = K rows (row c16 of the tile, dims 32s + 8*g4.. for step s, so that a load takes 64 bytes of each row),
//            B = Q (query head c16, same dims)  ->  lane holds S[row 4*g4+i][head c16]
//   output:  A = P (head c16, rows 4*g4+i of both tiles of the step: exactly the layout the scores come out in), B = V (the
//            same rows, dim (D/16)*c16 + t for output tile t)  ->  lane holds out[head 4*g4+i][that dim]
// Bound by memory and by what a launch cannot overlap, its first loads and last merges.  112 units of 6554 rows, 7 query
// heads (0.38 GB): 79.2 us as long as rows claimed the last-level cache, a load took 16 bytes in four places of a K row and
// products were of 16; 74.1 with these changed, all but 1 us of it for the loads past the cache, and 66.3 in order of the
// layers' budgets (see place_of); 896 units of 1638 rows, paged: 156 / 144 / 135.
template <int D, bool PAGED, bool FITS, bool WHOLE>
__global__ __launch_bounds__(kDecThreads, 2) void decode_mfma_partial_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ Kc, const uint16_t* __restrict__ Vc,
    const int* __restrict__ budgets, const long long* __restrict__ layer_offsets, int B, int L, int H, int G,
    long long rows_per_seq, float scale_log2e, int splits, bool spread, bool may_rank, float* __restrict__ partial,
    float* __restrict__ whole, PagedSrc pg) {
  constexpr int KS = D / 32;            // k-steps of the score product
  constexpr int KW = D / 8;             // dwords of a K row (and of a Q row) per lane: D/4 dims
  constexpr int VT = D / 16;            // output tiles = dims of a V row per lane
  constexpr int VW = VT / 2;            // dwords of a V row per lane
  constexpr int NW = kDecThreads / 64;
  constexpr int GP = 16;                // query heads per tile
  constexpr int kStepRows = 16 * kTilesPerStep;
  __shared__ float sm_m[NW][GP], sm_l[NW][GP];
  __shared__ float sm_o[NW][GP][D];
  const int split = spread ? blockIdx.y : blockIdx.x;
  const Place at = place_of<PAGED, FITS>(spread ? blockIdx.x : blockIdx.y, budgets, layer_offsets, B, L, H, splits, may_rank,
                                   D * (int)sizeof(*Kc));
  const int unit = at.unit, h = at.h, l = at.l, b = at.b, k = at.k;
  const long long off = at.off;
  float* rec = partial + ((size_t)unit * splits + split) * partial_floats(G, D);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c16 = lane & 15, g4 = lane >> 4;
  const bool bad = k < 0 || (!PAGED && (off < 0 || off + k > rows_per_seq));
  // the unit's steps of 32 rows, shared out evenly over the waves of its workgroups
  const int pieces = pieces_of(k, splits);
  if (split >= pieces) return;
  const int steps = bad ? 0 : (k + kStepRows - 1) / kStepRows, share = pieces * NW, w_id = split * NW + wave;
  const int s0 = (int)((int64_t)steps * w_id / share), s1 = (int)((int64_t)steps * (w_id + 1) / share);

  // B operand of the score product: query head c16 (zeros beyond G), dims 32 i + 8 g4 .. + 7
  uint32_t qw[KW];
#pragma unroll
  for (int i = 0; i < KW; ++i) qw[i] = 0u;
  if (c16 < G) {
    const uint16_t* qp = Q + (((size_t)b * L + l) * ((size_t)H * G) + (size_t)h * G + c16) * D + 8 * g4;
#pragma unroll
    for (int i = 0; i < KW / 4; ++i) {
      const uint4 u = *reinterpret_cast<const uint4*>(qp + 32 * i);
      qw[4 * i] = u.x; qw[4 * i + 1] = u.y; qw[4 * i + 2] = u.z; qw[4 * i + 3] = u.w;
    }
  }

  float m = -INFINITY, ls = 0.f;        // running maximum (common to the 4 lanes of a head) and this lane's sum
  float4v out[VT];
#pragma unroll
  for (int t = 0; t < VT; ++t) out[t] = float4v{0.f, 0.f, 0.f, 0.f};

  const long long packed_base = PAGED ? 0 : (long long)b * rows_per_seq + off;
  const uint16_t* kbase = Kc + 8 * g4;
  const uint16_t* vbase = Vc + VT * c16;
  // Loads of one step: K rows 16*tt+c16, V rows 16*tt+4*g4+i of it (clamped to the unit's last row; masked later).
  // vok: bit 4*tt+i set if V row i of tile tt has a page (always, in the packed layout).  In the paged layout
  // lane r looks up row r % 32 of the step, one step before the step's rows are requested, and the others take the
  // result from it: one lookup per lane and step, and no load waits for the block table.
  struct Rows {
    uint32_t kw[kTilesPerStep][KW], vw[kTilesPerStep][4][VW];
    unsigned vok;
  };
  constexpr uint32_t kNoRow = 0xFFFFFFFFu;
  auto lookup = [&](int st) -> uint32_t {
    bool ok;
    const long long ci = cache_row<true>(pg, 0, unit, min(st * kStepRows + (lane & (kStepRows - 1)), k - 1), ok);
    return ok ? (uint32_t)ci : kNoRow;
  };
  auto load_step = [&](auto keep, int st, uint32_t where, Rows& x) {
    x.vok = PAGED ? 0u : ~0u;
#pragma unroll
    for (int tt = 0; tt < kTilesPerStep; ++tt) {
      long long kr, vr[4];
      if constexpr (PAGED) {
        const uint32_t c = (uint32_t)__shfl((int)where, 16 * tt + c16, 64);
        kr = c == kNoRow ? 0u : c;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t v = (uint32_t)__shfl((int)where, 16 * tt + 4 * g4 + i, 64);
          x.vok |= (v != kNoRow ? 1u : 0u) << (4 * tt + i);
          vr[i] = v == kNoRow ? 0u : v;
        }
      } else {
        kr = packed_base + min(st * kStepRows + 16 * tt + c16, k - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) vr[i] = packed_base + min(st * kStepRows + 16 * tt + 4 * g4 + i, k - 1);
      }
      const uint16_t* kp = kbase + kr * D;
#pragma unroll
      for (int i = 0; i < KW / 4; ++i) {
        const u32x4 u = load_vec<keep, u32x4>(kp + 32 * i);
        x.kw[tt][4 * i] = u.x; x.kw[tt][4 * i + 1] = u.y; x.kw[tt][4 * i + 2] = u.z; x.kw[tt][4 * i + 3] = u.w;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint16_t* vp = vbase + vr[i] * D;
        if constexpr (VW == 4) {
          const u32x4 u = load_vec<keep, u32x4>(vp);
          x.vw[tt][i][0] = u.x; x.vw[tt][i][1] = u.y; x.vw[tt][i][2] = u.z; x.vw[tt][i][3] = u.w;
        } else {
          const u32x2 u = load_vec<keep, u32x2>(vp);
          x.vw[tt][i][0] = u.x; x.vw[tt][i][1] = u.y;
        }
      }
    }
  };
  auto work = [&](int st, const Rows& x) {
    const auto& kw = x.kw;
    const auto& vw = x.vw;
    const unsigned vok = x.vok;
    const int rb = st * kStepRows;
    // scores of the step, in log2 units
    float sc[kTilesPerStep][4];
    float mx = -INFINITY;
#pragma unroll
    for (int tt = 0; tt < kTilesPerStep; ++tt) {
      float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            as_bf16x8(kw[tt][4 * s], kw[tt][4 * s + 1], kw[tt][4 * s + 2], kw[tt][4 * s + 3]),
            as_bf16x8(qw[4 * s], qw[4 * s + 1], qw[4 * s + 2], qw[4 * s + 3]), acc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool valid = rb + 16 * tt + 4 * g4 + i < k && ((vok >> (4 * tt + i)) & 1u);
        sc[tt][i] = valid ? acc[i] * scale_log2e : -INFINITY;
        mx = fmaxf(mx, sc[tt][i]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // packed layout: row rb is valid and inputs are finite, so the new maximum is finite; paged
    // layout: a step whose rows all lack a page leaves the state as it is
    const float m_new = fmaxf(m, mx);
    const bool none = m_new == -INFINITY;
    const float alpha = none ? 1.f : exp2f(m - m_new);  // exp2(-inf) = 0 on the first step
    m = m_new;
    float psum = 0.f;
    uint32_t hi[2 * kTilesPerStep], lo[2 * kTilesPerStep];
#pragma unroll
    for (int tt = 0; tt < kTilesPerStep; ++tt)
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        const float p0 = none ? 0.f : exp2f(sc[tt][i] - m_new), p1 = none ? 0.f : exp2f(sc[tt][i + 1] - m_new);
        psum += p0;
        psum += p1;
        // high half = p truncated to bf16, low half = the rest rounded to nearest
        const uint32_t u0 = __float_as_uint(p0), u1 = __float_as_uint(p1);
        hi[2 * tt + i / 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        lo[2 * tt + i / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(
            (float2v{p0 - __uint_as_float(u0 & 0xFFFF0000u), p1 - __uint_as_float(u1 & 0xFFFF0000u)}), bf16x2));
      }
    const bf16x8 phi = as_bf16x8(hi[0], hi[1], hi[2], hi[3]), plo = as_bf16x8(lo[0], lo[1], lo[2], lo[3]);
    ls = fmaf(ls, alpha, psum);
    // the accumulators hold heads 4*g4+i: fetch their rescale factors from the lanes that own them
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a_i = __shfl(alpha, 4 * g4 + i, 64);
#pragma unroll
      for (int t = 0; t < VT; ++t) out[t][i] *= a_i;
    }
#pragma unroll
    for (int t = 0; t < VT; ++t) {
      // element t of this lane's V rows, four of each tile: dword t/2, low or high half
      const uint32_t sel = (t & 1) ? 0x07060302u : 0x05040100u;
      const int w = t >> 1;
      auto two = [&](int tt, int i) { return __builtin_amdgcn_perm(vw[tt][i + 1][w], vw[tt][i][w], sel); };
      const bf16x8 vb = as_bf16x8(two(0, 0), two(0, 2), two(1, 0), two(1, 2));
      out[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(phi, vb, out[t], 0, 0, 0);
      out[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plo, vb, out[t], 0, 0, 0);
    }
  };
  // two steps of rows under way; a step's registers are filled again in place
  auto walk = [&](auto keep) {
    Rows xa, xb;
    uint32_t where = 0;
    if (s0 < s1) {
      if (PAGED) where = lookup(s0);
      load_step(keep, s0, where, xa);
      if (s0 + 1 < s1) {
        if (PAGED) where = lookup(s0 + 1);
        load_step(keep, s0 + 1, where, xb);
        if (PAGED && s0 + 2 < s1) where = lookup(s0 + 2);
      }
    }
    auto turn = [&](int st, Rows& x) {
      work(st, x);
      if (st + 2 < s1) load_step(keep, st + 2, where, x);
      if (PAGED && st + 3 < s1) where = lookup(st + 3);
    };
    for (int st = s0; st < s1; st += 2) {
      turn(st, xa);
      if (st + 1 < s1) turn(st + 1, xb);
    }
  };
  if constexpr (FITS) walk(std::true_type{});
  else if (keep_rows<PAGED>(at, may_rank, B, H, D * (int)sizeof(*Kc))) walk(std::true_type{});
  else walk(std::false_type{});

  // the 4 lanes of a head add their sums; then the waves merge through LDS in a fixed order
  ls += __shfl_xor(ls, 16, 64);
  ls += __shfl_xor(ls, 32, 64);
  if (g4 == 0) { sm_m[wave][c16] = m; sm_l[wave][c16] = ls; }
#pragma unroll
  for (int t = 0; t < VT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) sm_o[wave][4 * g4 + i][VT * c16 + t] = out[t][i];
  __syncthreads();
  for (int item = tid; item < G * D; item += kDecThreads) {
    const int g = item / D, dim = item % D;
    float M = -INFINITY;
    for (int s2 = 0; s2 < NW; ++s2) M = fmaxf(M, sm_m[s2][g]);
    float acc = 0.f, lt = 0.f;
    if (M > -INFINITY) {
      for (int s2 = 0; s2 < NW; ++s2) {
        const float w = exp2f(sm_m[s2][g] - M);
        acc = fmaf(sm_o[s2][g][dim], w, acc);
        lt = fmaf(sm_l[s2][g], w, lt);
      }
    }
    if constexpr (WHOLE) {                                  // (what the merge makes of a single record)
      whole[((size_t)unit * G + g) * D + dim] = lt > 0.f ? acc / lt : 0.f;
    } else {
      rec[2 * G + (size_t)g * D + dim] = acc;
      if (dim == 0) { rec[g] = M; rec[G + g] = lt; }
    }
  }
}

// out[unit][g][:] = sum_s o_s w_s / sum_s l_s w_s with w_s = exp2(m_s - max m); zeros if no rows.
// grid = (G, units), one thread per feature and group of up to kAtOnce pieces, groups merged in order.  Bound by waiting for
// memory: a launch has groups for all pieces that its units may have, whose loads are under way together (8 units of 64 records:
// 10.9 -> 6.2 us, 112 units of 9 records: 6.8 -> 6.2, with events; an empty launch 6.1).  A unit whose budget makes no more than one
// group's pieces is done without LDS (28 units that keep 277 rows in a buffer for four times as many, both kernels: 8.1 -> 7.5).
constexpr int kMostPieces = 64;        // of a unit (see pick_splits)

template <int kAtOnce, int kGroups>
__global__ void decode_merge_kernel(const float* __restrict__ partial, const int* __restrict__ budgets, int H, int G,
                                    int d, int splits, float* __restrict__ out) {
  const int g = blockIdx.x, unit = blockIdx.y, group = threadIdx.x / d, dim = threadIdx.x - group * d;
  const int pieces = pieces_of(budgets[unit / H], splits);
  const size_t stride = partial_floats(G, d);
  const float* base = partial + (size_t)unit * splits * stride;
  float M = -INFINITY, acc = 0.f, lt = 0.f;
  const int s0 = group * kAtOnce;
  if (s0 < pieces) {
    float m[kAtOnce], l[kAtOnce], o[kAtOnce];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      const float* rec = base + (size_t)min(s0 + k, pieces - 1) * stride;
      m[k] = s0 + k < pieces ? rec[g] : -INFINITY;
      l[k] = rec[G + g];
      o[k] = rec[2 * G + (size_t)g * d + dim];
    }
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) M = fmaxf(M, m[k]);
    if (M > -INFINITY)
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const float w = exp2f(m[k] - M);
        acc = fmaf(o[k], w, acc);
        lt = fmaf(l[k], w, lt);
      }
  }
  if (kGroups > 1 && pieces > kAtOnce) {
    extern __shared__ float group_sums[];                  // [kGroups][3][d]: largest logit, sum, weighted sum
    float* mine = group_sums + (size_t)group * 3 * d + dim;
    mine[0] = M; mine[d] = lt; mine[2 * d] = acc;
    __syncthreads();
    if (group > 0) return;
    float top = M;
#pragma unroll
    for (int j = 1; j < kGroups; ++j) top = fmaxf(top, mine[j * 3 * d]);
    if (top > -INFINITY) {
      const float before = exp2f(M - top);
      acc *= before;
      lt *= before;
#pragma unroll
      for (int j = 1; j < kGroups; ++j) {
        const float w = exp2f(mine[j * 3 * d] - top);
        acc = fmaf(mine[(j * 3 + 2) * d], w, acc);
        lt = fmaf(mine[(j * 3 + 1) * d], w, lt);
      }
    }
  }
  if (group == 0) out[((size_t)unit * G + g) * d + dim] = lt > 0.f ? acc / lt : 0.f;
}

// Workgroups per unit.  A compute unit holds two, so the launch fills whole rounds of 512: two rounds for few
// units, four for many (their budgets differ, and shorter pieces even that out).  Where that many records would not
// fit the static array, one round of 1024 shared out among the units, which bounds what the array has to hold; the
// rule is the same for both kinds of scratch, so that their results agree to the bit.
int pick_splits(int units, int group, int d) {
  const int fine = std::min(kMostPieces, (units > 256 ? 2048 : 1024) / units);
  if (fine >= 1 && (size_t)units * fine * partial_floats(group, d) * sizeof(float) <= kStaticScratchBytes) return fine;
  return std::max(1, std::min(32, (1024 + units - 1) / units));
}

hipError_t launch_merge(const float* ws, const int32_t* budgets, int H, int G, int d, int splits, int units, float* out,
                        hipStream_t s) {
  ProfileScope ps("decode_merge_kernel", s);
  auto launch = [&](auto kern, int groups) {
    hipLaunchKernelGGL(kern, dim3(G, units), dim3(groups * d), groups > 1 ? (size_t)groups * 3 * d * sizeof(float) : 0, s, ws,
                       budgets, H, G, d, splits, out);
  };
  static_assert(kMostPieces <= 8 * 8, "a group for all pieces of a unit");
  if (splits <= 2) launch(decode_merge_kernel<2, 1>, 1);
  else if (splits <= 4) launch(decode_merge_kernel<4, 1>, 1);
  else if (splits <= 8) launch(decode_merge_kernel<8, 1>, 1);
  else if (splits <= 16) launch(decode_merge_kernel<8, 2>, 2);
  else launch(decode_merge_kernel<8, 8>, 8);
  return hipGetLastError();
}

// The pieces a launch provides for: what the largest budget there can be makes, one layer's heads keeping every row of
// the sequence or, in the paged layout, a unit as many as its part of the table reaches.  Where the mean budget makes
// fewer, surplus workgroups are among them, and the units' first pieces are launched before their second ones, so that
// those with rows spread over the compute units (fp32, 3 layers of 4 heads that keep 1463 rows, 8 query heads each: 17.3 ->
// 13.5 us; a unit's pieces side by side are better where all have rows: 18 layers of 8 heads, 1827 rows: 83 / 88).
// Layers may come by falling budget (see place_of) in launches of more than the 512 workgroups that are resident, so
// that the last to begin are the shortest (28 layers of 4 heads that keep 6554 rows: 66.3 us, as numbered 74.1, all layers
// alike 64).  The host knows what a budget can be, a table's reach for instance; what the budgets are is decided by on the
// device (by the reach alone eight sequences that keep 300 rows were ranked whatever their table: 41.3 us instead of 37.5).
// Launches of a single piece for each unit (budgets that cannot exceed 128 rows, or more than 1024 units) write the results themselves and
// need no merge: 13 layers of 2 heads that keep 73 rows, through tables that reach 128, 10.9 us with it, 8.0 without; 1280 units that keep 100
// 21.9 / 17.6, of fp32 31.5 / 27.1.  (Kernels of their own: asked at run time the others took 1 % longer.)
struct Cut {
  int splits;
  bool spread, long_pieces;
  dim3 grid(int units) const { return spread ? dim3(units, splits) : dim3(splits, units); }
  bool may_rank(int L, int units) const { return long_pieces && L > 1 && L <= 64 && (int64_t)units * splits > 512; }
};
Cut cut_splits(int splits, int L, int H, int64_t rows_per_seq, int row_bytes, const PagedSrc& pg) {
  const int64_t rows = pg.table ? (int64_t)pg.max_pages * pg.page_size : rows_per_seq / H;
  const int64_t most = (rows + 127) / 128, mean = pg.table ? rows : rows / L;
  const int cut = most < 1 ? 1 : (most < splits ? (int)most : splits);
  return {cut, mean < 128 * (int64_t)cut, ranks_by_budget(mean, 1, cut, row_bytes)};
}

// Whether the rows fit the last-level cache whatever the budgets are; else the kernels look at these (see keep_rows).
bool surely_fits(int B, int L, int H, int64_t rows_per_seq, int row_bytes, const PagedSrc& pg) {
  const int64_t rows = pg.table ? std::min<int64_t>(pg.num_pages, (int64_t)B * L * H * pg.max_pages) * pg.page_size
                                : B * rows_per_seq;
  return keeps_rows(rows, row_bytes);
}

template <typename T, int G, int LPR>
hipError_t decode_t(const void* Q, const void* Kc, const void* Vc, int B, int L, int H, const int32_t* budgets,
                    const int64_t* offs, int64_t rows_per_seq, float scale, float* out, float* ws,
                    const PagedSrc& pg, hipStream_t s) {
  const int units = B * L * H, d = LPR * 8;
  const Cut cut = cut_splits(pick_splits(units, G, d), L, H, rows_per_seq, d * (int)sizeof(T), pg);
  {
    ProfileScope ps("decode_partial_kernel", s);
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, cut.grid(units), dim3(kDecThreads), 0, s, static_cast<const T*>(Q),
                         static_cast<const T*>(Kc), static_cast<const T*>(Vc), budgets,
                         reinterpret_cast<const long long*>(offs), B, L, H, (long long)rows_per_seq,
                         scale * 1.4426950408889634f, cut.splits, cut.spread, cut.may_rank(L, units), ws, cut.splits == 1 ? out : nullptr, pg);
    };
    const bool fits = surely_fits(B, L, H, rows_per_seq, d * (int)sizeof(T), pg);
    auto choose = [&](auto single) {
      constexpr bool kWhole = decltype(single)::value;
      if (pg.table) fits ? launch(decode_partial_kernel<T, G, LPR, true, true, kWhole>) : launch(decode_partial_kernel<T, G, LPR, true, false, kWhole>);
      else fits ? launch(decode_partial_kernel<T, G, LPR, false, true, kWhole>) : launch(decode_partial_kernel<T, G, LPR, false, false, kWhole>);
    };
    cut.splits == 1 ? choose(std::true_type{}) : choose(std::false_type{});
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || cut.splits == 1) return e;
  return launch_merge(ws, budgets, H, G, d, cut.splits, units, out, s);
}

template <int D>
hipError_t decode_mfma_t(const void* Q, const void* Kc, const void* Vc, int B, int L, int H, int G,
                         const int32_t* budgets, const int64_t* offs, int64_t rows_per_seq, float scale,
                         float* out, float* ws, const PagedSrc& pg, hipStream_t s) {
  const int units = B * L * H;
  const Cut cut = cut_splits(pick_splits(units, G, D), L, H, rows_per_seq, D * (int)sizeof(uint16_t), pg);
  {
    ProfileScope ps("decode_mfma_partial_kernel", s);
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, cut.grid(units), dim3(kDecThreads), 0, s, static_cast<const uint16_t*>(Q),
                         static_cast<const uint16_t*>(Kc), static_cast<const uint16_t*>(Vc), budgets,
                         reinterpret_cast<const long long*>(offs), B, L, H, G, (long long)rows_per_seq,
                         scale * 1.4426950408889634f, cut.splits, cut.spread, cut.may_rank(L, units), ws, cut.splits == 1 ? out : nullptr, pg);
    };
    const bool fits = surely_fits(B, L, H, rows_per_seq, D * (int)sizeof(uint16_t), pg);
    auto choose = [&](auto single) {
      constexpr bool kWhole = decltype(single)::value;
      if (pg.table) fits ? launch(decode_mfma_partial_kernel<D, true, true, kWhole>) : launch(decode_mfma_partial_kernel<D, true, false, kWhole>);
      else fits ? launch(decode_mfma_partial_kernel<D, false, true, kWhole>) : launch(decode_mfma_partial_kernel<D, false, false, kWhole>);
    };
    cut.splits == 1 ? choose(std::true_type{}) : choose(std::false_type{});
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || cut.splits == 1) return e;
  return launch_merge(ws, budgets, H, G, D, cut.splits, units, out, s);
}

}  // namespace

bool decode_supported(int group, int d, int dtype) {
  if (d != 64 && d != 128) return false;
  if (dtype == FC_BF16) return group >= 1 && group <= 16;          // matrix-core kernel
  return group == 1 || group == 2 || group == 4 || group == 7 || group == 8;
}

size_t decode_static_scratch_bytes() { return kStaticScratchBytes; }

// Device address of this GPU's copy of `scratch` (looked up on the first call per device, with that
// device current; no allocation).
hipError_t decode_static_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

size_t decode_workspace_bytes(int B, int L, int H, int group, int d) {
  const int units = B * L * H;
  return units == 0 ? 0 : (size_t)units * pick_splits(units, group, d) * partial_floats(group, d) * sizeof(float);
}

hipError_t decode_launch(const void* Q, const void* Kc, const void* Vc, int B, int L, int H, int group, int d,
                         int dtype, const int32_t* budgets, const int64_t* offs, int64_t rows_per_seq,
                         float scale, float* out, void* ws, const int32_t* block_table, int32_t page_size,
                         int32_t max_pages, int64_t num_pages, hipStream_t s) {
  float* w = static_cast<float*>(ws);
  const PagedSrc pg{block_table, page_size, max_pages, (long long)num_pages};
  if (dtype == FC_BF16)
    return d == 128
               ? decode_mfma_t<128>(Q, Kc, Vc, B, L, H, group, budgets, offs, rows_per_seq, scale, out, w, pg, s)
               : decode_mfma_t<64>(Q, Kc, Vc, B, L, H, group, budgets, offs, rows_per_seq, scale, out, w, pg, s);
#define FC_DEC(GV)                                                                                          \
  if (group == GV)                                                                                          \
    return d == 128                                                                                         \
               ? decode_t<float, GV, 16>(Q, Kc, Vc, B, L, H, budgets, offs, rows_per_seq, scale, out, w, pg, s) \
               : decode_t<float, GV, 8>(Q, Kc, Vc, B, L, H, budgets, offs, rows_per_seq, scale, out, w, pg, s);
  FC_DEC(1) FC_DEC(2) FC_DEC(4) FC_DEC(7) FC_DEC(8)
#undef FC_DEC
  return hipErrorInvalidValue;
}

}  // namespace fc
