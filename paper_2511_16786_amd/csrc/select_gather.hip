// Selection of the b_l highest-scoring KV pairs of every unit and the packed gather (the rule in
// the sentence after Eq. 10: per layer, the pairs that deviate most, as many as the budget allows).
//
// select_kernel / select_large_kernel: one workgroup per unit.  Counting passes over the fp32 bit
//   patterns (a narrowing key range, or 8-bit digits) find the k-th largest key and how many keys
//   equal to it are still needed; a compaction in token order (prefix counts) then writes the kept
//   indices, which yields them ascending and gives ties to the lower index without any sort.  Up to
//   65536 tokens the keys stay in registers between the passes; beyond that they are re-read from L2.
//   Only integer atomics are used (LDS histogram), so the result is deterministic.  Small launches copy the rows as well.
// gather_kernel: rows are bit copies, 16 bytes a thread; one lookup a row.
#include <algorithm>

#include "fc_common.h"
#include "rules.h"

namespace fc {

namespace {

constexpr int kSelThreads = 1024;

// Monotone map float -> uint32 (larger float = larger key), valid for any sign.
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Score the selection is taken on.  Per-head mode: the unit's own score.  Layer-shared mode (the
// row-wide reading of Eq. 10, where the MSE runs over all H*d features of a token): the fp32 sum
// of the heads' scores in ascending head order divided by H, one correctly rounded division.
template <bool SHARED>
__device__ __forceinline__ float score_at(const float* __restrict__ s, int i, int n, int H) {
  if (!SHARED) return s[i];
  float acc = s[i];
  for (int h = 1; h < H; ++h) acc += s[(size_t)h * n + i];
  return __fdiv_rn(acc, (float)H);
}

template <bool SHARED>
__global__ __launch_bounds__(kSelThreads) void select_large_kernel(
    const float* __restrict__ scores, const int* __restrict__ budgets,
    const long long* __restrict__ layer_offsets, int L, int H, int n, long long rows_per_seq,
    int* __restrict__ idx_out) {
  __shared__ unsigned hist[256];
  __shared__ unsigned wave_gt[kSelThreads / 64], wave_eq[kSelThreads / 64];
  __shared__ unsigned sh_bucket, sh_need;
  __shared__ unsigned run_gt, run_eq;

  // per-head mode: one workgroup per (b,l,h); layer-shared mode: one per (b,l), writing H copies
  const int unit = SHARED ? blockIdx.x * H : blockIdx.x;
  const int h = unit % H, bl = unit / H, l = bl % L, b = bl / L;
  const int k = budgets[(size_t)b * L + l];
  const int copies = SHARED ? H : 1;
  const long long off = layer_offsets[(size_t)b * (L + 1) + l] + (long long)h * k;
  if (k <= 0 || k > n || off < 0 || off + (long long)copies * k > rows_per_seq) return;   // bad budgets
  const float* s = scores + (size_t)unit * n;
  int* out = idx_out + (size_t)b * rows_per_seq + off;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // ---- radix select: after the loop `prefix` is the k-th largest key
  uint32_t prefix = 0, mask = 0;
  unsigned need = (unsigned)k;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += kSelThreads) {
      uint32_t key = order_key(score_at<SHARED>(s, i, n, H));
      if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (wave == 0) {
      // suffix sums over the 256 buckets, 4 per lane (lane 63 holds the top buckets)
      unsigned c0 = hist[lane * 4 + 0], c1 = hist[lane * 4 + 1], c2 = hist[lane * 4 + 2],
               c3 = hist[lane * 4 + 3];
      unsigned mine = c0 + c1 + c2 + c3;
      unsigned above = 0;                      // keys in buckets of higher lanes
      unsigned run = mine;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        unsigned v = __shfl_down(run, d, 64);
        if (lane + d < 64) run += v;
      }
      above = run - mine;
      // the bucket holding the need-th largest key is in this lane iff above < need <= above+mine
      if (above < need && need <= above + mine) {
        unsigned a = above;
        unsigned bucket;
        if (a + c3 >= need) bucket = 3;
        else { a += c3; if (a + c2 >= need) bucket = 2;
        else { a += c2; if (a + c1 >= need) bucket = 1;
        else { a += c1; bucket = 0; } } }
        sh_bucket = lane * 4 + bucket;
        sh_need = need - a;
      }
    }
    __syncthreads();
    prefix |= sh_bucket << shift;
    mask |= 255u << shift;
    need = sh_need;
    __syncthreads();
  }
  const uint32_t tau = prefix;          // key of the k-th largest score
  // `need` = how many keys equal to tau are kept (those with the lowest token indices)

  // ---- compaction in token order
  if (tid == 0) { run_gt = 0; run_eq = 0; }
  __syncthreads();
  for (int base = 0; base < n; base += kSelThreads) {
    const int i = base + tid;
    uint32_t key = i < n ? order_key(score_at<SHARED>(s, i, n, H)) : 0u;
    const bool gt = i < n && key > tau;
    const bool eq = i < n && key == tau;
    const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const unsigned pre_gt = __popcll(bgt & below), pre_eq = __popcll(beq & below);
    if (lane == 0) { wave_gt[wave] = __popcll(bgt); wave_eq[wave] = __popcll(beq); }
    __syncthreads();
    unsigned ogt = run_gt, oeq = run_eq, tgt = 0, teq = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / 64; ++w) {
      unsigned g = wave_gt[w], e = wave_eq[w];
      if (w < wave) { ogt += g; oeq += e; }
      tgt += g; teq += e;
    }
    const unsigned gt_before = ogt + pre_gt, eq_before = oeq + pre_eq;
    if (gt || (eq && eq_before < need)) {
      const unsigned pos = gt_before + min(eq_before, need);
      for (int c = 0; c < copies; ++c) out[(size_t)c * k + pos] = i;
    }
    __syncthreads();
    if (tid == 0) { run_gt += tgt; run_eq += teq; }
    __syncthreads();
  }
}

// Register-resident variant for n <= 64*1024.  A wave keeps 64 * MAXC consecutive tokens, lane l the tokens
// 256 j + 4 l + e of them (coalesced 16-byte loads).  The k-th largest key is found by narrowing a key range:
// 2048 equal bins between the lowest and the highest key in question, counted in LDS, take a range of any width
// to a single key in three passes, usually in two (the search ends when a bin is kept whole); bins of equal width
// between the extremes spread the keys over many counters, where digits of the key put nearly all of them on a few.
// One workgroup per unit, a barrier per step: bound by latency and by how fast one CU's SIMDs issue the work on its keys
// (32768 tokens, 112 units: 19.7 us; 8192: 9.1; 4 units of 512: 7.1, 6 of them an empty launch).  Kept tokens are gathered
// in LDS and written as whole lines: stored from where they were found, with the loads one after another, it took 26.3 and
// 11.1 us (16384 tokens, 896 units: 52.4 / 26.5; 60000, 80 units: 62.6 / 29.4).
constexpr int kSelMaxChunk = 64;
constexpr int kSelBins = 2048;

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_u32(unsigned v) {       // 0 where there is no source lane
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
  v += dpp_u32<0x111, 0xF>(v);      // row_shr:1, 2, 4, 8
  v += dpp_u32<0x112, 0xF>(v);
  v += dpp_u32<0x114, 0xF>(v);
  v += dpp_u32<0x118, 0xF>(v);
  v += dpp_u32<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
  v += dpp_u32<0x143, 0xC>(v);      // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {  // valid in lane 63
  v = max(v, dpp_u32<0x111, 0xF>(v));
  v = max(v, dpp_u32<0x112, 0xF>(v));
  v = max(v, dpp_u32<0x114, 0xF>(v));
  v = max(v, dpp_u32<0x118, 0xF>(v));
  v = max(v, dpp_u32<0x142, 0xA>(v));
  return max(v, dpp_u32<0x143, 0xC>(v));
}
__device__ __forceinline__ unsigned below_me(unsigned long long mask, unsigned add) {   // set bits of lower lanes
  return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, add));
}

// a value that all lanes of the wave hold, in a scalar register
__device__ __forceinline__ unsigned uniform(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }

typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));

// Destination of the paged variant: kept row j of unit (b,l,h) goes to slot j % page_size of page
// block_table[b][l][h][j / page_size] of caches laid out [num_pages][page_size][d].
struct PagedDst {
  const int* block_table;
  int page_size, max_pages;
  long long num_pages;
};

// What the selection needs to copy the rows as well.
struct CopyArgs {
  const char *K, *V;
  KvStrides st;
  int lists, elem_bytes, vec_per_row, vpr_shift;
  char *K_out, *V_out;
  PagedDst pg;
};

// The index set that a workgroup works on, and which of how many shares of its kept rows.  A set has as many workgroups as
// its budget takes of equal shares of all sets' rows (one layer: budgets are alike); there are no more than 64 sets, a
// lane each.
struct Share {
  int list, at, of;
};
__device__ __forceinline__ Share share_of(int g, int all, int lists, int L, int sets_per_budget, int n, const int* __restrict__ budgets) {
  if (L == 1) return {g % lists, g / lists, all / lists};
  const int lane = threadIdx.x & 63;
  const unsigned k = lane < lists ? (unsigned)min(max(budgets[lane / sets_per_budget], 0), n) : 0u;
  const unsigned total = (unsigned)__builtin_amdgcn_readlane((int)wave_incl_scan(k), 63), spare = (unsigned)(all - lists);
  const unsigned rows = max(1u, (total + spare - 1) / spare), mine = (k + rows - 1) / rows, upto = wave_incl_scan(mine);
  const unsigned long long behind = __ballot(upto > (unsigned)g);
  if (!behind) return {0, 0, 0};
  const int list = __builtin_ctzll(behind), of = __builtin_amdgcn_readlane((int)mine, list);
  return {list, g - __builtin_amdgcn_readlane((int)upto, list) + of, of};
}

// COPY: workgroups that have a set in common make the same selection, and each writes the indices of its share of the kept rows and copies
// these.  For launches that leave most compute units idle, whose time is that of the launches themselves.
template <bool SHARED, int NT, int MAXC, bool COPY>
__global__ __launch_bounds__(NT) void select_kernel(
    const float* __restrict__ scores, const int* __restrict__ budgets,
    const long long* __restrict__ layer_offsets, int L, int H, int n, long long rows_per_seq,
    int* __restrict__ idx_out, CopyArgs cp) {
  constexpr int kWaves = NT / 64, kPer = kSelBins / NT;
  __shared__ union { unsigned hist[kSelBins]; unsigned short stage[NT * MAXC]; } lds;
  unsigned* const hist = lds.hist;
  unsigned short* const stage = lds.stage;
  __shared__ unsigned short list[COPY ? NT * MAXC : 1];    // this workgroup's share of the kept tokens
  __shared__ unsigned wave_a[kWaves], wave_b[kWaves];
  __shared__ unsigned sh_bin, sh_need, sh_count;

  // per-head mode: one workgroup per (b,l,h); layer-shared mode: one per (b,l), writing H copies
  Share share{(int)blockIdx.x, 0, 1};
  if (COPY) share = share_of(blockIdx.x, gridDim.x, cp.lists, L, SHARED ? 1 : H, n, budgets);
  if (share.of == 0) return;
  const int unit = SHARED ? share.list * H : share.list;
  const int h = unit % H, bl = unit / H, l = bl % L, b = bl / L;
  const int k = budgets[(size_t)b * L + l];
  const int copies = SHARED ? H : 1;
  const long long off = layer_offsets[(size_t)b * (L + 1) + l] + (long long)h * k;
  const float* s = scores + (size_t)unit * n;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int i0 = wave * 64 * MAXC + lane * 4;

  // tokens past n get key 0, which no score has but the NaN of all set bits; equal keys are kept lowest token first
  // and k <= n, so that the surplus tokens, which come last, are never among the kept
  uint32_t key[MAXC];
  // All loads are under way before the first is looked at.  Lanes whose four tokens are not all there load the unit's last
  // four and move them down.  (Units of an odd number of tokens begin at any multiple of 4 bytes, which is all that a load
  // of 16 needs.)
  constexpr int kAhead = SHARED && MAXC > 16 ? 16 : MAXC;
#pragma unroll
  for (int j0 = 0; j0 < MAXC; j0 += kAhead) {
    float4u f[kAhead / 4];
    if (n >= 4) {
#pragma unroll
      for (int q = 0; q < kAhead / 4; ++q)
        f[q] = *reinterpret_cast<const float4u*>(s + min(i0 + (j0 + 4 * q) * 64, n - 4));
      if (SHARED) {
        for (int hh = 1; hh < H; ++hh) {
          const float* sh = s + (size_t)hh * n;
#pragma unroll
          for (int q = 0; q < kAhead / 4; ++q)
            f[q] += *reinterpret_cast<const float4u*>(sh + min(i0 + (j0 + 4 * q) * 64, n - 4));
        }
#pragma unroll
        for (int q = 0; q < kAhead / 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) f[q][e] = __fdiv_rn(f[q][e], (float)H);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) f[0][e] = score_at<SHARED>(s, max(n - 4 + e, 0), n, H);
#pragma unroll
      for (int q = 1; q < kAhead / 4; ++q) f[q] = f[0];
    }
#pragma unroll
    for (int q = 0; q < kAhead / 4; ++q) {
      uint32_t* g = key + j0 + 4 * q;
      const int past = i0 + (j0 + 4 * q) * 64 + 4 - n;     // tokens of the four that are past the last
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = order_key(f[q][e]);
      if (past > 0) {
        if (past & 1) { g[0] = g[1]; g[1] = g[2]; g[2] = g[3]; g[3] = 0u; }
        if (past & 2) { g[0] = g[2]; g[1] = g[3]; g[2] = g[3] = 0u; }
        if (past > 3) { g[0] = g[1] = g[2] = g[3] = 0u; }
      }
    }
  }
  if (k <= 0 || k > n || off < 0 || off + (long long)copies * k > rows_per_seq) return;   // bad budgets
  int* out = idx_out + (size_t)b * rows_per_seq + off;

#pragma unroll
  for (int q = 0; q < kPer; ++q) hist[tid * kPer + q] = 0;
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int j = 0; j < MAXC; ++j) {
    lo = min(lo, i0 + (j >> 2) * 256 + (j & 3) < n ? key[j] : 0xFFFFFFFFu);
    hi = max(hi, key[j]);
  }
  lo = wave_max_u32(~lo);                      // (~ of the lowest)
  hi = wave_max_u32(hi);
  if (lane == 63) { wave_a[wave] = ~lo; wave_b[wave] = hi; }
  lo = ~0u;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) { lo = min(lo, wave_a[w]); hi = max(hi, wave_b[w]); }
  lo = uniform(lo);
  hi = uniform(hi);

  // the k-th largest key is the need-th largest of the keys in [lo, hi]; `whole`: all of [lo, hi] is kept
  unsigned need = (unsigned)k;
  bool whole = false;
  while (hi > lo) {
    const uint32_t width = hi - lo;
    const int shift = max(0, 21 - __clz((int)width));          // width >> shift < 2048
#pragma unroll
    for (int j = 0; j < MAXC; ++j) {
      const uint32_t rel = key[j] - lo;
      if (rel <= width) atomicAdd(&hist[rel >> shift], 1u);
    }
    __syncthreads();
    // counts from the top: thread t has the kPer bins from 2047 - t kPer downwards
    unsigned c[kPer], mine = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      c[q] = hist[kSelBins - 1 - tid * kPer - q];
      hist[kSelBins - 1 - tid * kPer - q] = 0;
      mine += c[q];
    }
    const unsigned incl = wave_incl_scan(mine);
    if (lane == 63) wave_a[wave] = incl;
    __syncthreads();
    unsigned above = incl - mine;
    for (int w = 0; w < wave; ++w) above += wave_a[w];
    if (above < need && need <= above + mine) {
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        if (above < need && need <= above + c[q]) {
          sh_bin = kSelBins - 1 - tid * kPer - q;
          sh_need = need - above;
          sh_count = c[q];
        }
        above += c[q];
      }
    }
    __syncthreads();
    lo += uniform(sh_bin) << shift;
    hi = min(hi, lo + ((1u << shift) - 1u));
    need = uniform(sh_need);
    if (uniform(sh_count) == need) { whole = true; break; }
  }
  // kept: all keys from tau upwards
  uint32_t tau = lo;
  __syncthreads();                              // (wave_a and wave_b are still being read above)
  if (!whole) {
    // of the keys equal to tau only the `need` with the lowest token indices: keys are marked as kept or not
    uint32_t equal = 0;                         // of this wave
#pragma unroll
    for (int j = 0; j < MAXC; ++j) equal += __popcll(__ballot(key[j] == tau));
    if (lane == 0) wave_b[wave] = equal;
    __syncthreads();
    unsigned before = 0;
    for (int w = 0; w < wave; ++w) before += wave_b[w];
    before = uniform(before);
#pragma unroll
    for (int j = 0; j < MAXC; j += 4) {
      asm volatile("" : "+s"(tau));             // (or all groups' masks are made at once, in registers a second workgroup needs)
      unsigned mine = before;                   // before this lane's first token of the group
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned long long me = __ballot(key[j + e] == tau);
        mine = below_me(me, mine);
        before += __popcll(me);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool eq = key[j + e] == tau;
        key[j + e] = key[j + e] > tau || (eq && mine < need) ? 1u : 0u;
        mine += eq ? 1u : 0u;
      }
    }
    tau = 1u;
  }
  unsigned short* mine = stage + wave * 64 * MAXC;
  unsigned held = 0;                            // kept tokens of this wave, in `mine`
#pragma unroll
  for (int j = 0; j < MAXC; j += 4) {
    asm volatile("" : "+s"(tau));
    unsigned at = held;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned long long mk = __ballot(key[j + e] >= tau);
      at = below_me(mk, at);
      held += __popcll(mk);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool keep = key[j + e] >= tau;
      if (keep) mine[at] = (unsigned short)(i0 + j * 64 + e);
      at += keep ? 1u : 0u;
    }
  }
  if (lane == 0) wave_a[wave] = held;
  __syncthreads();
  unsigned pos = 0;                             // kept by lower waves
  for (int w = 0; w < wave; ++w) pos += wave_a[w];
  pos = uniform(pos);
  const unsigned r0 = COPY ? (unsigned)k * share.at / share.of : 0u, r1 = COPY ? (unsigned)k * (share.at + 1) / share.of : (unsigned)k;
  for (unsigned t = lane; t < held; t += 64) {
    const int token = mine[t];
    if (pos + t >= r0 && pos + t < r1) {
      if (COPY) list[pos + t - r0] = (unsigned short)token;
      for (int c = 0; c < copies; ++c) out[(size_t)c * k + pos + t] = token;
    }
  }
  if constexpr (COPY) {
    __syncthreads();
    const long long filled = layer_offsets[(size_t)b * (L + 1) + L];       // (no rows beyond what the budgets fill)
    const unsigned rows = r1 - r0, all = rows * (unsigned)copies * (unsigned)cp.vec_per_row;
    for (unsigned v = tid; v < all; v += NT) {
      const unsigned at = cp.vpr_shift >= 0 ? v >> cp.vpr_shift : v / (unsigned)cp.vec_per_row, part = (v - at * cp.vec_per_row) * 16;
      const unsigned c = SHARED ? at / rows : 0, i = at - c * rows;
      const int j = (int)(r0 + i), token = list[i];                        // kept row j of head h + c
      const long long packed = off + (long long)c * k + j;
      if (packed >= filled) continue;
      const long long src = (long long)b * cp.st.sb + (long long)l * cp.st.sl + (long long)(h + (int)c) * cp.st.sh + (long long)token * cp.st.sn;
      long long dst = (long long)b * rows_per_seq + packed;
      if (cp.pg.block_table) {
        const int slot_page = j / cp.pg.page_size;
        const long long page = slot_page < cp.pg.max_pages ? cp.pg.block_table[(long long)(unit + (int)c) * cp.pg.max_pages + slot_page] : -1;
        if (page < 0 || page >= cp.pg.num_pages) continue;                 // not a valid page: row skipped
        dst = page * cp.pg.page_size + (j - slot_page * cp.pg.page_size);
      }
      const size_t from = (size_t)src * cp.elem_bytes + part, to = (size_t)dst * cp.vec_per_row * 16 + part;
      const uint4v kv = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(cp.K + from));
      const uint4v vv = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(cp.V + from));
      __builtin_nontemporal_store(kv, reinterpret_cast<uint4v*>(cp.K_out + to));
      __builtin_nontemporal_store(vv, reinterpret_cast<uint4v*>(cp.V_out + to));
    }
  }
}

// A workgroup copies the `rows` kept rows from blockIdx.x * rows on (blockIdx.y is the sequence): a thread looks up where
// one of them is and goes, then each copies a 16-byte vector of a K row and the matching one of V (more than one vector of a
// long row).  Rows are read once and written once, so both sides bypass the caches' retention (non-temporal): the scores,
// budgets and indices the other workgroups need stay resident instead.  Bound by memory: 112 units that keep 6554 rows
// 128 us, 5.9 TB/s; with a lookup for each vector 152, with two, four or eight vectors of each tensor under way in a thread
// 133, 137 and 140, with K and V in workgroups of their own 163.
constexpr int kGatherThreads = 256;

template <bool PAGED>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(
    const char* __restrict__ K, const char* __restrict__ V, KvStrides st, int n, int elem_bytes,
    int vec_per_row, int vpr_shift, int rows, const int* __restrict__ budgets,
    const long long* __restrict__ layer_offsets, const int* __restrict__ idx, long long rows_per_seq,
    char* __restrict__ K_out, char* __restrict__ V_out, PagedDst pg) {
  __shared__ long long from[kGatherThreads], to[kGatherThreads];
  extern __shared__ long long offs[];                    // [L + 1]: the sequence's layer_offsets
  const int b = blockIdx.y, tid = threadIdx.x;
  const long long j = (long long)blockIdx.x * rows + tid;   // packed row of the sequence
  const bool mine = tid < rows && j < rows_per_seq;
  const long long grow = (long long)b * rows_per_seq + j;
  const int token = mine ? idx[grow] : -1;
  for (int i = tid; i <= st.L; i += kGatherThreads) offs[i] = layer_offsets[(size_t)b * (st.L + 1) + i];
  __syncthreads();
  if (tid < rows) {
    long long src = -1, dst = grow;
    if (mine && token >= 0 && token < n && j < offs[st.L]) {   // (no rows beyond what the budgets fill)
      // largest l with offs[l] <= j
      int lo = 0, hi = st.L;                             // invariant: offs[lo] <= j < offs[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offs[mid] <= j) lo = mid; else hi = mid;
      }
      const int l = lo, k = budgets[(size_t)b * st.L + l];
      const long long in_layer = j - offs[l];            // < H * k
      if (k > 0 && in_layer < (long long)st.H * k) {
        const int h = (int)((unsigned)in_layer / (unsigned)k);
        src = ((long long)b * st.sb + (long long)l * st.sl + (long long)h * st.sh + (long long)token * st.sn) * elem_bytes;
        if (PAGED) {
          const long long jj = in_layer - (long long)h * k;            // row within the unit
          const long long slot_page = jj / pg.page_size;
          const long long unit = ((long long)b * st.L + l) * st.H + h;
          const long long page = slot_page < pg.max_pages ? pg.block_table[unit * pg.max_pages + slot_page] : -1;
          if (page < 0 || page >= pg.num_pages) src = -1;              // not a valid page: row skipped
          dst = page * pg.page_size + jj % pg.page_size;
        }
      }
    }
    from[tid] = src;
    to[tid] = dst * vec_per_row * 16;
  }
  __syncthreads();
  for (int v = tid; v < rows * vec_per_row; v += kGatherThreads) {
    const int r = vpr_shift >= 0 ? v >> vpr_shift : v / vec_per_row, part = (v - r * vec_per_row) * 16;
    if (from[r] < 0) continue;
    const uint4v kv = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(K + from[r] + part));
    const uint4v vv = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(V + from[r] + part));
    __builtin_nontemporal_store(kv, reinterpret_cast<uint4v*>(K_out + to[r] + part));
    __builtin_nontemporal_store(vv, reinterpret_cast<uint4v*>(V_out + to[r] + part));
  }
}

}  // namespace

hipError_t select_gather_launch(const void* K, const void* V, const fc_kv_desc& d, const float* scores,
                                const int32_t* budgets, const int64_t* layer_offsets,
                                int64_t rows_per_seq, bool shared, int32_t* idx_out, void* K_out,
                                void* V_out, const int32_t* block_table, int32_t page_size,
                                int32_t max_pages, int64_t num_pages, hipStream_t s) {
  const int units = d.batch * d.layers * d.kv_heads;
  if (units == 0 || rows_per_seq == 0) return hipSuccess;
  const long long* offs = reinterpret_cast<const long long*>(layer_offsets);
  const int elem_bytes = d.dtype == FC_BF16 ? 2 : 4;
  const int vec_per_row = d.head_dim * elem_bytes / 16;
  int vpr_shift = -1;
  if ((vec_per_row & (vec_per_row - 1)) == 0)
    for (vpr_shift = 0; (1 << vpr_shift) < vec_per_row; ++vpr_shift) {}
  const PagedDst pg{block_table, page_size, max_pages, (long long)num_pages};
  const int lists = shared ? units / d.kv_heads : units;           // index sets to be found
  const int groups = copy_groups(lists, d.layers, d.n_tokens, shared ? d.kv_heads : 1, (long long)rows_per_seq * d.batch, vec_per_row,
                                 block_table != nullptr);
  {
    ProfileScope ps(shared ? "select_shared_kernel" : "select_kernel", s);
    const dim3 grid(groups ? groups : lists);
    const CopyArgs cp{static_cast<const char*>(K), static_cast<const char*>(V), strides_of(d), lists, elem_bytes, vec_per_row, vpr_shift,
                      static_cast<char*>(K_out), static_cast<char*>(V_out), pg};
    const long long rows = (long long)rows_per_seq;
    const int n = d.n_tokens;
#define FC_SELECT(SH, NT, MAXC)                                                                               \
  hipLaunchKernelGGL((select_kernel<SH, NT, MAXC, false>), grid, dim3(NT), 0, s, scores, budgets, offs,        \
                     d.layers, d.kv_heads, n, rows, idx_out, cp)
#define FC_SELECT_COPY(SH, NT, MAXC)                                                                          \
  if (groups)                                                                                                 \
    hipLaunchKernelGGL((select_kernel<SH, NT, MAXC, true>), grid, dim3(NT), 0, s, scores, budgets, offs,       \
                       d.layers, d.kv_heads, n, rows, idx_out, cp);                                           \
  else FC_SELECT(SH, NT, MAXC)
    // The fewest keys per thread that cover n, and more waves while the barriers they wait at cost less than the keys
    // they share out (us at 16 and at 896 units): 2048 tokens, 512 threads of 4 keys 7.8 / 12.2, 256 of 16 11.2 / 15.5;
    // 4096 tokens, 512 threads of 8 9.4 / 15.6, 1024 of 4 8.9 / 19.8; 8192 tokens, 1024 of 8 11.4 / 26.6, 512 of 16
    // 12.1 / 25.9; 16384 tokens, 1024 of 16 15.3 / 52.6, 512 of 32 19.2 / 48.7.
#define FC_SELECT_N(SH)                                                                                        \
  static_assert(select_threads(1024) == 256 && select_threads(4096) == 512 && select_threads(4097) == 1024);                    \
  if (n <= 1024) { FC_SELECT_COPY(SH, 256, 4); }                                                               \
  else if (n <= 2048) { FC_SELECT_COPY(SH, 512, 4); }                                                          \
  else if (n <= 4096) { FC_SELECT_COPY(SH, 512, 8); }                                                          \
  else if (n <= 8192) { FC_SELECT_COPY(SH, 1024, 8); }                                                         \
  else if (n <= 16384) { FC_SELECT_COPY(SH, 1024, 16); }                                                       \
  else FC_SELECT(SH, 1024, 32)
    if (n <= 32 * kSelThreads) {
      if (shared) { FC_SELECT_N(true); } else { FC_SELECT_N(false); }
    } else if (n <= kSelMaxChunk * kSelThreads) {
      if (shared) FC_SELECT(true, 1024, 64); else FC_SELECT(false, 1024, 64);
#undef FC_SELECT_N
#undef FC_SELECT_COPY
#undef FC_SELECT
    } else if (shared) {
      hipLaunchKernelGGL(select_large_kernel<true>, grid, dim3(kSelThreads), 0, s, scores, budgets, offs, d.layers,
                         d.kv_heads, n, rows, idx_out);
    } else {
      hipLaunchKernelGGL(select_large_kernel<false>, grid, dim3(kSelThreads), 0, s, scores, budgets, offs, d.layers,
                         d.kv_heads, n, rows, idx_out);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || groups) return e;
  // rows of a workgroup: one turn of its threads' copies, if it has a thread for each of them
  const int rows = std::min(kGatherThreads, std::max(1, kGatherThreads / vec_per_row));
  const long long blocks = (rows_per_seq + rows - 1) / rows;
  if (blocks > 0x7FFFFFFFll || d.batch > 65535) return hipErrorInvalidValue;
  ProfileScope ps("gather_kernel", s);
  const dim3 grid((unsigned)blocks, (unsigned)d.batch);
  const size_t lds = (size_t)(d.layers + 1) * sizeof(long long);
  if (block_table)
    hipLaunchKernelGGL(gather_kernel<true>, grid, dim3(kGatherThreads), lds, s, static_cast<const char*>(K),
                       static_cast<const char*>(V), strides_of(d), d.n_tokens, elem_bytes, vec_per_row,
                       vpr_shift, rows, budgets, offs, idx_out, (long long)rows_per_seq, static_cast<char*>(K_out),
                       static_cast<char*>(V_out), pg);
  else
    hipLaunchKernelGGL(gather_kernel<false>, grid, dim3(kGatherThreads), lds, s, static_cast<const char*>(K),
                       static_cast<const char*>(V), strides_of(d), d.n_tokens, elem_bytes, vec_per_row,
                       vpr_shift, rows, budgets, offs, idx_out, (long long)rows_per_seq, static_cast<char*>(K_out),
                       static_cast<char*>(V_out), pg);
  return hipGetLastError();
}

}  // namespace fc
