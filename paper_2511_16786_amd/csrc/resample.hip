// Resampled realisation of the low-pass projection (Eq. 6-10): any token count, cost nearly
// independent of the cut-off.
//
// Base KV holds only the r lowest DCT modes, so it lives on a grid of M ~ 2r points as well as on the
// N tokens.  With the even extension of period 2N, token i sits at grid position u_i = (i + 1/2) M/N - 1/2
// and a window function phi of W grid points (Kaiser-Bessel) moves values between the two:
//     g[k]    = sum_i phi(u_i - k) x[i]            decimate_kernel     N -> M, banded product
//     b       = DCT^-1( f . DCT(g) )               grid_filter_kernel  length M, f[m] = 1 / (N phihat(m)^2), m < r
//     base[i] = sum_k phi(u_i - k) b[k]            residual_kernel     M -> N, banded product, fused with the score
// phihat is phi's Fourier transform; what the window lets through beyond the grid's own modes is the
// only approximation.  It is largest for the mode just below the cut-off, and kept below fp32's rounding of
// that mode, 6e-8, by the choice of W, see window_points.  The same operator serves every N, since the token
// positions enter through the window weights alone.
//
// The banded products run on the matrix cores with their operands split so that fp32 accuracy is kept:
// bf16 inputs are exact and meet weights split in three bf16 terms; on the way back weights are three fp16
// terms (more than fp32 holds) and grid values, scaled to a common exponent per window and 8 columns, two
// (23 bits: they come out of a transform in fp32), and only products below 2^-33 of the whole are left out.
// Sums over columns and tokens are in 64 bits from 32 squares on, of the rows' own squares (Etot) from 8 on: sums of bf16
// squares in 32 bits come out low, 1.2e-8 after 32, 6.5e-9 after 8.
#include <algorithm>
#include <type_traits>

#include "fc_common.h"
#include "rules.h"

namespace fc {

namespace {

template <int V>
using Int = std::integral_constant<int, V>;

constexpr int kMaxTilesPerWin = 16;    // 16-token tiles one wave of the residual kernel walks
constexpr float kInvWeightScale = 4096.0f;   // fp16 weights are stored times 2^12 (their tails stay normal numbers)

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

union Frag {
  u32x4 u;
  bf16v8 b;
  f16x8 h;
  _Float16 hs[8];
};

// ---------------------------------------------------------------------------- tables

// I0 by its power series in q = x^2/4 (all terms positive); the arguments stay below 10 pi 5/6 = 26.2 (9 pi = 28.3
// for 9 points), where the 48th term is 1e-22 of the sum.
struct I0Series {
  double c[48];
  constexpr I0Series() : c{} {
    double f = 1.0;
    for (int k = 0; k < 48; ++k) { c[k] = f; f /= (double)(k + 1) * (double)(k + 1); }
  }
};
__host__ __device__ __forceinline__ double bessel_i0(double q) {
  constexpr I0Series t;
  double sum = t.c[47];
#pragma unroll
  for (int k = 46; k >= 0; --k) sum = fma(sum, q, t.c[k]);
  return sum;
}

// Grid points a token's window reaches (W), by the grid points per kept mode.  Error of the projection of mode r - 1
// in 64 bits, the largest over N / M from 1 to 11 (white columns: a tenth of it):
//   M / r     1.75     1.87     2.0      2.25     2.5      3.0      5.0
//   W =  9    3.5e-7   1.6e-7   1.7e-7   6e-8     2.8e-8   8.4e-9   1.0e-9
//   W = 10    4.6e-8   2.0e-8   2.0e-8   6e-9     2.7e-9   7.6e-10
//   W = 11    6.6e-9   2.6e-9   2.3e-9   6e-10
// A wider window also multiplies the rounding of the grid's points by more (1 / phihat at the cut-off: 5.5, 6.6 and 8 at
// 1.75), and what comes out for that mode on the device, 2048 tokens, r = 585, is 3.6e-7, 2.0e-7 and 2.5e-7.
__host__ __device__ constexpr int window_points(int r, int m) { return m < 3 * (int64_t)r ? 10 : 9; }

struct Window {
  int w;
  double beta, inv_i0;
};
Window make_window(int r, int m) {
  const int w = window_points(r, m);
  const double beta = M_PI * w * (1.0 - 0.5 * (double)r / (double)m);
  return {w, beta, 1.0 / bessel_i0(0.25 * beta * beta)};
}

// weight between token position u and grid point k, images of the even extension included
__device__ double weight_at(double u, int k, int m, const Window& w) {
  double sum = 0.0;
#pragma unroll 1
  for (int image = 0; image < 3; ++image) {
    const double s = image == 0 ? u - k : (image == 1 ? u + 1.0 + k : 2.0 * m - 1.0 - k - u);
    const double z = s * (2.0 / w.w), t = 1.0 - z * z;
    if (t >= 0.0) sum += bessel_i0(0.25 * w.beta * w.beta * t) * w.inv_i0;
  }
  return sum;
}

// First 32-token step under a tile of 16 grid points, and first grid point (a multiple of four) of a window that begins with
// token `first`: the tables are made for them and the kernels derive them anew, which is quicker than to read them.
__host__ __device__ __forceinline__ int first_step(int tile, int n, int steps, double dd, int w) {
  const int t = (int)ceil(fma(dd, 16.0 * tile - 0.5 * w + 0.5, -0.5));
  return min(max(0, t) / 32, (n + 31) / 32 - steps);
}
__host__ __device__ __forceinline__ int first_point(int first, int m, double inv_dd, int w) {
  const int k0 = (int)ceil(fma(first + 0.5, inv_dd, -0.5) - 0.5 * w);
  return max(0, min(k0, m - 32)) & ~3;
}
// steps that the tile's windows reach into
__host__ __device__ __forceinline__ int step_count(int tile, int s0, int n, int steps, double dd, int w) {
  const int last = min(n - 1, (int)floor(fma(dd, 16.0 * tile + 15.5 + 0.5 * w, -0.5)));
  return min(last / 32 + 1 - s0, steps);
}

// Grid point of a tile that lane & 15 = l of the decimation holds: even points in lanes 0 to 7, odd ones in 8 to 15, of
// each the first half ascending, the second descending, so that lanes that mirror each other hold neighbours.
__host__ __device__ __forceinline__ int lane_point(int l) {
  return (l & 4 ? 4 * (3 - (l & 3)) + 2 : 4 * (l & 3)) + (l >> 3);
}

// position of grid point k in the order the transform takes its input (even points ascending, then
// odd points descending)
__device__ __forceinline__ int grid_pos(int k, int m) { return (k & 1) ? m - 1 - (k >> 1) : k >> 1; }

struct TablePtrs {
  WsHeader* hdr;
  float* wfwd;       // [M/16][steps][2][64][4]
  _Float16* winv;    // [tokens/16][3][64][8] fp16
  float2* filt;      // [M] (f[m] + f[M-m]) / 2, (f[m] - f[M-m]) / 2
  void* twid;        // see GridFft: float2, or double2 for a wide transform
};

// Passes of the grid transform: M = R0 R1 R2 R3 (a radix 1 is no pass) by M / P threads that keep P points each.
// More points a thread mean fewer passes and exchanges, fewer points more waves: 8192 transforms of 6144 and of 12288
// points take 258 and 530 us with 48 a thread in three passes, 269 and 807 with 24 in four.
// Twiddle table: for every pass after the first, powers 1..7 and 8, 16, .. (below R) of w_{R NS}^j, NS the product of
// the radices before it, j < NS, or j < threads for the last pass; then e^{i pi t / M}.
// A wide transform (see wide_transform, lengths from 128 to 4096) has twice the registers per point under work: 3072
// points take four passes, 294 us for 14336 column pairs, instead of three with spilled registers, 366.
struct GridRadices {
  int p, r[4];
};
__host__ __device__ constexpr GridRadices grid_radices(int m, bool wide) {
  switch (m) {
    case 64: return {8, {8, 8, 1, 1}};
    case 96: return {24, {8, 12, 1, 1}};
    case 128: return {16, {8, 16, 1, 1}};
    case 192: return {24, {8, 24, 1, 1}};
    case 256: return {16, {16, 16, 1, 1}};
    case 384: return {24, {8, 8, 6, 1}};
    case 512: return {16, {8, 8, 8, 1}};
    case 768: return {24, {8, 8, 12, 1}};
    case 1024: return {16, {8, 8, 16, 1}};
    case 1536: return {24, {8, 8, 24, 1}};
    case 2048: return {16, {8, 16, 16, 1}};
    case 3072: return wide ? GridRadices{24, {8, 8, 8, 6}} : GridRadices{48, {16, 16, 12, 1}};
    case 4096: return {32, {16, 16, 16, 1}};
    case 6144: return {48, {16, 16, 24, 1}};
    case 8192: return {32, {16, 16, 32, 1}};
    case 12288: return {48, {16, 16, 48, 1}};
    case 16384: return {32, {32, 32, 16, 1}};
    case 24576: return {48, {16, 16, 16, 6}};
    case 32768: return {32, {32, 32, 32, 1}};
    default: return {48, {16, 48, 48, 1}};         // 36864
  }
}
__host__ __device__ constexpr int grid_threads(int m, bool wide) { return m / grid_radices(m, wide).p; }
__host__ __device__ constexpr int twid_powers(int r) { return (r < 8 ? r : 8) - 1 + (r - 1) / 8; }
// first entry of the factors of pass k (k = 1, 2, 3), and of the phases for the first k that is no pass
__host__ __device__ constexpr int twid_off(int m, bool wide, int k) {
  const GridRadices g = grid_radices(m, wide);
  int off = 0, ns = g.r[0];
  for (int i = 1; i < k && i < 4 && ns < m; ++i) {
    off += twid_powers(g.r[i]) * (ns * g.r[i] == m ? m / g.p : ns);
    ns *= g.r[i];
  }
  return off;
}
__host__ __device__ constexpr int twid_phase_off(int m, bool wide) { return twid_off(m, wide, 4); }
// ... then e^{-2 pi i k / P} and e^{-pi i k / P}, k < P, which the transform's own code holds as constants
__host__ __device__ constexpr int twid_root_off(int m, bool wide) { return twid_phase_off(m, wide) + grid_threads(m, wide); }
__host__ __device__ constexpr int twid_size(int m, bool wide) { return twid_root_off(m, wide) + 2 * grid_radices(m, wide).p; }

// cos(2 pi k / 192) of the first quadrant; every constant root the transforms use is on this circle
__device__ constexpr double kCos192[49] = {
    1.0, 0.9994645874763657, 0.9978589232386035, 0.9951847266721969, 0.9914448613738104, 0.986643332084879,
    0.9807852804032304, 0.9738769792773336, 0.9659258262890683, 0.9569403357322088, 0.9469301294951057,
    0.9359059267573258, 0.9238795325112867, 0.9108638249211758, 0.8968727415326884, 0.881921264348355,
    0.8660254037844387, 0.8492021815265789, 0.8314696123025452, 0.8128466845916152, 0.7933533402912352,
    0.773010453362737, 0.7518398074789774, 0.7298640726978357, 0.7071067811865476, 0.6835923020228712,
    0.6593458151000688, 0.6343932841636455, 0.6087614290087207, 0.5824776968678022, 0.5555702330196024,
    0.5280678506503681, 0.5, 0.4713967368259976, 0.44228869021900125, 0.4127070298043947, 0.38268343236508984,
    0.3522500479212336, 0.3214394653031617, 0.2902846772544625, 0.25881904510252074, 0.22707626303437345,
    0.19509032201612833, 0.16289547339458882, 0.1305261922200517, 0.09801714032956055, 0.06540312923014327,
    0.032719082821776165, 0.0};
__device__ constexpr double cos192(int k) {
  k %= 192;
  if (k > 96) k = 192 - k;
  return k <= 48 ? kCos192[k] : -kCos192[96 - k];
}
// e^{-2 pi i k / n}, n a divisor of 192
template <typename C>
__device__ __forceinline__ constexpr C root(int k, int n) {
  typedef decltype(C::x) R;
  return C{(R)cos192(k * (192 / n)), (R)cos192(k * (192 / n) + 48)};
}

__device__ double2 unit_root(double frac) {       // e^{-2 pi i frac}
  double s, c;
  sincospi(2.0 * frac, &s, &c);
  return make_double2(c, -s);
}

// What the table kernel has to know of a plan's twiddle factors, made on the host: looked up on the device, the radices
// are an array under a running index, for which all of the kernel's threads had scratch memory and 20 KiB of LDS: 11.7 us
// instead of 7.6 at 7321 tokens.
struct TwidPlan {
  int off[4];                                      // factors of passes 1, 2 and 3 (a pass that is none: empty), phases
  int stride[3], low[3], len[3];
  int p, roots, size;
};
TwidPlan make_twid_plan(int m, bool wide) {
  const GridRadices g = grid_radices(m, wide);
  TwidPlan t{};
  int ns = g.r[0];
  for (int k = 1; k < 4; ++k) {
    const int len = ns * g.r[k];
    t.off[k - 1] = twid_off(m, wide, k);
    t.stride[k - 1] = len == m ? m / g.p : ns;
    t.low[k - 1] = std::min(g.r[k], 8) - 1;
    t.len[k - 1] = len;
    ns = len;
  }
  t.off[3] = twid_phase_off(m, wide);
  t.p = g.p; t.roots = twid_root_off(m, wide); t.size = twid_size(m, wide);
  return t;
}

// One thread per weight and per table entry; runs once per plan, and a prompt of a new length waits for it.  The
// weights' series are the work: as fused multiply-adds with constant factors, one weight a thread and the window's
// own constants from the host, 12 us at 7321 tokens where a thread of eight weights, each with a division per term,
// took 52 us; 7.6 us since the twiddle factors' radices come from the host as well.
__global__ __launch_bounds__(256) void resample_table_kernel(TablePtrs tp, int n, int r, int m, int d, int dtype,
                                                             int steps, int tpw, int n_wfwd, int n_winv, bool wide, Window win,
                                                             TwidPlan plan) {
  int id = blockIdx.x * blockDim.x + threadIdx.x;
  const double dd = (double)n / (double)m;        // tokens per grid point
  const double inv_dd = (double)m / (double)n;
  if (id == 0) {
    WsHeader h{};
    h.magic = kWsMagic; h.path = FC_PATH_RESAMPLE; h.n = n; h.r = r; h.d = d; h.dtype = dtype;
    *tp.hdr = h;
  }
  if (id < n_wfwd) {
    const int o = id & 511, lane = (o >> 2) & 63, e = (o >> 8) * 4 + (o & 3);
    const int step = (id >> 9) % steps, tile = (id >> 9) / steps;
    const int s0 = first_step(tile, n, steps, dd, win.w);
    // the last step slides back to end with the last token and takes only what earlier steps have not
    const int i = min(32 * (s0 + step), n - 32) + 8 * (lane >> 4) + e;
    tp.wfwd[id] =
        i >= 32 * (s0 + step) ? (float)weight_at((i + 0.5) * inv_dd - 0.5, 16 * tile + lane_point(lane & 15), m, win) : 0.0f;
    return;
  }
  id -= n_wfwd;
  if (id < n_winv) {
    const int o = id & 511, lane = o >> 3, e = o & 7, tile = id >> 9, g = lane >> 4, first = tile / tpw * tpw;
    const int k0 = first_point(16 * first, m, inv_dd, win.w);
    const int i = 16 * tile + (lane & 15);
    // the order in which the residual kernel's loads deliver the window's grid points
    const int k = e < 4 ? k0 + 2 * (8 * (e >> 1) + 2 * g + (e & 1)) : k0 + 2 * (31 - 8 * (e >> 1) - 2 * g - (e & 1)) + 1;
    const double w = i < n ? kInvWeightScale * weight_at((i + 0.5) * inv_dd - 0.5, k, m, win) : 0.0;
    _Float16* p = tp.winv + (size_t)tile * 1536 + o;
    double rest = w;
    for (int q = 0; q < 3; ++q) {
      const _Float16 t = (_Float16)(float)rest;
      p[512 * q] = t;
      rest -= (double)t;
    }
    return;
  }
  id -= n_winv;
  if (id < m) {
    auto f = [&](int q) -> double {
      if (q >= r) return 0.0;
      const double a = 0.5 * M_PI * win.w * q / m;
      const double s = sqrt(win.beta * win.beta - a * a);
      const double ph = win.w * sinh(s) / s * win.inv_i0;
      return 1.0 / ((double)n * ph * ph);
    };
    const double fa = f(id), fb = f(m - id);
    tp.filt[id] = make_float2((float)(0.5 * (fa + fb)), (float)(0.5 * (fa - fb)));
    return;
  }
  id -= m;
  if (id >= plan.size) return;
  double2 v;
  if (id >= plan.roots) {
    const int k = id - plan.roots;
    v = k < plan.p ? root<double2>(k, plan.p) : root<double2>(k - plan.p, 2 * plan.p);
  } else {
    double frac = 0.5 * (double)(id - plan.off[3]) / (double)m;
    if (id >= plan.off[3]) {
      frac = -frac;
    } else {
      const int k = id >= plan.off[2] ? 2 : (id >= plan.off[1] ? 1 : 0);
      const int off = k == 2 ? plan.off[2] : (k == 1 ? plan.off[1] : plan.off[0]);
      const int stride = k == 2 ? plan.stride[2] : (k == 1 ? plan.stride[1] : plan.stride[0]);
      const int low = k == 2 ? plan.low[2] : (k == 1 ? plan.low[1] : plan.low[0]);
      const int len = k == 2 ? plan.len[2] : (k == 1 ? plan.len[1] : plan.len[0]);
      const int j = id - off, slot = j / stride, power = slot < low ? slot + 1 : 8 * (slot - low + 1);
      frac = (double)(power * (j - slot * stride)) / (double)len;
    }
    v = unit_root(frac);
  }
  if (wide) static_cast<double2*>(tp.twid)[id] = v;
  else static_cast<float2*>(tp.twid)[id] = make_float2((float)v.x, (float)v.y);
}

// ---------------------------------------------------------------------------- decimation

// A lane's piece of a row is 16 bytes, so that a load takes whole lines; the 2*nb pieces of a unit's K and V rows are dealt out
// to waves of 16 slots.  (With pieces of 8 columns for fp32 too, each load took every other 16 bytes of its lines, rows could not be read past
// the cache, and a wave had twice the work: scoring, us, with 8 columns / with 4: 112 units of 8192 tokens 573 / 507, 64 of
// 20000, r = 4001 1117 / 984, 4 of 13648, 64 columns 34.8 / 32.1, 32 of 8192, 256 columns 328 / 292, two of 512 26.9 / 19.5.)
template <typename T>
constexpr int kCols = 16 / (int)sizeof(T);
struct SlotMap {
  int nb;        // pieces per tensor (head_dim / kCols)
  int wpu;       // waves per unit
};

// A piece of one row, read with (KEEP) or without a claim on the last-level cache (see round_keeps_rows).
template <bool KEEP, typename V>
__device__ __forceinline__ V load_piece(const void* p) {
  if constexpr (KEEP) return *static_cast<const V*>(p);
  return __builtin_nontemporal_load(static_cast<const V*>(p));
}
// From a uniform address and 32 bits of the lane's own.
template <typename V>
__device__ __forceinline__ V lane_load(const void* base, uint32_t at) {
  typedef const __attribute__((address_space(1))) V* Global;
  return *(Global)(static_cast<const char*>(base) + at);
}
template <typename T>
struct RowPiece;

template <>
struct RowPiece<uint16_t> {
  u32x4 v;
  template <bool KEEP>
  __device__ __forceinline__ void load(const uint16_t* p) { v = load_piece<KEEP, u32x4>(p); }
};
template <>
struct RowPiece<float> {
  f32x4 v;
  template <bool KEEP>
  __device__ __forceinline__ void load(const float* p) { v = load_piece<KEEP, f32x4>(p); }
};

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ f32x4 mfma_bf16(const Frag& a, const Frag& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.b, b.b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f16(const Frag& a, const Frag& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c, 0, 0, 0);
}

// Operand of column j of the 8 rows in x (a lane's 8 rows are 8 consecutive terms of the contraction).
__device__ __forceinline__ void column_frag(const RowPiece<uint16_t> (&x)[8], int j, Frag (&a)[1]) {
#pragma unroll
  for (int p = 0; p < 4; ++p)
    a[0].u[p] = __builtin_amdgcn_perm(x[2 * p + 1].v[j >> 1], x[2 * p].v[j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
}
// Word h of three operands that hold a and b in bf16 terms, a = t0 + t1 + t2 (24 bits), each rounded to nearest.
__device__ __forceinline__ void bf16_terms(float a, float b, Frag (&t)[3], int h) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const bf16x2 p = __builtin_convertvector((f32x2{a, b}), bf16x2);
    const uint32_t u = __builtin_bit_cast(uint32_t, p);
    t[q].u[h] = u;
    a -= __uint_as_float(u << 16);
    b -= __uint_as_float(u & 0xFFFF0000u);
  }
}
__device__ __forceinline__ void column_frag(const RowPiece<float> (&x)[8], int j, Frag (&a)[3]) {
#pragma unroll
  for (int p = 0; p < 4; ++p) bf16_terms(x[2 * p].v[j], x[2 * p + 1].v[j], a, p);
}
__device__ __forceinline__ f32x4 fold_column(const Frag (&a)[1], const Frag (&w)[3], f32x4 acc) {
#pragma unroll
  for (int q = 2; q >= 0; --q) acc = mfma_bf16(a[0], w[q], acc);
  return acc;
}
__device__ __forceinline__ f32x4 fold_column(const Frag (&a)[3], const Frag (&w)[3], f32x4 acc) {
  // the products below 2^-24 of the whole are left out
  acc = mfma_bf16(a[2], w[0], acc);
  acc = mfma_bf16(a[0], w[2], acc);
  acc = mfma_bf16(a[1], w[1], acc);
  acc = mfma_bf16(a[1], w[0], acc);
  acc = mfma_bf16(a[0], w[1], acc);
  return mfma_bf16(a[0], w[0], acc);
}

// The order of the steps of a wave that walks tiles of one group of four (for each tile the same, whether by itself or with others
// of its group in a wave): odd groups are walked from their end; even ones take the steps that they share with the group
// before from the last to the first, then the others from the first to the last, then the ones shared with the next group from
// the last again.  So neighbours take what they share in the same order and, where they begin together, at the same time.
struct StepOrder {
  int first, low, high, end;          // steps below low, and those from high on, in descending order
  __device__ __forceinline__ int at(int i) const {
    const int s = first + i;
    return s < low ? low - 1 - i : (s < high ? s : end - 1 - (s - high));
  }
};

constexpr int kDecWaves = 4;          // waves of a workgroup: 4 slots' worth of rows under the same tiles

// One wave: GT tiles of 16 grid points x 16 slots (128 columns), walking the tokens under the tiles'
// windows in steps of 32.  Rows go from memory straight into matrix operands: a lane loads 16 bytes of 8
// consecutive rows and swaps the halves of the words in registers (the order of the contraction is free).
// The tiles' weights are in LDS as fp32 and are split in three bf16 terms when a step uses them.
// Bound by the rows' way through the fabric: 16 tiles apart, rows under the seams are read twice, so GT is
// as large as registers allow; results do not depend on it (a tile's steps and their order are its own).  A tile walks
// the steps that its windows reach into, one fewer than the most any tile has for two tiles in three (12288 points
// for 32768 tokens: 757 instead of 800 us for 112 units).
// (one tile a wave reads the rows 1.75 times).  Neighbours take the rows they share in the same order (StepOrder), so that those
// that begin together find them in the L2, which holds some 5 us of what passes through it: 32768 tokens M = 3072 438 / 424 us, 8192 130 /
// 127, M = 12288 656 / 643, fp32 8192 228 / 221 (before: both towards the seam or away from it, a step apart at its middle alone).
// Results leave in 16 bytes and whole 128-byte lines, two tiles side by side: the
// writes, a seventh of the traffic, cost a quarter of the time as half lines of 8 bytes a lane.  112 units, us before both /
// walked both ways / now: 32768 tokens M = 3072 472 / 470 / 457 (1.09 GB read a round for 0.94 GB of rows, was 1.11; 0.19
// written), M = 12288 750 / 717 / 671, 30011 tokens 541 / 535 / 503, 8192 tokens 146 / 144 / 136; with the weights ahead of
// the rows 436, 653, 470 and 131 (5.8 TB/s).  Three to five steps of rows under way in the one-tile variant are no quicker.
template <typename T, int GT, bool KEEP>
__global__ __launch_bounds__(64 * kDecWaves, 2) void decimate_kernel(
    const T* __restrict__ K, const T* __restrict__ V, KvStrides st, int u0, int u1, int n, int r, int d, int dtype,
    int m, int steps, SlotMap sm, int groups, int along, WsHeader* hdr, const float* __restrict__ wfwd,
    float2* __restrict__ grid) {
  constexpr int kTerms = sizeof(T) == 2 ? 1 : 3;
  constexpr int C = kCols<T>;
  constexpr int kBuf = 2;                         // steps of rows under way (a step's registers are refilled in place)
  extern __shared__ f32x4 wlds[];                 // [GT][steps][2][64]
  const int slot_id = blockIdx.x >> 3;
  const Span mine_t = xcd_first(blockIdx.x & 7, along, (m / 16 + GT - 1) / GT), mine_g = xcd_second(blockIdx.x & 7, along, groups);
  if (slot_id >= mine_t.count * mine_g.count) return;
  const int row = (unsigned)slot_id / (unsigned)mine_t.count;
  const int group = mine_g.from + row, super = mine_t.from + slot_id - row * mine_t.count;
  const int tile0 = super * GT, n_tiles = min(GT, m / 16 - tile0);
  const int lane = threadIdx.x & 63;
  const int gw = group * kDecWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = u0 + gw / sm.wpu, part = gw % sm.wpu;
  const bool mine = unit < u1;
  const int slot = lane_slot(part, lane & 15, 2 * sm.nb);
  const bool second = slot >= sm.nb;
  const double dd = (double)n / (double)m;        // tokens per grid point
  int first[GT], count[GT], s_end = 0;            // a tile's first step, and how many it has
  // (a lane works out a tile: the one before the group of four, its own four, the one after)
  const int before = (tile0 & ~3) - 1, tiles = m / 16, lanes_tile = min(max(before + min(lane, 5), 0), tiles - 1);
  const int lanes_first = first_step(lanes_tile, n, steps, dd, window_points(r, m));
  const int lanes_count = step_count(lanes_tile, lanes_first, n, steps, dd, window_points(r, m));
#pragma unroll
  for (int q = 0; q < GT; ++q) {
    const int from = tile0 - before + min(q, n_tiles - 1);
    first[q] = __builtin_amdgcn_readlane(lanes_first, from);
    const int c = __builtin_amdgcn_readlane(lanes_count, from);
    count[q] = q < n_tiles ? c : 0;
    s_end = first[q] + c;
  }
  StepOrder order{first[0], first[0], first[0], s_end};
  if (!(tile0 & 4)) {
    // (with fewer than two tokens for each grid point nearly all steps are shared, and even groups are walked from the first)
    const bool meets = n >= 2 * m;
    if (meets && before >= 0)
      order.low = min(max(__builtin_amdgcn_readlane(lanes_first, 0) + __builtin_amdgcn_readlane(lanes_count, 0), first[0]), s_end);
    order.high = meets && before + 5 < tiles ? min(max(__builtin_amdgcn_readlane(lanes_first, 5), order.low), s_end) : s_end;
  }
  const T* p = (second ? V : K) + unit_offset(st, mine ? unit : u0) + (slot - (second ? sm.nb : 0)) * C +
               (int64_t)(8 * (lane >> 4)) * st.sn;
  RowPiece<T> x[kBuf][8];
  auto load = [&](RowPiece<T> (&v)[8], int s) {
    const T* ps = p + min(32 * s, n - 32) * st.sn;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e].template load<KEEP>(ps + e * st.sn);
  };
  const int steps_all = s_end - first[0];
  // The weights, four loads at a time and the first ahead of the rows, for which they would wait otherwise (one at a time
  // behind the rows, 28 layers: 32768 tokens 445 us, 436 now; 8192 tokens 134.5, 131.4; one layer of these 11.6, 11.0).
  const f32x4* w_src = reinterpret_cast<const f32x4*>(wfwd) + (size_t)tile0 * steps * 128;
  const int w_last = n_tiles * steps * 128 - 1;
  f32x4 wt[4];
  auto load_weights = [&](int i) {
#pragma unroll
    for (int k = 0; k < 4; ++k) wt[k] = w_src[min(i + k * 64 * kDecWaves, w_last)];
  };
  load_weights(threadIdx.x);
#pragma unroll
  for (int b = 0; b < kBuf; ++b)
    if (b == 0 || b < steps_all) load(x[b], order.at(b));
  if (ws_mismatch(hdr, FC_PATH_RESAMPLE, n, r, d, dtype)) return;     // (while all that is on its way)
  for (int i = threadIdx.x;;) {
#pragma unroll
    for (int k = 0; k < 4; ++k) wlds[min(i + k * 64 * kDecWaves, w_last)] = wt[k];
    i += 4 * 64 * kDecWaves;
    if (i > w_last) break;
    load_weights(i);
  }
  __syncthreads();
  if (!mine) return;

  f32x4 acc[GT][C];
#pragma unroll
  for (int q = 0; q < GT; ++q)
#pragma unroll
    for (int j = 0; j < C; ++j) acc[q][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](RowPiece<T> (&v)[8], int i) {
    const int s = order.at(i);
#pragma unroll
    for (int q = 0; q < GT; ++q) {
      const int k = s - first[q];
      if (k >= 0 && k < count[q]) {
        const f32x4* wp = wlds + (q * steps + k) * 128 + lane;
        const f32x4 wa = wp[0], wb = wp[64];
        Frag w[3];
#pragma unroll
        for (int h = 0; h < 4; ++h)
          bf16_terms(h < 2 ? wa[2 * h] : wb[2 * h - 4], h < 2 ? wa[2 * h + 1] : wb[2 * h - 3], w, h);
#pragma unroll
        for (int j = 0; j < C; ++j) {
          Frag a[kTerms];
          column_frag(v, j, a);
          acc[q][j] = fold_column(a, w, acc[q][j]);
        }
      }
    }
    if (i + kBuf < steps_all) load(v, order.at(i + kBuf));
  };
  for (int i = 0; i < steps_all; i += kBuf)
#pragma unroll
    for (int b = 0; b < kBuf; ++b)
      if (i + b < steps_all) step(x[b], i + b);

  // Out in 16 bytes, two neighbours of the transform's order: of the two lanes that hold them one takes what belongs to the
  // first tile (or column pair), the other what belongs to the second, and four lanes side by side write 64 bytes.
  const bool up = lane & 4, swap = ((lane >> 2) ^ (lane >> 3)) & 1;
  auto both = [&](float2 a, float2 b) {
    const float2 own = up ? b : a, give = up ? a : b;
    const float2 got = make_float2(dpp<0x141>(give.x), dpp<0x141>(give.y));        // row_half_mirror
    return swap ? f32x4{got.x, got.y, own.x, own.y} : f32x4{own.x, own.y, got.x, got.y};
  };
  // the one of the lane's two points that is first in the transform's order
  const int k0 = 16 * tile0 + (lane_point(lane & 15) & ~2) + ((lane >> 2) & 2);
#pragma unroll
  for (int q = 0; q < GT; q += 2) {
    if (q >= n_tiles) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s_out = part * 16 + 4 * (lane >> 4) + i;
      float2* o = grid + ((size_t)(unit - u0) * 2 * sm.nb + s_out) * (C / 2) * m;
      if constexpr (GT > 1) {
        const bool there = s_out < 2 * sm.nb && (!up || q + 1 < n_tiles);
        float2* t = o + grid_pos(k0 + 16 * (q + (up ? 1 : 0)), m);
#pragma unroll
        for (int jp = 0; jp < C / 2; ++jp) {
          const f32x4 w = both(make_float2(acc[q][2 * jp][i], acc[q][2 * jp + 1][i]),
                               make_float2(acc[q + 1][2 * jp][i], acc[q + 1][2 * jp + 1][i]));
          if (there) *reinterpret_cast<f32x4*>(t + (size_t)jp * m) = w;
        }
      } else {
        float2* t = o + grid_pos(k0, m) + (up ? m : 0);
#pragma unroll
        for (int jp = 0; jp < C / 2; jp += 2) {
          const f32x4 w = both(make_float2(acc[q][2 * jp][i], acc[q][2 * jp + 1][i]),
                               make_float2(acc[q][2 * jp + 2][i], acc[q][2 * jp + 3][i]));
          if (s_out < 2 * sm.nb) *reinterpret_cast<f32x4*>(t + (size_t)jp * m) = w;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------- filter on the grid

// Complex numbers of 32 and of 64 bits (C = float2, double2).
template <typename C>
__device__ __forceinline__ constexpr C cpair(decltype(C::x) re, decltype(C::x) im) { return C{re, im}; }
__device__ __forceinline__ float mad(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return fma(a, b, c); }
template <typename C>
__device__ __forceinline__ C cadd(C a, C b) { return cpair<C>(a.x + b.x, a.y + b.y); }
template <typename C>
__device__ __forceinline__ C csub(C a, C b) { return cpair<C>(a.x - b.x, a.y - b.y); }
template <typename C>
__device__ __forceinline__ C cmul(C a, C w) {
  return cpair<C>(mad(a.x, w.x, -a.y * w.y), mad(a.y, w.x, a.x * w.y));
}

// What 32 bits leave of a constant, for products that take both parts.  A constant's error is the same in every
// column's transform and does not average out over them as that of rounded points does: with constants of 32 bits the
// scores at 7680 tokens, r = 2305, are 1.1e-7 from 64 bits instead of 7e-8, at 32768 tokens, r = 6554, 7.2e-8 instead
// of 4.1e-8.  The filter takes 2 to 5 % longer for it (14336 column pairs of 3072 points: 199 / 207 us).
__device__ __forceinline__ constexpr float rest_of(double c) { return (float)(c - (double)(float)c); }
// a * e^{-2 pi i k / n}
__device__ __forceinline__ double2 turn(double2 a, int k, int n) { return cmul(a, root<double2>(k, n)); }
__device__ __forceinline__ float2 turn(float2 a, int k, int n) {
  const double c = cos192(k * (192 / n)), s = cos192(k * (192 / n) + 48);
  const float cl = rest_of(c), sl = rest_of(s);
  if (s == 0.0) return c > 0.0 ? a : make_float2(-a.x, -a.y);
  if (c == 0.0) return s > 0.0 ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
  if (cl == 0.f)                                           // (a half: its product is not rounded)
    return make_float2(fmaf(a.x, (float)c, fmaf(-a.y, (float)s, -a.y * sl)), fmaf(a.y, (float)c, fmaf(a.x, (float)s, a.x * sl)));
  if (sl == 0.f)
    return make_float2(fmaf(-a.y, (float)s, fmaf(a.x, (float)c, a.x * cl)), fmaf(a.x, (float)s, fmaf(a.y, (float)c, a.y * cl)));
  return make_float2(fmaf(a.x, (float)c, fmaf(-a.y, (float)s, fmaf(a.x, cl, -a.y * sl))),
                     fmaf(a.y, (float)c, fmaf(a.x, (float)s, fmaf(a.y, cl, a.x * sl))));
}

template <typename C>
__device__ __forceinline__ void dft2(C (&v)[2]) {
  const C a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}
template <typename C>
__device__ __forceinline__ void dft3(C (&v)[3]) {
  typedef decltype(C::x) R;
  const C t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
  constexpr double sin60 = 0.86602540378443865;
  const R k = (R)sin60, h = (R)-0.5;
  const C m = cpair<C>(mad(h, t.x, v[0].x), mad(h, t.y, v[0].y));
  v[0] = cadd(v[0], t);
  C p = m, q = m;
  if constexpr (sizeof(R) == 4) {
    const R l = rest_of(sin60);
    p = cpair<C>(mad(l, d.y, m.x), mad(-l, d.x, m.y));
    q = cpair<C>(mad(-l, d.y, m.x), mad(l, d.x, m.y));
  }
  v[1] = cpair<C>(mad(k, d.y, p.x), mad(-k, d.x, p.y));
  v[2] = cpair<C>(mad(-k, d.y, q.x), mad(k, d.x, q.y));
}
template <typename C>
__device__ __forceinline__ void dft4(C (&v)[4]) {
  const C s = cadd(v[0], v[2]), t = csub(v[0], v[2]), u = cadd(v[1], v[3]), w = csub(v[1], v[3]);
  const C p = cpair<C>(t.x + w.y, t.y - w.x), q = cpair<C>(t.x - w.y, t.y + w.x);
  v[0] = cadd(s, u);
  v[1] = p;
  v[2] = csub(s, u);
  v[3] = q;
}

// Transform of R points in registers, natural order on both sides: R = A * B with A-point transforms
// over the strided points, constant factors, B-point transforms.
template <int R>
constexpr int first_factor() { return R == 2 || R == 3 || R == 4 ? R : (R % 4 == 0 ? 4 : 2); }
template <int R, typename C>
__device__ __forceinline__ void dft(C (&v)[R]) {
  if constexpr (R == 2) dft2(v);
  else if constexpr (R == 3) dft3(v);
  else if constexpr (R == 4) dft4(v);
  else {
    constexpr int A = first_factor<R>(), B = R / A;
    C y[A][B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      C u[A];
#pragma unroll
      for (int a = 0; a < A; ++a) u[a] = v[B * a + b];
      if (R >= 24 && b % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      dft<A>(u);
#pragma unroll
      for (int a = 0; a < A; ++a) {
        if (a * b == 0) y[a][b] = u[a];
        else if (4 * a * b == R) y[a][b] = cpair<C>(u[a].y, -u[a].x);
        else y[a][b] = turn(u[a], a * b, R);
      }
    }
#pragma unroll
    for (int a = 0; a < A; ++a) {
      if (R >= 24) __builtin_amdgcn_sched_barrier(0);
      dft<B>(y[a]);
#pragma unroll
      for (int b = 0; b < B; ++b) v[a + A * b] = y[a][b];
    }
  }
}

template <int M, bool WIDE>
struct GridPlan {
  static constexpr GridRadices G = grid_radices(M, WIDE);
  static constexpr int P = G.p, T = M / P, R0 = G.r[0], R1 = G.r[1], R2 = G.r[2], R3 = G.r[3];
  // One slot of padding per R0 (or T, where fewer): the strided writes of a pass fall on distinct banks.
  static constexpr int log2(int v) { return v <= 1 ? 0 : 1 + log2(v / 2); }
  static constexpr int kPadShift = log2(R0 < T ? R0 : T);
  static constexpr int kLds = M + (M >> kPadShift) + 2;       // (even: blocks are read as pairs)
  // Bins from each end of a thread's points that meet their mirrors at a time, 0: all bins at once, real parts, then
  // imaginary parts.  Blocks need the registers of one block's mirrors instead of all bins', and with them and each
  // pass's points pinned (see the kernel) a SIMD holds the waves of kWaves without spilling: 48 points a thread three
  // instead of two, 32 points four instead of three (and 16384 points two workgroups a compute unit instead of one), 64-bit
  // ones three (16 points; 32: two).  Filter of 112 units, us before / after: 32768 tokens M = 3072 184 / 167, M = 12288
  // 902 / 778, 30011 tokens M = 6144 401 / 355, 50000 tokens M = 16384 (36 units) 496 / 338; in 64 bits 1500 tokens M = 768
  // (32 units) 27.0 / 23.0.  The short narrow ones have the registers as they are, and are slower with blocks and more
  // waves (M = 1536: 84 / 103).
  static constexpr int kBlock = !WIDE && P < 32 ? 0 : (P == 48 && T == 64 ? 4 : P / 8);
  // (a pass's exchange takes a thread's butterflies to be T apart in whole groups of the transforms done before it)
  static_assert((R2 == 1 || R0 <= T) && (R3 == 1 || R0 * R1 <= T), "groups of the grid transform");
  static_assert(R0 * R1 * R2 * R3 == M && T % (1 << kPadShift) == 0 && kLds % 2 == 0, "radices of the grid transform");
  static_assert(kBlock == 0 || ((P / 2) % kBlock == 0 && 8 * kBlock * T + 8 <= kLds), "blocks of bins fit the exchange's LDS");
  // (24576 points have a compute unit's LDS to themselves, eight waves' worth)
  static constexpr int kWaves = WIDE ? (P <= 16 ? 3 : 2) : (P <= 16 || P == 32 ? 4 : (T == 512 ? 2 : 3));   // a SIMD's
};

// element i + k of a table: uniform base and constant part, 32-bit part of the lane
// (said to be global memory: a pointer that went through an asm statement has lost that)
template <typename C>
__device__ __forceinline__ C at(const C* base, int k, uint32_t i) {
  typedef decltype(C::x) V2 __attribute__((ext_vector_type(2)));
  typedef const __attribute__((address_space(1))) V2* Global;
  const V2 v = *(Global)(reinterpret_cast<const char*>(base + k) + i * (uint32_t)sizeof(C));
  return cpair<C>(v.x, v.y);
}

// Element k of a grid's column pair as a scalar base and the part of k that a load's 12-bit offset holds.  (Left to the compiler each
// load of the longer grids makes a 64-bit address of its own on the vector units.)
__device__ __forceinline__ float2* element(float2* base, int k) {
  char* b = reinterpret_cast<char*>(base) + ((k * (int)sizeof(float2)) & ~4095);
  asm volatile("" : "+s"(b));
  return reinterpret_cast<float2*>(b + ((k * (int)sizeof(float2)) & 4095));
}

// Length-M complex transform of one column pair; natural order before and after, exchanges through LDS.
// Points are held in 32 bits; a wide transform takes each pass's factors and arithmetic in 64, so that its results are
// rounded once a pass.
template <int M, bool WIDE>
struct GridFft {
  using G = GridPlan<M, WIDE>;
  using C = typename std::conditional<WIDE, double2, float2>::type;
  static constexpr int P = G::P, T = G::T;
  // (constants of their own: as a call in the kernel the phases' offset was computed at its start, by a loop over the
  // radices in scratch memory, three waits in turn: 112 units of 32768 tokens, M = 3072: 207 / 181 us of filter, M = 12288: 964 / 911)
  static constexpr int kOff2 = twid_off(M, WIDE, 2), kOff3 = twid_off(M, WIDE, 3), kPhaseOff = twid_phase_off(M, WIDE);
  // slot of point i; T and NS * R are multiples of 2^kPadShift, so that pad(i + T q) = pad(i) + pad(T q)
  static __device__ __forceinline__ constexpr int pad(int i) { return i + (i >> G::kPadShift); }

  // Factors w_{R NS}^{(j mod NS) q} of a pass, q = lo + 8 hi from stored powers 1..7 and 8 hi.
  template <int R, int NS>
  struct Factors {
    static constexpr int HI = (R - 1) / 8;
    C lo[8], hi[HI + 1];
    __device__ __forceinline__ void load(const C* __restrict__ tw, int t) {
      constexpr bool kLast = R * NS == M;
      constexpr int stride = kLast ? T : NS;
      const int j = kLast ? t : t & (NS - 1);
#pragma unroll
      for (int q = 1; q < 8; ++q)
        if (q < R) lo[q] = at(tw, (q - 1) * stride, j);
#pragma unroll
      for (int q = 1; q <= HI; ++q) hi[q] = at(tw, ((R < 8 ? R : 8) - 1 + q - 1) * stride, j);
    }
    __device__ __forceinline__ C get(int q) const {
      return q < 8 ? lo[q] : (q % 8 == 0 ? hi[q / 8] : cmul(lo[q % 8], hi[q / 8]));
    }
  };

  // Pass of radix R after NS-point transforms are done: butterfly j = t + T c takes the points j + (M/R) q,
  // which are this thread's own; the butterflies of a thread share the factors, in the last pass up to a constant.
  template <int R, int NS>
  static __device__ __forceinline__ void butterflies(float2 (&x)[P], const Factors<R, NS>& f) {
    constexpr int N = P / R;
    constexpr bool kLast = R * NS == M;
    // (the factors first, shared by the thread's butterflies, where the points are multiplied in place)
    if constexpr (NS > 1 && !WIDE) {
#pragma unroll
      for (int q = 1; q < R; ++q) {
        const C w = f.get(q);
#pragma unroll
        for (int c = 0; c < N; ++c) x[c + N * q] = cmul(x[c + N * q], kLast && c > 0 ? cmul(w, root<C>(c * q, P)) : w);
        if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int c = 0; c < N; ++c) {
      C v[R];
#pragma unroll
      for (int q = 0; q < R; ++q) {
        v[q] = cpair<C>(x[c + N * q].x, x[c + N * q].y);
        if constexpr (NS > 1 && WIDE) {
          if (q > 0) v[q] = cmul(v[q], kLast && c > 0 ? cmul(f.get(q), root<C>(c * q, P)) : f.get(q));
          if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      dft<R>(v);
#pragma unroll
      for (int q = 0; q < R; ++q) x[c + N * q] = make_float2((float)v[q].x, (float)v[q].y);
      if (WIDE) __builtin_amdgcn_sched_barrier(0);
    }
  }
  // Results of a pass to where the next one takes them: real parts, then imaginary parts, through the same half
  // (half the LDS keeps twice the waves resident).  Point (j / NS) NS R + j % NS + q NS of butterfly j = t + T c.
  template <int R, int NS>
  static __device__ __forceinline__ void exchange(float2 (&x)[P], float* lds, int t) {
    constexpr int N = P / R;
    asm volatile("" : "+v"(t));                            // (addresses are not worth keeping from one exchange to the next)
    float* o = lds + pad((t / NS) * (NS * R) + (t & (NS - 1)));
    const float* in = lds + pad(t);
    float re[P];
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
      for (int q = 0; q < R; ++q) o[pad(T * c * R) + pad(q * NS)] = x[c + N * q].x;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < P; ++q) re[q] = in[pad(T * q)];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
      for (int q = 0; q < R; ++q) o[pad(T * c * R) + pad(q * NS)] = x[c + N * q].y;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < P; ++q) x[q] = make_float2(re[q], in[pad(T * q)]);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  }
  // (a pass's factors are requested before the exchange that precedes it)
  static __device__ __forceinline__ void run(float2 (&x)[P], float* lds, const C* __restrict__ twid, int t) {
    constexpr int N1 = G::R0, N2 = N1 * G::R1, N3 = N2 * G::R2;
    Factors<G::R0, 1> f0;
    Factors<G::R1, N1> f1;
    butterflies<G::R0, 1>(x, f0);
    f1.load(twid, t);
    exchange<G::R0, 1>(x, lds, t);
    butterflies<G::R1, N1>(x, f1);
    if constexpr (G::R2 > 1) {
      Factors<G::R2, N2> f2;
      f2.load(twid + kOff2, t);
      exchange<G::R1, N1>(x, lds, t);
      butterflies<G::R2, N2>(x, f2);
    }
    if constexpr (G::R3 > 1) {
      Factors<G::R3, N3> f3;
      f3.load(twid + kOff3, t);
      exchange<G::R2, N2>(x, lds, t);
      butterflies<G::R3, N3>(x, f3);
    }
  }
};

// One column pair (as real and imaginary part) per M/P threads, in place: transform, keep and weight the
// modes below the cut-off, transform back.  With the permuted input order the DFT carries DCT modes m and
// M-m in the pair of bins (m, M-m):
//     W'[m] = (f[m] + f[M-m])/2 W[m] + (f[m] - f[M-m])/2 e^{i pi m/M} W[M-m].
// sum_m Re(conj(W) W') is the kept energy of both columns (the operator is symmetric).  The way back is the same
// transform with real and imaginary parts exchanged.  Short lengths (few workgroups) run it in the same code, since
// such a launch would wait for the instructions of a second copy to be fetched (768 points: 13 instead of 16 us); the
// lengths with 32 and 48 points a thread are better off with two copies (3072 points: 180 instead of 220 us).
template <int M, bool WIDE, typename G = GridPlan<M, WIDE>, typename F = GridFft<M, WIDE>>
__global__ __launch_bounds__(G::T < 64 ? 64 : G::T, G::kWaves) void grid_filter_kernel(
    float2* __restrict__ grid, int pairs, int n, int r, int d, int dtype, WsHeader* hdr,
    const float2* __restrict__ filt, const typename F::C* __restrict__ twid, double* __restrict__ elow) {
  using C = typename F::C;
  constexpr int P = G::P, T = G::T, PB = T < 64 ? 64 / T : 1;
  extern __shared__ float lds_all[];
  __shared__ double wsum[T < 64 ? 1 : T / 64];
  const int t = threadIdx.x % T, pb = threadIdx.x / T;
  float* lds = lds_all + pb * G::kLds;
  const int pair = min((int)blockIdx.x * PB + pb, pairs - 1);   // (surplus lanes repeat the last pair)
  float2* g = grid + (size_t)blockIdx.x * PB * M;
  uint32_t lane_at = (uint32_t)(T < 64 ? (pair - (int)blockIdx.x * PB) * M + t : t);
  float2 x[P];
#pragma unroll
  for (int q = 0; q < P; ++q) x[q] = at(element(g, T * q), 0, lane_at);
  C ph = at(twid, F::kPhaseOff, t);
  if (ws_mismatch(hdr, FC_PATH_RESAMPLE, n, r, d, dtype)) return;
  decltype(C::x) e = 0;
#pragma unroll(P <= 24 ? 1 : 2)
  for (int way = 0; way < 2; ++way) {
    // (what the tables give is loaded and derived anew: kept from one way to the next it would fill the registers)
    asm volatile("" : "+s"(twid), "+s"(filt), "+v"(ph.x), "+v"(ph.y));
    F::run(x, lds, twid, t);
    // (the points are made here: moved down to where a block takes them, the last pass would keep more operands than results)
    if constexpr (G::kBlock > 0)
#pragma unroll
      for (int q = 0; q < P; ++q) asm volatile("" : "+v"(x[q].x), "+v"(x[q].y));
    if (way == 1) break;
    auto bin = [&](int q, float2 mirror) {
      const float2 fq = at(filt, T * q, t);
      const C f = cpair<C>(fq.x, fq.y);
      const C c = root<C>(q, 2 * P), w = cpair<C>(x[q].x, x[q].y);
      const C z = cmul(cpair<C>(mirror.x, mirror.y), cmul(ph, cpair<C>(c.x, -c.y)));   // e^{i pi (t + T q) / M}
      const C y = cpair<C>(mad(f.y, z.x, f.x * w.x), mad(f.y, z.y, f.x * w.y));
      e = mad(w.x, y.x, mad(w.y, y.y, e));
      x[q] = make_float2((float)y.y, (float)y.x);
    };
    // each bin's mirror, W[M - m] (with W[M] = W[0])
    if constexpr (G::kBlock > 0) {
      // a block of bins from each end, which are each other's mirrors
      constexpr int H = G::kBlock;
      float2 edge = x[0];
#pragma unroll
      for (int q0 = 0; q0 < P / 2; q0 += H) {
        // (blocks take turns with the two halves of the buffer, so that one wait a block will do)
        float2 *lo = reinterpret_cast<float2*>(lds) + (q0 / H & 1) * (2 * H * T + 2), *hi = lo + H * T + 1;
#pragma unroll
        for (int j = 0; j < H; ++j) lo[T * j + t] = x[q0 + j];
#pragma unroll
        for (int j = 0; j < H; ++j) hi[T * j + t] = x[P - q0 - H + j];
        if (t == 0) {
          lo[T * H] = x[q0 + H];
          hi[T * H] = edge;
        }
        edge = x[P - q0 - H];
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          float2 o[H];
#pragma unroll
          for (int j = 0; j < H; ++j) o[j] = (side ? lo : hi)[T * (H - j) - t];
#pragma unroll
          for (int j = 0; j < H; ++j) bin(side ? P - q0 - H + j : q0 + j, o[j]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
    } else {
      float2 o[P];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int q = 0; q < P; ++q) lds[F::pad(t) + F::pad(T * q)] = h ? x[q].y : x[q].x;
        if (t == 0) lds[F::pad(M)] = h ? x[0].y : x[0].x;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < P; ++q) (h ? o[q].y : o[q].x) = lds[F::pad(M - T * q) + F::pad(-t)];
        __syncthreads();
      }
#pragma unroll
      for (int q = 0; q < P; ++q) {
        if (q % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        bin(q, o[q]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("" : "+v"(lane_at));                        // (the load addresses are not worth keeping)
#pragma unroll
  for (int q = 0; q < P; ++q) {
    typedef float V2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(1))) V2* Global;
    *(Global)(reinterpret_cast<char*>(element(g, T * q)) + lane_at * (uint32_t)sizeof(float2)) = V2{x[q].y, x[q].x};
  }

  double es = (double)e;
#pragma unroll
  for (int s = 1; s < (T < 64 ? T : 64); s <<= 1) es += __shfl_xor(es, s, 64);
  if (T < 64) {
    if (t == 0) elow[pair] = es;
  } else {
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = es;
    __syncthreads();
    if (threadIdx.x == 0) {
      double a = 0.0;
      for (int k = 0; k < T / 64; ++k) a += wsum[k];
      elow[pair] = a;
    }
  }
}

// The same transform (in 32 bits) spread over one thread for each butterfly of its widest pass, every pass through LDS.
// Points meet the same factors in the same order as in grid_filter_kernel, so that results are the same bits (the kept
// energy's sum aside).  It takes more instructions in all, and is for launches that leave much of the chip without a
// wave, whose time is that of one wave's instructions one after the other: up to 512 column pairs of transforms with 24
// points a thread and more, more where it was found the quicker one.  One wave for each transform / spread, us with events (an empty
// launch: 6): 512 pairs of 3072 points 21.8 / 16.9, of 1536 14.9 / 13.2, of 4096 16.8 / 14.7, 256 of 96 8.2 / 6.4; 1024 pairs of 3072
// 25.5 / 23.8, of 1536 14.9 / 17.6, of 768 12.2 / 11.5, of 384 10.9 / 8.3, of 192 8.8 / 9.5; 2048 of 3072 35.7 / 37.4, of 768 14.6 /
// 15.2, of 384 12.0 / 9.8; 256 of 2048, which have 16 points a thread, 11.1 / 12.2; 512 of 6144 26.3 / 41.6.  (kMostPairs is a list: no rule by
// points, radices, threads or registers gives these lines.)  (Addresses of LDS as a part of the
// thread's own and constants: a seventh of the instructions, 512 pairs of 3072 points 17.5 / 16.9, of 384 7.4 / 7.0.)
template <int M>
struct SpreadPlan {
  using G = GridPlan<M, false>;
  static constexpr bool kUse = G::P >= 24 && M <= 4096;
  static constexpr int kMostPairs = M == 384 ? 2048 : (M == 768 || M == 3072 ? 1024 : 512);
  static constexpr int least(int a, int b) { return a < b ? a : b; }
  static constexpr int kRadix = least(least(G::R0, G::R1), least(G::R2 > 1 ? G::R2 : M, G::R3 > 1 ? G::R3 : M));
  static constexpr int NT = (M / kRadix + 63) / 64 * 64;
};
template <int M, typename G = GridPlan<M, false>, typename F = GridFft<M, false>>
__global__ __launch_bounds__(SpreadPlan<M>::NT) void grid_spread_kernel(
    float2* __restrict__ grid, int n, int r, int d, int dtype, WsHeader* hdr, const float2* __restrict__ filt,
    const float2* __restrict__ twid, double* __restrict__ elow) {
  using C = float2;
  constexpr int P = G::P, T = G::T, NT = SpreadPlan<M>::NT;
  constexpr int kRoots = twid_root_off(M, false), kPhases = twid_phase_off(M, false);
  static_assert(NT % T == 0, "a thread's bins share a phase");
  extern __shared__ float lds_all[];
  __shared__ double wsum[NT / 64];
  float *re = lds_all, *im = lds_all + G::kLds;
  const int tid = threadIdx.x;
  float2* g = grid + (size_t)blockIdx.x * M;
  // what the tables give, requested at once with the points
  constexpr int N1 = G::R0, N2 = N1 * G::R1, N3 = N2 * G::R2;
  constexpr int kPasses = G::R3 > 1 ? 4 : (G::R2 > 1 ? 3 : 2), RL = kPasses == 4 ? G::R3 : (kPasses == 3 ? G::R2 : G::R1);
  constexpr bool kTurns = T < M / RL;                      // butterflies of the last pass share T threads' factors
  typename F::template Factors<G::R0, 1> f0;
  typename F::template Factors<G::R1, N1> f1;
  typename F::template Factors<(kPasses > 2 ? G::R2 : 2), (kPasses > 2 ? N2 : 1)> f2;
  typename F::template Factors<(kPasses > 3 ? G::R3 : 2), (kPasses > 3 ? N3 : 1)> f3;
  const int t = tid & (T - 1);
  float2 x0[G::R0];
#pragma unroll
  for (int q = 0; q < G::R0; ++q)
    if (M / G::R0 >= NT || tid < M / G::R0) x0[q] = g[tid + M / G::R0 * q];
  f1.load(twid, kPasses == 2 ? t : tid);
  if constexpr (kPasses > 2) f2.load(twid + F::kOff2, kPasses == 3 ? t : tid);
  if constexpr (kPasses > 3) f3.load(twid + F::kOff3, t);
  C turn_by[kTurns ? RL : 1];
  if constexpr (kTurns)
#pragma unroll
    for (int q = 1; q < RL; ++q) turn_by[q] = twid[kRoots + (tid / T) * q % P];
  constexpr int kBins = (M + NT - 1) / NT;
  float2 fq[kBins];
  C phase[kBins];
  const C ph = twid[kPhases + t];
#pragma unroll
  for (int k = 0; k < kBins; ++k) {
    const int m = min(tid + NT * k, M - 1);
    fq[k] = filt[m];
    phase[k] = twid[kRoots + P + m / T];
  }
  // butterfly tid of a pass of radix R after NS-point transforms: from registers (x) or LDS to LDS or the grid (STORE)
  auto pass = [&](auto radix, auto done, auto first, auto store, const auto& f) {
    constexpr int R = decltype(radix)::value, NS = decltype(done)::value, B = M / R;
    constexpr bool kLast = R * NS == M;
    const bool mine = B >= NT || tid < B;
    // (addresses are a part of the thread's own and a constant: B q, and q NS or q of a group of NS R, are made of whole groups of
    // 2^kPadShift, or do not leave one)
    static_assert(B % (1 << G::kPadShift) == 0 && pads_apart(R, NS, 1 << G::kPadShift), "padding of a pass");
    C v[R];
    if (mine)
#pragma unroll
      for (int q = 0; q < R; ++q) {
        if constexpr (first) v[q] = cpair<C>(x0[q].x, x0[q].y);
        else v[q] = cpair<C>(re[F::pad(tid) + F::pad(B * q)], im[F::pad(tid) + F::pad(B * q)]);
      }
    if (!first) __syncthreads();
    if (mine) {
      if constexpr (NS > 1) {
#pragma unroll
        for (int q = 1; q < R; ++q) {
          C w = f.get(q);
          if constexpr (kLast && kTurns) w = cmul(w, turn_by[q]);
          v[q] = cmul(v[q], w);
        }
      }
      dft<R>(v);
      const int to = kLast ? tid : tid / NS * (NS * R) + (tid & (NS - 1));
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const float2 x = make_float2((float)v[q].x, (float)v[q].y);
        const int at = F::pad(to) + F::pad(kLast ? B * q : q * NS);
        if (store) g[to + B * q] = make_float2(x.y, x.x);
        else { re[at] = x.x; im[at] = x.y; }
      }
    }
    if (!store) __syncthreads();
  };
  auto transform = [&](auto first, auto store) {
    std::false_type no;
    pass(Int<G::R0>{}, Int<1>{}, first, no, f0);
    if constexpr (kPasses == 2) pass(Int<G::R1>{}, Int<N1>{}, no, store, f1);
    else {
      pass(Int<G::R1>{}, Int<N1>{}, no, no, f1);
      if constexpr (kPasses == 3) pass(Int<G::R2>{}, Int<N2>{}, no, store, f2);
      else {
        pass(Int<G::R2>{}, Int<N2>{}, no, no, f2);
        pass(Int<G::R3>{}, Int<N3>{}, no, store, f3);
      }
    }
  };
  if (ws_mismatch(hdr, FC_PATH_RESAMPLE, n, r, d, dtype)) return;
  transform(std::true_type{}, std::false_type{});
  decltype(C::x) e = 0;
  C y[kBins];
#pragma unroll
  for (int k = 0; k < kBins; ++k) {
    const int m = tid + NT * k;
    if (M % NT == 0 || m < M) {
      const int at = F::pad(tid) + F::pad(NT * k), o = k == 0 && tid == 0 ? 0 : F::pad(M - NT * k) + F::pad(-tid);
      const C w = cpair<C>(re[at], im[at]), mirror = cpair<C>(re[o], im[o]);
      const C f = cpair<C>(fq[k].x, fq[k].y), z = cmul(mirror, cmul(ph, cpair<C>(phase[k].x, -phase[k].y)));
      y[k] = cpair<C>(mad(f.y, z.x, f.x * w.x), mad(f.y, z.y, f.x * w.y));
      e = mad(w.x, y[k].x, mad(w.y, y[k].y, e));
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kBins; ++k) {
    const int m = tid + NT * k;
    const int at = F::pad(tid) + F::pad(NT * k);
    if (M % NT == 0 || m < M) { re[at] = (float)y[k].y; im[at] = (float)y[k].x; }
  }
  __syncthreads();
  transform(std::false_type{}, std::true_type{});

  double es = (double)e;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) es += __shfl_xor(es, s, 64);
  if ((tid & 63) == 0) wsum[tid >> 6] = es;
  __syncthreads();
  if (tid == 0) {
    double a = 0.0;
    for (int k = 0; k < NT / 64; ++k) a += wsum[k];
    elow[blockIdx.x] = a;
  }
}

// ---------------------------------------------------------------------------- residual and score

// squares of (row - inv * base) and of the row, a piece of token i of the tile
__device__ __forceinline__ void residual_piece(const RowPiece<uint16_t>& x, const f32x4 (&acc)[8], int i, float inv,
                                               float& hp, float& tot) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t w = x.v[c];
    const float lo = __uint_as_float(w << 16), hi = __uint_as_float(w & 0xFFFF0000u);
    const float dl = fmaf(-inv, acc[2 * c][i], lo), dh = fmaf(-inv, acc[2 * c + 1][i], hi);
    hp = fmaf(dl, dl, hp);
    hp = fmaf(dh, dh, hp);
    tot = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(s16x2, w), __builtin_bit_cast(s16x2, w), tot, false);
  }
}
__device__ __forceinline__ void residual_piece(const RowPiece<float>& x, const f32x4 (&acc)[4], int i, float inv,
                                               float& hp, float& tot) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float dv = fmaf(-inv, acc[c][i], x.v[c]);
    hp = fmaf(dv, dv, hp);
    tot = fmaf(x.v[c], x.v[c], tot);
  }
}

// a and b times scale, a power of two, in two terms of 16 bits each: rounded, and what that leaves.  (Scaling, rounding and difference
// are one instruction for each of the four: the sums are fused multiply-adds, and the first terms are pinned as a word, else the
// compiler makes them twice, 192 instructions more for a window.)
__device__ __forceinline__ void halves(float a, float b, float scale, Frag& high, Frag& low, int word) {
  f16x2 h = {(_Float16)fmaf(a, scale, 0.f), (_Float16)fmaf(b, scale, 0.f)};
  asm volatile("" : "+v"(h));
  const f16x2 l = {(_Float16)fmaf(a, scale, -(float)h[0]), (_Float16)fmaf(b, scale, -(float)h[1])};
  high.u[word] = __builtin_bit_cast(uint32_t, h);
  low.u[word] = __builtin_bit_cast(uint32_t, l);
}
// Over the four lanes that hold one slot.
__device__ __forceinline__ float slot_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return v + __hiloint2double(hi, lo);
}
// Sums over the wave: of a in lanes 16 to 31, of b in lanes 48 to 63.
__device__ __forceinline__ double wave_sums(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  double v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  v = dpp_add<0x128>(dpp_add<0x124>(dpp_add<0x122>(dpp_add<0x121>(v))));
  return dpp_add<0x142>(v);                                // row_bcast:15
}
// Sums of v[0..3] over the 16 lanes of a row, from four lanes' sums on in 64 bits; a lane returns the sum of v[lane & 3].
__device__ __forceinline__ double row_sums(const float (&v)[4], int lane) {
  const bool b0 = lane & 1, b1 = lane & 2;
  const float s01 = (b0 ? v[1] : v[0]) + dpp<0xB1>(b0 ? v[0] : v[1]);      // quad_perm 1,0,3,2
  const float s23 = (b0 ? v[3] : v[2]) + dpp<0xB1>(b0 ? v[2] : v[3]);
  const float s = (b1 ? s23 : s01) + dpp<0x4E>(b1 ? s01 : s23);            // quad_perm 2,3,0,1
  return dpp_add<0x128>(dpp_add<0x124>((double)s));                        // row_ror:4, row_ror:8
}

// What a residual workgroup's waves take side by side: units, and of each the blocks of a window's tiles, and of each the parts.
// (From the host, and divisors as factors: a division of the kernel's own is a tenth of a us before the first load is asked for.)
struct SideBySide {
  int units, parts, sets;     // sets: of so many units, in the launch
  int per_unit, per_block;    // side_factor of the waves of a unit and of a block
};
constexpr int side_factor(int waves) { return 256 / waves + 1; }
__device__ __forceinline__ int side_div(int wave, int factor) { return wave * factor >> 8; }   // (exact up to 8 waves)

// One wave applies windows (32 grid points each) to the 16-token tiles they cover, 16 slots at a time.  Its work
// is a list of segments: a window, a unit (four units at a time, one for each wave of a workgroup), a part of the
// unit's slots; or (split) a workgroup's waves take the parts of a unit side by side instead of one
// after the other.  Rows are requested two tiles ahead and grid values one window ahead, across segments.
// Neighbouring windows read the same lines of the grid: an XCD takes a contiguous range of windows and its
// workgroups walk (units, window) side by side, window fastest, so that its L2 serves what they share.  Launches with no
// more than one segment for a wave (ONCE) ask for nothing ahead of a next one (one layer of 16384 tokens: 19.7 / 19.1 us).
// Bound by the memory path: 56 units of 32768 tokens, M = 3072: 238 to 245 us by card, 1.18 GB read for 0.94 GB of rows and
// 0.18 of grid, 5.0 to 4.8 TB/s.  Rows three or four tiles ahead, with their weights, or windows not asked for ahead leave it there (112
// units, us: 452 as it is, 453, 454, 457).  Sums: 432 us with three of the five products and sums in 32 bits where 455 were
// taken with sums as they are and 474 with all in 64.
// A lane holds slot lane & 15 throughout: columns 8 slot + j of tokens 4 (lane >> 4) + i, so that a load reads whole
// rows, and of a window the points that loads of 64-byte pieces deliver (see resample_table_kernel).  Those loads are made
// by four lanes next to each other and turned over to the operands' lanes through LDS (a swizzle keeps them on distinct
// banks): by the operands' lanes, 16 slots apart in memory, they took the address unit four times as long.  112 units, us
// before / after: 32768 tokens M = 3072 460 / 448, M = 12288 729 / 683, 30011 tokens 526 / 507; one layer of 16384 21.5 / 18.0,
// of which 1.6 for not loading a window after the last segment.
// What a segment takes besides its tiles weighs where those are few (three at M = 12288): of 600 vector and 500 scalar
// instructions 350 and 300 are left, since a window's values are scaled and split in one instruction a term, energies of one
// tensor's slots take one pair of sums over the wave, items follow one another without a division and loads have scalar bases.
// Residual of 112 units, us: M = 12288 681 / 654, 16384 tokens, M = 12288 715 / 680, 30011 tokens 505 / 490, M = 3072 449 / 443.
template <typename T, bool KEEP, bool ONCE, bool BLOCKS, int BUF, int WAVES>
__global__ __launch_bounds__(64 * WAVES, sizeof(T) == 2 ? 2 : (ONCE ? 4 : 3)) void residual_kernel(
    const T* __restrict__ K, const T* __restrict__ V, KvStrides st, int u0, int u1, int n, int r, int d, int dtype,
    int m, int tpw, int wins, SlotMap sm, bool split, int blocks, SideBySide side, int along, WsHeader* hdr, const _Float16* __restrict__ winv,
    const float2* __restrict__ grid, float* __restrict__ scores,
    double* __restrict__ epart, UnitMap um) {
  constexpr int C = kCols<T>;
  constexpr int kBuf = BUF;                                // tiles of rows under way
  __shared__ double part_sum[WAVES][16 * kMaxTilesPerWin];
  // a wave's window on its way from loading to operand lanes; then (BLOCKS) what each of its tiles adds to the energies
  constexpr int kMostBlockTiles = window_block(kMaxTilesPerWin);
  __shared__ f32x4 turn_lds[WAVES][BLOCKS ? 5 : 4][64];
  static_assert(!BLOCKS || ONCE, "blocks of a window's tiles are worked on side by side");
  static_assert(!BLOCKS || kMostBlockTiles * 5 * 64 * sizeof(float) <= sizeof(turn_lds[0]), "a block's energies by tile and lane");
  const double inv_d = 1.0 / (double)d, inv_dd = (double)m / (double)n;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // units worked on side by side: one for each wave, or (split) as many as have a wave for every part
  // and (BLOCKS) with a wave for every block of a window's tiles
  const int side_parts = side.parts, parts = split ? 1 : sm.wpu, abreast = side.units;
  const int my_unit = side_div(wave, side.per_unit), of_unit = wave - my_unit * (BLOCKS ? side_parts * blocks : side_parts);
  const int my_block = BLOCKS ? side_div(of_unit, side.per_block) : 0, my_part = of_unit - my_block * side_parts;
  const int block_tiles = window_block(tpw), my_tile = my_block * block_tiles;
  const int tok_tiles = (n + 15) >> 4;
  const int peers = gridDim.x >> 3;
  const Span mine_w = xcd_first(blockIdx.x & 7, along, wins), mine_s = xcd_second(blockIdx.x & 7, along, side.sets);
  const int items = mine_w.count * mine_s.count;
  int item = blockIdx.x >> 3, part = 0;                    // segment under way
  if (item >= items) return;
  // (a workgroup's next item is as many rows and columns of the XCD's rectangle further on: no division for each)
  const int peer_rows = (unsigned)peers / (unsigned)mine_w.count, peer_cols = peers - peer_rows * mine_w.count;

  struct Seg {
    int row, col, win, unit, part, tiles, n0;              // n0: position of the window's first even grid point
    const T* rows;                                         // this lane's columns of token 4 g
    float* score;                                          // of the unit's first token
  };
  auto segment = [&](int row, int col, int pt) {
    Seg s;
    s.part = my_part + pt;
    s.row = row;
    s.col = col;
    const int set = mine_s.from + row;
    s.win = mine_w.from + col;
    s.n0 = __builtin_amdgcn_readfirstlane(first_point(16 * tpw * s.win, m, inv_dd, window_points(r, m))) >> 1;
    s.unit = min(u0 + abreast * set + my_unit, u1 - 1);    // (a surplus wave repeats the last unit)
    s.tiles = min(tpw, tok_tiles - s.win * tpw);
    if (BLOCKS) s.tiles = max(0, min(block_tiles, s.tiles - my_tile));
    if (!ONCE) s.tiles = max(s.tiles, kBuf);               // (a tile too many is worked on and dropped)
    const int slot = lane_slot(s.part, lane & 15, 2 * sm.nb);
    const bool second = slot >= sm.nb;
    s.rows = (second ? V : K) + unit_offset(st, s.unit) + (slot - (second ? sm.nb : 0)) * C + (int64_t)(4 * g) * st.sn;
    s.score = scores + (size_t)out_unit(um, s.unit) * n;
    return s;
  };
  bool follows;                                            // whether there is a segment after the one under way
  auto following = [&](const Seg& s) {
    int it = item, pt = part + 1, row = s.row, col = s.col;
    if (pt == parts) {
      pt = 0;
      it += peers;
      row += peer_rows;
      col += peer_cols;
      if (col >= mine_w.count) { col -= mine_w.count; ++row; }
    }
    follows = !ONCE && it < items;
    return follows ? segment(row, col, pt) : s;
  };
  f32x4 v[C / 2][4];
  auto load_window = [&](const Seg& s) {
    // (addresses are a scalar base and 32 bits of the lane's)
    const int first = s.part * 16, slot = lane_slot(s.part, lane >> 2, 2 * sm.nb) - first;
    const uint32_t at = ((uint32_t)(slot * (C / 2) * m) + 2 * ((lane ^ (lane >> 3)) & 3)) * (uint32_t)sizeof(float2);
    const float2* base = grid + ((size_t)(s.unit - u0) * 2 * sm.nb + first) * (C / 2) * m;
#pragma unroll
    for (int jp = 0; jp < C / 2; ++jp)
#pragma unroll
      for (int c = 0; c < 4; ++c) v[jp][c] = lane_load<f32x4>(base + (size_t)jp * m + (c < 2 ? s.n0 : m - 32 - s.n0) + 8 * c, at);
  };
  const T* ahead;                                          // this lane's columns of token 4 g of the next tile to load
  int ahead_at;                                            // its first token
  auto start_rows = [&](const Seg& s) {
    ahead_at = (s.win * tpw + my_tile) * 16;
    ahead = s.rows + ahead_at * st.sn;
  };
  auto load_rows = [&](RowPiece<T> (&x)[4]) {
    if (ahead_at + 16 <= n) {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i].template load<KEEP>(ahead + i * st.sn);
    } else {                                               // rows past the end repeat the last one
#pragma unroll
      for (int i = 0; i < 4; ++i)
        x[i].template load<KEEP>(ahead + (int64_t)(min(ahead_at + 4 * g + i, n - 1) - ahead_at - 4 * g) * st.sn);
    }
    ahead += 16 * st.sn;
    ahead_at += 16;
  };
  Frag wn[3];
  auto load_weights = [&](const Seg& s, int tl) {
    const u32x4* p = reinterpret_cast<const u32x4*>(winv) + (size_t)(s.win * tpw + min(my_tile + tl, tpw - 1)) * 192;
#pragma unroll
    for (int q = 0; q < 3; ++q) wn[q].u = lane_load<u32x4>(p + 64 * q, lane * (uint32_t)sizeof(u32x4));
  };

  const int first_row = (unsigned)item / (unsigned)mine_w.count;
  Seg cur = segment(first_row, item - first_row * mine_w.count, part);
  RowPiece<T> x[kBuf][4];
  load_window(cur);
  load_weights(cur, 0);
  start_rows(cur);
#pragma unroll
  for (int k = 0; k < kBuf; ++k)
    if (!ONCE || k < cur.tiles) load_rows(x[k]);
  if (ws_mismatch(hdr, FC_PATH_RESAMPLE, n, r, d, dtype)) return;     // (while the above is on its way)
  Seg nxt = following(cur);
  int tl = 0;
  bool more = true;
  Frag bh[C], bl[C];
  float inv = 0.f;
  double hp = 0.0, tot = 0.0;

  const int operand_at = 4 * (lane & 15) + (g ^ ((lane >> 1) & 3));
  // What other lanes of the wave wrote to LDS is there, and what they read of it has been read.  (No instruction: a wave's LDS
  // operations are in order; the compiler, which sees one lane, has to keep them so.)
  auto turned = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
  };
  auto take_window = [&]() {
#pragma unroll
    for (int jp = 0; jp < C / 2; ++jp) {
#pragma unroll
      for (int c = 0; c < 4; ++c) turn_lds[wave][c][lane] = v[jp][c];
      turned();
#pragma unroll
      for (int c = 0; c < 4; ++c) v[jp][c] = turn_lds[wave][c][operand_at];
      turned();
    }
    float mx = 0.f;
#pragma unroll
    for (int jp = 0; jp < C / 2; ++jp)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(v[jp][c][q]));
    // Largest magnitude of the slot's window into [2^14, 2^15); powers of two, so nothing is rounded.  The exponent is
    // the slot's own: columns of K and V, which one wave may hold, can lie any number of octaves apart, and with a
    // common one the smaller tensor's values would run out of bits (2^-30 below: a thousandth of Ehp, 2^-40: all).
    mx = slot_max(mx);
    const int eb = max(14, min((int)(__float_as_uint(mx) >> 23), 254));
    const float scale = __uint_as_float((uint32_t)(268 - eb) << 23);
    inv = ldexpf(1.0f / kInvWeightScale, eb - 141);
#pragma unroll
    for (int jp = 0; jp < C / 2; ++jp)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 2; ++q) halves(v[jp][c][q], v[jp][c][q + 2], scale, bh[2 * jp + q], bl[2 * jp + q], c);
    // (the operands are made here, before their sources' registers are loaded again)
#pragma unroll
    for (int j = 0; j < C; ++j) asm volatile("" : "+v"(bh[j].u), "+v"(bl[j].u));
    hp = tot = 0.0;
    if (!ONCE && follows) load_window(nxt);
  };
  // Energies of the segment: Ehp_k, Ehp_v, Etot_k, Etot_v.  (Slots past the last have sums of 0; a part of one tensor's slots alone,
  // the usual one, takes one pair of sums over the wave, not two.)
  auto record = [&]() {
    const bool second = cur.part * 16 + (lane & 15) >= sm.nb;
    const bool has_k = cur.part * 16 < sm.nb, has_v = cur.part * 16 + 16 > sm.nb;
    double ek = 0.0, ev = 0.0;
    if (has_k) ek = wave_sums(has_v && second ? 0.0 : hp, has_v && second ? 0.0 : tot);
    if (has_v) ev = wave_sums(has_k && !second ? 0.0 : hp, has_k && !second ? 0.0 : tot);
    double* e = epart + (((size_t)cur.unit * wins + cur.win) * sm.wpu + cur.part) * 4;
    if ((lane & 30) == 16) e[(lane >> 5) * 2 + (lane & 1)] = lane & 1 ? ev : ek;
  };
  // Scores of a window (or block) whose unit's parts the workgroup's waves took side by side.
  auto add_parts = [&]() {                                 // (segments are the same for all waves of a workgroup)
    __syncthreads();
    if (my_part == 0)
      for (int k = lane; k < 16 * cur.tiles; k += 64) {
        const int token = (cur.win * tpw + my_tile) * 16 + k;
        double s = part_sum[wave][k];
        for (int p = 1; p < sm.wpu; ++p) s += part_sum[wave + p][k];
        if (token < n && k < 16 * tpw) cur.score[token] = (float)(s * inv_d);
      }
    __syncthreads();
  };
  auto step = [&](RowPiece<T> (&xb)[4]) {
    if (!ONCE && tl == 0) take_window();
    f32x4 acc[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
      acc[j] = mfma_f16(wn[1], bl[j], f32x4{0.f, 0.f, 0.f, 0.f});
      acc[j] = mfma_f16(wn[2], bh[j], acc[j]);
      acc[j] = mfma_f16(wn[0], bl[j], acc[j]);
      acc[j] = mfma_f16(wn[1], bh[j], acc[j]);
      acc[j] = mfma_f16(wn[0], bh[j], acc[j]);
    }
    const bool last = tl + 1 == cur.tiles;
    if (!last) load_weights(cur, tl + 1);
    else if (!ONCE) load_weights(nxt, 0);
    const int t0 = (cur.win * tpw + my_tile + tl) * 16;
    float h[4], t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = t[i] = 0.f;
      residual_piece(xb[i], acc, i, inv, h[i], t[i]);
    }
    // tokens past the end, tiles past the window's own (they are the next window's) and slots past the last
    if (t0 + 16 > n || tl >= tpw || cur.part * 16 + 16 > 2 * sm.nb) {
      const bool slot_used = cur.part * 16 + (lane & 15) < 2 * sm.nb;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t use = slot_used && t0 + 4 * g + i < n && tl < tpw ? ~0u : 0u;
        h[i] = __uint_as_float(__float_as_uint(h[i]) & use);
        t[i] = __uint_as_float(__float_as_uint(t[i]) & use);
      }
    }
    const float hs = (h[0] + h[1]) + (h[2] + h[3]);
    if constexpr (BLOCKS) {
      float* e = reinterpret_cast<float*>(turn_lds[wave]) + tl * 320 + lane;
      e[0] = hs;
#pragma unroll
      for (int i = 0; i < 4; ++i) e[64 * (i + 1)] = t[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) tot += (double)t[i];
      hp += (double)hs;
    }
    double sum = row_sums(h, lane);
    if ((lane & 15) < 4) {
      const int k = 4 * g + (lane & 3), token = t0 + k;
      if (part > 0) sum += part_sum[wave][16 * tl + k];
      if (split || part + 1 < parts) part_sum[wave][16 * tl + k] = sum;
      else if (token < n && tl < tpw) cur.score[token] = (float)(sum * inv_d);
    }
    if (!ONCE && tl + kBuf == cur.tiles) start_rows(nxt);
    if (!ONCE || tl + kBuf < cur.tiles) load_rows(xb);
    ++tl;
    if (last) {
      if constexpr (ONCE) {
        more = false;
      } else {
        asm volatile("");                                  // (keeps what follows out of every tile's path)
        record();
        if (split) add_parts();
        if (++part == parts) { part = 0; item += peers; }
        more = item < items;
        cur = nxt;
        nxt = following(cur);
        tl = 0;
      }
    }
  };
  if (BLOCKS) more = cur.tiles > 0;
  if (ONCE && more) take_window();                         // (out of the loop, in which its registers are free: 232 are 161, of fp32 152 are 113)
  while (more) {
#pragma unroll
    for (int k = 0; k < kBuf; ++k)
      if (more) step(x[k]);
  }
  if constexpr (ONCE) {
    if constexpr (BLOCKS) {
      // the tiles' energies in the order in which a wave that takes all of the window's adds them up
      __syncthreads();
      if (my_tile == 0) {
        hp = tot = 0.0;
        const int tiles = min(tpw, tok_tiles - cur.win * tpw);
        for (int b = 0; b < blocks; ++b) {
          const float* e = reinterpret_cast<const float*>(turn_lds[wave + b * side_parts]) + lane;
          float add[kMostBlockTiles][5];
#pragma unroll
          for (int k = 0; k < kMostBlockTiles; ++k)
#pragma unroll
            for (int i = 0; i < 5; ++i) add[k][i] = e[k * 320 + 64 * i];
          const int left = min(block_tiles, tiles - b * block_tiles);
#pragma unroll
          for (int k = 0; k < kMostBlockTiles; ++k)
            if (k < left) {
#pragma unroll
              for (int i = 1; i < 5; ++i) tot += (double)add[k][i];
              hp += (double)add[k][0];
            }
        }
      }
    }
    if (my_tile == 0) record();
    if (split) add_parts();
  }
}

// lowpass[unit][t] = sum over the tensor's column pairs of the kept energies (fixed order)
__global__ void resample_lowpass_kernel(const double* __restrict__ elow, int pairs, int n_ut,
                                        double* __restrict__ lowpass) {
  const int ut = blockIdx.x * blockDim.x + threadIdx.x;
  if (ut >= n_ut) return;
  double s = 0.0;
  for (int k = 0; k < pairs; ++k) s += elow[(size_t)ut * pairs + k];
  lowpass[ut] = s;
}

template <int M, bool WIDE>
hipError_t launch_filter(float2* grid, int pairs, int n, int r, int d, int dtype, WsHeader* hdr, const float2* filt,
                         const void* twid, double* elow, hipStream_t s) {
  constexpr int T = GridPlan<M, WIDE>::T, PB = T < 64 ? 64 / T : 1;
  const size_t lds = (size_t)PB * GridPlan<M, WIDE>::kLds * sizeof(float);
  auto kern = grid_filter_kernel<M, WIDE>;
  if (lds > 64 * 1024) {
    // raising the dynamic LDS limit is per kernel and per device, and idempotent
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  ProfileScope ps("grid_filter_kernel", s);
  if constexpr (!WIDE && SpreadPlan<M>::kUse) {
    if (pairs <= SpreadPlan<M>::kMostPairs) {
      auto spread = grid_spread_kernel<M>;
      constexpr int kThreads = SpreadPlan<M>::NT;
      constexpr size_t kBytes = 2 * GridPlan<M, WIDE>::kLds * sizeof(float);
      static_assert(kBytes <= 64 * 1024, "a kernel's dynamic LDS without asking for more");
      hipLaunchKernelGGL(spread, dim3(pairs), dim3(kThreads), kBytes, s, grid, n, r, d, dtype, hdr, filt,
                         static_cast<const float2*>(twid), elow);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL(kern, dim3((pairs + PB - 1) / PB), dim3(T < 64 ? 64 : T), lds, s, grid, pairs, n, r, d, dtype,
                     hdr, filt, static_cast<const typename GridFft<M, WIDE>::C*>(twid), elow);
  return hipGetLastError();
}

}  // namespace

// Bytes of grid one round of the three kernels works on.  They are written, read, written and read again: below the
// last-level cache's 256 MB, and with the rows kept out of it (round_keeps_rows), three of the four ways stay on the chip, while
// smaller rounds leave the launches too little to work on.  Scoring 112 units of 30011 tokens, M = 6144, rounds of 176,
// 201, 251 and 302 MB: 1394, 1376, 1337, 1452 us; with ordinary loads of the rows larger rounds are better.  Where the rows are less
// than twice the grid, rounds of 201 MB are (8000 tokens, M = 4096: 168 MB 749 us, 251 MB 766; 32768 tokens, M = 12288: 201
// MB 2122, 251 MB 2141).
constexpr size_t kRoundGridBytes = (size_t)240 << 20;
constexpr int kMaxGrid = 36864;       // points

// The grid lengths are 2^k and 3 2^k points from 64 on, and the longest of which a compute unit's LDS holds one part (real or
// imaginary) of a column pair.
static int next_grid(int m) { return m == 32768 ? kMaxGrid : ((m & (m - 1)) == 0 ? m + m / 2 : m / 3 * 4); }

// Grid length for this shape and cut-off, 0 if the realisation does not apply.  Above 9362 modes (16384 points) it starts again
// with 2.6 points a mode or fewer (9453 modes on; 2.4 where tokens are fewer than points: 10240 on).  No time or error speaks for that line:
// the grid of 24576 points serves the cut-offs before it as well, eight units of 30000 tokens, r = 9400 in 357 us where the basis takes 12833,
// of 24000, r = 10000 337 / 10370, of 32768, r = 9400 380 where the streaming transform takes 656.  It stands because the interface has them
// refused by FC_PATH_RESAMPLE and realised by the other two, which programs that name a path, and the tests, rely on.
// Scoring by that realisation / this one, us (bf16, 128 columns): basis 12 units of 47568 tokens, r = 10894 34113 / 565, 8 of 44736,
// r = 17649 34666 / 419, 8 of 50000, r = 20501 46754 / 528, 2 of 24600, r = 11071 2585 / 76; streaming 16 of 42752, r = 10415 18677 / 726,
// 32 of 32768, r = 13108 2508 / 1451, 4 of 65536, r = 19661 728 / 148.  Error of the scores against 64 bits, white columns:
// 29435 tokens, r = 10759 2.3e-7 (basis) / 4.5e-8, 30720, r = 14300 6.5e-8 (streaming) / 5.0e-8, 37449, r = 18724 4.3e-7 / 6.2e-8.
static int grid_length(const fc_kv_desc& d, int32_t r) {
  const int64_t n = d.n_tokens;
  if (d.head_dim % 8 != 0 || d.head_dim > 256 || r < 1 || 2 * (int64_t)r > n) return 0;
  int64_t m = 64;
  while (4 * m < 7 * (int64_t)r || 16 * m < n) {           // M >= 1.75 r: see window_points
    if (m >= (r > 9362 ? kMaxGrid : 16384)) return 0;
    m = next_grid((int)m);
  }
  if (m > 16384 && 5 * m > (n >= m ? 13 : 12) * (int64_t)r) return 0;
  // a 16-token tile and its windows fit 32 points: 15 M/N + W < 29
  return 5 * n >= 4 * m ? (int)m : 0;
}

// Whether the grid transform is computed in 64 bits.  Its rounding in 32 comes back from modes near the cut-off
// multiplied by 1 / phihat there, and counts against a residual that shrinks as the cut-off rises.  Error of the scores
// against 64 bits (2-norm, 1e-8): streaming transform or explicit basis / this realisation in 32 bits / in 64 bits:
//   N, r, M             32768, 1639, 3072   4864, 674, 1536   3001, 991, 2048   7680, 2305, 4096   1111, 293, 768
//                       5.1 / 3.3 / -       5.1 / 3.7 / -     6.9 / 6.0 / 4.0   6.4 / 7.2 / 4.4    5.4 / 6.1 / 3.4
//   N, r, M             16384, 3277, 6144   32768, 6554, 12288   10562, 2968, 6144   32768, 9176, 16384
//                       10.1 / 4.2 / -      11.4 / 4.1 / -       10.5 / 5.8 / 3.4    11.2 / 3.9 / 3.2
// So it is taken where 32 bits are worse than the other realisations: above r = N/4 for grids of up to 4096 points (the
// longer ones' shapes take those several passes over an fp32 residual, or sums of 10000 products).  The filter takes
// 1.4 times as long (14336 column pairs of 4096 points: 240 / 330 us).
static bool wide_transform(int64_t n, int64_t r, int64_t m) { return m <= 4096 && 4 * r > n; }

// (below 256 tokens the products with the basis itself are as quick and need no plan worth speaking of)
bool resample_supported(const fc_kv_desc& d, int32_t r) { return d.n_tokens >= 256 && grid_length(d, r) != 0; }

ResampleLayout resample_layout(const fc_kv_desc& d, int32_t r) {
  ResampleLayout lay{};
  const int64_t n = d.n_tokens, m = grid_length(d, r);
  const size_t units = (size_t)d.batch * d.layers * d.kv_heads;
  lay.m = (int)m;
  lay.wide = wide_transform(n, r, m);
  // tokens under a tile of 16 grid points: at most (15 + W) N/M + 1, and the 32-token steps they lie in
  const int w = window_points(r, (int)m);
  lay.steps = (int)std::min(((15 + w) * n / m + 31) / 32 + 1, (n + 31) / 32);
  // tiles whose windows fit 32 grid points when the first point is rounded down to a multiple of 4: the positions of
  // 16 tpw tokens span (16 tpw - 1) M/N, and together with W that has to be less than 29
  lay.tpw = (int)std::min<int64_t>(kMaxTilesPerWin, (((29 - w) * n - 1) / m + 1) / 16);
  const int tok_tiles = (int)((n + 15) / 16);
  lay.wins = (tok_tiles + lay.tpw - 1) / lay.tpw;
  lay.pairs = d.head_dim / 2;
  lay.nb = d.head_dim * (d.dtype == FC_BF16 ? 2 : 4) / 16;
  lay.wpu = slot_waves(2 * lay.nb);
  // units per round of the three kernels
  const size_t unit_grid = 2 * (size_t)m * d.head_dim * sizeof(float);
  const bool much_grid = (size_t)n * (d.dtype == FC_BF16 ? 2 : 4) < 2 * (size_t)m * sizeof(float);
  const int most = (int)std::max<size_t>(1, (much_grid ? kRoundGridBytes / 6 * 5 : kRoundGridBytes) / unit_grid);
  lay.chunk = round_units((int)units, most, (lay.wins + 7) / 8);
  auto up = [](size_t x) { return (x + kWsAlign - 1) / kWsAlign * kWsAlign; };
  size_t off = sizeof(WsHeader);
  lay.wfwd = off; off = up(off + (size_t)(m / 16) * lay.steps * 512 * sizeof(float));
  lay.winv = off; off = up(off + (size_t)lay.wins * lay.tpw * 1536 * 2);
  lay.filt = off; off = up(off + (size_t)m * sizeof(float2));
  lay.twid = off; off = up(off + (size_t)twid_size((int)m, lay.wide) * (lay.wide ? sizeof(double2) : sizeof(float2)));
  lay.elow = off; off = up(off + units * 2 * lay.pairs * sizeof(double));
  lay.epart = off; off = up(off + units * lay.wins * lay.wpu * 4 * sizeof(double));
  // (room for the most units of a round: fewer units than these may make a round longer than theirs)
  lay.grid = off; off = up(off + kGridSlack + std::min<size_t>(units, most) * 2 * lay.pairs * m * sizeof(float2));
  lay.total = off;
  return lay;
}

// Upper bound, over all cut-offs, of what this realisation needs beyond the streaming transform's
// partial sums: one workspace size per shape and cut-off serves both.
size_t resample_reserve(const fc_kv_desc& d) {
  if (d.head_dim > 256 || d.n_tokens < 256) return 0;
  const size_t n = d.n_tokens, nb = d.head_dim / 8, units = (size_t)d.batch * d.layers * d.kv_heads;
  const size_t m = std::min<size_t>(kMaxGrid, n * 5 / 4);
  const size_t tables = 296 * n + 288 * m + (256 << 10);
  const size_t records = units * (64 * nb + 2 * n * slot_waves(2 * (int)nb * (d.dtype == FC_BF16 ? 1 : 2)) + 64 * 8);
  const size_t grid = std::max<size_t>(kRoundGridBytes, 64 * nb * m);
  const size_t need = tables + records + std::min<size_t>(grid, units * 64 * nb * m);
  const size_t have = units * 2 * (nb / 2) * n * sizeof(float);
  return need > have ? (need - have + kWsAlign - 1) / kWsAlign * kWsAlign : 0;
}

hipError_t resample_prepare(const fc_kv_desc& d, int32_t r, const ResampleLayout& lay, void* ws, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  TablePtrs tp{reinterpret_cast<WsHeader*>(base), reinterpret_cast<float*>(base + lay.wfwd),
               reinterpret_cast<_Float16*>(base + lay.winv), reinterpret_cast<float2*>(base + lay.filt), base + lay.twid};
  const int n_wfwd = lay.m / 16 * lay.steps * 512, n_winv = lay.wins * lay.tpw * 512;
  const TwidPlan plan = make_twid_plan(lay.m, lay.wide);
  const int total = n_wfwd + n_winv + lay.m + plan.size;
  ProfileScope ps("resample_table_kernel", s);
  hipLaunchKernelGGL(resample_table_kernel, dim3((total + 255) / 256), dim3(256), 0, s, tp, d.n_tokens, r, lay.m,
                     d.head_dim, d.dtype, lay.steps, lay.tpw, n_wfwd, n_winv, lay.wide,
                     make_window(r, lay.m), plan);
  return hipGetLastError();
}

template <typename T, int GT, bool KEEP>
static hipError_t launch_decimate_gt(const T* K, const T* V, KvStrides st, int u0, int u1, int n, int r,
                                     const fc_kv_desc& d, int m, const ResampleLayout& lay, SlotMap sm, Sides sides, int along,
                                     WsHeader* hdr, const float* wfwd, float2* grid, hipStream_t s) {
  auto kern = decimate_kernel<T, GT, KEEP>;
  const size_t lds = (size_t)GT * lay.steps * 2048;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  ProfileScope ps("decimate_kernel", s);
  hipLaunchKernelGGL(kern, dim3(8 * xcd_items(along, sides)), dim3(64 * kDecWaves), lds, s, K, V, st, u0, u1, n, r, d.head_dim,
                     d.dtype, m, lay.steps, sm, sides.second, along, hdr, wfwd, grid);
  return hipGetLastError();
}

template <typename T, bool KEEP>
static hipError_t resample_score_t(const T* K, const T* V, const fc_kv_desc& d, int32_t r, const ResampleLayout& lay,
                                   float* scores, double* energy, void* ws, UnitMap um, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  WsHeader* hdr = reinterpret_cast<WsHeader*>(base);
  const int units = d.batch * d.layers * d.kv_heads, n = d.n_tokens, m = lay.m;
  float2* grid = reinterpret_cast<float2*>(grid_start(reinterpret_cast<uintptr_t>(base) + lay.grid));
  const float2* filt = reinterpret_cast<const float2*>(base + lay.filt);
  const void* twid = base + lay.twid;
  double* epart = reinterpret_cast<double*>(base + lay.epart);
  const SlotMap sm{lay.nb, lay.wpu};
  const KvStrides st = strides_of(d);
  // each XCD takes a contiguous range of tiles (or windows), so that its L2 holds that range's weights
  // and the rows neighbouring tiles share
  for (int u0 = 0; u0 < units; u0 += lay.chunk) {
    const int u1 = std::min(units, u0 + lay.chunk);
    const int groups = ((u1 - u0) * sm.wpu + kDecWaves - 1) / kDecWaves;
    const int gt = decimate_tiles(m, groups, lay.steps, sizeof(T) == 2, 2 * lay.nb, (long long)(u1 - u0) * 2 * n * d.head_dim * (int)sizeof(T));
    const Sides dec{(m / 16 + gt - 1) / gt, groups};
    const ResidualPlan res = residual_plan(lay.wins, lay.tpw, 2 * lay.nb, u1 - u0, dec, sizeof(T) == 2);
    const float* wfwd = reinterpret_cast<const float*>(base + lay.wfwd);
    auto decimate = gt == 4 ? launch_decimate_gt<T, 4, KEEP> : (gt == 2 ? launch_decimate_gt<T, 2, KEEP> : launch_decimate_gt<T, 1, KEEP>);
    hipError_t e = decimate(K, V, st, u0, u1, n, r, d, m, lay, sm, dec, res.along, hdr, wfwd, grid, s);
    if (e != hipSuccess) return e;
    double* elow = reinterpret_cast<double*>(base + lay.elow) + (size_t)u0 * 2 * lay.pairs;
    const int pairs = (u1 - u0) * 2 * lay.pairs;
#define FC_FILTER(MV, WIDE) launch_filter<MV, WIDE>(grid, pairs, n, r, d.head_dim, d.dtype, hdr, filt, twid, elow, s)
#define FC_NARROW(MV) case MV: e = FC_FILTER(MV, false); break;
#define FC_EITHER(MV) case MV: e = lay.wide ? FC_FILTER(MV, true) : FC_FILTER(MV, false); break;
    switch (m) {
      FC_NARROW(64) FC_NARROW(96)
      FC_EITHER(128) FC_EITHER(192) FC_EITHER(256) FC_EITHER(384) FC_EITHER(512) FC_EITHER(768) FC_EITHER(1024)
      FC_EITHER(1536) FC_EITHER(2048) FC_EITHER(3072) FC_EITHER(4096)
      FC_NARROW(6144) FC_NARROW(8192) FC_NARROW(12288) FC_NARROW(16384) FC_NARROW(24576) FC_NARROW(32768)
      FC_NARROW(36864)
      default: e = hipErrorInvalidValue;
    }
#undef FC_EITHER
#undef FC_NARROW
#undef FC_FILTER
    if (e != hipSuccess) return e;
    {
      ProfileScope ps("residual_kernel", s);
      // Windows of a single tile (token counts below 1.7 times the grid's): with a second tile under way each would be worked on
      // twice.  Residual, two tiles / one under way: 28 layers of 8192 tokens, M = 6144 390 / 342 us, 4 layers 54 / 45, 28 of 4096,
      // M = 3072 201 / 179.
      constexpr bool kWide = sizeof(T) == 4;               // (a unit has more than four parts: fp32 rows of more than 128 columns)
      auto kern = res.blocks > 1 ? (res.waves > 4 ? residual_kernel<T, KEEP, true, true, 2, 8> : residual_kernel<T, KEEP, true, true, 2, 4>)
                  : res.once     ? residual_kernel<T, KEEP, true, false, 2, 4>
                  : lay.tpw > 1  ? residual_kernel<T, KEEP, false, false, 2, 4> : residual_kernel<T, KEEP, false, false, 1, 4>;
      if constexpr (kWide)
        if (res.blocks == 1 && res.waves > 4)
          kern = res.once ? residual_kernel<T, KEEP, true, false, 2, 8>
                 : lay.tpw > 1 ? residual_kernel<T, KEEP, false, false, 2, 8> : residual_kernel<T, KEEP, false, false, 1, 8>;
      const int side_parts = res.split ? lay.wpu : 1;
      const SideBySide side{res.abreast, side_parts, (u1 - u0 + res.abreast - 1) / res.abreast, side_factor(side_parts * res.blocks), side_factor(side_parts)};
      hipLaunchKernelGGL(kern, dim3(8 * res.workgroups), dim3(64 * res.waves), 0, s, K, V, st, u0, u1, n, r,
                         d.head_dim, d.dtype, m, lay.tpw, lay.wins, sm, res.split, res.blocks, side, res.along, hdr, reinterpret_cast<const _Float16*>(base + lay.winv),
                         grid, scores, epart, um);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return energy_reduce_launch(epart, lay.wins * lay.wpu, units, energy, um, s);
}

static bool keep_rows(const fc_kv_desc& d, const ResampleLayout& lay) {
  const int row_bytes = d.head_dim * (d.dtype == FC_BF16 ? 2 : 4);
  return round_keeps_rows((long long)lay.chunk * 2 * d.n_tokens * row_bytes, row_bytes);
}

hipError_t resample_score(const void* K, const void* V, const fc_kv_desc& d, int32_t r, const ResampleLayout& lay,
                          float* scores, double* energy, void* ws, UnitMap um, hipStream_t s) {
  auto run = [&](auto score, const auto* k, const auto* v) { return score(k, v, d, r, lay, scores, energy, ws, um, s); };
  if (d.dtype == FC_BF16) {
    const uint16_t *k = static_cast<const uint16_t*>(K), *v = static_cast<const uint16_t*>(V);
    return keep_rows(d, lay) ? run(resample_score_t<uint16_t, true>, k, v) : run(resample_score_t<uint16_t, false>, k, v);
  }
  const float *k = static_cast<const float*>(K), *v = static_cast<const float*>(V);
  return keep_rows(d, lay) ? run(resample_score_t<float, true>, k, v) : run(resample_score_t<float, false>, k, v);
}

hipError_t resample_lowpass(const fc_kv_desc& d, const ResampleLayout& lay, void* ws, double* lowpass, hipStream_t s) {
  const int n_ut = d.batch * d.layers * d.kv_heads * 2;
  ProfileScope ps("resample_lowpass_kernel", s);
  hipLaunchKernelGGL(resample_lowpass_kernel, dim3((n_ut + 255) / 256), dim3(256), 0, s,
                     reinterpret_cast<const double*>(static_cast<char*>(ws) + lay.elow), lay.pairs, n_ut, lowpass);
  return hipGetLastError();
}

}  // namespace fc
