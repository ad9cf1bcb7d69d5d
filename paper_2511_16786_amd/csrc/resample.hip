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
// only approximation, below 1e-8 of the signal for M >= 1.75 r and W = 9 (fp32 rounding is 1e-7).  The
// same operator serves every N, since the token positions enter through the window weights alone.
//
// The banded products run on the matrix cores with their operands split so that fp32 accuracy is kept:
// bf16 inputs are exact and meet weights split in three bf16 terms; grid values, scaled to a common
// exponent per window, and weights are split in two fp16 terms each (22 bits and the rounding of the
// second term) and the product of the two second terms, 2^-24 of the whole, is left out.
#include <algorithm>

#include "fc_common.h"

namespace fc {

namespace {

constexpr int kW = 9;                  // grid points a token's window reaches
constexpr int kPathResample = 3;       // header tag of a workspace prepared for this realisation
constexpr int kMaxTilesPerWin = 16;    // 16-token tiles one wave of the residual kernel walks
constexpr float kInvWeightScale = 4096.0f;   // fp16 weights are stored times 2^12 (their tails stay normal numbers)

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
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

__device__ double bessel_i0(double x) {          // power series, all terms positive
  const double q = 0.25 * x * x;
  double term = 1.0, sum = 1.0;
  for (int k = 1; k < 200; ++k) {
    term *= q / ((double)k * (double)k);
    sum += term;
    if (term < sum * 1e-18) break;
  }
  return sum;
}

__device__ double window(double s, double beta, double inv_i0) {
  const double z = s * (2.0 / kW);
  const double t = 1.0 - z * z;
  return t >= 0.0 ? bessel_i0(beta * sqrt(t)) * inv_i0 : 0.0;
}

// weight between token position u and grid point k, images of the even extension included
__device__ double weight_at(double u, int k, int m, double beta, double inv_i0) {
  return window(u - k, beta, inv_i0) + window(u + 1.0 + k, beta, inv_i0) +
         window(2.0 * m - 1.0 - k - u, beta, inv_i0);
}

__device__ __forceinline__ uint32_t bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u + ((u >> 16) & 1u) + 0x7FFFu) >> 16;
}

// position of grid point k in the order the transform takes its input (even points ascending, then
// odd points descending)
__device__ __forceinline__ int grid_pos(int k, int m) { return (k & 1) ? m - 1 - (k >> 1) : k >> 1; }

struct TablePtrs {
  WsHeader* hdr;
  uint16_t* wfwd;    // [M/16][steps][3][64][8] bf16
  _Float16* winv;    // [tokens/16][2][64][8] fp16
  int* t0;           // [M/16] first token of a grid tile
  int* k0;           // [windows] first grid point of a window
  float2* filt;      // [M] (f[m] + f[M-m]) / 2, (f[m] - f[M-m]) / 2
  float2* twid;      // see GridFft
};

// twiddle table: six powers (1,2,3,4,8,12) of w_{16 Ns} for Ns = 16 and 256, then the last pass's
// powers w_M^{t q}, q = 1..R-1, then e^{i pi t / M}, t < M/16 each
__host__ __device__ constexpr int last_radix(int m) { return m % 4096 == 0 ? (m == 4096 ? 1 : m / 4096) : m / 256; }
__host__ __device__ constexpr int twid16_off() { return 0; }
__host__ __device__ constexpr int twid256_off() { return 6 * 16; }
__host__ __device__ constexpr int twid_last_off(int m) { return 6 * 16 + (m >= 4096 ? 6 * 256 : 0); }
__host__ __device__ constexpr int twid_phase_off(int m) {
  return twid_last_off(m) + (last_radix(m) > 1 ? (last_radix(m) - 1) * (m / 16) : 0);
}
__host__ __device__ constexpr int twid_size(int m) { return twid_phase_off(m) + m / 16; }

__device__ float2 unit_root(double frac) {        // e^{-2 pi i frac}
  double s, c;
  sincospi(2.0 * frac, &s, &c);
  return make_float2((float)c, (float)-s);
}

// One thread per 8-weight fragment piece and per table entry; runs once per plan.
__global__ __launch_bounds__(256) void resample_table_kernel(TablePtrs tp, int n, int r, int m, int d, int dtype,
                                                             int steps, int tpw, int n_wfwd, int n_winv) {
  int id = blockIdx.x * blockDim.x + threadIdx.x;
  const double dd = (double)n / (double)m;        // tokens per grid point
  const double inv_dd = (double)m / (double)n;
  const double beta = M_PI * kW * (1.0 - 0.5 * (double)r / (double)m);
  const double inv_i0 = 1.0 / bessel_i0(beta);
  if (id == 0) {
    WsHeader h{};
    h.magic = kWsMagic; h.path = kPathResample; h.n = n; h.r = r; h.d = d; h.dtype = dtype;
    *tp.hdr = h;
  }
  if (id < n_wfwd) {
    const int lane = id & 63, step = (id >> 6) % steps, tile = (id >> 6) / steps;
    int t0 = (int)ceil(dd * (16.0 * tile - 0.5 * kW + 0.5) - 0.5);
    t0 = max(0, min(t0, n - 32 * steps));
    if (lane == 0 && step == 0) tp.t0[tile] = t0;
    const int k = 16 * tile + (lane & 15);
    const int i0 = t0 + 32 * step + 8 * (lane >> 4);
    uint16_t p[3][8];
    for (int e = 0; e < 8; ++e) {
      const double w = weight_at((i0 + e + 0.5) * inv_dd - 0.5, k, m, beta, inv_i0);
      double rest = w;
      for (int q = 0; q < 3; ++q) {
        const uint32_t b = bf16_rne((float)rest);
        p[q][e] = (uint16_t)b;
        rest -= (double)bf16_to_f32(b);
      }
    }
    for (int q = 0; q < 3; ++q)
      for (int e = 0; e < 8; ++e) tp.wfwd[((size_t)(tile * steps + step) * 3 + q) * 512 + lane * 8 + e] = p[q][e];
    return;
  }
  id -= n_wfwd;
  if (id < n_winv) {
    const int lane = id & 63, tile = id >> 6, win = tile / tpw;
    const double uf = (16.0 * tpw * win + 0.5) * inv_dd - 0.5;
    int k0 = (int)ceil(uf - 0.5 * kW);
    k0 = max(0, min(k0, m - 32)) & ~3;
    if (lane == 0 && tile == win * tpw) tp.k0[win] = k0;
    const int i = 16 * tile + (lane & 15), g = lane >> 4;
    const double u = (i + 0.5) * inv_dd - 0.5;
    for (int e = 0; e < 8; ++e) {
      // the order in which the residual kernel's loads deliver the window's grid points
      const int k = g < 2 ? k0 + 2 * (8 * g + e) : k0 + 2 * (7 + 8 * (g - 2) - e) + 1;
      const double w = i < n ? kInvWeightScale * weight_at(u, k, m, beta, inv_i0) : 0.0;
      const _Float16 hi = (_Float16)(float)w;
      tp.winv[(size_t)tile * 1024 + lane * 8 + e] = hi;
      tp.winv[(size_t)tile * 1024 + 512 + lane * 8 + e] = (_Float16)(float)(w - (double)hi);
    }
    return;
  }
  id -= n_winv;
  if (id < m) {
    auto f = [&](int q) -> double {
      if (q >= r) return 0.0;
      const double a = 0.5 * M_PI * kW * q / m;
      const double s = sqrt(beta * beta - a * a);
      const double ph = kW * sinh(s) / s * inv_i0;
      return 1.0 / ((double)n * ph * ph);
    };
    const double fa = f(id), fb = f(m - id);
    tp.filt[id] = make_float2((float)(0.5 * (fa + fb)), (float)(0.5 * (fa - fb)));
    return;
  }
  id -= m;
  if (id >= twid_size(m)) return;
  const int pw[6] = {1, 2, 3, 4, 8, 12};
  float2 v;
  if (id < twid256_off()) {
    v = unit_root((double)(pw[id / 16] * (id % 16)) / 256.0);
  } else if (id < twid_last_off(m)) {
    const int j = id - twid256_off();
    v = unit_root((double)(pw[j / 256] * (j % 256)) / 4096.0);
  } else if (id < twid_phase_off(m)) {
    const int j = id - twid_last_off(m), t = m / 16;
    v = unit_root((double)((long long)(j / t + 1) * (j % t)) / (double)m);
  } else {
    v = unit_root(-0.5 * (double)(id - twid_phase_off(m)) / (double)m);
  }
  tp.twid[id] = v;
}

// ---------------------------------------------------------------------------- decimation

// The 2*nb column blocks (8 columns each) of a unit's K and V rows are dealt out to waves of 16 slots.
struct SlotMap {
  int nb;        // blocks per tensor (head_dim / 8)
  int wpu;       // waves per unit: 1, 2 or 4
};

template <typename T>
struct RowPiece;                                   // 8 columns of one row

template <>
struct RowPiece<uint16_t> {
  u32x4 v;
  __device__ __forceinline__ void load(const uint16_t* p) { v = *reinterpret_cast<const u32x4*>(p); }
};
template <>
struct RowPiece<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
};

__device__ __forceinline__ f32x4 mfma_bf16(const Frag& a, const Frag& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.b, b.b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f16(const Frag& a, const Frag& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c, 0, 0, 0);
}

// acc[j] += (column j of the 8 rows in x, for 16 slots) x (weights of this step)
__device__ __forceinline__ void fold_rows(const RowPiece<uint16_t> (&x)[8], const Frag (&w)[3], f32x4 (&acc)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    Frag a;
#pragma unroll
    for (int p = 0; p < 4; ++p)
      a.u[p] = __builtin_amdgcn_perm(x[2 * p + 1].v[j >> 1], x[2 * p].v[j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
    for (int q = 2; q >= 0; --q) acc[j] = mfma_bf16(a, w[q], acc[j]);
  }
}

__device__ __forceinline__ void fold_rows(const RowPiece<float> (&x)[8], const Frag (&w)[3], f32x4 (&acc)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    // x = x0 + x1 + x2 in bf16 terms; the products below 2^-24 of the whole are left out
    Frag a[3];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t t[3][2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float v = j < 4 ? x[2 * p + h].a[j & 3] : x[2 * p + h].b[j & 3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          t[q][h] = bf16_rne(v);
          v -= bf16_to_f32(t[q][h]);
        }
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q].u[p] = t[q][0] | (t[q][1] << 16);
    }
    acc[j] = mfma_bf16(a[2], w[0], acc[j]);
    acc[j] = mfma_bf16(a[0], w[2], acc[j]);
    acc[j] = mfma_bf16(a[1], w[1], acc[j]);
    acc[j] = mfma_bf16(a[1], w[0], acc[j]);
    acc[j] = mfma_bf16(a[0], w[1], acc[j]);
    acc[j] = mfma_bf16(a[0], w[0], acc[j]);
  }
}

// One wave: 16 grid points x 16 slots (128 columns), walking the tokens under the tile's windows 32
// at a time.  Rows go from memory straight into matrix operands: a lane loads 16 bytes of 8 consecutive
// rows and swaps the two halves of the words in registers (the order of the contraction is free).
template <typename T>
__global__ __launch_bounds__(256) void decimate_kernel(const T* __restrict__ K, const T* __restrict__ V,
                                                       KvStrides st, int u0, int u1, int n, int r, int d,
                                                       int dtype, int m, int steps, SlotMap sm, int tiles_per_xcd,
                                                       WsHeader* hdr, const uint16_t* __restrict__ wfwd,
                                                       const int* __restrict__ t0s, float2* __restrict__ grid) {
  if (ws_mismatch(hdr, kPathResample, n, r, d, dtype)) return;
  const int xcd = blockIdx.x & 7, slot_id = blockIdx.x >> 3;
  const int tile = xcd * tiles_per_xcd + slot_id % tiles_per_xcd;
  if (tile >= m / 16) return;
  const int lane = threadIdx.x & 63;
  const int gw = (slot_id / tiles_per_xcd) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = u0 + gw / sm.wpu, part = gw % sm.wpu;
  if (unit >= u1) return;
  const int s_mine = part * 16 + (lane & 15);
  const int slot = s_mine < 2 * sm.nb ? s_mine : 0;
  const bool second = slot >= sm.nb;
  const int t0 = t0s[tile];
  const T* p = (second ? V : K) + unit_offset(st, unit) + (slot - (second ? sm.nb : 0)) * 8 +
               (int64_t)(t0 + 8 * (lane >> 4)) * st.sn;
  const u32x4* wp = reinterpret_cast<const u32x4*>(wfwd) + (size_t)tile * steps * 192 + lane;

  f32x4 acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  RowPiece<T> x[8];
  Frag w[3];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e].load(p + e * st.sn);
#pragma unroll
  for (int q = 0; q < 3; ++q) w[q].u = wp[q * 64];
  for (int s = 1; s < steps; ++s) {
    p += 32 * st.sn;
    wp += 192;
    RowPiece<T> xn[8];
    Frag wn[3];
#pragma unroll
    for (int e = 0; e < 8; ++e) xn[e].load(p + e * st.sn);
#pragma unroll
    for (int q = 0; q < 3; ++q) wn[q].u = wp[q * 64];
    fold_rows(x, w, acc);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = xn[e];
#pragma unroll
    for (int q = 0; q < 3; ++q) w[q] = wn[q];
  }
  fold_rows(x, w, acc);

  const int pos = grid_pos(16 * tile + (lane & 15), m);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s_out = part * 16 + 4 * (lane >> 4) + i;
    if (s_out < 2 * sm.nb) {
      float2* o = grid + ((size_t)(unit - u0) * 2 * sm.nb + s_out) * 4 * m + pos;
#pragma unroll
      for (int jp = 0; jp < 4; ++jp) o[(size_t)jp * m] = make_float2(acc[2 * jp][i], acc[2 * jp + 1][i]);
    }
  }
}

// ---------------------------------------------------------------------------- filter on the grid

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
template <bool INV>
__device__ __forceinline__ float2 cmul(float2 a, float2 w) {      // a * w, or a * conj(w)
  return INV ? make_float2(fmaf(a.x, w.x, a.y * w.y), fmaf(a.y, w.x, -a.x * w.y))
             : make_float2(fmaf(a.x, w.x, -a.y * w.y), fmaf(a.y, w.x, a.x * w.y));
}
template <bool INV>
__device__ __forceinline__ void fft4(float2& a, float2& b, float2& c, float2& d) {
  const float2 s = cadd(a, c), t = csub(a, c), u = cadd(b, d), v = csub(b, d);
  a = cadd(s, u);
  c = csub(s, u);
  const float2 p = make_float2(t.x + v.y, t.y - v.x), q = make_float2(t.x - v.y, t.y + v.x);
  b = INV ? q : p;
  d = INV ? p : q;
}
// w_16^k, k < 16, as e^{-2 pi i k / 16}
__device__ constexpr float kCos16[16] = {1.f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f,
                                         0.f, -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f,
                                         -1.f, -0.92387953251128674f, -0.70710678118654752f, -0.38268343236508977f,
                                         0.f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f};
__device__ __forceinline__ constexpr float2 w16(int k) { return float2{kCos16[k & 15], kCos16[(k + 4) & 15]}; }

// x[q] -> X[q], result q at x[4 (q % 4) + q / 4]
template <bool INV>
__device__ __forceinline__ void fft16(float2 (&x)[16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) fft4<INV>(x[i], x[i + 4], x[i + 8], x[i + 12]);
#pragma unroll
  for (int k = 1; k < 4; ++k)
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      float2& v = x[i + 4 * k];
      if (i * k == 4) v = INV ? make_float2(-v.y, v.x) : make_float2(v.y, -v.x);
      else v = cmul<INV>(v, w16(i * k));
    }
#pragma unroll
  for (int k = 0; k < 4; ++k) fft4<INV>(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
}
__device__ __forceinline__ constexpr int rev16(int q) { return 4 * (q & 3) + (q >> 2); }

__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 4); }   // keeps stride-16 writes off one bank

// Length-M complex transform of one column pair by M/16 threads; thread t holds the points t + (M/16) q
// before and after (natural order both sides), exchanges go through LDS.
template <int M, bool INV>
struct GridFft {
  static constexpr int T = M / 16, R = last_radix(M);
  static __device__ __forceinline__ void exchange(float2 (&x)[16], float2* lds, int base, int ns, int t) {
#pragma unroll
    for (int q = 0; q < 16; ++q) lds[lds_pad(base + q * ns)] = x[rev16(q)];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = lds[lds_pad(t + T * q)];
    __syncthreads();
  }
  static __device__ __forceinline__ void twiddle(float2 (&x)[16], const float2* __restrict__ tw, int ns, int j) {
    float2 p[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = tw[i * ns + j];
#pragma unroll
    for (int q = 1; q < 16; ++q) {
      const int lo = q & 3, hi = q >> 2;
      if (hi == 0) x[q] = cmul<INV>(x[q], p[lo - 1]);
      else if (lo == 0) x[q] = cmul<INV>(x[q], p[2 + hi]);
      else x[q] = cmul<INV>(x[q], cmul<false>(p[lo - 1], p[2 + hi]));
    }
  }
  static __device__ __forceinline__ void run(float2 (&x)[16], float2* lds, const float2* __restrict__ twid, int t) {
    fft16<INV>(x);
    exchange(x, lds, t * 16, 1, t);
    twiddle(x, twid + twid16_off(), 16, t & 15);
    fft16<INV>(x);
    exchange(x, lds, (t >> 4) * 256 + (t & 15), 16, t);
    if (M >= 4096) {
      twiddle(x, twid + twid256_off(), 256, t & 255);
      fft16<INV>(x);
      if (M > 4096) {
        exchange(x, lds, (t >> 8) * 4096 + (t & 255), 256, t);
      } else {
        float2 y[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) y[q] = x[rev16(q)];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = y[q];
      }
    }
    if (R > 1) {
      constexpr int C = 16 / (R > 1 ? R : 2);       // butterflies of this thread: points c + C q
      float2 b[R > 1 ? R : 2];
#pragma unroll
      for (int q = 1; q < R; ++q) b[q] = twid[twid_last_off(M) + (q - 1) * T + t];
#pragma unroll
      for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int q = 1; q < R; ++q) {
          // w_M^{(t + T c) q} = w_M^{t q} w_16^{c q}
          const float2 w = (c == 0) ? b[q] : cmul<false>(b[q], w16(c * q));
          x[c + C * q] = cmul<INV>(x[c + C * q], w);
        }
        if (R == 2) {
          const float2 a = x[c], v = x[c + C];
          x[c] = cadd(a, v);
          x[c + C] = csub(a, v);
        } else if (R == 4) {
          fft4<INV>(x[c], x[c + C], x[c + 2 * C], x[c + 3 * C]);
        } else if (R == 8) {
          // even and odd inputs, then the eighth-root butterflies
          float2 e0 = x[c], e1 = x[c + 2 * C], e2 = x[c + 4 * C], e3 = x[c + 6 * C];
          float2 o0 = x[c + C], o1 = x[c + 3 * C], o2 = x[c + 5 * C], o3 = x[c + 7 * C];
          fft4<INV>(e0, e1, e2, e3);
          fft4<INV>(o0, o1, o2, o3);
          o1 = cmul<INV>(o1, w16(2));
          o2 = INV ? make_float2(-o2.y, o2.x) : make_float2(o2.y, -o2.x);
          o3 = cmul<INV>(o3, w16(6));
          x[c] = cadd(e0, o0); x[c + 4 * C] = csub(e0, o0);
          x[c + C] = cadd(e1, o1); x[c + 5 * C] = csub(e1, o1);
          x[c + 2 * C] = cadd(e2, o2); x[c + 6 * C] = csub(e2, o2);
          x[c + 3 * C] = cadd(e3, o3); x[c + 7 * C] = csub(e3, o3);
        }
      }
    }
  }
};

// One column pair (as real and imaginary part) per M/16 threads, in place: transform, keep and weight the
// modes below the cut-off, transform back.  With the permuted input order the DFT carries DCT modes m and
// M-m in the pair of bins (m, M-m):
//     W'[m] = (f[m] + f[M-m])/2 W[m] + (f[m] - f[M-m])/2 e^{i pi m/M} W[M-m].
// sum_m Re(conj(W) W') is the kept energy of both columns (the operator is symmetric).
template <int M>
__global__ __launch_bounds__(M / 16 < 64 ? 64 : M / 16) void grid_filter_kernel(
    float2* __restrict__ grid, int pairs, int n, int r, int d, int dtype, WsHeader* hdr,
    const float2* __restrict__ filt, const float2* __restrict__ twid, double* __restrict__ elow) {
  constexpr int T = M / 16, PB = T < 64 ? 64 / T : 1;
  extern __shared__ float2 lds_all[];
  __shared__ double wsum[T < 64 ? 1 : T / 64];
  if (ws_mismatch(hdr, kPathResample, n, r, d, dtype)) return;
  const int t = threadIdx.x % T, pb = threadIdx.x / T;
  float2* lds = lds_all + pb * (M + M / 16);
  const int pair = min(blockIdx.x * PB + pb, pairs - 1);   // (a surplus half wave repeats the last pair)
  float2* g = grid + (size_t)pair * M;
  float2 x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = g[t + T * q];
  GridFft<M, false>::run(x, lds, twid, t);

#pragma unroll
  for (int q = 0; q < 16; ++q) lds[lds_pad(t + T * q)] = x[q];
  __syncthreads();
  const float2 ph = twid[twid_phase_off(M) + t];
  float e = 0.f;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int m = t + T * q;
    const float2 o = lds[lds_pad((M - m) & (M - 1))];
    const float2 f = filt[m];
    // e^{i pi q / 16} as a constant: cos and sin of q/32 turns
    constexpr float cq[16] = {1.f, 0.98078528040323044f, 0.92387953251128674f, 0.83146961230254524f,
                              0.70710678118654752f, 0.55557023301960222f, 0.38268343236508977f,
                              0.19509032201612827f, 0.f, -0.19509032201612827f, -0.38268343236508977f,
                              -0.55557023301960222f, -0.70710678118654752f, -0.83146961230254524f,
                              -0.92387953251128674f, -0.98078528040323044f};
    constexpr float sq[16] = {0.f, 0.19509032201612827f, 0.38268343236508977f, 0.55557023301960222f,
                              0.70710678118654752f, 0.83146961230254524f, 0.92387953251128674f,
                              0.98078528040323044f, 1.f, 0.98078528040323044f, 0.92387953251128674f,
                              0.83146961230254524f, 0.70710678118654752f, 0.55557023301960222f,
                              0.38268343236508977f, 0.19509032201612827f};
    const float2 w = cmul<false>(ph, make_float2(cq[q], sq[q]));
    const float2 z = cmul<false>(o, w);
    const float2 y = make_float2(fmaf(f.y, z.x, f.x * x[q].x), fmaf(f.y, z.y, f.x * x[q].y));
    e = fmaf(x[q].x, y.x, fmaf(x[q].y, y.y, e));
    x[q] = y;
  }
  __syncthreads();
  GridFft<M, true>::run(x, lds, twid, t);
#pragma unroll
  for (int q = 0; q < 16; ++q) g[t + T * q] = x[q];

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

// ---------------------------------------------------------------------------- residual and score

__device__ __forceinline__ void residual8(const RowPiece<uint16_t>& x, const f32x4 (&acc)[8], int i, float inv,
                                          float& hp, float& tot) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t w = x.v[c];
    const float lo = __uint_as_float(w << 16), hi = __uint_as_float(w & 0xFFFF0000u);
    const float dl = fmaf(-inv, acc[2 * c][i], lo), dh = fmaf(-inv, acc[2 * c + 1][i], hi);
    hp = fmaf(dl, dl, hp);
    hp = fmaf(dh, dh, hp);
    tot = fmaf(lo, lo, tot);
    tot = fmaf(hi, hi, tot);
  }
}
__device__ __forceinline__ void residual8(const RowPiece<float>& x, const f32x4 (&acc)[8], int i, float inv,
                                          float& hp, float& tot) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float v = c < 4 ? x.a[c & 3] : x.b[c & 3];
    const float dv = fmaf(-inv, acc[c][i], v);
    hp = fmaf(dv, dv, hp);
    tot = fmaf(v, v, tot);
  }
}

// One wave: one window of 32 grid points x 16 slots, applied to the 16-token tiles it covers.  The four
// waves of a workgroup share the window (their weights come from L1) and hold different slots or units.
template <typename T>
__global__ __launch_bounds__(256) void residual_kernel(const T* __restrict__ K, const T* __restrict__ V, KvStrides st,
                                                       int u0, int u1, int n, int r, int d, int dtype, int m, int tpw,
                                                       int wins, SlotMap sm, int wins_per_xcd, WsHeader* hdr,
                                                       const _Float16* __restrict__ winv, const int* __restrict__ k0s,
                                                       const float2* __restrict__ grid, float* __restrict__ scores,
                                                       double* __restrict__ epart, UnitMap um) {
  __shared__ float part_sum[4][16 * kMaxTilesPerWin];
  __shared__ double part_e[4][4];
  if (ws_mismatch(hdr, kPathResample, n, r, d, dtype)) return;
  const int xcd = blockIdx.x & 7, slot_id = blockIdx.x >> 3;
  const int win = xcd * wins_per_xcd + slot_id % wins_per_xcd;
  if (win >= wins) return;
  const int lane = threadIdx.x & 63, g = lane >> 4, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gw0 = (slot_id / wins_per_xcd) * 4, gw = gw0 + wave;
  const int unit = u0 + gw / sm.wpu, part = gw % sm.wpu;
  const int tiles = min(tpw, (n + 15) / 16 - win * tpw);
  if (unit < u1) {
    // grid values of the window: lane holds 8 points of the columns of slot 4 (row & 3) + (row >> 2)
    const int row = lane & 15;
    const int s_mine = part * 16 + 4 * (row & 3) + (row >> 2);
    const int slot = s_mine < 2 * sm.nb ? s_mine : 0;
    const int n0 = k0s[win] >> 1;
    const int pos = g < 2 ? n0 + 8 * g : m - 8 - n0 - 8 * (g - 2);
    const float2* gp = grid + ((size_t)(unit - u0) * 2 * sm.nb + slot) * 4 * m + pos;
    Frag bh[8], bl[8];
    float inv;
    {
      f32x4 v[4][4];
#pragma unroll
      for (int jp = 0; jp < 4; ++jp)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[jp][c] = *reinterpret_cast<const f32x4*>(gp + (size_t)jp * m + 2 * c);
      float mx = 0.f;
#pragma unroll
      for (int jp = 0; jp < 4; ++jp)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(v[jp][c][q]));
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) mx = fmaxf(mx, __shfl_xor(mx, s, 64));
      // largest magnitude of the window into [2^14, 2^15); powers of two, so nothing is rounded
      const int eb = max(14, min((int)(__float_as_uint(mx) >> 23), 254));
      const float scale = __uint_as_float((uint32_t)(268 - eb) << 23);
      inv = ldexpf(1.0f / kInvWeightScale, eb - 141);
#pragma unroll
      for (int jp = 0; jp < 4; ++jp)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float b = v[jp][c][q] * scale;
            const _Float16 h = (_Float16)b;
            bh[2 * jp + (q & 1)].hs[2 * c + (q >> 1)] = h;
            bl[2 * jp + (q & 1)].hs[2 * c + (q >> 1)] = (_Float16)(b - (float)h);
          }
    }
    // rows: register i of a lane belongs to slot 4 i + g of token lane & 15
    const int tok0 = win * tpw * 16 + (lane & 15);
    const int64_t ubase = unit_offset(st, unit);
    const T* px[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int so = part * 16 + 4 * i + g;
      const int sl = so < 2 * sm.nb ? so : 0;
      const bool second = sl >= sm.nb;
      px[i] = (second ? V : K) + ubase + (sl - (second ? sm.nb : 0)) * 8;
    }
    const u32x4* wp = reinterpret_cast<const u32x4*>(winv) + (size_t)win * tpw * 128 + lane;
    float hp[4] = {0.f, 0.f, 0.f, 0.f}, tot[4] = {0.f, 0.f, 0.f, 0.f};
    RowPiece<T> x[4];
    Frag wh, wl;
    {
      const int64_t off = (int64_t)min(tok0, n - 1) * st.sn;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i].load(px[i] + off);
      wh.u = wp[0];
      wl.u = wp[64];
    }
    for (int tl = 0; tl < tiles; ++tl) {
      const int nx = min(tl + 1, tiles - 1);
      const int64_t off = (int64_t)min(tok0 + 16 * nx, n - 1) * st.sn;
      RowPiece<T> xn[4];
      Frag whn, wln;
#pragma unroll
      for (int i = 0; i < 4; ++i) xn[i].load(px[i] + off);
      whn.u = wp[nx * 128];
      wln.u = wp[nx * 128 + 64];
      f32x4 acc[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        acc[j] = mfma_f16(bl[j], wh, f32x4{0.f, 0.f, 0.f, 0.f});
        acc[j] = mfma_f16(bh[j], wl, acc[j]);
        acc[j] = mfma_f16(bh[j], wh, acc[j]);
      }
      const bool in = tok0 + 16 * tl < n;
      float row_sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float h = 0.f, t2 = 0.f;
        residual8(x[i], acc, i, inv, h, t2);
        const bool use = in && part * 16 + 4 * i + g < 2 * sm.nb;
        h = use ? h : 0.f;
        t2 = use ? t2 : 0.f;
        hp[i] += h;
        tot[i] += t2;
        row_sum += h;
      }
      row_sum += __shfl_xor(row_sum, 16, 64);
      row_sum += __shfl_xor(row_sum, 32, 64);
      if (lane < 16) part_sum[wave][16 * tl + lane] = row_sum;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = xn[i];
      wh = whn;
      wl = wln;
    }
    double ev[4] = {0.0, 0.0, 0.0, 0.0};                // Ehp_k, Ehp_v, Etot_k, Etot_v
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool second = part * 16 + 4 * i + g >= sm.nb;
      ev[second ? 1 : 0] += (double)hp[i];
      ev[second ? 3 : 2] += (double)tot[i];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) ev[k] += __shfl_xor(ev[k], s, 64);
      if (lane == 0) part_e[wave][k] = ev[k];
    }
  }
  __syncthreads();
  const int upw = 4 / sm.wpu;                            // units of this workgroup
  const int span = 16 * tiles, tokens = min(span, n - win * tpw * 16);
  for (int k = threadIdx.x; k < upw * span; k += 256) {
    const int ul = k / span, tk = k % span, u = u0 + gw0 / sm.wpu + ul;
    if (u < u1 && tk < tokens) {
      float s = part_sum[ul * sm.wpu][tk];
      for (int p = 1; p < sm.wpu; ++p) s += part_sum[ul * sm.wpu + p][tk];
      scores[(size_t)out_unit(um, u) * n + win * tpw * 16 + tk] = s / (float)d;
    }
  }
  if (threadIdx.x < 4 * upw) {
    const int ul = threadIdx.x >> 2, k = threadIdx.x & 3, u = u0 + gw0 / sm.wpu + ul;
    if (u < u1) {
      double s = 0.0;
      for (int p = 0; p < sm.wpu; ++p) s += part_e[ul * sm.wpu + p][k];
      epart[((size_t)u * wins + win) * 4 + k] = s;
    }
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

template <int M>
hipError_t launch_filter(float2* grid, int pairs, int n, int r, int d, int dtype, WsHeader* hdr, const float2* filt,
                         const float2* twid, double* elow, hipStream_t s) {
  constexpr int T = M / 16, PB = T < 64 ? 64 / T : 1;
  const size_t lds = (size_t)PB * (M + M / 16) * sizeof(float2);
  auto kern = grid_filter_kernel<M>;
  if (lds > 64 * 1024) {
    // raising the dynamic LDS limit is per kernel and per device, and idempotent
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  ProfileScope ps("grid_filter_kernel", s);
  hipLaunchKernelGGL(kern, dim3((pairs + PB - 1) / PB), dim3(T < 64 ? 64 : T), lds, s, grid, pairs, n, r, d, dtype,
                     hdr, filt, twid, elow);
  return hipGetLastError();
}

}  // namespace

// Bytes of input rows and grid one round of the three kernels works on (see resample_layout).
static size_t resample_chunk_bytes() {
  return (size_t)1 << 30;
}

// Grid length for this shape and cut-off, 0 if the realisation does not apply.
static int grid_length(const fc_kv_desc& d, int32_t r) {
  if (d.head_dim % 8 != 0 || d.head_dim > 256 || r < 1 || 2 * (int64_t)r > d.n_tokens) return 0;
  for (int m = 512; m <= 16384; m *= 2)
    if (4 * (int64_t)m >= 7 * (int64_t)r)                       // M >= 1.75 r: see the accuracy note above
      return 5 * (int64_t)d.n_tokens >= 4 * (int64_t)m ? m : 0;  // a 16-token tile and its windows fit 32 points
  return 0;
}

bool resample_supported(const fc_kv_desc& d, int32_t r) { return grid_length(d, r) != 0; }

ResampleLayout resample_layout(const fc_kv_desc& d, int32_t r) {
  ResampleLayout lay{};
  const int64_t n = d.n_tokens, m = grid_length(d, r);
  const size_t units = (size_t)d.batch * d.layers * d.kv_heads;
  lay.m = (int)m;
  // tokens under a tile of 16 grid points: at most (15 + W) N/M + 1
  lay.steps = (int)(((15 + kW) * n / m + 2 + 31) / 32);
  // tiles whose windows fit 32 grid points when the first point is rounded down to a multiple of 4
  lay.tpw = (int)std::min<int64_t>(kMaxTilesPerWin, ((28 - kW) * n / m + 1) / 16);
  if (lay.tpw < 1) lay.tpw = 1;
  const int tok_tiles = (int)((n + 15) / 16);
  lay.wins = (tok_tiles + lay.tpw - 1) / lay.tpw;
  lay.nb = d.head_dim / 8;
  const int waves = (2 * lay.nb + 15) / 16;
  lay.wpu = waves <= 2 ? waves : 4;
  // units per round of the three kernels (bounds the memory the grid takes; measured, smaller rounds
  // gain less from the last-level cache than their launches cost)
  const size_t eb = d.dtype == FC_BF16 ? 2 : 4;
  const size_t unit_bytes = 2 * (size_t)n * d.head_dim * eb + 2 * (size_t)m * d.head_dim * 4;
  lay.chunk = (int)std::max<size_t>(1, std::min(std::max<size_t>(units, 1), resample_chunk_bytes() / unit_bytes));
  auto up = [](size_t x) { return (x + kWsAlign - 1) / kWsAlign * kWsAlign; };
  size_t off = sizeof(WsHeader);
  lay.wfwd = off; off = up(off + (size_t)(m / 16) * lay.steps * 3 * 512 * 2);
  lay.winv = off; off = up(off + (size_t)lay.wins * lay.tpw * 1024 * 2);
  lay.t0 = off; off = up(off + (size_t)(m / 16) * 4);
  lay.k0 = off; off = up(off + (size_t)lay.wins * 4);
  lay.filt = off; off = up(off + (size_t)m * sizeof(float2));
  lay.twid = off; off = up(off + (size_t)twid_size((int)m) * sizeof(float2));
  lay.elow = off; off = up(off + units * 2 * lay.nb * 4 * sizeof(double));
  lay.epart = off; off = up(off + units * lay.wins * 4 * sizeof(double));
  lay.grid = off; off = up(off + (size_t)lay.chunk * 2 * lay.nb * 4 * m * sizeof(float2));
  lay.total = off;
  return lay;
}

hipError_t resample_prepare(const fc_kv_desc& d, int32_t r, const ResampleLayout& lay, void* ws, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  TablePtrs tp{reinterpret_cast<WsHeader*>(base), reinterpret_cast<uint16_t*>(base + lay.wfwd),
               reinterpret_cast<_Float16*>(base + lay.winv), reinterpret_cast<int*>(base + lay.t0),
               reinterpret_cast<int*>(base + lay.k0), reinterpret_cast<float2*>(base + lay.filt),
               reinterpret_cast<float2*>(base + lay.twid)};
  const int n_wfwd = lay.m / 16 * lay.steps * 64, n_winv = lay.wins * lay.tpw * 64;
  const int total = n_wfwd + n_winv + lay.m + twid_size(lay.m);
  ProfileScope ps("resample_table_kernel", s);
  hipLaunchKernelGGL(resample_table_kernel, dim3((total + 255) / 256), dim3(256), 0, s, tp, d.n_tokens, r, lay.m,
                     d.head_dim, d.dtype, lay.steps, lay.tpw, n_wfwd, n_winv);
  return hipGetLastError();
}

template <typename T>
static hipError_t resample_score_t(const T* K, const T* V, const fc_kv_desc& d, int32_t r, const ResampleLayout& lay,
                                   float* scores, double* energy, void* ws, UnitMap um, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  WsHeader* hdr = reinterpret_cast<WsHeader*>(base);
  const int units = d.batch * d.layers * d.kv_heads, n = d.n_tokens, m = lay.m;
  float2* grid = reinterpret_cast<float2*>(base + lay.grid);
  const float2* filt = reinterpret_cast<const float2*>(base + lay.filt);
  const float2* twid = reinterpret_cast<const float2*>(base + lay.twid);
  double* epart = reinterpret_cast<double*>(base + lay.epart);
  const SlotMap sm{lay.nb, lay.wpu};
  const KvStrides st = strides_of(d);
  // each XCD takes a contiguous range of tiles (or windows), so that its L2 holds that range's weights
  // and the rows neighbouring tiles share
  const int tpx = (m / 16 + 7) / 8, wpx = (lay.wins + 7) / 8;
  for (int u0 = 0; u0 < units; u0 += lay.chunk) {
    const int u1 = std::min(units, u0 + lay.chunk);
    const int groups = ((u1 - u0) * lay.wpu + 3) / 4;
    {
      ProfileScope ps("decimate_kernel", s);
      hipLaunchKernelGGL(decimate_kernel<T>, dim3(8 * tpx * groups), dim3(256), 0, s, K, V, st, u0, u1, n, r,
                         d.head_dim, d.dtype, m, lay.steps, sm, tpx, hdr,
                         reinterpret_cast<const uint16_t*>(base + lay.wfwd),
                         reinterpret_cast<const int*>(base + lay.t0), grid);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    double* elow = reinterpret_cast<double*>(base + lay.elow) + (size_t)u0 * 2 * lay.nb * 4;
    const int pairs = (u1 - u0) * 2 * lay.nb * 4;
#define FC_FILTER(MV) case MV: e = launch_filter<MV>(grid, pairs, n, r, d.head_dim, d.dtype, hdr, filt, twid, elow, s); break;
    switch (m) {
      FC_FILTER(512) FC_FILTER(1024) FC_FILTER(2048) FC_FILTER(4096) FC_FILTER(8192) FC_FILTER(16384)
      default: e = hipErrorInvalidValue;
    }
#undef FC_FILTER
    if (e != hipSuccess) return e;
    {
      ProfileScope ps("residual_kernel", s);
      hipLaunchKernelGGL(residual_kernel<T>, dim3(8 * wpx * groups), dim3(256), 0, s, K, V, st, u0, u1, n, r,
                         d.head_dim, d.dtype, m, lay.tpw, lay.wins, sm, wpx, hdr,
                         reinterpret_cast<const _Float16*>(base + lay.winv),
                         reinterpret_cast<const int*>(base + lay.k0), grid, scores, epart, um);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return energy_reduce_launch(epart, lay.wins, units, energy, um, s);
}

hipError_t resample_score(const void* K, const void* V, const fc_kv_desc& d, int32_t r, const ResampleLayout& lay,
                          float* scores, double* energy, void* ws, UnitMap um, hipStream_t s) {
  return d.dtype == FC_BF16
             ? resample_score_t(static_cast<const uint16_t*>(K), static_cast<const uint16_t*>(V), d, r, lay, scores,
                                energy, ws, um, s)
             : resample_score_t(static_cast<const float*>(K), static_cast<const float*>(V), d, r, lay, scores, energy,
                                ws, um, s);
}

hipError_t resample_lowpass(const fc_kv_desc& d, const ResampleLayout& lay, void* ws, double* lowpass, hipStream_t s) {
  const int n_ut = d.batch * d.layers * d.kv_heads * 2;
  ProfileScope ps("resample_lowpass_kernel", s);
  hipLaunchKernelGGL(resample_lowpass_kernel, dim3((n_ut + 255) / 256), dim3(256), 0, s,
                     reinterpret_cast<const double*>(static_cast<char*>(ws) + lay.elow), lay.nb * 4, n_ut, lowpass);
  return hipGetLastError();
}

}  // namespace fc
