// Device helpers shared by the edge kernels: compile-time path lists, edge
// geometry (directions, real harmonics), MFMA operand helpers
// and the radial tables with the MFMA operands read from them.
#pragma once
#include <utility>

#include "kernels.h"

namespace mpip {

template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
// f(integral_constant<int, 0>), ..., f(integral_constant<int, N-1>), fully unrolled
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// ------------------------------------------------------------ path lists

struct P3 { int l1, l2, l3; };

constexpr bool natural3(int a, int b, int c) {
  return ((a + b + c) % 2 == 0) && c >= (a > b ? a - b : b - a) && c <= a + b;
}

template <int L, int KIND>
struct PathList {
  static constexpr int l1max() { return (KIND == KIND_ONLY || KIND == KIND_FIRST) ? 0 : L; }
  static constexpr bool keep(int a, int b, int c) {
    if (!natural3(a, b, c)) return false;
    if (KIND == KIND_ONLY || KIND == KIND_LAST) return c == 0;
    return true;
  }
  static constexpr int count() {
    int n = 0;
    for (int a = 0; a <= l1max(); ++a)
      for (int b = 0; b <= L; ++b)
        for (int c = 0; c <= L; ++c)
          if (keep(a, b, c)) ++n;
    return n;
  }
  static constexpr P3 get(int i) {
    int n = 0;
    for (int a = 0; a <= l1max(); ++a)
      for (int b = 0; b <= L; ++b)
        for (int c = 0; c <= L; ++c)
          if (keep(a, b, c)) {
            if (n == i) return P3{a, b, c};
            ++n;
          }
    return P3{0, 0, 0};
  }
  static constexpr int nin() { return (KIND == KIND_ONLY || KIND == KIND_FIRST) ? 1 : (L + 1) * (L + 1); }
  static constexpr int nout() { return (KIND == KIND_ONLY || KIND == KIND_LAST) ? 1 : (L + 1) * (L + 1); }
};

// ------------------------------------------------------------ geometry

struct Geo {
  float u[3];
  float d, inv;      // length and its inverse
  float Y[kMaxNlm];
};

// Direction, length and harmonics of an edge.  Tail lanes of a tile (valid ==
// false) evaluate a unit vector along x and get zeros, so the code has no
// divergent branch.
__device__ __forceinline__ void edge_direction(float4 v, bool valid, Geo& g) {
  const float vx = valid ? v.x : 1.f, vy = valid ? v.y : 0.f, vz = valid ? v.z : 0.f;
  const float d2 = vx * vx + vy * vy + vz * vz;
  const float inv = __builtin_amdgcn_rsqf(d2);
  const float d = d2 * inv;
  const float x = vx * inv, y = vy * inv, z = vz * inv;
  const float msk = valid ? 1.f : 0.f;
  g.u[0] = msk * x; g.u[1] = msk * y; g.u[2] = msk * z; g.d = d; g.inv = inv;
  const float s3 = 1.7320508075688772f, s5 = 2.23606797749979f, s15 = 3.872983346207417f;
  g.Y[0] = msk;
  g.Y[1] = msk * s3 * y; g.Y[2] = msk * s3 * z; g.Y[3] = msk * s3 * x;
  g.Y[4] = msk * s15 * x * y; g.Y[5] = msk * s15 * y * z; g.Y[6] = msk * 0.5f * s5 * (3.f * z * z - 1.f);
  g.Y[7] = msk * s15 * x * z; g.Y[8] = msk * 0.5f * s15 * (x * x - y * y);
}

// Tabulated radial MLP (BF16 form).  The second hidden layer a(d) in R^64
// of one layer's radial MLP is a function of the edge length alone; the
// table holds, for the kRadTab intervals [d_k, d_k+1) of [0, r_c]
// (d_k = k r_c / kRadTab), a(d_k) and the increment a(d_k+1) - a(d_k) as a
// BF16 pair per hidden unit (value in the low half), [kRadTab][64] words.
// Between the knots a is interpolated linearly:
//   a(d) = a(d_k) + tau (a(d_k+1) - a(d_k)),  tau = d kRadTab / r_c - k,
// and its derivative is the interval's slope, (a(d_k+1) - a(d_k)) kRadTab / r_c.
// Lengths at or past r_c take the last interval at tau = 1 (a = 0 there).
struct RadPos {
  int k;
  float tau;
};
__device__ __forceinline__ RadPos rad_pos(float d, float scale) {
  const float t = fminf(d * scale, (float)kRadTab);
  const int k = min((int)t, kRadTab - 1);
  return {k, fminf(t - (float)k, 1.f)};
}
// The table words of a lane's D tiles in the features x edges layout (lane
// (g, el): hidden 16 mt + 4 g + r of the lane's edge, of 16 NH in a row), with
// tau.  The directions' tables (NH = 2, and Radial<3>) hold the value at the
// middle of the interval: its BF16 rounding and the operand's then leave no
// bias, where a value at the left end lags by up to half an interval wherever
// the increment is below half a unit in the last place (4.0e-4 of R on average
// over a shell of neighbours, against 1.7e-4).
template <int NH>
struct RadRowN {
  uint4 w[NH];
  float tau;
};
typedef RadRowN<4> RadRow;
template <int NH>
__device__ __forceinline__ RadRowN<NH> rad_load(const uint32_t* tab, RadPos rp, int g) {
  const uint4* row = (const uint4*)(tab + (size_t)rp.k * (16 * NH)) + g;
  RadRowN<NH> rr;
#pragma unroll
  for (int mt = 0; mt < NH; ++mt) rr.w[mt] = row[4 * mt];
  rr.tau = NH == 2 ? rp.tau - 0.5f : rp.tau;
  return rr;
}
// a(d) in that layout and, when sl is given, the increments
template <int NH>
__device__ __forceinline__ void rad_eval(const RadRowN<NH>& rr, f32x4* a2, f32x4* sl) {
#pragma unroll
  for (int mt = 0; mt < NH; ++mt) {
    const unsigned w[4] = {rr.w[mt].x, rr.w[mt].y, rr.w[mt].z, rr.w[mt].w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = __uint_as_float(w[r] << 16), inc = __uint_as_float(w[r] & 0xffff0000u);
      a2[mt][r] = fmaf(rr.tau, inc, v);
      if (sl) sl[mt][r] = inc;
    }
  }
}
// |v| as edge_direction forms it (tail lanes carry a unit vector)
__device__ __forceinline__ float edge_length(float4 v) {
  const float d2 = v.x * v.x + v.y * v.y + v.z * v.z;
  return d2 * __builtin_amdgcn_rsqf(d2);
}
// dE/dd of the lane's edge from dE/da (ab2, same layout) and the increments:
// sum over the hidden units, the four lane groups of an edge combined
template <int NH>
__device__ __forceinline__ float rad_dbar(const f32x4* ab2, const f32x4* sl, float scale) {
  float s = 0.f;
#pragma unroll
  for (int mt = 0; mt < NH; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) s = fmaf(ab2[mt][r], sl[mt][r], s);
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  return s * scale;
}

// FP32 form: the same function as a cubic in tau per interval, [rn][64]
// coefficients (value, first, second, third order) and a zero row, and its derivative.
struct RadTab32 {
  const float4* c;
  int n;               // intervals
  float scale, scale_lo; // n / r_c: rounded to FP32, and what the rounding left
};
template <int N>   // functions of a lane: 16 hidden units, or 12 directions
struct Rad32N {
  float4 c[N];
  float tau;
  // interval k and tau of the length of v; d, inv: the length and its inverse
  // in FP32 (what d leaves of the length is far below the table's spacing,
  // but not below its accuracy, so it goes into tau)
  static __device__ __forceinline__ RadPos pos(const RadTab32& t, float4 v, float d, float inv) {
    const double q = fma((double)v.z, (double)v.z, fma((double)v.y, (double)v.y, (double)v.x * (double)v.x));
    const float rest = 0.5f * inv * (float)fma(-(double)d, (double)d, q);
    const int k = min((int)(d * t.scale), t.n - 1);
    return {k, fminf(fmaf(d, t.scale, -(float)k) + fmaf(d, t.scale_lo, rest * t.scale), 1.f)};
  }
  // the lane's four D tiles in the features x edges layout (hidden 16 mt + 4 g + r)
  // (unless valid: the zero row past the last interval)
  __device__ __forceinline__ void load(const RadTab32& t, float4 v, float d, float inv, int g, bool valid) {
    const RadPos rp = pos(t, v, d, inv);
    tau = rp.tau;
    const float4* row = t.c + (size_t)(valid ? rp.k : t.n) * (4 * N) + 4 * g;
#pragma unroll
    for (int q4 = 0; q4 < N; ++q4) c[q4] = row[16 * (q4 / 4) + q4 % 4];
  }
  static __device__ __forceinline__ float value(float4 c, float tau) { return fmaf(tau, fmaf(tau, fmaf(tau, c.w, c.z), c.y), c.x); }
  // a(d) and, when da is given, da/dd / scale
  __device__ __forceinline__ void eval(f32x4* a2, f32x4* da) const {
    const float t2 = 2.f * tau, t3 = 3.f * tau * tau;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      a2[q / 4][q % 4] = value(c[q], tau);
      if (da) da[q / 4][q % 4] = fmaf(t3, c[q].w, fmaf(t2, c[q].z, c[q].y));
    }
  }
};

typedef Rad32N<16> Rad32;

// gu = (dP/du)^T Ybar for the polynomials above
__device__ __forceinline__ void sh_grad_contract(const float* Yb, const float* u, float* gu) {
  const float s3 = 1.7320508075688772f, s5 = 2.23606797749979f, s15 = 3.872983346207417f;
  const float x = u[0], y = u[1], z = u[2];
  gu[0] = s3 * Yb[3] + s15 * (y * Yb[4] + z * Yb[7] + x * Yb[8]);
  gu[1] = s3 * Yb[1] + s15 * (x * Yb[4] + z * Yb[5] - y * Yb[8]);
  gu[2] = s3 * Yb[2] + s15 * (y * Yb[5] + x * Yb[7]) + 3.f * s5 * z * Yb[6];
}

// ------------------------------------------------------------ MFMA helpers

template <int PREC> struct Op;

template <> struct Op<1> {  // BF16 operands, K = 32 per instruction
  typedef bf16x8 T;
  __device__ static f32x4 mma(T a, T b, f32x4 c) { return mfma_bf16(a, b, c); }
  // operand of k-chunk kc from four D tiles (hidden 16*t + 4*g + r)
  __device__ static T from_tiles(const f32x4* t, int kc) {
    T v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)t[2 * kc + j / 4][j % 4];
    return v;
  }
};

template <> struct Op<0> {  // FP32 operands, K = 4 per instruction
  typedef float T;
  __device__ static f32x4 mma(T a, T b, f32x4 c) { return mfma_f32(a, b, c); }
  __device__ static T from_tiles(const f32x4* t, int q) { return t[q / 4][q % 4]; }
};

// MFMA operand of one hidden chunk (32 of the 64 units): BF16, or FP32 as
// three BF16 parts
template <int PREC>
struct Parts {
  static constexpr int N = PREC == 1 ? 1 : 3;
  bf16x8 p[N];
  // hidden units of chunk kc from four D tiles
  static __device__ __forceinline__ Parts from(const f32x4* t, int kc) {
    Parts o;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float x = t[2 * kc + j / 4][j % 4];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const __bf16 h = (__bf16)x;
        o.p[k][j] = h;
        x -= (float)h;
      }
    }
    return o;
  }
};

// R = W3^T a(d) of an edge tile on the MFMA, by form F = (BF16 ? 1 : 0) + (compressed ? 2 : 0).
// All 64 hidden units: two k-chunks (BF16), or six products of BF16 parts of
// each (FP32).  Compressed (LayerDev::comp): a(d) = V b(d) with b in order of
// falling size, R = (V^T W3)^T b.
//   BF16: one chunk.  Lane group g holds directions 4 q + g, q < 6, the weights of
//   the first two (the largest eight) in two parts: weights round the same way
//   for every edge, and their error adds up in the energy and the virial.
// Half of the MFMA, table and LDS traffic of all units (BF16), 5/12 of the MFMA
// (FP32).  13,824 atoms, K = 6, a layer: BF16 forward 257 -> 225 us, adjoint
// 430 -> 386; FP32 499 -> 414 and 822 -> 623 us.
//   FP32: five chunks.  Lane group g holds directions 4 g .. 4 g + 3 of each of
//   the groups A, B, C (0.., 16.., 32..).  A takes all six products that reach
//   2^-24 of it, B (at most 2^-5 of a(d): radial_basis) three, C (2^-13) one:
//     W1A (A1, A2)   W2A (A1, A2)   W1A A3, W3A A1   W1B (B1, B2)   W2B B1, W1C C1.
template <int F>
struct HidForm {
  static constexpr bool BF = F & 1, COMP = F & 2;
  static constexpr int NT = COMP ? (BF ? 1 : 5) : (BF ? 2 : 6);   // weight tiles
  static constexpr int NB = COMP ? (BF ? 1 : 4) : NT;             // operands of the edge
};
template <int F>
struct Hid {
  typedef HidForm<F> H;
  bf16x8 p[H::NB];
  // W^T of one output tile, smallest products first
  __device__ __forceinline__ f32x4 mma(const bf16x8 (&w)[H::NT]) const {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (F == 3) {
      acc = mfma_bf16(w[0], p[0], acc);
    } else if constexpr (F == 2) {
      acc = mfma_bf16(w[4], p[3], acc);
      acc = mfma_bf16(w[2], p[1], acc);
      acc = mfma_bf16(w[1], p[0], acc);
      acc = mfma_bf16(w[3], p[2], acc);
      acc = mfma_bf16(w[0], p[0], acc);
    } else {
      constexpr int P = H::NT / 2;   // [chunk][part]
#pragma unroll
      for (int o = P - 1; o >= 0; --o)
#pragma unroll
        for (int i = 0; i <= o; ++i)
#pragma unroll
          for (int kc = 0; kc < 2; ++kc) acc = mfma_bf16(w[kc * P + i], p[kc * P + o - i], acc);
    }
    return acc;
  }
};

struct RadSrc {
  const uint32_t* rtab;   // BF16 form
  RadTab32 t32;           // FP32 form; its scale in both
};
// The table words of a lane's edge, and the operands of a and (NR = 2) da/dd
// (without the table's scale) from them
template <int F>
struct Radial;
template <>
struct Radial<1> {
  RadRow rr;
  // tail lanes read the zero row past the table's last interval
  __device__ __forceinline__ void load(const RadSrc& t, float4, float d, float, int g, bool valid) {
    RadPos rp = rad_pos(d, t.t32.scale);
    rp.k = valid ? rp.k : kRadTab;
    rr = rad_load<4>(t.rtab, rp, g);
  }
  template <int NR>
  __device__ __forceinline__ void operands(Hid<1> (&b)[NR]) const {
    f32x4 a2[4];
    rad_eval<4>(rr, a2, nullptr);
#pragma unroll
    for (int k = 0; k < 2; ++k) b[0].p[k] = Parts<1>::from(a2, k).p[0];
    if constexpr (NR == 2) {   // the BF16 increments in the table's high halves
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint4 p = rr.w[2 * k], q = rr.w[2 * k + 1];
        const uint4 u = {__builtin_amdgcn_perm(p.y, p.x, 0x07060302u), __builtin_amdgcn_perm(p.w, p.z, 0x07060302u),
                         __builtin_amdgcn_perm(q.y, q.x, 0x07060302u), __builtin_amdgcn_perm(q.w, q.z, 0x07060302u)};
        b[1].p[k] = __builtin_bit_cast(bf16x8, u);
      }
    }
  }
};
template <>
struct Radial<3> {
  uint4 w;      // six (value, increment) pairs
  uint2 w2;
  float tau;
  __device__ __forceinline__ void load(const RadSrc& t, float4, float d, float, int g, bool valid) {
    const RadPos rp = rad_pos(d, t.t32.scale);
    const uint32_t* row = t.rtab + (size_t)(valid ? rp.k : kRadTab) * 32 + 8 * g;
    w = *(const uint4*)row;
    w2 = *(const uint2*)(row + 4);
    tau = rp.tau - 0.5f;
  }
  template <int NR>
  __device__ __forceinline__ void operands(Hid<3> (&b)[NR]) const {
    const unsigned u[6] = {w.x, w.y, w.z, w.w, w2.x, w2.y};
    bf16x8& o = b[0].p[0];
#pragma unroll
    for (int q = 0; q < 6; ++q)
      o[q < 2 ? q : q + 2] = (__bf16)fmaf(tau, __uint_as_float(u[q] & 0xffff0000u), __uint_as_float(u[q] << 16));
    o[2] = o[0];
    o[3] = o[1];
    if constexpr (NR == 2) {   // the increments, in the high halves
      const unsigned top = __builtin_amdgcn_perm(u[1], u[0], 0x07060302u);
      const uint4 v = {top, top, __builtin_amdgcn_perm(u[3], u[2], 0x07060302u), __builtin_amdgcn_perm(u[5], u[4], 0x07060302u)};
      b[1].p[0] = __builtin_bit_cast(bf16x8, v);
    }
  }
};
template <>
struct Radial<0> {
  Rad32 r;
  __device__ __forceinline__ void load(const RadSrc& t, float4 v, float d, float inv, int g, bool valid) {
    r.load(t.t32, v, d, inv, g, valid);
  }
  template <int NR>
  __device__ __forceinline__ void operands(Hid<0> (&b)[NR]) const {
    f32x4 a2[4], da[4];
    r.eval(a2, NR == 2 ? da : nullptr);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const Parts<0> t = Parts<0>::from(i ? da : a2, k);
#pragma unroll
        for (int q = 0; q < 3; ++q) b[i].p[3 * k + q] = t.p[q];
      }
  }
};
template <>
struct Radial<2> {
  Rad32N<12> r;
  __device__ __forceinline__ void load(const RadSrc& t, float4 v, float d, float inv, int g, bool valid) {
    r.load(t.t32, v, d, inv, g, valid);
  }
  template <int NR>
  __device__ __forceinline__ void operands(Hid<2> (&b)[NR]) const {
    f32x4 x[NR == 2 ? 6 : 3];
    r.eval(x, NR == 2 ? x + 3 : nullptr);
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float v = x[3 * i][j];
        const __bf16 a1 = (__bf16)v;
        v -= (float)a1;
        const __bf16 a2 = (__bf16)v;
        v -= (float)a2;
        const __bf16 b1 = (__bf16)x[3 * i + 1][j];
        b[i].p[0][j] = a1;
        b[i].p[0][4 + j] = a2;
        b[i].p[1][j] = (__bf16)v;
        b[i].p[1][4 + j] = a1;
        b[i].p[2][j] = b1;
        b[i].p[2][4 + j] = (__bf16)(x[3 * i + 1][j] - (float)b1);
        b[i].p[3][j] = b1;
        b[i].p[3][4 + j] = (__bf16)x[3 * i + 2][j];
      }
  }
};

__device__ __forceinline__ int64_t edges_total(const LayerArgs& a) { return (int64_t)a.row_ptr[a.n]; }

// Rows of the calling wave.  Workgroups are dispatched to the 8 XCDs in
// round-robin order, so workgroup b runs on XCD b % 8: each XCD takes a
// contiguous eighth of the spatially sorted rows and its waves walk that
// range side by side, so the sender rows they gather stay within one L2.
// The grid is a multiple of 8 workgroups.
struct RowWalk {
  int64_t i, end, step;
};
template <int NW>
__device__ __forceinline__ RowWalk row_walk(int64_t n) {
  const int b = blockIdx.x, x = b & 7, lb = b >> 3, BX = gridDim.x >> 3;
  const int64_t r0 = n * x / 8, r1 = n * (x + 1) / 8;
  return {r0 + (int64_t)lb * NW + (threadIdx.x >> 6), r1, (int64_t)BX * NW};
}

// Edge ranges of a wave's current row and of its next row along a RowWalk
// (the next row's bounds are read a row ahead), so that a tile loop can
// request the first tile of the next row while it works on its last one.
// row_end: the walked prefix of each row (receptive-field trimming), or null.
struct RowAhead {
  int64_t i, end, step;
  int e0, e1, n0, n1;
  __device__ __forceinline__ RowAhead(const RowWalk& rw, const int32_t* row_ptr, const int32_t* row_end)
      : i(rw.i), end(rw.end), step(rw.step), e0(0), e1(0), n0(0), n1(0) {
    if (i < end) { e0 = row_ptr[i]; e1 = row_end ? row_end[i] : row_ptr[i + 1]; }
    if (i + step < end) { n0 = row_ptr[i + step]; n1 = row_end ? row_end[i + step] : row_ptr[i + step + 1]; }
  }
  __device__ __forceinline__ bool has_row() const { return i < end; }
  __device__ __forceinline__ bool has_next() const { return i + step < end; }
  __device__ __forceinline__ void advance(const int32_t* row_ptr, const int32_t* row_end) {
    i += step;
    e0 = n0;
    e1 = n1;
    if (i + step < end) { n0 = row_ptr[i + step]; n1 = row_end ? row_end[i + step] : row_ptr[i + step + 1]; }
  }
};


}  // namespace mpip
