// Node kernels between two layers (any form, depth and path set): channel
// mixing, gates, residual and the next layer's features in one pass over an
// atom's rows, and their adjoint; and the last layer's node update with the
// readout and its adjoint.
//
//   forward, layer t < K:  z = A W_down (layer 1 species-factorised: Q (V W_down)),
//     h_0 += silu(z_0), h_l += sigmoid(gate_l) z_l, h~(t+1) = h W_up(t+1);
//   adjoint: hbar += h~bar(t+1) W_up(t+1)^T, the gates' adjoint, and
//     dE/dA = zbar W_down^T (P = zbar (V W_down)^T);
//   last layer: z_0, E_i = e0 + (h_0 + silu(z_0)) w_read, dE/dA.
//
// A wave takes 16 atoms.  Products are features x atoms: the weights are the
// MFMA A operand, an atom's row the B operand, so lane (g, n) holds features
// 16 t + 4 g + r of atom n; gates and residuals are lane-local and a
// product's tiles are the next one's operand (weights packed in that order),
// with nothing exchanged between lanes or waves.  FP32 form: operands split
// into three BF16 parts, six products on the BF16 MFMA (edge_common.h).
// The weights of a phase (a degree's W_up, its W_down) sit in LDS, shared by
// the eight waves of a persistent workgroup.  Read from L2 instead, with one
// wave per SIMD, each tile's loads waited for the stores before them (one
// in-order counter), and the passes were bound by that latency.  Now: by the
// latency of the rows with few waves to cover it (13,824 atoms are 864 tiles:
// 1.1 to 1.4 waves per SIMD, VALU 7 to 16 % and MFMA 2 to 11 % active), and by
// the passes over Q, h, z and h~.
//   103,635 atoms, FP32, 128 channels, l_max 2: forward 2.16 -> 0.88 ms,
//   adjoint 2.06 -> 0.92 ms; 13,824 atoms, 64 channels: BF16 56 -> 41 and
//   61 -> 48 us a layer, FP32 93 -> 50 and 93 -> 55; 4,096 atoms, FP32: 99 -> 44
//   and 88 -> 37 us.
// The separate launches before (one product per degree, one for the gates: 14
// per layer and direction pair) were bound by their number and by the passes
// over h, z and A between them: 4,096 atoms, FP32, 17 launches fewer.
#include "edge_common.h"

namespace mpip {

namespace {

// eight consecutive values of an atom's row as an operand
template <int PREC>
__device__ __forceinline__ Parts<PREC> row_parts(const float* x) {
  const f32x4 t[2] = {*(const f32x4*)x, *(const f32x4*)(x + 4)};
  return Parts<PREC>::from(t, 0);
}

// BF16 parts of a weight: three in the FP32 form, one in the BF16 form, and
// there two of V W_down of the first layer's directions (LayerDev::kh1), which
// are those of its BF16 weights of all hidden units.
template <int PREC>
constexpr int kWP = PREC == 1 ? 1 : 3;
// weight tile: w[part], 64 lanes apart
template <int PREC, int WP>
struct Tile {
  bf16x8 v[WP];
  __device__ __forceinline__ explicit Tile(const bf16x8* w) {
#pragma unroll
    for (int q = 0; q < WP; ++q) v[q] = w[q * 64];
  }
  // acc += (tile) b over its chunk of 32, smallest products first
  __device__ __forceinline__ f32x4 mma(const Parts<PREC>& b, f32x4 acc) const {
#pragma unroll
    for (int o = WP - 1; o >= 0; --o)
#pragma unroll
      for (int i = 0; i <= o; ++i)
        if (o - i < Parts<PREC>::N) acc = mfma_bf16(v[i], b.p[o - i], acc);
    return acc;
  }
};

template <int NM, int NT>
__device__ __forceinline__ void clear(f32x4 (&D)[NM][NT]) {
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int t = 0; t < NT; ++t) D[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// D[m][t] += sum over kc of W[kc][t] x_m for NM rows of an atom in memory,
// xs bytes apart: each weight tile is read once for all of them.  w: this
// lane's part of the first tile, LD tiles per chunk
template <int PREC, int WP, int NT, int NM, int LD>
__device__ __forceinline__ void mix_rows(const bf16x8* w, const char* x, int64_t xs, bool x_bf16, int kch, int lane,
                                         f32x4 (&D)[NM][NT]) {
  const int g = lane >> 4;
#pragma unroll 1
  for (int kc = 0; kc < kch; ++kc) {
    Parts<PREC> b[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if (PREC == 1 && x_bf16) b[m].p[0] = *(const bf16x8*)(x + m * xs + 2 * (32 * kc + 8 * g));
      else b[m] = row_parts<PREC>((const float*)(x + m * xs) + 32 * kc + 8 * g);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const Tile<PREC, WP> v(w + (kc * LD + t) * WP * 64);
#pragma unroll
      for (int m = 0; m < NM; ++m) D[m][t] = v.mma(b[m], D[m][t]);
    }
  }
}

// operand chunks from a product's tiles
template <int PREC, int NT>
__device__ __forceinline__ void tile_parts(const f32x4 (&t)[NT], Parts<PREC>* b) {
#pragma unroll
  for (int kc = 0; kc < NT / 2; ++kc) b[kc] = Parts<PREC>::from(t, kc);
}

// tile t of W[t][kc] b_m
template <int PREC, int WP, int KCH, int NM>
__device__ __forceinline__ void mix_tile(const bf16x8* w, int t, const Parts<PREC> (&b)[NM][KCH], f32x4 (&D)[NM]) {
#pragma unroll
  for (int m = 0; m < NM; ++m) D[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < KCH; ++kc) {
    const Tile<PREC, WP> v(w + (t * KCH + kc) * WP * 64);
#pragma unroll
    for (int m = 0; m < NM; ++m) D[m] = v.mma(b[m][kc], D[m]);
  }
}

// rows of a degree taken together: as many as 256 registers hold
template <int PREC, int C>
constexpr int rows_together() { return C == 128 ? 1 : PREC == 1 ? 3 : 2; }
// f(first row, integral_constant<rows>) over the chunks sub, sub + split, ..
// of N rows out of TOTAL
template <int N, int TOTAL, typename F>
__device__ __forceinline__ void row_chunks(int sub, int split, F&& f) {
#pragma unroll 1
  for (int at = N * sub; at < TOTAL; at += N * split) {
    if (at + N <= TOTAL) f(at, std::integral_constant<int, N < TOTAL ? N : TOTAL>{});
    else if constexpr (TOTAL % N != 0) f(at, std::integral_constant<int, TOTAL % N>{});
  }
}

// the weights of a phase: nt tiles of 1 KB
__device__ __forceinline__ void stage(bf16x8* dst, const void* src, int nt) {
  const int lane = threadIdx.x & 63, nw = (int)(blockDim.x >> 6);
  for (int t = (int)(threadIdx.x >> 6); t < nt; t += nw)
    __builtin_amdgcn_global_load_lds((const void*)((const uint4*)src + (size_t)t * 64 + lane),
                                     (__attribute__((address_space(3))) void*)(dst + t * 64), 16, 0, 0);
}

// LDS of a workgroup, in tiles of 1 KB
template <int PREC, int C>
constexpr int lds_tiles() { return PREC == 1 && C <= 64 ? 80 : 160; }

// which 16-atom tiles this wave walks, and its share of a tile's rows
struct Walk {
  int sub, split;
  int64_t t, dt, nt;
  __device__ __forceinline__ explicit Walk(const MixArgs& a) {
    const int w = threadIdx.x >> 6, per = (int)(blockDim.x >> 6) / a.split;
    split = a.split;
    sub = w % split;
    t = (int64_t)blockIdx.x * per + w / split;
    dt = (int64_t)gridDim.x * per;
    nt = (a.n + 15) / 16;
  }
};

__device__ __forceinline__ void store4(void* y, int64_t o, f32x4 v, bool bf16) {
  if (bf16) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    *(bf16x4*)((__bf16*)y + o) = __builtin_convertvector(v, bf16x4);
  } else {
    *(f32x4*)((float*)y + o) = v;
  }
}

}  // namespace

// BOTH: see mix_launch
template <int PREC, int C, int L, int ND, bool BOTH>
__global__ __launch_bounds__(512) void k_mix_fwd(MixArgs a) {
  constexpr int NT = C / 16, KC = C / 32, NLM = (L + 1) * (L + 1), NU = kWP<PREC>;   // parts of W_up; of W_down: ND
  __shared__ __align__(16) bf16x8 sW[64 * lds_tiles<PREC, C>()];
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int kch = a.kx / 32;
  const int64_t es = (PREC == 1 && a.x_bf16) ? 2 : 4;   // bytes per value of x
  const int kg = BOTH ? kch : lds_tiles<PREC, C>() / (NT * ND);   // chunks of W_down in LDS at a time
  const Walk wk(a);
  // z rows of an atom (NT tiles each, LD per chunk in W), chunks k0 .. k0 + nk
  // of x with W in LDS from the first of them on
  auto down = [&](auto LDC, const bf16x8* w, const char* x, int k0, int nk, float* zm, int64_t zs, bool ok, auto& z) {
    constexpr int NM = sizeof(z) / sizeof(z[0]);
    clear(z);
    if (k0 > 0)
#pragma unroll
      for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) z[m][t] = *(const f32x4*)(zm + m * zs + 16 * t + 4 * g);
    mix_rows<PREC, ND, NT, NM, decltype(LDC)::value>(w + lane, x + 32 * k0 * es, a.kx * es, a.x_bf16, nk, lane, z);
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (ok) *(f32x4*)(zm + m * zs + 16 * t + 4 * g) = z[m][t];
  };
  // scalars: z_0 and the gates' logits
  static_for<BOTH ? 1 : 1 + L>([&](auto QC) {
    constexpr int q0 = decltype(QC)::value;
    for (int k0 = 0; k0 < kch; k0 += kg) {
      const int nk = kch - k0 < kg ? kch - k0 : kg;
      if (q0 > 0 || k0 > 0) __syncthreads();
      if constexpr (BOTH) stage(sW, a.dn[0], kch * NT * (1 + L) * ND);
      else
        for (int k = 0; k < nk; ++k)
          stage(sW + k * NT * ND * 64, (const bf16x8*)a.dn[0] + ((k0 + k) * (1 + L) + q0) * NT * ND * 64, NT * ND);
      lds_dma_sync();
      for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
        const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
        const bool ok = i0 < a.n;
#pragma unroll 1
        for (int q = BOTH ? wk.sub : q0; q <= (BOTH ? L : q0 - (wk.sub > 0)); q += wk.split) {
          const char* x = (const char*)a.x + i * NLM * a.kx * es;
          f32x4 z[1][NT];
          down(std::integral_constant<int, BOTH ? NT * (1 + L) : NT>{}, sW + (BOTH ? q * NT * ND * 64 : 0), x, k0, nk,
               a.z0 + (i * (1 + L) + q) * C, 0, ok, z);
          if (q == 0 && k0 + nk == kch) {
            float* h = a.h + i * NLM * C;
            const float* hin = a.first ? a.emb + (int64_t)a.spec_s[i] * C : h;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              f32x4 hv = *(const f32x4*)(hin + 16 * t + 4 * g);
#pragma unroll
              for (int r = 0; r < 4; ++r) hv[r] += silu(z[0][t][r]);
              if (ok) *(f32x4*)(h + 16 * t + 4 * g) = hv;
            }
          }
        }
      }
    }
  });
  __syncthreads();
  stage(sW, a.up[0], KC * NT * NU);
  lds_dma_sync();
  for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
    const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
    const bool ok = i0 < a.n;
    f32x4 hv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) hv[t] = *(const f32x4*)(a.h + i * NLM * C + 16 * t + 4 * g);
    Parts<PREC> b[1][KC];
    tile_parts<PREC, NT>(hv, b[0]);
#pragma unroll 1
    for (int t = wk.sub; t < NT; t += wk.split) {
      f32x4 v[1];
      mix_tile<PREC, NU, KC, 1>(sW + lane, t, b, v);
      if (ok) store4(a.ht, i * NLM * C + 16 * t + 4 * g, v[0], a.ht_bf16);
    }
  }
  static_for<L>([&](auto LC) {
    constexpr int l = decltype(LC)::value + 1;
    __syncthreads();
    if constexpr (!BOTH)
      for (int k0 = 0; k0 < kch; k0 += kg) {
        const int nk = kch - k0 < kg ? kch - k0 : kg;
        if (k0 > 0) __syncthreads();
        stage(sW, (const bf16x8*)a.dn[l] + k0 * NT * ND * 64, nk * NT * ND);
        lds_dma_sync();
        for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
          const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
          row_chunks<rows_together<PREC, C>(), 2 * l + 1>(wk.sub, wk.split, [&](int at, auto MC) {
            const int lm0 = l * l + at;
            f32x4 z[decltype(MC)::value][NT];
            down(std::integral_constant<int, NT>{}, sW, (const char*)a.x + (i * NLM + lm0) * a.kx * es, k0, nk,
                 a.zl + (i * (NLM - 1) + lm0 - 1) * C, C, i0 < a.n, z);
          });
        }
      }
    if constexpr (!BOTH) __syncthreads();
    stage(sW, a.up[l], KC * NT * NU);
    if constexpr (BOTH) stage(sW + KC * NT * NU * 64, a.dn[l], kch * NT * ND);
    lds_dma_sync();
    for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
      const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
      const bool ok = i0 < a.n;
      float* h = a.h + i * NLM * C;
      row_chunks<rows_together<PREC, C>(), 2 * l + 1>(wk.sub, wk.split, [&](int at, auto MC) {
        constexpr int NM = decltype(MC)::value;
        const int lm0 = l * l + at;
        f32x4 z[NM][NT];
        float* zl = a.zl + (i * (NLM - 1) + lm0 - 1) * C;
        if constexpr (BOTH) {
          down(std::integral_constant<int, NT>{}, sW + KC * NT * NU * 64, (const char*)a.x + (i * NLM + lm0) * a.kx * es, 0,
               kch, zl, C, ok, z);
        } else {
#pragma unroll
          for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t) z[m][t] = *(const f32x4*)(zl + m * C + 16 * t + 4 * g);
        }
        Parts<PREC> b[NM][KC];
        f32x4 gate[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          gate[t] = *(const f32x4*)(a.z0 + (i * (1 + L) + l) * C + 16 * t + 4 * g);
#pragma unroll
          for (int r = 0; r < 4; ++r) gate[t][r] = sigm(gate[t][r]);
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          f32x4 hv[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t)
            hv[t] = a.first ? f32x4{0.f, 0.f, 0.f, 0.f} : *(const f32x4*)(h + (lm0 + m) * C + 16 * t + 4 * g);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const int o = (lm0 + m) * C + 16 * t + 4 * g;
#pragma unroll
            for (int r = 0; r < 4; ++r) hv[t][r] = fmaf(gate[t][r], z[m][t][r], hv[t][r]);
            if (ok) *(f32x4*)(h + o) = hv[t];
          }
          tile_parts<PREC, NT>(hv, b[m]);
        }
#pragma unroll 2
        for (int t = 0; t < NT; ++t) {
          f32x4 v[NM];
          mix_tile<PREC, NU, KC, NM>(sW + lane, t, b, v);
#pragma unroll
          for (int m = 0; m < NM; ++m)
            if (ok) store4(a.ht, (i * NLM + lm0 + m) * C + 16 * t + 4 * g, v[m], a.ht_bf16);
        }
      });
    }
  });
}

// z0 and zl hold the forward's values and are overwritten (zl with each wave's
// share of the gates' adjoint, z0 with zbar_0, h~bar with zbar unless BOTH); y: dE/dA [N][nlm][C] or P [N][nlm][kx]
template <int PREC, int C, int L, int ND, bool BOTH>
__global__ __launch_bounds__(512) void k_mix_bwd(MixArgs a) {
  constexpr int NT = C / 16, KC = C / 32, NLM = (L + 1) * (L + 1), NU = kWP<PREC>;   // parts of W_up; of W_down: ND
  __shared__ __align__(16) bf16x8 sW[64 * lds_tiles<PREC, C>()];
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int nty = a.kx / 16;   // even: C/16, 4 S or (32 directions) 2 S
  const Walk wk(a);
  // hbar of rows lm0 ..: the next layer's share, and the residual's (of the
  // last layer: w_read on the scalars of root atoms)
  auto hbar_rows = [&](int64_t i, bool ok, int lm0, auto& hb) {
    constexpr int NM = sizeof(hb) / sizeof(hb[0]);
    clear(hb);
    mix_rows<PREC, NU, NT, NM, NT>(sW + lane, (const char*)(a.htbar + (i * NLM + lm0) * C), 4 * C, false, KC, lane, hb);
    float* hbar = a.hbar + i * NLM * C;
    const float seed = a.seed && lm0 == 0 && a.owned_s[i] ? 1.f : 0.f;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      f32x4 res[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        res[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (a.seed) {
          if (lm0 + m == 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) res[t][r] = seed * a.w_read[16 * t + 4 * g + r];
        } else if (i < a.n_res) {
          res[t] = *(const f32x4*)(hbar + (lm0 + m) * C + 16 * t + 4 * g);
        }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) hb[m][t][r] += res[t][r];
        if (ok && a.keep_hbar) *(f32x4*)(hbar + (lm0 + m) * C + 16 * t + 4 * g) = hb[m][t];
      }
    }
  };
  // operands of one row of a lane's own values
  auto row_tiles = [&](const float* x, Parts<PREC>* b) {
    f32x4 z[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) z[t] = *(const f32x4*)(x + 16 * t + 4 * g);
    tile_parts<PREC, NT>(z, b);
  };
  // tiles t0 .. t1 (an even number) of y's rows from row on
  auto rows_out = [&](int t0, int t1, const bf16x8* w, auto& b, int64_t row, bool ok) {
    constexpr int NM = sizeof(b) / sizeof(b[0]), KB = sizeof(b[0]) / sizeof(b[0][0]);
#pragma unroll 1
    for (int tt = t0; tt < t1; tt += 2)
#pragma unroll
      for (int t = tt; t < tt + 2; ++t) {
        f32x4 v[NM];
        mix_tile<PREC, ND, KB, NM>(w + lane, t - t0, b, v);
#pragma unroll
        for (int m = 0; m < NM; ++m)
          if (ok) store4(a.y, (row + m) * a.kx + 16 * t + 4 * g, v[m], a.x_bf16);
      }
  };
  static_for<L>([&](auto LC) {
    constexpr int l = decltype(LC)::value + 1, N = rows_together<PREC, C>(), M = 2 * l + 1;
    if (l > 1) __syncthreads();
    stage(sW, a.up[l], KC * NT * NU);
    if constexpr (BOTH) stage(sW + KC * NT * NU * 64, a.dn[l], nty * KC * ND);
    lds_dma_sync();
    for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
      const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
      const bool ok = i0 < a.n;
      float* zl = a.zl + (i * (NLM - 1) + l * l - 1) * C;
      f32x4 dg[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) dg[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      row_chunks<N, M>(wk.sub, wk.split, [&](int at, auto MC) {
        constexpr int NM = decltype(MC)::value;
        const int lm0 = l * l + at;
        f32x4 hb[NM][NT];
        hbar_rows(i, ok, lm0, hb);
        Parts<PREC> b[NM][KC];
        f32x4 s[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) s[t] = *(const f32x4*)(a.z0 + (i * (1 + L) + l) * C + 16 * t + 4 * g);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          f32x4 z[NT];
#pragma unroll
          for (int t = 0; t < NT; ++t) z[t] = *(const f32x4*)(zl + (at + m) * C + 16 * t + 4 * g);
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              if (m == 0) s[t][r] = sigm(s[t][r]);
              dg[t][r] = fmaf(hb[m][t][r], z[t][r], dg[t][r]);
              hb[m][t][r] *= s[t][r];
            }
          if constexpr (BOTH) tile_parts<PREC, NT>(hb[m], b[m]);
        }
        if constexpr (BOTH) {
          rows_out(0, nty, sW + KC * NT * NU * 64, b, i * NLM + lm0, ok);
        } else {
#pragma unroll
          for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t)
              if (ok) *(f32x4*)(a.htbar + (i * NLM + lm0 + m) * C + 16 * t + 4 * g) = hb[m][t];
        }
      });
      // this wave's share of the gate's adjoint, in its first row's slot
      if (ok && N * wk.sub < M)
#pragma unroll
        for (int t = 0; t < NT; ++t) *(f32x4*)(zl + N * wk.sub * C + 16 * t + 4 * g) = dg[t];
    }
    if constexpr (!BOTH) {
      // zbar W_down^T alone, from the zbar left in the rows of h~bar
      const int tg = lds_tiles<PREC, C>() / (KC * ND) & ~1;
      for (int t0 = 0; t0 < nty; t0 += tg) {
        const int t1 = nty - t0 < tg ? nty : t0 + tg;
        __syncthreads();
        stage(sW, (const bf16x8*)a.dn[l] + t0 * KC * ND * 64, (t1 - t0) * KC * ND);
        lds_dma_sync();
        for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
          const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
          row_chunks<N, M>(wk.sub, wk.split, [&](int at, auto MC) {
            constexpr int NM = decltype(MC)::value;
            Parts<PREC> b[NM][KC];
#pragma unroll
            for (int m = 0; m < NM; ++m) row_tiles(a.htbar + (i * NLM + l * l + at + m) * C, b[m]);
            rows_out(t0, t1, sW, b, i * NLM + l * l + at, i0 < a.n);
          });
        }
      }
    }
  });
  __syncthreads();
  stage(sW, a.up[0], KC * NT * NU);
  lds_dma_sync();
  for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
    const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
    const bool ok = i0 < a.n;
    float* z0 = a.z0 + i * (1 + L) * C;
    if (wk.sub == 0) {
      f32x4 hb[1][NT];
      hbar_rows(i, ok, 0, hb);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f32x4 z = *(const f32x4*)(z0 + 16 * t + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) hb[0][t][r] *= dsilu(z[r]);
        if (ok) *(f32x4*)(z0 + 16 * t + 4 * g) = hb[0][t];
      }
    }
    static_for<L>([&](auto LC) {
      constexpr int l = decltype(LC)::value + 1, N = rows_together<PREC, C>(), M = 2 * l + 1;
      if (wk.sub == (l < wk.split ? l : wk.split - 1)) {
        const float* zl = a.zl + (i * (NLM - 1) + l * l - 1) * C;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          f32x4 dg = *(const f32x4*)(zl + 16 * t + 4 * g), s = *(const f32x4*)(z0 + l * C + 16 * t + 4 * g);
          for (int q = 1; q < wk.split && N * q < M; ++q) {
            const f32x4 d = *(const f32x4*)(zl + N * q * C + 16 * t + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) dg[r] += d[r];
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            s[r] = sigm(s[r]);
            dg[r] *= s[r] * (1.f - s[r]);
          }
          if (ok) *(f32x4*)(z0 + l * C + 16 * t + 4 * g) = dg;
        }
      }
    });
  }
  // zbar_0 and the gates' adjoint through degree 0's W_down
  constexpr int K0 = KC * (1 + L);
  const int tg = BOTH ? nty : lds_tiles<PREC, C>() / (K0 * ND);
  for (int t0 = 0; t0 < nty; t0 += tg) {
    const int t1 = nty - t0 < tg ? nty : t0 + tg;
    __syncthreads();
    stage(sW, (const bf16x8*)a.dn[0] + t0 * K0 * ND * 64, (t1 - t0) * K0 * ND);
    lds_dma_sync();
    for (int64_t tile = wk.t; tile < wk.nt; tile += wk.dt) {
      const int64_t i0 = 16 * tile + (lane & 15), i = i0 < a.n ? i0 : a.n - 1;
      const bool ok = i0 < a.n;
      Parts<PREC> b[1][K0];
#pragma unroll
      for (int l = 0; l <= L; ++l) row_tiles(a.z0 + (i * (1 + L) + l) * C, b[0] + l * KC);
#pragma unroll 1
      for (int t = t0 + wk.sub; t < t1; t += wk.split) {
        f32x4 v[1];
        mix_tile<PREC, ND, K0, 1>(sW + lane, t - t0, b, v);
        if (ok) store4(a.y, i * NLM * a.kx + 16 * t + 4 * g, v[0], a.x_bf16);
      }
    }
  }
}

// Last layer: A [N][C] in, dE/dA out (root atoms seed the adjoint)
template <int PREC, int C>
__global__ __launch_bounds__(256) void k_mix_last(MixArgs a) {
  constexpr int NT = C / 16, KC = C / 32;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int64_t i0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 16 + (lane & 15);
  const bool ok = i0 < a.n;
  const int64_t i = ok ? i0 : a.n - 1;
  const int sp = a.spec_s[i];
  // chosen before the product: with the branch between the last MFMA and the
  // first read of its result the compiler leaves out the wait that read needs
  // (it looks past the empty block of one side)
  const float* hin = a.first ? a.emb + (int64_t)sp * C : a.h + i * a.nlm * C;
  asm volatile("" : "+v"(hin));
  f32x4 zm[1][NT];
  clear(zm);
  mix_rows<PREC, kWP<PREC>, NT, 1, NT>((const bf16x8*)a.up[0] + lane, (const char*)((const float*)a.x + i * C), 0, false, KC, lane, zm);
  f32x4 (&z)[NT] = zm[0];
  const float seed = a.owned_s[i] ? 1.f : 0.f;
  double e = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const f32x4 hv = *(const f32x4*)(hin + 16 * t + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float w = a.w_read[16 * t + 4 * g + r];
      e += (double)(hv[r] + silu(z[t][r])) * (double)w;
      z[t][r] = seed * w * dsilu(z[t][r]);
    }
  }
  e += __shfl_xor(e, 16);
  e += __shfl_xor(e, 32);
  if (ok && g == 0) a.atom_e[i] = (double)a.e0[sp] + e;
  Parts<PREC> b[1][KC];
  tile_parts<PREC, NT>(z, b[0]);
  const bf16x8* dn = (const bf16x8*)a.dn[0] + lane;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    f32x4 v[1];
    mix_tile<PREC, kWP<PREC>, KC, 1>(dn, t, b, v);
    if (ok) *(f32x4*)((float*)a.y + i * C + 16 * t + 4 * g) = v[0];
  }
}

// Eight waves share the weights.  With fewer tiles than the waves of the chip
// 2, 4 or 8 waves share a tile's rows, so that every CU has eight waves (a
// wave per tile with 4,096 atoms: one wave on a CU, each row's latency exposed;
// 76 instead of 44 us forward, 87 instead of 37 back).
template <int PREC, int C, int L>
static void mix_launch(int which, MixArgs a, hipStream_t s) {
  const int64_t tiles = (a.n + 15) / 16;
  if (which == 2) {
    if constexpr (L == 1) {
      // a wave alone on its CU while the tiles do not fill the chip (512 atoms of
      // 128 channels: 24.7 us, four to a workgroup 26.6), the same from 4,096 atoms on
      const int nw = a.n > 4096 ? 4 : 1;
      k_mix_last<PREC, C><<<(unsigned)((tiles + nw - 1) / nw), 64 * nw, 0, s>>>(a);
    }
    return;
  }
  constexpr int kWaves = 8, kCus = 256;
  a.split = 1;
  while (a.split < kWaves && 2 * a.split * tiles <= (int64_t)kWaves * kCus) a.split *= 2;
  const int64_t need = (tiles * a.split + kWaves - 1) / kWaves;
  const unsigned g = (unsigned)(need < kCus ? need : kCus);
  // BOTH: LDS holds a degree's W_down beside its W_up (degree 0: all of its
  // columns alone).  Else they are staged in turn, as many chunks of W_down as
  // fit at a time, and z (zbar) goes through memory in between.
  auto parts = [&](auto DC) {
    constexpr int nd = decltype(DC)::value;
    const int nt = C / 16, dn = a.kx / 32 * nt * nd, up = C / 32 * nt * kWP<PREC>;
    const bool fits = dn * (1 + L) <= lds_tiles<PREC, C>() && dn + up <= lds_tiles<PREC, C>();
    if (which == 0) {
      if (fits) k_mix_fwd<PREC, C, L, nd, true><<<g, 64 * kWaves, 0, s>>>(a);
      else k_mix_fwd<PREC, C, L, nd, false><<<g, 64 * kWaves, 0, s>>>(a);
    } else {
      if (fits) k_mix_bwd<PREC, C, L, nd, true><<<g, 64 * kWaves, 0, s>>>(a);
      else k_mix_bwd<PREC, C, L, nd, false><<<g, 64 * kWaves, 0, s>>>(a);
    }
  };
  if constexpr (PREC == 1) {
    if (a.dn_parts == 2) return parts(std::integral_constant<int, 2>{});
  }
  parts(std::integral_constant<int, kWP<PREC>>{});
}

template <int PREC>
static void mix_prec(int which, int C, int L, const MixArgs& a, hipStream_t s) {
  if (which == 2) L = 1;   // the last layer's kernel has no degrees
  if (C == 32 && L == 1) mix_launch<PREC, 32, 1>(which, a, s);
  else if (C == 32) mix_launch<PREC, 32, 2>(which, a, s);
  else if (C == 64 && L == 1) mix_launch<PREC, 64, 1>(which, a, s);
  else if (C == 64) mix_launch<PREC, 64, 2>(which, a, s);
  else if (L == 1) mix_launch<PREC, 128, 1>(which, a, s);
  else mix_launch<PREC, 128, 2>(which, a, s);
}

void launch_mix(int which, int prec, int C, int L, const MixArgs& a, hipStream_t s) {
  if (a.n <= 0) return;
  if (prec == MPIP_BF16_MIXED) mix_prec<1>(which, C, L, a, s);
  else mix_prec<0>(which, C, L, a, s);
}

}  // namespace mpip
