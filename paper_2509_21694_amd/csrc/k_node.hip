// Output reductions (forces, virial, energy: fixed order, FP64) and the fill
// kernel.
#include "kernels.h"

namespace mpip {

// ------------------------------------------------------------ outputs

// Per atom: F_i = sum_{e in row i} G_e - G_rev(e) (FP64), written in input
// order, with G_e = g[e] (dE/dr_e, or the h_e of FastArgs::g2p, which gives
// the same sums); per block: sum of root energies and of r_e (x) G_e, fixed
// order.
// A wave takes 16 rows, 4 at a time with 16 lanes over each row's edges
// (three edges per lane in flight, so a row of up to 48 edges costs one
// round of dependent loads) and a 16-lane butterfly per row; each lane keeps
// its virial partial sums, reduced over the wave by shuffles and over the
// block's 4 waves in LDS, always in the same order.
__global__ __launch_bounds__(256) void k_forces(OutArgs a) {
  __shared__ double sh[4][10];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, q = lane >> 4, el = lane & 15;
  double loc[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) loc[k] = 0.0;
  const bool run = (a.status[ST_FLAGS] == 0) && ((int64_t)a.row_ptr[a.n] <= a.capacity);
  if (run) {
    const int64_t r0 = (int64_t)blockIdx.x * kOutRowsPerBlock + w * 16;
#pragma unroll 1
    for (int64_t ib = r0; ib < r0 + 16; ib += 4) {
      const int64_t i = ib + q;
      double F[3] = {0.0, 0.0, 0.0};
      if (i < a.n) {
        const int e1 = a.row_ptr[i + 1];
        for (int e = a.row_ptr[i] + el; e < e1; e += 48) {
          int rv[3];
          float4 ge[3], gr[3], r[3];
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            const int eu = e + 16 * u;
            const bool ok = eu < e1;
            rv[u] = ok ? a.e_rev[eu] : -1;
            ge[u] = ok ? a.g[eu] : make_float4(0.f, 0.f, 0.f, 0.f);
            r[u] = ok ? a.e_vec[eu] : make_float4(0.f, 0.f, 0.f, 0.f);
          }
#pragma unroll
          for (int u = 0; u < 3; ++u) gr[u] = rv[u] >= 0 ? a.g[rv[u]] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            F[0] += (double)ge[u].x - (double)gr[u].x;
            F[1] += (double)ge[u].y - (double)gr[u].y;
            F[2] += (double)ge[u].z - (double)gr[u].z;
            const double rr[3] = {r[u].x, r[u].y, r[u].z}, gg[3] = {ge[u].x, ge[u].y, ge[u].z};
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
              for (int c = 0; c < 3; ++c) loc[1 + 3 * p + c] += rr[p] * gg[c];
          }
        }
      }
#pragma unroll
      for (int off = 8; off > 0; off >>= 1)
#pragma unroll
        for (int d = 0; d < 3; ++d) F[d] += __shfl_xor(F[d], off);
      if (el == 0 && i < a.n) {
        const int o = a.perm[i];
        a.forces[3 * (int64_t)o + 0] = F[0];
        a.forces[3 * (int64_t)o + 1] = F[1];
        a.forces[3 * (int64_t)o + 2] = F[2];
        if (a.atom_energy) a.atom_energy[o] = a.atom_e[i];
        if (a.owned_s[i]) loc[0] += a.atom_e[i];
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < 10; ++k) loc[k] += __shfl_xor(loc[k], off);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 10; ++k) sh[w][k] = loc[k];
  __syncthreads();
  if (threadIdx.x < 10)
    a.partials[(int64_t)blockIdx.x * 10 + threadIdx.x] =
        ((sh[0][threadIdx.x] + sh[1][threadIdx.x]) + sh[2][threadIdx.x]) + sh[3][threadIdx.x];
}

__global__ void k_final(OutArgs a) {
  __shared__ double sh[10][256];
  double loc[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) loc[k] = 0.0;
  for (int b = threadIdx.x; b < a.nblocks; b += 256)
#pragma unroll
    for (int k = 0; k < 10; ++k) loc[k] += a.partials[(int64_t)b * 10 + k];
#pragma unroll
  for (int k = 0; k < 10; ++k) sh[k][threadIdx.x] = loc[k];
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off)
#pragma unroll
      for (int k = 0; k < 10; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + off];
    __syncthreads();
  }
  // a data-dependent error (the passes skipped their work) leaves NaN in the
  // energy and virial, visible to callers that cannot read the status word
  const bool ok = (a.status[ST_FLAGS] == 0) && ((int64_t)a.row_ptr[a.n] <= a.capacity);
  const double nan = __longlong_as_double(0x7ff8000000000000ll);
  if (threadIdx.x == 0) a.energy[0] = ok ? sh[0][0] : nan;
  if (threadIdx.x < 9) a.virial[threadIdx.x] = ok ? -sh[1 + threadIdx.x][0] : nan;
}

void launch_outputs(const OutArgs& a, hipStream_t s) {
  k_forces<<<a.nblocks, 256, 0, s>>>(a);
  k_final<<<1, 256, 0, s>>>(a);
}

__global__ void k_fill(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// a kernel rather than hipMemsetAsync, so that a captured graph holds only kernel nodes
void launch_fill32(void* p, uint32_t value, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 4);
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  k_fill<<<(unsigned)blocks, 256, 0, s>>>((uint32_t*)p, n, value);
}

void launch_zero(void* p, size_t bytes, hipStream_t s) { launch_fill32(p, 0u, bytes, s); }

}  // namespace mpip
