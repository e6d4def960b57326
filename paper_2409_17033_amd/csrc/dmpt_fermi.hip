// Reductions and outputs of the finite-temperature path (Sec. V.B).  The products
// of the recursion and everything elementwise between them run in the general
// product kernels (ProdArgs).
#include <hip/hip_runtime.h>

#include "dmpt_device.h"
#include "dmpt_fermi.h"

namespace dmpt {

namespace {

// Block b of matrix k sums the squares of its share of the 16-byte pieces, in a
// fixed order, and the diagonal entries i = b (mod nblk).  Padding is zero, so
// the layout does not matter for the squares.
__global__ __launch_bounds__(256) void k_trace_sq(const float* m, size_t stride, int n, int n_pad, int tiled, double* part) {
  __shared__ double s_tr[4], s_sq[4];
  const float* mk = m + (size_t)blockIdx.y * stride;
  const f32x4* m4 = (const f32x4*)mk;
  const size_t n4 = (size_t)n_pad * n_pad / 4;
  double sq[2] = {0.0, 0.0}, tr = 0.0;
  const size_t step = (size_t)gridDim.x * 256;
  size_t q = (size_t)blockIdx.x * 256 + threadIdx.x;
  for (; q + step < n4; q += 2 * step) {
    const f32x4 x0 = m4[q], x1 = m4[q + step];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sq[0] += (double)x0[e] * (double)x0[e];
      sq[1] += (double)x1[e] * (double)x1[e];
    }
  }
  if (q < n4) {
    const f32x4 x0 = m4[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) sq[0] += (double)x0[e] * (double)x0[e];
  }
  for (int i = blockIdx.x + (int)threadIdx.x * gridDim.x; i < n; i += 256 * gridDim.x) tr += mk[m_off(tiled, i, i, n_pad)];
  const double s = wave_sum(sq[0] + sq[1]), t = wave_sum(tr);
  if ((threadIdx.x & 63) == 0) {
    s_tr[threadIdx.x >> 6] = t;
    s_sq[threadIdx.x >> 6] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* o = part + 2 * ((size_t)blockIdx.y * gridDim.x + blockIdx.x);
    o[0] = s_tr[0] + s_tr[1] + s_tr[2] + s_tr[3];
    o[1] = s_sq[0] + s_sq[1] + s_sq[2] + s_sq[3];
  }
}

// A wave takes 16 x 16 pieces: 4 columns of a row per lane, 16 lanes down the
// rows of a tiled matrix (256-byte reads) or along a row-major one's.
__global__ __launch_bounds__(256) void k_fermi_output(const float* em, const float* e2, const float* y, size_t ystride,
                                                      const float* a, int n, int n_pad, int nobs, int tiled,
                                                      FermiShift shift, double scale, float* d_out, float* chi_out,
                                                      double* a0_part) {
  __shared__ double s_red[4];
  const size_t n2 = (size_t)n * n;
  const int k = blockIdx.y, lane = threadIdx.x & 63;
  // row-major: 4 rows x 64 columns a piece
  const int pr = tiled ? 16 : 4, pc = tiled ? 16 : 64;
  const int cg = (n + pc - 1) / pc, rg = (n + pr - 1) / pr;
  const size_t pieces = (size_t)rg * cg;
  double acc = 0.0;
  for (size_t p = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); p < pieces; p += (size_t)gridDim.x * 4) {
    const int i = (int)(p / cg) * pr + (tiled ? lane & 15 : lane >> 4);
    const int j = (int)(p % cg) * pc + 4 * (tiled ? lane >> 4 : lane & 15);
    if (i >= n || j >= n) continue;
    const size_t o = m_off(tiled, i, j, n_pad), e = (size_t)i * n + j;
    f32x4 dv = *(const f32x4*)(em + o);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i == j + q) dv[q] += 0.5f;
    if (k == 0 && d_out)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (j + q < n) d_out[e + q] = dv[q];
    if (nobs > 0) {
      f32x4 yv = *(const f32x4*)(y + (size_t)k * ystride + o);
      const float g = shift.g[k];
      const f32x4 ev = *(const f32x4*)(e2 + o);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (j + q >= n) break;
        const float v = yv[q] - g * ev[q] + (i == j + q ? 0.25f * g : 0.0f);
        if (chi_out) chi_out[(size_t)k * n2 + e + q] = (float)(scale * (double)v);
        acc += (double)dv[q] * (double)a[(size_t)k * n2 + e + q];
      }
    }
  }
  if (nobs > 0) {
    acc = wave_sum(acc);
    if (lane == 0) s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) a0_part[(size_t)k * gridDim.x + blockIdx.x] = s_red[0] + s_red[1] + s_red[2] + s_red[3];
  }
}

}  // namespace

hipError_t launch_trace_sq(const float* m, size_t stride, int nmat, int n, int n_pad, int tiled, double* part, int nblk,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_trace_sq, dim3(nblk, nmat), dim3(256), 0, s, m, stride, n, n_pad, tiled, part);
  return hipGetLastError();
}

hipError_t launch_fermi_output(const float* e, const float* e2, const float* y, size_t ystride, const float* a, int n,
                               int n_pad, int nobs, int tiled, FermiShift shift, double scale, float* d_out,
                               float* chi_out, double* a0_part, int nblk, hipStream_t s) {
  hipLaunchKernelGGL(k_fermi_output, dim3(nblk, nobs > 0 ? nobs : 1), dim3(256), 0, s, e, e2, y, ystride, a, n, n_pad, nobs,
                     tiled, shift, scale, d_out, chi_out, a0_part);
  return hipGetLastError();
}

}  // namespace dmpt
