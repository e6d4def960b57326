// gfx950 kernels of the self-consistent response loop (Eq. CP_SCF): the
// vector steps on the diagonal state v = diag(chi'), and the learned mixer.
//
// The mixer network is applied site by site with shared weights: for a
// state vector x in R^n, site i sees z_i = [x_{i-w} .. x_{i+w}, e_{i-w} ..
// e_{i+w}, U_i] with e the on-site energies (k = 4w + 3 features, zeros
// beyond the ends) and outputs
//   y_i = w2 . tanh(W1 z_i + b1) + b2          (hidden width h).
// Parameters (FP32 masters and the BF16 copy alike): [W1 (h x k, row-major) |
// b1 (h) | w2 (h) | b2 (1)].  Training: MSE loss, Adam (Kingma & Ba, 2015).
// Shapes are small next to the SP2 products (B n ~ 1e4-1e5 site rows,
// k ~ 131, h = 256).  Up to h = 256 and w = 64 one fused kernel forms outputs,
// loss and gradients; beyond, the products use one LDS-tiled FP32 kernel with
// an optional deterministic split over K.  Weights are read as BF16 and widened.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dmpt_internal.h"
#include "dmpt_scf.h"

namespace dmpt {

namespace {

__device__ __forceinline__ float ld(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float ld(const uint16_t* p, size_t i) {
  return __builtin_bit_cast(float, ((unsigned int)p[i]) << 16);
}
__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

constexpr int GT = 32;   // output tile edge; 256 threads, 4 outputs each

// C_z[m][c] = sum_{k in split z} a(m, k) b(k, c), C_z = C + z * zstride
//   a(m, k) = TRA ? A[k * lda + m] : A[m * lda + k]
//   b(k, c) = TRB ? B[c * ldb + k] : B[k * ldb + c]
template <class TA, class TB, bool TRA, bool TRB>
__global__ __launch_bounds__(256) void k_gemm(const TA* A, int lda, const TB* B, int ldb, float* C, int ldc,
                                              size_t zstride, int M, int N, int K, int kc) {
  __shared__ float sa[GT][GT + 1];
  __shared__ float sb[GT][GT + 1];
  const int t = threadIdx.x;
  const int m0 = blockIdx.y * GT, c0 = blockIdx.x * GT;
  const int kbeg = blockIdx.z * kc, kend = min(K, kbeg + kc);
  const int tr = t / 8, tc = (t % 8) * 4;   // this thread: row tr, columns tc..tc+3
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = kbeg; k0 < kend; k0 += GT) {
    for (int e = t; e < GT * GT; e += 256) {
      const int i = e / GT, j = e % GT;
      // sa[i][j] = a(m0 + i, k0 + j); sb[i][j] = b(k0 + i, c0 + j)
      const int am = m0 + i, ak = k0 + j;
      sa[i][j] = (am < M && ak < kend) ? ld(A, TRA ? (size_t)ak * lda + am : (size_t)am * lda + ak) : 0.f;
      const int bk = k0 + i, bc = c0 + j;
      sb[i][j] = (bk < kend && bc < N) ? ld(B, TRB ? (size_t)bc * ldb + bk : (size_t)bk * ldb + bc) : 0.f;
    }
    __syncthreads();
#pragma unroll 8
    for (int k = 0; k < GT; ++k) {
      const float av = sa[tr][k];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] += av * sb[k][tc + q];
    }
    __syncthreads();
  }
  float* cz = C + blockIdx.z * zstride;
  const int m = m0 + tr;
  if (m < M)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (c0 + tc + q < N) cz[(size_t)m * ldc + c0 + tc + q] = acc[q];
}

// C[e] = sum_z P[z][e] for e < count (fixed order)
__global__ void k_sum_splits(const float* part, int splits, size_t count, float* c) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  float acc = 0.f;
  for (int z = 0; z < splits; ++z) acc += part[(size_t)z * count + e];
  c[e] = acc;
}

unsigned blocks(size_t total, unsigned per) { return (unsigned)((total + per - 1) / per); }

template <class TA, class TB, bool TRA, bool TRB>
hipError_t gemm(const TA* A, int lda, const TB* B, int ldb, float* C, int ldc, int M, int N, int K,
                hipStream_t s) {
  dim3 grid((N + GT - 1) / GT, (M + GT - 1) / GT, 1);
  hipLaunchKernelGGL((k_gemm<TA, TB, TRA, TRB>), grid, dim3(256), 0, s, A, lda, B, ldb, C, ldc, (size_t)0, M, N,
                     K, K);
  return hipGetLastError();
}

// Long-K products (weight gradients over all site rows): K split into
// `splits` ranges, partial products into `scratch` (splits x M x N), then
// summed in a fixed order into the dense C (ldc = N).
constexpr int kSplits = 64;
template <class TA, class TB, bool TRA, bool TRB>
hipError_t gemm_splitk(const TA* A, int lda, const TB* B, int ldb, float* C, int M, int N, int K, float* scratch,
                       hipStream_t s) {
  const int kc = ((K + kSplits - 1) / kSplits + GT - 1) / GT * GT;
  const int splits = (K + kc - 1) / kc;
  dim3 grid((N + GT - 1) / GT, (M + GT - 1) / GT, splits);
  hipLaunchKernelGGL((k_gemm<TA, TB, TRA, TRB>), grid, dim3(256), 0, s, A, lda, B, ldb, scratch, N,
                     (size_t)M * N, M, N, K, kc);
  hipLaunchKernelGGL(k_sum_splits, dim3(blocks((size_t)M * N, 256)), dim3(256), 0, s, scratch, splits,
                     (size_t)M * N, C);
  return hipGetLastError();
}

// Column sums of a rows x c matrix: chunk z of the rows into part[z][c]
// (then k_sum_splits over the chunks, fixed order).
__global__ void k_colsum_part(const float* m, size_t rows, int c, size_t chunk, float* part) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= c) return;
  const size_t r0 = (size_t)blockIdx.y * chunk, r1 = r0 + chunk < rows ? r0 + chunk : rows;
  float acc = 0.f;
  for (size_t r = r0; r < r1; ++r) acc += m[r * c + j];
  part[(size_t)blockIdx.y * c + j] = acc;
}

hipError_t colsum(const float* m, size_t rows, int c, float* out, float* scratch, hipStream_t s) {
  const size_t chunk = (rows + kSplits - 1) / kSplits;
  const int nchunk = (int)((rows + chunk - 1) / chunk);
  hipLaunchKernelGGL(k_colsum_part, dim3(blocks(c, 256), nchunk), dim3(256), 0, s, m, rows, c, chunk, scratch);
  hipLaunchKernelGGL(k_sum_splits, dim3(blocks(c, 256)), dim3(256), 0, s, scratch, nchunk, (size_t)c, out);
  return hipGetLastError();
}

// Z ((B n) x k): rows (b, i) = [x_b,i-w .. x_b,i+w, en_i-w .. en_i+w, U_i]
__global__ void k_site_inputs(const float* x, const float* u, const float* en, int B, int n, int w, float* z) {
  const int m = 2 * w + 1, k = 2 * m + 1;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)B * n * k) return;
  const size_t row = e / k;
  const int f = (int)(e % k);
  const int b = (int)(row / n), i = (int)(row % n);
  float v;
  if (f == k - 1) {
    v = u[i];
  } else if (f < m) {
    const int j = i + f - w;
    v = (j >= 0 && j < n) ? x[(size_t)b * n + j] : 0.0f;
  } else {
    const int j = i + (f - m) - w;
    v = (j >= 0 && j < n) ? en[j] : 0.0f;
  }
  z[e] = v;
}

__global__ void k_diag(const float* m, int n, float* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = m[(size_t)i * n + i];
}

// Z (rows x h) += b1, then A = tanh(Z) in place.
__global__ void k_bias_tanh(float* z, const uint16_t* b1, size_t rows, int h) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < rows * h) z[e] = tanhf(z[e] + ld(b1, e % h));
}

// y (rows) += b2
__global__ void k_bias1(float* y, const uint16_t* b2, size_t rows) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < rows) y[e] += ld(b2, 0);
}

// dY = 2 (Y - T) / m in place of Y; per-block FP64 partials of sum (Y - T)^2.
__global__ __launch_bounds__(256) void k_mse(float* y, const float* t, size_t m, double* part) {
  __shared__ double red[4];
  const double scale = 2.0 / (double)m;
  double acc = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < m; e += (size_t)gridDim.x * 256) {
    const double r = (double)y[e] - (double)t[e];
    acc += r * r;
    y[e] = (float)(scale * r);
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// loss = sum(part) * inv, written to out[idx] (fixed order, one block).
__global__ void k_loss_final(const double* part, int nblk, double inv, double* out, int idx) {
  double acc = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 64) acc += part[b];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (threadIdx.x == 0) out[idx] = acc * inv;
}

// dZ = dA * (1 - A^2) in place of dA (A = tanh(Z) kept from the forward pass).
__global__ void k_tanh_back(float* da, const float* a, size_t total) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < total) da[e] *= 1.0f - a[e] * a[e];
}

// Adam on the FP32 masters; refreshes the BF16 copy.
__global__ void k_adam(float* p, uint16_t* p16, float* m, float* v, const float* g, size_t count, float lr,
                       float beta1, float beta2, float eps, float c1, float c2) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
  const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
  p[i] = pi;
  p16[i] = to_bf16(pi);
}

// Initial weights: W ~ U(-r, r) with r = sqrt(6 / (fan_in + fan_out)) (Glorot),
// biases 0; the uniform numbers come from splitmix64 of (seed, index).
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
__global__ void k_init_params(float* p, uint16_t* p16, int k, int h, uint64_t seed) {
  const size_t count = (size_t)h * k + 2 * h + 1;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const size_t w1 = (size_t)h * k, b1 = w1 + h, w2 = b1 + h;
  float val = 0.0f;
  if (i < w1 || (i >= b1 && i < w2)) {
    const double u = (double)(splitmix64(seed * 0x100000001B3ull + i) >> 11) * (1.0 / 9007199254740992.0);
    const double r = i < w1 ? sqrt(6.0 / (double)(k + h)) : sqrt(6.0 / (double)(h + 1));
    val = (float)((2.0 * u - 1.0) * r);
  }
  p[i] = val;
  p16[i] = to_bf16(val);
}

// ---------------------------------------------------------------- fused network pass

// One workgroup takes 64 sites and, one after the other, its share of the
// batch: forward, loss and the gradients of those rows without writing Z, A or
// their gradients to memory.  Wave w owns the hidden units 32 w .. 32 w + 31.
// Products on v_mfma_f32_32x32x2_f32 (FP32 operands and sums; the weights are
// BF16 values, widened exactly):
//   * Z is a Toeplitz matrix of x: operand (i, f) is x_{i + f - w}, read from
//     one LDS row, so it is never formed.  The columns of E and U are the same
//     for every state of the batch: their part of W1 z (with b1) is formed once
//     per workgroup and starts every accumulator.
//   * The accumulator holds rows 8 (e / 4) + 4 h + e % 4 of hidden unit l32 in
//     register e of lane (h, l32), which is the operand layout of dZ^T for the
//     row pair (r, r + 4): the weight gradient takes it as it stands.
//   * The gradient's E and U columns are linear in dZ summed over the batch:
//     one product at the end.
// Each workgroup writes its own gradient (summed afterwards in order, in FP64).
// Covers h <= 256 and windows w <= 64 (FB blocks of 32 window columns and one
// column more); other shapes take the general products above.
// Bound by the FP32 MFMAs beside tanh on the vector ALU.  n = 1024, batch 64,
// w = 32, h = 256: loss and gradient 1145 -> 125 us (the pass 95 us, of which 35
// are its MFMAs; the sum over the workgroups 10), error of the gradient against
// 64 bits 1.3e-7 -> 3.6e-8.
typedef float f16v __attribute__((ext_vector_type(16)));
constexpr int kFusedSites = 64, kFusedHidden = 256, kFusedWGs = 256;

inline int fused_blocks(int w) { return (2 * w + 1) / 32 + ((2 * w + 1) % 32 > 1 ? 1 : 0); }   // FB (0: one column)
inline bool fused_shape(int w, int h) { return h <= kFusedHidden && fused_blocks(w) <= 4; }
// Few sites fill little of a block, whose rows cost the same: with several states a
// workgroup the general products, whose rows run on through the batch, win.  us,
// general / fused, w = 8, h = 64: forward n = 8 16384 states 131 / 241, n = 16 1024
// states 51 / 42, n = 8 64 states 41 / 31; gradient 16384 states n = 1 275 / 405, n = 3
// 533 / 414 (w = 2, h = 16: 351 / 383), n = 8 1180 / 427.
inline bool use_fused(int n, int w, int h, int B, bool grad) {
  const bool sparse = grad ? n < kFusedSites / 16 && B > 4 * kFusedWGs : n < kFusedSites / 4 && B > kFusedWGs;
  return fused_shape(w, h) && !sparse;
}
// Batch groups a 64-site block is cut into: about one workgroup per CU.
inline int fused_groups(int n, int B) {
  const int ib = (n + kFusedSites - 1) / kFusedSites;
  int g = kFusedWGs / ib;
  g = g < 1 ? 1 : g > B ? B : g;
  const int per = (B + g - 1) / g;
  return (B + per - 1) / per;
}

template <int FB, bool BWD, bool TAIL>
__global__ __launch_bounds__(512) void k_mixer_fused(const uint16_t* p16, int w, int h, const float* u, const float* en,
                                                     int n, const float* x, const float* t, int B, int per, float* y,
                                                     double* loss_part, float* gpart, double scale) {
  constexpr int KM = 32 * FB + 2;                  // window columns, padded to an even count
  constexpr int XS = kFusedSites + KM + 32;
  __shared__ uint16_t wx[KM * kFusedHidden];       // W1's x columns, [f][unit]
  __shared__ uint16_t we[KM * kFusedHidden];       // its E columns
  __shared__ float xs[XS], es[XS], us[kFusedSites], zeros[TAIL ? 32 * FB + 1 : 1];
  __shared__ float ysum[8][kFusedSites];
  __shared__ __attribute__((aligned(16))) float dys[kFusedSites];
  const int m = 2 * w + 1, k = 2 * m + 1, km = m + 1;
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, wave = tid >> 6;
  const int hf = lane >> 5, l32 = lane & 31, unit = wave * 32 + l32, hp = (nth >> 6) * 32;
  // the last block ends with the last site and passes over rows of the block before it
  const int own = blockIdx.x * kFusedSites, i0 = min(own, max(n - kFusedSites, 0));
  const uint16_t* b1 = p16 + (size_t)h * k;
  const uint16_t* w2 = b1 + h;
  const int b0 = blockIdx.y * per, be = b0 + per < B ? b0 + per : B;
  for (int q = tid; q < km * hp; q += nth) {
    const int f = q % km, c = q / km;              // along a row of W1
    const bool in = f < m && c < h;
    wx[f * hp + c] = in ? p16[(size_t)c * k + f] : (uint16_t)0;
    we[f * hp + c] = in ? p16[(size_t)c * k + m + f] : (uint16_t)0;
  }
  for (int q = tid; q < XS; q += nth) {
    const int j = i0 + q - w;
    es[q] = j >= 0 && j < n ? en[j] : 0.0f;
  }
  if (TAIL)
    for (int q = tid; q < 32 * FB + 1; q += nth) zeros[q] = 0.0f;
  for (int q = tid; q < kFusedSites; q += nth) us[q] = i0 + q < n ? u[i0 + q] : 0.0f;
  const float w2c = unit < h ? ld(w2, unit) : 0.0f, b1c = unit < h ? ld(b1, unit) : 0.0f;
  const float wuc = unit < h ? ld(p16, (size_t)unit * k + 2 * m) : 0.0f, b2 = ld(w2 + h, 0);
  __syncthreads();
  // row of register e, block bi: 32 bi + 8 (e / 4) + 4 hf + e % 4
  f16v site[2];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int e = 0; e < 16; ++e) site[bi][e] = b1c + us[32 * bi + 8 * (e >> 2) + 4 * hf + (e & 3)] * wuc;
  auto forward = [&](const float* v, const uint16_t* wt, f16v (&acc)[2]) {
#pragma unroll 4
    for (int s = 0; s < km / 2 - 1; ++s) {
      const int f = 2 * s + hf;
      const float bv = ld(wt, f * hp + unit);
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[l32 + f], bv, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[32 + l32 + f], bv, acc[1], 0, 0, 0);
    }
    // columns m - 1 and m: the padding one's input lies outside the window (zero times Inf or NaN is NaN)
    const float bv = ld(wt, (m - 1 + hf) * hp + unit);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(hf ? 0.0f : v[l32 + m - 1], bv, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(hf ? 0.0f : v[32 + l32 + m - 1], bv, acc[1], 0, 0, 0);
  };
  forward(es, we, site);
  constexpr int GB = FB > 0 ? FB : 1;
  f16v g[GB];
  f16v sdz[2];
  float grem = 0.0f, gw2 = 0.0f;
#pragma unroll
  for (int q = 0; q < GB; ++q) g[q] = f16v{0};
  sdz[0] = f16v{0};
  sdz[1] = f16v{0};
  double loss = 0.0;
  float gb2 = 0.0f;
  // g[fb] += (dZ rows of this wave's units)^T (window columns of v); rem: column 32 FB.
  // TAIL (fewer sites than a block): rows past the last site read zeros, so that an
  // Inf or NaN near the end does not meet their zero gradients.  Rows that a last
  // block shares with the one before it need no such care: what a zero gradient
  // meets there, the site's own row meets too.
  const int left = n - i0;
  auto backward = [&](const f16v (&dz)[2], const float* v, float& rem) {
    int lf = left;
    if (TAIL) asm volatile("" : "+s"(lf));   // the 32 row addresses are formed here, not kept in registers
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = 32 * bi + 8 * (e >> 2) + 4 * hf + (e & 3);
        const float* vr = !TAIL || row < lf ? v + row : zeros;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
          g[fb] = __builtin_amdgcn_mfma_f32_32x32x2f32(dz[bi][e], vr[32 * fb + l32], g[fb], 0, 0, 0);
        rem += dz[bi][e] * vr[32 * FB];
      }
  };
  for (int b = b0; b < be; ++b) {
    for (int q = tid; q < XS; q += nth) {
      const int j = i0 + q - w;
      xs[q] = j >= 0 && j < n ? x[(size_t)b * n + j] : 0.0f;
    }
    __syncthreads();
    f16v a[2] = {site[0], site[1]};
    forward(xs, wx, a);
    float v[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      a[q >> 4][q & 15] = tanhf(a[q >> 4][q & 15]);
      v[q] = a[q >> 4][q & 15] * w2c;
    }
    if (hp != h) {   // padding units add nothing, whatever their zero weights met
#pragma unroll
      for (int q = 0; q < 32; ++q) v[q] = unit < h ? v[q] : 0.0f;
    }
    if (TAIL) {
#pragma unroll
      for (int q = 0; q < 32; ++q)
        if (32 * (q >> 4) + 8 * ((q & 15) >> 2) + 4 * hf + (q & 3) >= left) a[q >> 4][q & 15] = 0.0f;
    }
    // sums over the 32 units: halve the values a lane holds with each exchange;
    // lane l32 ends with value l32.  The steps have constant indices: in a loop over
    // `off` some instances kept v as one 32-register vector with an index chain of
    // selects per access (forward, 64 states a workgroup: 0.99 ms, and now 0.18).
    auto halve = [&](auto step) {
      constexpr int off = decltype(step)::value;
      const bool up = (l32 & off) != 0;
#pragma unroll
      for (int q = 0; q < off; ++q) {
        const float keep = up ? v[q + off] : v[q], send = up ? v[q] : v[q + off];
        v[q] = keep + __shfl_xor(send, off, 64);
      }
    };
    halve(std::integral_constant<int, 16>{});
    halve(std::integral_constant<int, 8>{});
    halve(std::integral_constant<int, 4>{});
    halve(std::integral_constant<int, 2>{});
    halve(std::integral_constant<int, 1>{});
    ysum[wave][32 * (l32 >> 4) + 8 * ((l32 & 15) >> 2) + 4 * hf + (l32 & 3)] = v[0];
    __syncthreads();
    if (tid < kFusedSites) {
      float yv = 0.0f;
      for (int q = 0; q < (nth >> 6); ++q) yv += ysum[q][tid];
      yv += b2;
      const bool in = i0 + tid >= own && i0 + tid < n;
      const size_t row = (size_t)b * n + i0 + tid;
      if (!BWD) {
        if (in) y[row] = yv;
      } else {
        const double r = in ? (double)yv - (double)t[row] : 0.0;
        loss += r * r;
        const float d = (float)(scale * r);
        dys[tid] = d;
        gb2 += d;
      }
    }
    __syncthreads();
    if (BWD) {
#pragma unroll
      for (int q = 0; q < 32; ++q) {
        const int bi = q >> 4, e = q & 15;
        const float d = dys[32 * bi + 8 * (e >> 2) + 4 * hf + (e & 3)], av = a[bi][e];
        gw2 += av * d;
        const float dz = d * w2c * (1.0f - av * av);
        sdz[bi][e] += dz;
        a[bi][e] = dz;
      }
      backward(a, xs, grem);
      __syncthreads();   // xs is read: the next state may take its place
    }
  }
  if (!BWD) return;
  const int wg = blockIdx.y * gridDim.x + blockIdx.x;
  float* gp = gpart + (size_t)wg * ((size_t)h * k + 2 * h + 1);
  // accumulator of a weight block: row = unit, column = window column
  auto store = [&](int c0, float rem) {
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int un = wave * 32 + 8 * (e >> 2) + 4 * hf + (e & 3), f = 32 * fb + l32;
        if (un < h && f < m) gp[(size_t)un * k + c0 + f] = g[fb][e];
      }
    rem += __shfl_xor(rem, 32, 64);
    if (hf == 0 && unit < h && 32 * FB < m) gp[(size_t)unit * k + c0 + 32 * FB] = rem;
  };
  store(0, grem);
#pragma unroll
  for (int q = 0; q < GB; ++q) g[q] = f16v{0};
  grem = 0.0f;
  backward(sdz, es, grem);
  store(m, grem);
  float gu = 0.0f, gb1 = 0.0f;
#pragma unroll
  for (int q = 0; q < 32; ++q) {
    const int bi = q >> 4, e = q & 15;
    gu += sdz[bi][e] * us[32 * bi + 8 * (e >> 2) + 4 * hf + (e & 3)];
    gb1 += sdz[bi][e];
  }
  gu += __shfl_xor(gu, 32, 64);
  gb1 += __shfl_xor(gb1, 32, 64);
  gw2 += __shfl_xor(gw2, 32, 64);
  if (hf == 0 && unit < h) {
    gp[(size_t)unit * k + 2 * m] = gu;
    gp[(size_t)h * k + unit] = gb1;
    gp[(size_t)h * k + h + unit] = gw2;
  }
  if (tid < 64) {
    for (int off = 32; off > 0; off >>= 1) {
      loss += __shfl_xor(loss, off, 64);
      gb2 += __shfl_xor(gb2, off, 64);
    }
    if (tid == 0) {
      loss_part[wg] = loss;
      gp[(size_t)h * k + 2 * h] = gb2;
    }
  }
}

// grad[p] = sum over the workgroups' gradients (FP64, fixed order: four
// interleaved runs), and in workgroup 0 the loss.
__global__ __launch_bounds__(256) void k_mixer_reduce(const float* gpart, int nwg, size_t count, float* grad,
                                                      const double* loss_part, double inv, double* loss_out, int idx) {
  __shared__ double red[4][64];
  const size_t p = (size_t)blockIdx.x * 64 + (threadIdx.x & 63);
  const int q = threadIdx.x >> 6;
  double acc = 0.0;
  if (p < count)
#pragma unroll 8
    for (int z = q; z < nwg; z += 4) acc += (double)gpart[(size_t)z * count + p];
  red[q][threadIdx.x & 63] = acc;
  __syncthreads();
  if (q == 0 && p < count) grad[p] = (float)(red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x]);
  if (blockIdx.x == 0 && q == 1) {
    double l = 0.0;
    for (int z = threadIdx.x - 64; z < nwg; z += 64) l += loss_part[z];
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (threadIdx.x == 64) loss_out[idx] = l * inv;
  }
}

// The fused pass over B states; gradient and loss with t, outputs y without.
hipError_t launch_fused(const uint16_t* p16, int w, int h, const float* u, const float* en, int n, const float* x,
                        const float* t, int B, float* y, double* loss_part, float* gpart, hipStream_t s) {
  const int groups = fused_groups(n, B), per = (B + groups - 1) / groups;
  const dim3 grid((n + kFusedSites - 1) / kFusedSites, groups), block((h + 31) / 32 * 64);
  const double scale = 2.0 / ((double)B * n);
#define DMPT_FUSED(FB)                                                                                              \
  case FB:                                                                                                          \
    if (!t) hipLaunchKernelGGL((k_mixer_fused<FB, false, false>), grid, block, 0, s, p16, w, h, u, en, n, x, t, B, per, y, \
                               loss_part, gpart, scale);                                                            \
    else if (n >= kFusedSites) hipLaunchKernelGGL((k_mixer_fused<FB, true, false>), grid, block, 0, s, p16, w, h, u, en, n, \
                                                      x, t, B, per, y, loss_part, gpart, scale);                    \
    else hipLaunchKernelGGL((k_mixer_fused<FB, true, true>), grid, block, 0, s, p16, w, h, u, en, n, x, t, B, per, y,  \
                            loss_part, gpart, scale);                                                               \
    break;
  switch (fused_blocks(w)) {
    DMPT_FUSED(0)
    DMPT_FUSED(1)
    DMPT_FUSED(2)
    DMPT_FUSED(3)
    DMPT_FUSED(4)
    default: return hipErrorInvalidValue;
  }
#undef DMPT_FUSED
  return hipGetLastError();
}

}  // namespace

size_t mixer_param_count(int w, int h) { return (size_t)h * mixer_features(w) + 2 * h + 1; }

hipError_t mixer_diag(const float* m, int n, float* out, hipStream_t s) {
  hipLaunchKernelGGL(k_diag, dim3(blocks(n, 256)), dim3(256), 0, s, m, n, out);
  return hipGetLastError();
}

size_t mixer_scratch_floats(int n, int w, int h, int B) {
  const size_t rows = (size_t)B * n, k = mixer_features(w);
  // z, a, y, da, split partials of the weight gradients
  const size_t general = rows * k + rows * h + rows + rows * h + (size_t)kSplits * (h * k + h + 1);
  if (!fused_shape(w, h)) return general;
  // the fused pass: one gradient per workgroup.  A bound on fused_groups that does not
  // fall with B (the groups themselves do: 256 for B = 256, 129 for B = 257), since a
  // workspace sized for a batch serves the smaller ones too.
  const size_t ib = (n + kFusedSites - 1) / kFusedSites;
  const size_t groups = std::min<size_t>(B, std::max<size_t>(1, kFusedWGs / ib));
  return std::max(general, ib * groups * mixer_param_count(w, h));
}

// forward: y (B x n) for states x (B x n).  scratch: mixer_scratch_floats.
hipError_t mixer_forward(const uint16_t* p16, int w, int h, const float* u, const float* en, int n, const float* x,
                         int B, float* y, float* scratch, hipStream_t s) {
  if (use_fused(n, w, h, B, false)) return launch_fused(p16, w, h, u, en, n, x, nullptr, B, y, nullptr, nullptr, s);
  const int k = mixer_features(w);
  const size_t rows = (size_t)B * n;
  const uint16_t* w1 = p16;
  const uint16_t* b1 = w1 + (size_t)h * k;
  const uint16_t* w2 = b1 + h;
  const uint16_t* b2 = w2 + h;
  float* z = scratch;
  float* a = z + rows * k;
  hipLaunchKernelGGL(k_site_inputs, dim3(blocks(rows * k, 256)), dim3(256), 0, s, x, u, en, B, n, w, z);
  hipError_t e = gemm<float, uint16_t, false, true>(z, k, w1, k, a, h, (int)rows, h, k, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bias_tanh, dim3(blocks(rows * h, 256)), dim3(256), 0, s, a, b1, rows, h);
  e = gemm<float, uint16_t, false, false>(a, h, w2, 1, y, 1, (int)rows, 1, h, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bias1, dim3(blocks(rows, 256)), dim3(256), 0, s, y, b2, rows);
  return hipGetLastError();
}

constexpr int kMseBlocks = 256;

// loss (device double at loss_out[idx]) and gradient (FP32, packed layout).
hipError_t mixer_loss_grad(const uint16_t* p16, int w, int h, const float* u, const float* en, int n, const float* x,
                           const float* t, int B, float* scratch, double* part, float* grad, double* loss_out,
                           int idx, hipStream_t s) {
  const int k = mixer_features(w);
  const size_t rows = (size_t)B * n;
  if (use_fused(n, w, h, B, true)) {
    const int nwg = (n + kFusedSites - 1) / kFusedSites * fused_groups(n, B);
    hipError_t e = launch_fused(p16, w, h, u, en, n, x, t, B, nullptr, part, scratch, s);
    if (e != hipSuccess) return e;
    const size_t np = mixer_param_count(w, h);
    hipLaunchKernelGGL(k_mixer_reduce, dim3(blocks(np, 64)), dim3(256), 0, s, scratch, nwg, np, grad, part,
                       1.0 / (double)rows, loss_out, idx);
    return hipGetLastError();
  }
  float* z = scratch;
  float* a = z + rows * k;
  float* y = a + rows * h;
  float* da = y + rows;
  float* split = da + rows * h;
  hipError_t e = mixer_forward(p16, w, h, u, en, n, x, B, y, scratch, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mse, dim3(kMseBlocks), dim3(256), 0, s, y, t, rows, part);   // y := dY
  hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(64), 0, s, part, kMseBlocks, 1.0 / (double)rows, loss_out, idx);
  const uint16_t* w2 = p16 + (size_t)h * k + h;
  float* gw1 = grad;
  float* gb1 = gw1 + (size_t)h * k;
  float* gw2 = gb1 + h;
  float* gb2 = gw2 + h;
  // gw2 (h) = A^T dY ; gb2 = sum dY
  e = gemm_splitk<float, float, true, false>(a, h, y, 1, gw2, h, 1, (int)rows, split, s);
  if (e != hipSuccess) return e;
  e = colsum(y, rows, 1, gb2, split, s);
  if (e != hipSuccess) return e;
  // dA (rows x h) = dY w2^T (outer product), then dZ = dA (1 - A^2)
  e = gemm<float, uint16_t, false, false>(y, 1, w2, h, da, h, (int)rows, h, 1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_tanh_back, dim3(blocks(rows * h, 256)), dim3(256), 0, s, da, a, rows * h);
  // gW1 (h x k) = dZ^T Z ; gb1 = colsum(dZ)
  e = gemm_splitk<float, float, true, false>(da, h, z, k, gw1, h, k, (int)rows, split, s);
  if (e != hipSuccess) return e;
  e = colsum(da, rows, h, gb1, split, s);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t mixer_adam(float* p, uint16_t* p16, float* m, float* v, const float* g, size_t count, float lr,
                      int step, hipStream_t s) {
  const double beta1 = 0.9, beta2 = 0.999;
  const float c1 = (float)(1.0 / (1.0 - std::pow(beta1, step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow(beta2, step)));
  hipLaunchKernelGGL(k_adam, dim3(blocks(count, 256)), dim3(256), 0, s, p, p16, m, v, g, count, lr, (float)beta1,
                     (float)beta2, 1e-8f, c1, c2);
  return hipGetLastError();
}

hipError_t mixer_init(float* p, uint16_t* p16, int w, int h, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(k_init_params, dim3(blocks(mixer_param_count(w, h), 256)), dim3(256), 0, s, p, p16,
                     mixer_features(w), h, seed);
  return hipGetLastError();
}

// ---------------------------------------------------------------- SCF vectors

namespace {

// out[i] = c[i * ld + i]
__global__ void k_get_diag(const float* c, int n, size_t ld, double* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = c[(size_t)i * ld + i];
}

// W = diag(U_i s v_i) as a full n x n matrix (off-diagonal zeros written too).
__global__ void k_set_diag(float* w, int n, const float* u, const double* v, double s) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  const int i = (int)(e / n), j = (int)(e % n);
  w[e] = i == j ? (float)((double)u[i] * s * v[i]) : 0.0f;
}

// chi = s (a + b) (b may be null)
__global__ void k_combine(float* chi, const float* a, const float* b, double s, size_t n2) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n2) chi[e] = (float)(s * ((double)a[e] + (b ? (double)b[e] : 0.0)));
}

// One 1024-thread block: out[q] = x_q . y_q for q < nq pairs of n-vectors (FP64).
__global__ __launch_bounds__(1024) void k_dots(const double* const* xs, const double* const* ys, int nq, int n,
                                               double* out) {
  __shared__ double red[16];
  for (int q = 0; q < nq; ++q) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) acc += xs[q][i] * ys[q][i];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < 16; ++w) t += red[w];
      out[q] = t;
    }
    __syncthreads();
  }
}

// out = sum_q c_q x_q over nq vectors (coefficients on the device).
__global__ void k_lincomb(double* out, const double* const* xs, const double* c, int nq, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int q = 0; q < nq; ++q) acc += c[q] * xs[q][i];
  out[i] = acc;
}

// x = (float)(r * inv)
__global__ void k_to_float(float* x, const double* r, double inv, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = (float)(r[i] * inv);
}

// out = v + alpha r + scale y  (y FP32, may be null)
__global__ void k_step_vec(double* out, const double* v, const double* r, double alpha, const float* y,
                           double scale, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = v[i] + alpha * r[i] + (y ? scale * (double)y[i] : 0.0);
}

// r = f - v ; record (FP32 copies) when the pointers are set
__global__ void k_residual(double* r, const double* f, const double* v, int n, float* rec_v, float* rec_r) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  r[i] = f[i] - v[i];
  if (rec_v) rec_v[i] = (float)v[i];
  if (rec_r) rec_r[i] = (float)r[i];
}

// f = d_a + diag(cw) (cw may be null)
__global__ void k_fvec(double* f, const double* da, const float* cw, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) f[i] = da[i] + (cw ? (double)cw[(size_t)i * n + i] : 0.0);
}

// Training pairs of the learned mixer: for kept record row j = rows[b],
// x_b = sqrt(n) r_j / ||r_j||, t_b = sqrt(n) (v* - v_j - mix r_j) / ||r_j||
// (||r_j|| in FP64).  One workgroup per output row.
__global__ __launch_bounds__(256) void k_mixer_pairs(const float* v, const float* r, const float* vstar,
                                                     const int* rows, int n, float mix, float* x, float* t) {
  __shared__ double s_red[4];
  __shared__ double s_inv;
  const int j = rows[blockIdx.x];
  const float* rj = r + (size_t)j * n;
  const float* vj = v + (size_t)j * n;
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) acc += (double)rj[i] * (double)rj[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double nrm = sqrt((s_red[0] + s_red[1] + s_red[2] + s_red[3]) / (double)n);   // ||r|| / sqrt(n)
    s_inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
  }
  __syncthreads();
  const float inv = (float)s_inv;
  float* xb = x + (size_t)blockIdx.x * n;
  float* tb = t + (size_t)blockIdx.x * n;
  for (int i = threadIdx.x; i < n; i += 256) {
    xb[i] = rj[i] * inv;
    tb[i] = (vstar[i] - vj[i] - mix * rj[i]) * inv;
  }
}

// dst row b = src row perm[b] (rows of n floats).
__global__ __launch_bounds__(256) void k_gather_rows(const float* src, const int* perm, int n, float* dst) {
  const float* sr = src + (size_t)perm[blockIdx.x] * n;
  float* dr = dst + (size_t)blockIdx.x * n;
  for (int i = threadIdx.x; i < n; i += 256) dr[i] = sr[i];
}

}  // namespace

hipError_t mixer_pairs(const float* v, const float* r, const float* vstar, const int* rows, int nrows, int n,
                       float mix, float* x, float* t, hipStream_t s) {
  if (nrows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mixer_pairs, dim3(nrows), dim3(256), 0, s, v, r, vstar, rows, n, mix, x, t);
  return hipGetLastError();
}

hipError_t mixer_gather_rows(const float* src, const int* perm, int nrows, int n, float* dst, hipStream_t s) {
  if (nrows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rows, dim3(nrows), dim3(256), 0, s, src, perm, n, dst);
  return hipGetLastError();
}

hipError_t scf_get_diag(const float* c, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_get_diag, dim3(blocks(n, 256)), dim3(256), 0, s, c, n, (size_t)n, out);
  return hipGetLastError();
}
hipError_t scf_set_diag(float* w, int n, const float* u, const double* v, double spin, hipStream_t s) {
  hipLaunchKernelGGL(k_set_diag, dim3(blocks((size_t)n * n, 256)), dim3(256), 0, s, w, n, u, v, spin);
  return hipGetLastError();
}
hipError_t scf_combine(float* chi, const float* a, const float* b, double spin, size_t n2, hipStream_t s) {
  hipLaunchKernelGGL(k_combine, dim3(blocks(n2, 256)), dim3(256), 0, s, chi, a, b, spin, n2);
  return hipGetLastError();
}
hipError_t scf_dots(const double* const* xs, const double* const* ys, int nq, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_dots, dim3(1), dim3(1024), 0, s, xs, ys, nq, n, out);
  return hipGetLastError();
}
hipError_t scf_lincomb(double* out, const double* const* xs, const double* c, int nq, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_lincomb, dim3(blocks(n, 256)), dim3(256), 0, s, out, xs, c, nq, n);
  return hipGetLastError();
}
hipError_t scf_to_float(float* x, const double* r, double inv, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_to_float, dim3(blocks(n, 256)), dim3(256), 0, s, x, r, inv, n);
  return hipGetLastError();
}
hipError_t scf_step(double* out, const double* v, const double* r, double alpha, const float* y, double scale,
                    int n, hipStream_t s) {
  hipLaunchKernelGGL(k_step_vec, dim3(blocks(n, 256)), dim3(256), 0, s, out, v, r, alpha, y, scale, n);
  return hipGetLastError();
}
hipError_t scf_residual(double* r, const double* f, const double* v, int n, float* rec_v, float* rec_r,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_residual, dim3(blocks(n, 256)), dim3(256), 0, s, r, f, v, n, rec_v, rec_r);
  return hipGetLastError();
}
hipError_t scf_fvec(double* f, const double* da, const float* cw, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_fvec, dim3(blocks(n, 256)), dim3(256), 0, s, f, da, cw, n);
  return hipGetLastError();
}

}  // namespace dmpt
