// Device helpers shared by the kernels that read and write the tiled operand
// copies (dmpt_kernels.hip, dmpt_small.hip): formats, the split terms of
// Eq. doubleHalf, the layout of a copy and its stores.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dmpt_internal.h"
#include "sp2_rule.h"

namespace dmpt {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define LDS_AS __attribute__((address_space(3)))
#define GLB_AS __attribute__((address_space(1)))

// Bytes per LDS row per pipeline stage: 16 k values of FP32 / packed split-2
// (BF16 or FP16; 64 B = 4 slots of 16 B), 32 k values of plain BF16 (64 B),
// 16 k values of packed split-3 (96 B = 6 slots).
template <int PREC> struct Fmt {
  static constexpr int RB = PREC == kSplit3 ? 96 : 64;
  static constexpr int S = RB / 16;
  static constexpr int K = PREC == kBF16 ? 32 : 16;
};
// Format of the operand copy in HBM (the same as the staged one).
template <int PREC> struct Store { static constexpr int F = PREC; };

constexpr int RBLK = 128;   // rows per chunk of the tiled operand layout

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ unsigned short bf16_bits(float x) {
  return __builtin_bit_cast(unsigned short, (__bf16)x);   // round to nearest even
}
__device__ __forceinline__ float bf16_val(unsigned short b) {
  return __builtin_bit_cast(float, ((unsigned int)b) << 16);
}
__device__ __forceinline__ unsigned short f16_bits(float x) {
  return __builtin_bit_cast(unsigned short, (_Float16)x);   // round to nearest even, subnormals kept
}
__device__ __forceinline__ float f16_val(unsigned short b) { return (float)__builtin_bit_cast(_Float16, b); }
// Eq. doubleHalf with BF16 terms: part_0 = RNE(x), part_t = RNE(x - sum_{s<t} part_s).
template <int T>
__device__ __forceinline__ void split_terms(float x, unsigned short (&p)[T]) {
  float r = x;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    p[t] = bf16_bits(r);
    r = r - bf16_val(p[t]);
  }
}
// Eq. doubleHalf with FP16 terms on the scaled value: hi = RNE(x sc),
// lo = RNE(x sc - hi); sc is a power of two, x sc - hi is exact in FP32.
__device__ __forceinline__ void split_terms_h(float x, float sc, unsigned short (&p)[2]) {
  const float xs = x * sc;
  p[0] = f16_bits(xs);
  p[1] = f16_bits(xs - f16_val(p[0]));
}
template <int PREC> struct Terms {
  static constexpr int T = PREC == kSplit3 ? 3 : (PREC == kSplit2 || PREC == kSplitH) ? 2 : 1;
};
// The split terms of one element in the operand format F (sc: kSplitH scale).
template <int F>
__device__ __forceinline__ void split_for(float v, float sc, unsigned short (&p)[Terms<F>::T]) {
  if constexpr (F == kSplitH) split_terms_h(v, sc, p);
  else split_terms<Terms<F>::T>(v, p);
}

// Sum over the 64 lanes, in every lane: the butterfly over lane bits 5 .. 0.  Lane
// moves inside the vector unit (the halves and 16-lane rows swapped, rotations and
// permutations within a row): the same sum through LDS permutes took 0.27 us, this
// 0.05.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const u32x2 u = __builtin_bit_cast(u32x2, v);
  const u32x2 r = {(unsigned)__builtin_amdgcn_update_dpp(0, (int)u[0], CTRL, 0xf, 0xf, true),
                   (unsigned)__builtin_amdgcn_update_dpp(0, (int)u[1], CTRL, 0xf, 0xf, true)};
  return __builtin_bit_cast(double, r);
}
__device__ __forceinline__ double wave_sum(double v) {
  u32x2 u = __builtin_bit_cast(u32x2, v);
  auto lo = __builtin_amdgcn_permlane32_swap(u[0], u[0], false, false);
  auto hi = __builtin_amdgcn_permlane32_swap(u[1], u[1], false, false);
  v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
  u = __builtin_bit_cast(u32x2, v);
  lo = __builtin_amdgcn_permlane16_swap(u[0], u[0], false, false);
  hi = __builtin_amdgcn_permlane16_swap(u[1], u[1], false, false);
  v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
  v += dpp_move<0x128>(v);   // row_ror:8 = lane ^ 8
  v += dpp_move<0x124>(v);   // row_ror:4 = lane ^ 4 (the row now repeats every 8 lanes)
  v += dpp_move<0x4e>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_move<0xb1>(v);    // quad_perm [1, 0, 3, 2]
  return v;
}

// kSplitH: exponent s of the scale 2^s of a Y copy whose entries are bounded
// by bound * nrm (nrm a Frobenius norm): the largest s with bound * nrm * 2^s
// <= kYTarget, clamped to [-100, 100]; 0 for a zero or non-finite norm.
__device__ __forceinline__ int yscale_exp(double nrm, double bound) {
  const double b = bound * nrm;
  if (!(b > 0.0) || !(b < 1e300)) return 0;
  const int e = (int)floor(log2(kYTarget / b));
  return e < -100 ? -100 : e > 100 ? 100 : e;
}

// Frobenius norm of a matrix from its producer's partials (count of them in
// meta->nrm, at most cap = the allocated number), summed in a fixed order by
// wave 0 of the block (every block gets the same value); the result is
// broadcast through *s_out.
__device__ __forceinline__ double meta_norm(const MatMeta* m, int cap, double* s_out) {
  if (threadIdx.x < 64) {
    const int cnt = m->count < cap ? m->count : cap;
    double t = 0.0;
    for (int i = threadIdx.x; i < cnt; i += 64 * 16) {   // 16 loads in flight, added in order
      double u[16];
#pragma unroll
      for (int z = 0; z < 16; ++z) u[z] = i + 64 * z < cnt ? m->nrm[i + 64 * z] : 0.0;
#pragma unroll
      for (int z = 0; z < 16; ++z) t += u[z];
    }
    t = wave_sum(t);
    if (threadIdx.x == 0) *s_out = sqrt(t);
  }
  __syncthreads();
  return *s_out;
}

// Physical 16-byte slot of logical slot ls in LDS row r.  4 slots/row:
// XOR with (r/4)&3; 6 slots/row: XOR with (r/8)&1.  Either way 16 lanes that
// read one logical slot of 16 consecutive rows hit 16 distinct 4-bank groups.
template <int S>
__device__ __forceinline__ int phys_slot(int r, int ls) {
  if constexpr (S == 4) return ls ^ ((r >> 2) & 3);
  else return ls ^ ((r >> 3) & 1);
}
template <int S>
__device__ __forceinline__ int swz(int r, int ls) { return r * (S * 16) + 16 * phys_slot<S>(r, ls); }

// Byte offset of element (r, c), split term `part`, in the tiled operand copy.
// small: the small-size kernels' layout, blocks of 32 rows x one stage whose
// 16-byte pieces (8 columns of one term) lie in the order an MFMA operand load
// takes them: register q (term, or k16 step of plain BF16), k-group, row.
template <int PREC>
__device__ __forceinline__ size_t op_off(int r, int c, int part, int nst, int small = 0) {
  constexpr int RB = Fmt<PREC>::RB, S = Fmt<PREC>::S, K = Fmt<PREC>::K, T = Terms<PREC>::T;
  const int rr = r & (RBLK - 1);
  const int st = c / K, kk = c % K;
  if (small) {
    const int piece = PREC == kBF16 ? (kk >> 3) : 2 * part + (kk >> 3);
    return ((size_t)(r >> 5) * nst + st) * (size_t)(32 * RB) + 512 * piece + 16 * (r & 31) + (kk & 7) * 2;
  }
  const int ls = PREC == kBF16 ? (kk >> 3) : T * (kk >> 3) + part;
  return ((size_t)(r / RBLK) * nst + st) * (size_t)(RBLK * RB) + (size_t)rr * RB + 16 * phys_slot<S>(rr, ls) +
         (kk & 7) * 2;
}

template <int PREC>
__device__ __forceinline__ void store_split1(char* oop, int nst, int r, int c, float v, float sc) {
  constexpr int T = Terms<PREC>::T;
  unsigned short part[T];
  split_for<PREC>(v, sc, part);
#pragma unroll
  for (int t = 0; t < T; ++t) *(unsigned short*)(oop + op_off<PREC>(r, c, t, nst)) = part[t];
}

// Element offset of (r, c) in a padded FP32 matrix: row-major, or (tiled, the
// small-size kernels' layout) 32-row x 16-column blocks of 2 KB, block row by
// block row, each block's 16-byte pieces of 4 columns ordered by column group,
// then row: the 16 bytes a lane of an FP32 MFMA operand load takes lie next to
// its neighbour's, where rows of a power-of-two length share one L2 channel.
__device__ __forceinline__ size_t m_off(int tiled, int r, int c, int n_pad) {
  if (!tiled) return (size_t)r * n_pad + c;
  return ((size_t)(r >> 5) * (n_pad >> 4) + (c >> 4)) * 512 + ((c >> 2) & 3) * 128 + (r & 31) * 4 + (c & 3);
}

// Operand copy of 8 consecutive columns c0..c0+7 (c0 % 8 == 0) of row r, in
// the tiled layout: each split term of the group is one 16-byte slot.
template <int PREC>
__device__ __forceinline__ void store_group8_t(char* op, int nst, int r, int c0, const float (&v)[8], float sc, int small = 0) {
  constexpr int T = Terms<PREC>::T;
  unsigned short part[8][T];
#pragma unroll
  for (int e = 0; e < 8; ++e) split_for<PREC>(v[e], sc, part[e]);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = part[2 * e][t] | ((unsigned)part[2 * e + 1][t] << 16);
    *(u32x4*)(op + op_off<PREC>(r, c0, t, nst, small)) = w;
  }
}

template <bool WG>
__device__ __forceinline__ void region_sync() {
  if constexpr (WG) {
    __syncthreads();
  } else {   // one wave: its LDS accesses in order
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
}

// Epilogue of a general product (ProdArgs) on one TS x TS region of V at
// (gr0, gc0), whose product sums stand in T (row stride LS): NTH threads (a
// workgroup, or with WG false one wave).  sym: the region is stored at its
// mirror place too; a region on the diagonal keeps its upper triangle.
// Returns this thread's part of ||V||_F^2 over the region and its mirror.
template <int PREC, int TS, int LS, int NTH, bool WG, int SMALL>
__device__ __forceinline__ double prod_region(const ProdArgs& a, int k, LDS_AS float* T, int tid, int gr0, int gc0,
                                              bool sym, float alpha, float sc) {
  constexpr int V4 = TS / 4, V8 = TS / 8;
  const bool diag = sym && gr0 == gc0;
  const float* x = a.x ? a.x + (size_t)k * a.sx : nullptr;
  double sq = 0.0;
  constexpr int NX = (TS * V4 + NTH - 1) / NTH;
  f32x4 xv[NX];   // all of X's loads in flight at once
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    const int e = tid + z * NTH, r = SMALL ? e % TS : e / V4, c = 4 * (SMALL ? e / TS : e % V4);
    xv[z] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if (x && e < TS * V4) xv[z] = *(const f32x4*)(x + m_off(SMALL, gr0 + r, gc0 + c, a.n_pad));
  }
#pragma unroll
  for (int z = 0; z < NX; ++z) {
    const int e = tid + z * NTH, r = SMALL ? e % TS : e / V4, c = 4 * (SMALL ? e / TS : e % V4);
    if (e >= TS * V4) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (diag && r > c + q) continue;
      const float v = alpha * T[r * LS + c + q] + a.beta * xv[z][q];
      T[r * LS + c + q] = v;
      if (a.mo) sq += (sym && !(diag && r == c + q) ? 2.0 : 1.0) * (double)v * (double)v;
    }
  }
  region_sync<WG>();
  auto at = [&](bool mir, int r, int c) { return mir || (diag && r > c) ? T[c * LS + r] : T[r * LS + c]; };
  const bool two = sym && !diag;   // also the mirror region
  float* m = a.m ? a.m + (size_t)k * a.sm : nullptr;
  if (m || a.m2) {
#pragma unroll 4
    for (int e = tid; e < (two ? 2 : 1) * TS * V4; e += NTH) {
      const bool mir = e >= TS * V4;
      const int g = mir ? e - TS * V4 : e, r = SMALL ? g % TS : g / V4, c = 4 * (SMALL ? g / TS : g % V4);
      const int gr = (mir ? gc0 : gr0) + r, gc = (mir ? gr0 : gc0) + c;
      f32x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = at(mir, r, c + q);
      const size_t o = m_off(SMALL, gr, gc, a.n_pad);
      if (m) *(f32x4*)(m + o) = v;
      if (a.m2) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = a.g1 * v[q] + (gr == gc + q && gr < a.n ? a.g0 : 0.0f);
        *(f32x4*)(a.m2 + o) = v;
      }
    }
  }
  if constexpr (PREC != kFP32) {
    char* cp = a.c ? a.c + (size_t)k * a.sc : nullptr;
    if (cp || a.c2) {
      const int nst = a.n_pad / Fmt<PREC>::K;
      const float sc2 = PREC == kSplitH ? ldexpf(1.0f, a.ec2) : 1.0f;
#pragma unroll 2
      for (int e = tid; e < (two ? 2 : 1) * TS * V8; e += NTH) {
        const bool mir = e >= TS * V8;
        const int g = mir ? e - TS * V8 : e, r = SMALL ? g % TS : g / V8, c = 8 * (SMALL ? g / TS : g % V8);
        const int gr = (mir ? gc0 : gr0) + r, gc = (mir ? gr0 : gc0) + c;
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = at(mir, r, c + q);
        if (cp) store_group8_t<PREC>(cp, nst, gr, gc, v, sc, SMALL);
        if (a.c2) {
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = a.g1 * v[q] + (gr == gc + q && gr < a.n ? a.g0 : 0.0f);
          store_group8_t<PREC>(a.c2, nst, gr, gc, v, sc2, SMALL);
        }
      }
    }
  }
  return sq;
}

// Scale of the product sums (undoes the copies' exponents) and exponent of V's
// copy, for kSplitH; nrm: the norm behind `bound`.
__device__ __forceinline__ float prod_scale(const ProdArgs& a, int k) {
  const int ea = a.ma ? ((const MatMeta*)(a.ma + (size_t)k * a.sma))->scale : a.ea;
  const int eb = a.mb ? ((const MatMeta*)(a.mb + (size_t)k * a.smb))->scale : a.eb;
  return ldexpf(1.0f, -(ea + eb));
}

// The step controller's decision at launch k = a.step from the sums of the
// previous launch's partials: Tr X_k, ||X_k||_F^2 and eps_{k-1}.  Every
// workgroup evaluates it on the same FP64 numbers; the one with `record` set
// writes it to the control block.  Returns sigma_k (+1 / -1) or a stop code;
// *zskip: the sweep has stopped (ytol2).  `in` holds what the decision reads
// of the control block (ctl_read, which a caller can issue early).
struct CtlIn {
  int nonfinite, ystop;
  double e1, e2, e3;   // eps of X_{k-2}, X_{k-3}, X_{k-4}: recorded at rec[j]
};
__device__ __forceinline__ CtlIn ctl_read(const StepArgs& a) {
  const Ctl* c = a.ctl;
  const int k = a.step;
  return CtlIn{c->nonfinite, c->ystop, k >= 3 ? c->rec[k - 2].eps : 0.0, k >= 4 ? c->rec[k - 3].eps : 0.0,
               k >= 5 ? c->rec[k - 4].eps : 0.0};
}
__device__ __forceinline__ int step_decide(const StepArgs& a, const CtlIn& in, double tr, double sq, double eps,
                                           bool record, int* zskip) {
  Ctl* c = a.ctl;
  const int k = a.step;
  int code = 1, m = -1;   // m >= 0: the recursion ends with X_{m+1}
  if (in.nonfinite) {
    code = kDecideNonfinite;
    m = k - 1;
  } else {
    if (k >= 2) {
      // eps of X_{k-1} is this launch's
      if (sp2_should_stop(eps, in.e1, in.e2, in.e3, k - 2, a.n, a.min_iter, a.idem_tol, a.unit)) {
        code = kDecideStop;
        m = k - 2;
      } else if (k - 2 >= a.max_iter) {
        code = kDecideNotConverged;
        m = k - 2;
      }
    }
    if (m < 0) {
      if (!sp2_bounds_ok(tr, sq, a.n)) {
        code = kDecideBounds;
        m = k - 1;
      } else {
        code = sp2_sigma(tr, sq, a.nocc);
      }
    }
  }
  // Sweep stop (ytol2 > 0): the Z-jobs of this launch would form Y_{k+1}
  // from X_k; once X_{k-1} (the operand of Y_k) is within the tolerance
  // they are skipped here and in every later launch, and Y_k is the
  // result.  Every workgroup evaluates the same test on the same eps;
  // the recording workgroup writes k.
  int zs = 0;
  if (a.ytol2 > 0.0 && k >= 2 && m < 0) {
    zs = (in.ystop != 0 || eps <= a.ytol2) ? 1 : 0;
    if (zs && record && in.ystop == 0) c->ystop = k;
  }
  *zskip = zs;
  if (record) {
    c->rec[k].tr = tr;
    c->rec[k].sq = sq;
    if (k >= 2) c->rec[k - 1].eps = eps;
    c->rec[k].sigma = m < 0 ? code : 0;
    if (m >= 0) {
      c->m = m;
      c->code = code;
      __threadfence();
      c->done = 1;
    }
  }
  return m < 0 ? code : (code == kDecideStop ? 2 : code);
}

}  // namespace dmpt
