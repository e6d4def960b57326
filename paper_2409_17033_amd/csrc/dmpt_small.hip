// gfx950 kernels of the matrix products at small sizes: the same SP2 /
// susceptibility step and general product as dmpt_kernels.hip on square tiles
// of 64 (or 32) with the K range split over the waves of a workgroup.
//
// The 256 x 128 tiles of the large-size kernels leave most of the chip idle
// when the matrix is small: n = 1000 has 20 of them per product on 256 CUs,
// and a launch then takes as long as one tile's serial K loop.  Here a
// workgroup owns one TS x TS tile and each of its waves forms the whole tile
// over its own part of the K range, so a tile's loop is NWV times shorter and
// there are 8 times as many tiles.  Such waves share no operand bytes (different
// k), so operands go straight from memory to registers: no LDS ring, no barrier in
// the loop, D stages in flight.  (FP32 64 x 64 tiles, whose waves keep FP64 sums
// beside their accumulators: a wave forms half of the tile's rows, and two waves read
// the same columns' operands.)  The partial sums meet in LDS (added in
// FP64, in wave order), and the workgroup runs the tile's epilogue.
//
// What bounds it, and what it measured (one step of one observable, us; the
// 256 x 128 tiles before): n = 128 FP32 77 -> 7.8, of which the chain of a few
// dependent memory round trips (operands and partials, the current matrix, the
// stores) and the launch; n = 1000 FP32 248 -> 51, FP16 split 86 -> 27; n = 2048
// FP32 562 -> 276, FP16 split 162 -> 114.  At n = 128 the controller's sums and its
// decision took 2.3 of them; with the sums inside the vector unit (wave_sum) and the
// decision beside the main loop the whole solve went from 0.65 to 0.58 ms (four waves
// a workgroup included).  From n = 1000 on the operand loads
// bound the split formats (n = 2048: 0.9 GB of operands a launch; the same loop
// without its MFMAs takes as long) and the FP32 MFMAs the FP32 ones (0.6 of
// their peak at n = 2048).  Loads in the order of the 128-row chunks of the
// large-size kernels (half of each 128-byte line per instruction) ran at 14.8,
// in the layout here at 22 TB/s; FP32 rows of a row-major matrix slower still.
//
// n_pad is a multiple of 64 on this path, and the FP32 masters and operand
// copies are laid out for these loads (m_off, op_off in dmpt_device.h).
#include <hip/hip_runtime.h>

#include "dmpt_device.h"
#include "dmpt_internal.h"
#include "dmpt_tiles.h"
#include "sp2_rule.h"

namespace dmpt {

namespace {

// ---------------------------------------------------------------- operand loads and products

// 16-byte operand registers of one stage: Q per 32 rows of A and of B.
template <int PREC> struct SFmt {
  static constexpr int Q = PREC == kSplit3 ? 3 : 2;
  static constexpr int D = PREC == kFP32 ? 4 : PREC == kSplit3 ? 2 : 3;   // stages in registers
  static constexpr int BLK = 32 * Fmt<PREC>::RB;   // bytes of a 32-row block of one stage
};
template <int PREC, int BA, int B> struct SOps { u32x4 a[BA][SFmt<PREC>::Q], b[B][SFmt<PREC>::Q]; };

// Byte offset of row r0 (a multiple of 32), stage 0 of an operand copy.
template <int PREC>
__device__ __forceinline__ size_t panel_off(int r0, int n_pad) { return (size_t)r0 * n_pad * operand_bytes(PREC); }

// One stage's operands: 32-row group i of a panel starts i * rstep bytes on;
// within a group's block register q of lane l is the 16 bytes at 1024 q + 16 l
// (row l % 32; split: k-group l / 32 of term q; BF16: k16 step q; FP32: columns
// 8 q + 4 (l / 32), the same k permutation on A and B).
template <int PREC, int BA, int B>
__device__ __forceinline__ void s_load(SOps<PREC, BA, B>& o, const char* pa, const char* pb, size_t rstep,
                                       uint32_t off) {
#pragma unroll
  for (int i = 0; i < BA; ++i)
#pragma unroll
    for (int q = 0; q < SFmt<PREC>::Q; ++q) o.a[i][q] = *(const u32x4*)(pa + i * rstep + q * 1024 + off);
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int q = 0; q < SFmt<PREC>::Q; ++q) o.b[i][q] = *(const u32x4*)(pb + i * rstep + q * 1024 + off);
}

// acc[i][j] += A_i B_j^T for one stage; the products and their order are those
// of the large-size kernels (split-3: mm, hl, lh, hm, mh, hh; two terms: hl, lh, hh).
// The blocks are taken in the order F, F + 1, ... (FP32 flushes block F after it).
template <int PREC, int BA, int B, int F>
__device__ __forceinline__ void s_mma(const SOps<PREC, BA, B>& o, f32x16 (&acc)[BA][B]) {
#pragma unroll
  for (int t = 0; t < BA * B; ++t) {
    const int blk = (F + t) % (BA * B), i = blk / B, j = blk % B;
    f32x16 c = acc[i][j];
    if constexpr (PREC == kFP32) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4 x = __builtin_bit_cast(f32x4, o.a[i][q]), y = __builtin_bit_cast(f32x4, o.b[j][q]);
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], c, 0, 0, 0);
      }
    } else if constexpr (PREC == kSplitH) {
      constexpr int pa[3] = {0, 1, 0}, pb[3] = {1, 0, 0};
#pragma unroll
      for (int q = 0; q < 3; ++q)
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, o.a[i][pa[q]]),
                                                   __builtin_bit_cast(f16x8, o.b[j][pb[q]]), c, 0, 0, 0);
    } else {
      constexpr int np = PREC == kSplit3 ? 6 : PREC == kSplit2 ? 3 : 2;
      constexpr int pa3[6] = {1, 0, 2, 0, 1, 0}, pb3[6] = {1, 2, 0, 1, 0, 0};
      constexpr int pa2[3] = {0, 1, 0}, pb2[3] = {1, 0, 0};
#pragma unroll
      for (int q = 0; q < np; ++q) {
        const int pa = PREC == kSplit3 ? pa3[q] : PREC == kSplit2 ? pa2[q % 3] : q;
        const int pb = PREC == kSplit3 ? pb3[q] : PREC == kSplit2 ? pb2[q % 3] : q;
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o.a[i][pa]),
                                                    __builtin_bit_cast(bf16x8, o.b[j][pb]), c, 0, 0, 0);
      }
    }
    acc[i][j] = c;
  }
}

// W waves: KP parts of the K range x WR row parts of the tile.  FP32 keeps
// FP64 partial sums beside its accumulators: at TS = 64 a wave takes 32 rows.
template <int PREC, int B, int W> struct SGeo {
  static constexpr int NWV = W, NTH = NWV * 64;
  static constexpr int WR = PREC == kFP32 ? B : 1, KP = NWV / WR, BA = B / WR;
  static constexpr int TS = 32 * B, LS = TS + 1;
  using P = typename std::conditional<PREC == kFP32, double, float>::type;
  static constexpr int SUMS = KP * B * B * 16 * 64 * (int)sizeof(P);
  static constexpr int PART = SUMS > TS * LS * 8 ? SUMS : TS * LS * 8;   // the tile (FP64 in a fold) takes the sums' place
  static constexpr int VX = (TS * TS / 4 + NTH - 1) / NTH;   // 16-byte pieces of the tile per thread
};

// This wave's part of the tile sum over stages [0, nst) of the K stream: stages
// below spass come from panels (a0, b0), the rest from (a1, b1).  Adds the
// waves' sums in `part` and leaves the tile (times the scales) there, row stride LS.
// Two-level accumulation as in the large-size kernels: FP32 operands go into
// FP64 sums every 4 stages, the split formats into a second FP32 level every
// 4 x flush stages (within the wave's range); the waves' sums add in FP64.
// kr, kc: the tile's rows and columns in units of 32 (32 x 32 tiles).
// fold: the tile of P + P^T (a diagonal tile of Z from Y X alone), still in FP64.
// ov runs while the first loads are in flight (false: leave, in every thread
// alike); pre runs before the partial sums are exchanged.
template <int PREC, int B, int W, class Ov, class Pre>
__device__ __forceinline__ bool tile_sum(const char* a0, const char* b0, const char* a1, const char* b1, int spass,
                                         int nst, int n_pad, int flush, int kr, int kc, float scale, float scale2, bool fold,
                                         LDS_AS char* part_, int wave, int lane, Ov ov, Pre pre) {
  using G = SGeo<PREC, B, W>;
  constexpr int D = SFmt<PREC>::D, BA = G::BA, NB = BA * B;
  const int h = lane >> 5, l32 = lane & 31;
  const int kp = wave / G::WR, wr = wave % G::WR;
  const size_t step_b = SFmt<PREC>::BLK, rstep = (size_t)32 * n_pad * operand_bytes(PREC);
  const uint32_t off = 16u * (uint32_t)lane;
  // FP32 ranges begin with a multiple of 4 stages (their chains end at fixed columns, see
  // below): of two ranges the first takes the odd pair; four of them, of fewer stages
  // each, may begin anywhere, and the loop passes over the stages before.
  constexpr bool PASS = PREC == kFP32 && (NB == 1 || G::KP > 2);
  int per = (nst + G::KP - 1) / G::KP;
  if (PREC == kFP32 && !PASS) per = (per + 3) & ~3;
  const int s0 = kp * per;
  const int cnt = s0 >= nst ? 0 : (nst - s0 < per ? nst - s0 : per);
  const size_t arow = (size_t)(wr * BA) * rstep;
  auto load = [&](SOps<PREC, BA, B>& o, int s) {   // past the end: the last stage again (never multiplied)
    const int sc = s < nst ? s : nst - 1;
    const bool first = sc < spass;
    const size_t ko = (size_t)(first ? sc : sc - spass) * step_b;
    s_load<PREC, BA, B>(o, (first ? a0 : a1) + ko + arow, (first ? b0 : b1) + ko, rstep, off);
  };
  SOps<PREC, BA, B> o[D];
  f32x16 acc[BA][B];
#pragma unroll
  for (int q = 0; q < NB; ++q) acc[q / B][q % B] = f32x16{0};
  const int skip = PASS ? s0 & 3 : 0, t0 = s0 - skip;
#pragma unroll
  for (int d = 0; d < D - 1; ++d) load(o[d], t0 + d);
  __builtin_amdgcn_sched_barrier(0);
  if (!ov()) return false;
  LDS_AS typename G::P* part = (LDS_AS typename G::P*)part_;
  const int pbase = (kp * B * B + wr * NB) * 16;   // this wave's first register row of the exchange
  if constexpr (PREC == kFP32) {
    double td[NB][16];
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int e = 0; e < 16; ++e) td[q][e] = 0.0;
    // Each block goes into its FP64 sum once in 4 stages, so that no FP32 chain is longer
    // (64 columns).  Where the chains end matters: X and Y have their largest entries
    // on and near the diagonal, so a tile's largest terms are those of its own rows'
    // and columns' k range, and every addition after them in their chain rounds at
    // their size.  So the chains end at fixed columns, whatever stage a wave's range begins
    // with.  Two blocks of columns a wave: each after its own 32 columns.  One (32 x 32 tiles): after every
    // other 32 columns, the tile's own among them, and after its rows'.  Ended every 4
    // stages of a wave's range instead, errors in D and chi were 1.1 - 1.5 times these
    // (FP32, n = 128 - 1100).
    static_assert(NB == 1 || NB == 2, "FP32 waves take one or two blocks");
#define DMPT_SSTAGE(K)                                                              \
  {                                                                                 \
    load(o[((K) + D - 1) % D], t0 + s + (K) + D - 1);                               \
    __builtin_amdgcn_sched_barrier(0);                                              \
    if ((!PASS || s + (K) >= skip) && s + (K) < cnt + skip) {                       \
      constexpr int blk = (K) * NB / 4;                                             \
      s_mma<PREC, BA, B, blk>(o[K], acc);                                           \
      bool end = ((K) & 1) != 0;                                                    \
      if constexpr (NB == 1 && ((K) & 1) != 0) {                                    \
        const int t = t0 + s + (K), c = (t < spass ? t : t - spass) >> 1;           \
        end = ((c ^ kc) & 1) == 0 || c == kr;                                       \
      }                                                                             \
      if (end) {                                                                    \
        _Pragma("unroll") for (int e = 0; e < 16; ++e) td[blk][e] += (double)acc[blk / B][blk % B][e]; \
        acc[blk / B][blk % B] = f32x16{0};                                          \
      }                                                                             \
    }                                                                               \
  }
    for (int s = 0; s < cnt + skip; s += 4) {
      DMPT_SSTAGE(0)
      DMPT_SSTAGE(1)
      DMPT_SSTAGE(2)
      DMPT_SSTAGE(3)
    }
#undef DMPT_SSTAGE
    pre();
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int e = 0; e < 16; ++e) part[(pbase + q * 16 + e) * 64 + lane] = td[q][e] + (double)acc[q / B][q % B][e];
  } else {
    f32x16 tot[BA][B];
#pragma unroll
    for (int q = 0; q < NB; ++q) tot[q / B][q % B] = f32x16{0};
    const int fl = flush > 0 ? 4 * flush : 1 << 30;
    int since = 0;
    for (int s = 0; s < cnt; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(o[(d + D - 1) % D], s0 + s + d + D - 1);
        __builtin_amdgcn_sched_barrier(0);
        if (s + d < cnt) {
          s_mma<PREC, BA, B, 0>(o[d], acc);
          if (++since == fl) {
            since = 0;
#pragma unroll
            for (int q = 0; q < NB; ++q) {
              tot[q / B][q % B] += acc[q / B][q % B];
              acc[q / B][q % B] = f32x16{0};
            }
          }
        }
      }
    }
    pre();
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int e = 0; e < 16; ++e) part[(pbase + q * 16 + e) * 64 + lane] = tot[q / B][q % B][e] + acc[q / B][q % B][e];
  }
  __syncthreads();
  // register e of a 32 x 32 block: row 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32
  constexpr int PER = B * B * 16 / G::NWV;
  auto row = [&](int idx) { return ((idx >> 4) / B) * 32 + 8 * ((idx & 15) >> 2) + 4 * h + (idx & 3); };
  auto col = [&](int idx) { return ((idx >> 4) % B) * 32 + l32; };
  double v[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int idx = wave * PER + k;
    v[k] = 0.0;
#pragma unroll
    for (int w = 0; w < G::KP; ++w) v[k] += (double)part[(w * B * B * 16 + idx) * 64 + lane];
  }
  __syncthreads();   // the sums are read: the tile takes their place
  if (fold) {
    LDS_AS double* T = (LDS_AS double*)part_;
#pragma unroll
    for (int k = 0; k < PER; ++k) T[row(wave * PER + k) * G::LS + col(wave * PER + k)] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) v[k] += T[col(wave * PER + k) * G::LS + row(wave * PER + k)];
    __syncthreads();
  }
  LDS_AS float* T = (LDS_AS float*)part_;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    float f = (float)v[k];
    f *= scale;
    f *= scale2;
    T[row(wave * PER + k) * G::LS + col(wave * PER + k)] = f;
  }
  return true;
}

// This thread's part of the sum of a matrix's norm partials, four loads in flight.
template <int NTH>
__device__ __forceinline__ double meta_part(const MatMeta* m, int cap, int tid) {
  const int cnt = m->count < cap ? m->count : cap;
  double s = 0.0;
  for (int q = tid; q < cnt; q += 4 * NTH) {
    double u[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) u[z] = q + z * NTH < cnt ? m->nrm[q + z * NTH] : 0.0;
#pragma unroll
    for (int z = 0; z < 4; ++z) s += u[z];
  }
  return s;
}

// ---------------------------------------------------------------- step kernel

// One SP2 / sweep step (see the step kernel of dmpt_kernels.hip): workgroup =
// one tile of Z = Y_n X_n + X_n Y_n (nz observables, first: twice the work) or
// of P = X_n X_n (with_p).  The controller's reduction of the previous
// launch's partials overlaps the main loop; the decision is needed only by
// the epilogue, which every workgroup reaches or leaves together.  The tile's
// partials go to entry `slot` of its matrix's `slots` (next: the one after it is 0).
template <int PREC, int B, int W, bool MIX>
__device__ __forceinline__ void small_job(const StepArgs& a, const int kind, const int obs, const int ti, const int tj,
                                          const int slot, const bool next, const int slots, const bool halve,
                                          LDS_AS char* part,
                                          double* s_ctl, double* s_red, int* s_code) {
  using G = SGeo<PREC, B, W>;
  LDS_AS float* T = (LDS_AS float*)part;
  constexpr int TS = G::TS, LS = G::LS, NTH = G::NTH, V4 = TS / 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int spass = a.n_pad / Fmt<PREC>::K;
  const bool zk = kind == kJobZ;
  const bool diag = ti == tj;
  const bool fold = zk && diag && halve;   // Z's diagonal tile as Y X and its transpose
  const int nst = zk && !fold ? 2 * spass : spass;

  const char* xop = (const char*)(MIX && zk ? a.x_in.op2 : a.x_in.op);
  const char* yop = (const char*)a.y_in.op + obs * a.y_in.stride_op;
  // kSplitH: products scaled by 2^(s_a + s_b), outputs by 2^s_out (Z: from ||Y_n||_F)
  float usc = 1.0f, sc_out = 1.0f;
  int s_out = 0;
  if constexpr (PREC == kSplitH) {
    if (zk) {
      usc = ldexpf(1.0f, -(kXScaleExp + ((const MatMeta*)(a.y_in.meta + obs * a.y_in.stride_op))->scale));
    } else {
      usc = ldexpf(1.0f, -2 * kXScaleExp);
      s_out = kXScaleExp;
    }
  }
  // while the first operands are on their way: leave after the stop, and the
  // FP64 sums (lane-strided, fixed order) of the controller's partials and of ||Y_n||^2
  auto ov = [&]() {
    if constexpr (PREC == kSplitH) {
      if (zk) {
        const MatMeta* mi = (const MatMeta*)(a.y_in.meta + obs * a.y_in.stride_op);
        const double s = wave_sum(meta_part<NTH>(mi, meta_entries(a.n_pad), tid));
        if (lane == 0) s_red[wave] = s;
      }
    }
    if (!a.decide) return true;
    // everything the decision reads is asked for at once
    const CtlIn ci = ctl_read(a);
    const int done = a.ctl->done;
    double tr = 0.0, sq = 0.0, eps = 0.0;
    for (int q = tid; q < a.nparts; q += 4 * NTH) {
      Part p[4];
#pragma unroll
      for (int z = 0; z < 4; ++z) p[z] = q + z * NTH < a.nparts ? a.part_in[q + z * NTH] : Part{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        tr += p[z].tr;
        sq += p[z].sq;
        eps += p[z].eps;
      }
    }
    tr = wave_sum(tr);
    sq = wave_sum(sq);
    eps = wave_sum(eps);
    if (lane == 0) {
      s_ctl[3 * wave] = tr;
      s_ctl[3 * wave + 1] = sq;
      s_ctl[3 * wave + 2] = eps;
    }
    // sweep stop (ytol2): recorded by an earlier launch, or by this one, whose Z
    // tiles are then dropped either way.  One thread's reading counts, so that the
    // workgroup leaves as a whole.
    if (tid == 0) s_code[2] = done || (zk && a.ytol2 > 0.0 && ci.ystop != 0) ? 1 : 0;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the operand loads stay in flight
    if (s_code[2]) return false;
    // the first wave decides while the others start their loop
    if (tid == 0) {
      tr = sq = eps = 0.0;
      for (int w = 0; w < G::NWV; ++w) {
        tr += s_ctl[3 * w];
        sq += s_ctl[3 * w + 1];
        eps += s_ctl[3 * w + 2];
      }
      int zs = 0;
      s_code[0] = step_decide(a, ci, tr, sq, eps, blockIdx.x == gridDim.x - 1, &zs);
      s_code[1] = zs;
    }
    return true;
  };
  // this thread's pieces of the current matrix, for the update
  const float* cur = zk ? a.y_in.f32 + obs * a.y_in.stride_f32 : a.x_in.f32;
  const int gr0 = ti * TS, gc0 = tj * TS;
  f32x4 xc[G::VX];
  auto pre = [&]() {
    if (zk && !a.decide && !a.sigma_src && a.fixed_sigma > 0) return;   // not read
#pragma unroll
    for (int q = 0; q < G::VX; ++q) {
      const int e = tid + q * NTH;
      if (TS * V4 % NTH == 0 || e < TS * V4) xc[q] = *(const f32x4*)(cur + m_off(1, gr0 + e % TS, gc0 + 4 * (e / TS), a.n_pad));
    }
  };
  const size_t rI = panel_off<PREC>(ti * TS, a.n_pad), rJ = panel_off<PREC>(tj * TS, a.n_pad);
  const int fl = MIX && zk && a.flush_z > 0 ? a.flush_z : a.flush;
  if (!tile_sum<PREC, B, W>((zk ? yop : xop) + rI, xop + rJ, xop + rI, yop + rJ, spass, nst, a.n_pad, fl, ti, tj, usc,
                         a.oscale != 0.0f ? a.oscale : 1.0f, fold, part, wave, lane, ov, pre))
    return;
  if constexpr (PREC == kSplitH) {
    if (zk) {   // s_red was written before tile_sum's barrier
      double s = 0.0;
      for (int w = 0; w < G::NWV; ++w) s += s_red[w];
      s_out = yscale_exp(sqrt(s), kYBound);
    }
    sc_out = ldexpf(1.0f, s_out);
  }
  __syncthreads();
  int sigma;
  if (a.decide) {
    sigma = s_code[0];
    if (!(sigma == 1 || sigma == -1) || (zk && s_code[1])) return;
  } else {
    sigma = a.sigma_src ? a.sigma_src[a.step].sigma : a.fixed_sigma;
  }

  // epilogue: sigma-update in T, then rows, mirror rows and operand copies
  float* o32 = zk ? a.y_out.f32 + obs * a.y_out.stride_f32 : a.x_out.f32;
  char* oop = zk ? (char*)a.y_out.op + obs * a.y_out.stride_op : (char*)a.x_out.op;
  char* oop2 = nullptr;
  if constexpr (MIX) {
    char* o2 = (char*)(zk ? a.y_out.op2 : a.x_out.op2);
    oop2 = o2 ? o2 + (zk ? obs * a.y_out.stride_op : 0) : nullptr;
  }
  char* hop = !zk && a.hist ? a.hist + (size_t)(a.step + 1) * a.hist_stride : nullptr;
  const bool wsplit = a.write_split && PREC != kFP32;
  double tr = 0.0, sq = 0.0, ep = 0.0;
#pragma unroll
  for (int q = 0; q < G::VX; ++q) {
    const int e = tid + q * NTH;
    if (TS * V4 % NTH != 0 && e >= TS * V4) break;
    const int r = e % TS, c = 4 * (e / TS);
    const f32x4 x = xc[q];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (diag && r > c + k) continue;   // a diagonal tile keeps its upper triangle and mirrors it
      const float p = T[r * LS + c + k];
      const float v = sigma > 0 ? p : 2.0f * x[k] - p;
      T[r * LS + c + k] = v;
      const double w = diag && r == c + k ? 1.0 : 2.0;
      if (!zk) {
        const double d = x[k] - p;         // X_n - X_n^2
        if (diag && r == c + k) tr += v;
        sq += w * (double)v * (double)v;
        ep += w * d * d;
      } else if constexpr (PREC == kSplitH) {
        sq += w * (double)v * (double)v;
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < TS * V4; e += NTH) {
    const int r = e % TS, c = 4 * (e / TS);
    f32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = diag && r > c + k ? T[(c + k) * LS + r] : T[r * LS + c + k];
    *(f32x4*)(o32 + m_off(1, gr0 + r, gc0 + c, a.n_pad)) = v;
    if (!diag) {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = T[(c + k) * LS + r];
      *(f32x4*)(o32 + m_off(1, gc0 + r, gr0 + c, a.n_pad)) = v;
    }
  }
  if (wsplit || hop) {
    const int nstp = a.n_pad / Fmt<PREC>::K, nsth = a.n_pad / Fmt<kBF16>::K;
    constexpr int V8 = TS / 8;
    const int groups = diag ? TS * V8 : 2 * TS * V8;
    for (int e = tid; e < groups; e += NTH) {
      const bool mir = e >= TS * V8;
      const int g = mir ? e - TS * V8 : e;
      const int r = g % TS, c = 8 * (g / TS);
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = mir || (diag && r > c + k) ? T[(c + k) * LS + r] : T[r * LS + c + k];
      const int gr = (mir ? gc0 : gr0) + r, gc = (mir ? gr0 : gc0) + c;
      if (wsplit) {
        if constexpr (PREC != kFP32) store_group8_t<PREC>(oop, nstp, gr, gc, v, sc_out, 1);
        if constexpr (MIX) {
          if (oop2) store_group8_t<kSplit2>(oop2, nstp, gr, gc, v, 1.0f, 1);
        }
      }
      if (hop) store_group8_t<kBF16>(hop, nsth, gr, gc, v, 1.0f, 1);
    }
  }
  if (!zk || PREC == kSplitH) {
    sq = wave_sum(sq);
    if (!zk) {
      tr = wave_sum(tr);
      ep = wave_sum(ep);
    }
    if (lane == 0) {
      s_ctl[3 * wave] = tr;
      s_ctl[3 * wave + 1] = sq;
      s_ctl[3 * wave + 2] = ep;
    }
    __syncthreads();
    if (tid == 0) {
      Part p = {0.0, 0.0, 0.0, 0.0};
      for (int w = 0; w < G::NWV; ++w) {
        p.tr += s_ctl[3 * w];
        p.sq += s_ctl[3 * w + 1];
        p.eps += s_ctl[3 * w + 2];
      }
      if (!zk) {
        a.part_out[slot] = p;
        if (next) a.part_out[slot + 1] = Part{0.0, 0.0, 0.0, 0.0};
      } else {
        MatMeta* mo = (MatMeta*)(a.y_out.meta + obs * a.y_out.stride_op);
        mo->nrm[slot] = p.sq;
        if (next) mo->nrm[slot + 1] = 0.0;
        if (slot == 0) {
          mo->scale = s_out;
          mo->count = slots;
        }
      }
    }
  }
}

// Job b of a kind (small_place).
template <int PREC, int B, int W, bool MIX>
__device__ __forceinline__ void small_jobs(const StepArgs& a, const int kind, int b, const int whole, const bool quarter, const bool spread,
                                           LDS_AS char* part, double* s_ctl, double* s_red, int* s_code) {
  const SmallPlace p = small_place(a.n_pad, 32 * B, b, whole, quarter, spread);
  if (p.none) return;
  small_job<PREC, B, W, MIX>(a, kind, p.obs, p.ti, p.tj, p.slot, p.next, p.slots, spread, part, s_ctl, s_red, s_code);
}

// Workgroups: the first zw of the nz observables' Z tiles, the others in quarters, the
// first pw of the P tiles, the others in quarters (B = 2; small_split).
template <int PP, int PZ, int B, int W>
__global__ __launch_bounds__((W * 64)) __attribute__((amdgpu_waves_per_eu((B == 1 ? 4 : 2), (B == 1 ? 4 : 2))))
void k_step_small(StepArgs a, int nz, int zw, int pw) {
  using G = SGeo<PP, B, W>;
  constexpr int PART = G::PART > SGeo<PZ, B, W>::PART ? G::PART : SGeo<PZ, B, W>::PART;
  __shared__ __attribute__((aligned(1024))) char part_[PART];
  __shared__ double s_ctl[3 * 8];
  __shared__ double s_red[8];
  __shared__ int s_code[3];
  LDS_AS char* part = (LDS_AS char*)part_;
  const int nt = a.n_pad / G::TS, zt = nz * (nt * (nt + 1) / 2);
  const int zq = 4 * (zt - zw);
  const int b = blockIdx.x;
  constexpr bool MIX = PP != PZ;
  if (b < zw) small_jobs<PZ, B, W, MIX>(a, kJobZ, b, zw, false, nz <= 1, part, s_ctl, s_red, s_code);
  else if (b >= zw + zq && b < zw + zq + pw)
    small_jobs<PP, B, W, MIX>(a, kJobP, b - zw - zq, pw, false, nz <= 1, part, s_ctl, s_red, s_code);
  else if constexpr (B == 2 && W == 4) {
    if (b < zw + zq) small_jobs<PZ, 1, W, MIX>(a, kJobZ, b - zw, zw, true, nz <= 1, part, s_ctl, s_red, s_code);
    else small_jobs<PP, 1, W, MIX>(a, kJobP, b - zw - zq - pw, pw, true, nz <= 1, part, s_ctl, s_red, s_code);
  }
}

// Waves of a tile's workgroup: four, so that several workgroups share a CU (64 KB of
// sums at most, two to four of them) and one's prologue and epilogue run under the
// other's loop.  With eight a tile's own loop is shorter, but the sums cost more:
// whole solve, ms, eight / four waves on 32 x 32 tiles: n = 128 FP32 0.61 / 0.58, n =
// 700 1.14 / 1.03, n = 1000 FP16 split 1.44 / 1.32.  Eight on 64 x 64 tiles in FP32
// only where the tiles fill the chip once and a bit: there the few extra ones would
// double up on some CUs for the whole launch, while one workgroup a CU leaves them to
// the CUs that finish first: n = 1000 (272 tiles) 1.99 against 2.41 with four, n =
// 1050 (306) 2.23 / 2.76, n = 1100 (342) 2.74 / 2.67.
inline bool eight_waves(int grid) { return grid > 256 && grid <= 320; }

}  // namespace

hipError_t launch_step_small(int prec, int ts, const StepArgs& args, int nz, int with_p, hipStream_t s) {
  if (args.n_pad <= 0 || args.n_pad % 64 != 0 || (ts != 32 && ts != 64) || (args.decide && !with_p))
    return hipErrorInvalidValue;
  const SmallSplit sp = small_split(prec == kFP32, args.n_pad, ts, nz, with_p);
  const int tri = small_tile_count(args.n_pad, ts);
  const int grid = sp.zw + 4 * (nz * tri - sp.zw) + (with_p ? sp.pw + 4 * (tri - sp.pw) : 0);
  if (grid <= 0) return hipSuccess;
#define DMPT_SMALL(PP, PZ)                                                                                          \
  if (ts == 32) hipLaunchKernelGGL((k_step_small<PP, PZ, 1, 4>), dim3(grid), dim3(256), 0, s, args, nz, sp.zw, sp.pw);            \
  else hipLaunchKernelGGL((k_step_small<PP, PZ, 2, 4>), dim3(grid), dim3(256), 0, s, args, nz, sp.zw, sp.pw);                     \
  break;
  switch (prec) {
    case kFP32:
      if (ts == 64 && eight_waves(grid)) {
        hipLaunchKernelGGL((k_step_small<kFP32, kFP32, 2, 8>), dim3(grid), dim3(512), 0, s, args, nz, sp.zw, sp.pw);
        break;
      }
      DMPT_SMALL(kFP32, kFP32)
    case kSplit2: DMPT_SMALL(kSplit2, kSplit2)
    case kSplit3: DMPT_SMALL(kSplit3, kSplit3)
    case kSplit32: DMPT_SMALL(kSplit3, kSplit2)
    case kBF16: DMPT_SMALL(kBF16, kBF16)
    case kSplitH: DMPT_SMALL(kSplitH, kSplitH)
    default: return hipErrorInvalidValue;
  }
#undef DMPT_SMALL
  return hipGetLastError();
}

// ---------------------------------------------------------------- general product

// One tile of a general product (ProdArgs) per workgroup.
namespace {
template <int PREC, int B, int W>
__global__ __launch_bounds__((W * 64)) __attribute__((amdgpu_waves_per_eu((B == 1 ? 4 : 2), (B == 1 ? 4 : 2))))
void k_prod_small(ProdArgs a) {
  using G = SGeo<PREC, B, W>;
  constexpr int TS = G::TS, NTH = G::NTH;
  __shared__ __attribute__((aligned(1024))) char part[G::PART];
  __shared__ double s_red[8], s_nrm[8];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = a.n_pad / TS, tiles = a.kind == kProdFull ? nt * nt : nt * (nt + 1) / 2;
  const int k = blockIdx.x / tiles, t = xcd_order(blockIdx.x - k * tiles, tiles);
  int ti, tj;
  if (a.kind == kProdFull) full_tile(t, nt, &ti, &tj);
  else tri_tile(t, nt, &ti, &tj);
  const int spass = a.n_pad / Fmt<PREC>::K, nst = a.kind == kProdAnti ? 2 * spass : spass;
  const char* pa = a.a + (size_t)k * a.sa;
  const char* pb = a.b + (size_t)k * a.sb;
  const size_t rI = panel_off<PREC>(ti * TS, a.n_pad), rJ = panel_off<PREC>(tj * TS, a.n_pad);
  float usc = 1.0f;
  auto ov = [&]() {   // while the first operands are on their way: the norm behind the copy's exponent
    if constexpr (PREC == kSplitH) {
      usc = prod_scale(a, k);
      if (a.mn) {
        const MatMeta* mi = (const MatMeta*)(a.mn + (size_t)k * a.smn);
        const double v = wave_sum(meta_part<NTH>(mi, meta_entries(a.n_pad), tid));
        if (lane == 0) s_nrm[wave] = v;
      }
    }
    return true;
  };
  tile_sum<PREC, B, W>(pa + rI, pb + rJ, pb + rI, pa + rJ, spass, nst, a.n_pad, a.flush, ti, tj, 1.0f, 1.0f, false, (LDS_AS char*)part,
                       wave, lane, ov, [] {});
  int ec = a.ec;
  if constexpr (PREC == kSplitH) {
    if (a.mn) {
      double v = 0.0;
      for (int w = 0; w < G::NWV; ++w) v += s_nrm[w];
      ec = yscale_exp(sqrt(v), a.bound);
    }
  }
  __syncthreads();
  double sq = prod_region<PREC, TS, G::LS, NTH, true, 1>(a, k, (LDS_AS float*)part, tid, ti * TS, tj * TS,
                                                         a.kind != kProdFull, a.alpha * usc,
                                                         PREC == kSplitH ? ldexpf(1.0f, ec) : 1.0f);
  if (a.mo && a.kind == kProdFull) {   // the exponent only
    if (t == 0 && tid == 0) {
      MatMeta* mo = (MatMeta*)(a.mo + (size_t)k * a.smo);
      mo->scale = ec;
      mo->count = 0;
    }
  } else if (a.mo) {
    sq = wave_sum(sq);
    if (lane == 0) s_red[wave] = sq;
    __syncthreads();
    if (tid == 0) {
      double v = 0.0;
      for (int w = 0; w < G::NWV; ++w) v += s_red[w];
      MatMeta* mo = (MatMeta*)(a.mo + (size_t)k * a.smo);
      mo->nrm[t] = v;
      if (t == 0) {
        mo->scale = ec;
        mo->count = tiles;
      }
    }
  }
}
}  // namespace

hipError_t launch_prod_small(int prec, int ts, const ProdArgs& a, hipStream_t s) {
  if (a.n_pad <= 0 || a.n_pad % 64 != 0 || (ts != 32 && ts != 64) || a.nb < 1) return hipErrorInvalidValue;
  const int nt = a.n_pad / ts, grid = a.nb * (a.kind == kProdFull ? nt * nt : nt * (nt + 1) / 2);
  // Always four waves, so that an observable's sums do not depend on how many share a launch.
#define DMPT_PSMALL(P)                                                                                         \
  if (ts == 32) hipLaunchKernelGGL((k_prod_small<P, 1, 4>), dim3(grid), dim3(256), 0, s, a);                   \
  else hipLaunchKernelGGL((k_prod_small<P, 2, 4>), dim3(grid), dim3(256), 0, s, a);                            \
  break;
  switch (prec) {
    case kFP32: DMPT_PSMALL(kFP32)
    case kSplit2: DMPT_PSMALL(kSplit2)
    case kSplit3: DMPT_PSMALL(kSplit3)
    case kSplitH: DMPT_PSMALL(kSplitH)
    default: return hipErrorInvalidValue;
  }
#undef DMPT_PSMALL
  return hipGetLastError();
}

}  // namespace dmpt
