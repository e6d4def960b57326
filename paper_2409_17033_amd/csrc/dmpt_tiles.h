// Which tile a workgroup of the small-size kernels takes, and where its partials
// go.  Integer functions of the workgroup's index, compiled for the device and for
// the host (where a test runs them over many shapes).
#pragma once

#include <hip/hip_runtime.h>

#define DMPT_TILE __host__ __device__ __forceinline__

namespace dmpt {

// Tile t of the upper triangle (J >= I) of an nt x nt grid: bands of 4 tile
// rows, first the band's own triangle, then its columns from left to right,
// so that a run of tiles shares few row panels.
DMPT_TILE void tri_tile(int t, int nt, int* ti, int* tj) {
  const float m = (float)nt + 0.5f;
  int i = (int)(m - sqrtf(m * m - 2.0f * (float)t));
  i = i < 0 ? 0 : i > nt - 1 ? nt - 1 : i;
  while (i > 0 && i * nt - i * (i - 1) / 2 > t) --i;
  while (i + 1 < nt && (i + 1) * nt - (i + 1) * i / 2 <= t) ++i;
  const int r0 = i & ~3, hb = nt - r0 < 4 ? nt - r0 : 4;   // the band's first row and height
  int local = t - (r0 * nt - r0 * (r0 - 1) / 2);
  if (local < hb * (hb + 1) / 2) {
    int r = 0;
    while (local >= hb - r) {
      local -= hb - r;
      ++r;
    }
    *ti = r0 + r;
    *tj = r0 + r + local;
  } else {
    local -= hb * (hb + 1) / 2;
    *ti = r0 + local % hb;
    *tj = r0 + hb + local / hb;
  }
}

// Tile t of a whole nt x nt grid in the same bands.
DMPT_TILE void full_tile(int t, int nt, int* ti, int* tj) {
  const int r0 = t / (4 * nt) * 4, hb = nt - r0 < 4 ? nt - r0 : 4;
  const int local = t - r0 * nt;
  *ti = r0 + local % hb;
  *tj = local / hb;
}

// Position p of cnt tiles as workgroups are dealt to the XCDs in turn: each
// XCD takes a contiguous run of tiles, which share row panels in its L2.
DMPT_TILE int xcd_order(int p, int cnt) {
  const int x = p & 7, per = cnt >> 3, rest = cnt & 7;
  return x * per + (x < rest ? x : rest) + (p >> 3);
}

// Tiles of the upper triangle in the order of a step launch: the first diagonal tiles
// (a multiple of 8 up to half of them), those above the diagonal, the other
// diagonal tiles.  Z's diagonal tiles take half as long as its others: spread over the
// XCDs and over both ends of the launch they even out the CUs that take one tile more:
// n = 1024, FP32, 528 tiles of 32 x 32 on 256 CUs: the self-consistent loop, whose
// launches are sweeps, 21.8 -> 16.8 ms (with the diagonal tiles in one run, which goes to
// one XCD, no gain).
// Launches over several observables keep the bands' own order and whole diagonal
// tiles: n = 1500, four of them, FP16 split 4.3 ms, spread 4.6; n = 1000 2.1, and 2.3 with
// the shorter diagonal tiles in the bands' order.
struct StepOrder {
  int nt, first, off;
  bool spread;
  DMPT_TILE StepOrder(int nt_, bool spread_)
      : nt(nt_), first((nt_ / 2) & ~7), off(nt_ * (nt_ - 1) / 2), spread(spread_) {}
  // workgroup b of the first cw tiles: its tile
  DMPT_TILE int at(int b, int cw) const {
    if (!spread) return xcd_order(b, cw);
    const int w = cw - first < 0 ? 0 : cw - first < off ? cw - first : off;   // of those above the diagonal
    return b >= first && b < first + w ? first + xcd_order(b - first, w) : b;
  }
  DMPT_TILE void tile(int t, int* ti, int* tj) const {
    if (!spread) {
      tri_tile(t, nt, ti, tj);
    } else if (t >= first && t < first + off) {
      tri_tile(t - first, nt - 1, ti, tj);
      ++*tj;
    } else {
      *ti = *tj = t < first ? t : t - off;
    }
  }
};

// Job b of one kind of a step launch (Z of the observables, or P): tile b of the
// `whole` whole tiles (edge ts), or with `quarter` (tiles of 64, ts = 32) quarter b of
// the tiles after them.  none: nothing to do; next: the entry after `slot`, of the
// matrix's `slots`, is cleared too.
struct SmallPlace {
  int obs, ti, tj, slot, slots;   // ti, tj in units of ts
  bool next, none;
};
DMPT_TILE SmallPlace small_place(int n_pad, int ts, int b, int whole, bool quarter, bool spread) {
  const int nt = n_pad / (quarter ? 64 : ts), tri = nt * (nt + 1) / 2;
  const StepOrder order(nt, spread);
  SmallPlace p;
  const int f = quarter ? whole + (b >> 2) : b;
  p.obs = f < tri ? 0 : f / tri;
  const int left = whole - p.obs * tri, cw = left < 0 ? 0 : left < tri ? left : tri;   // the observable's whole tiles
  int t = f - p.obs * tri;
  p.slot = t;
  p.slots = cw + 4 * (tri - cw);
  p.next = p.none = false;
  if (!quarter) p.slot = t = order.at(t, cw);
  order.tile(t, &p.ti, &p.tj);
  if (quarter) {
    const int q = b & 3;
    p.slot = cw + 4 * (t - cw) + q;
    if (p.ti == p.tj) {
      p.none = q == 2;   // below the diagonal: the mirror of quarter 1, which clears its entry
      p.next = q == 1;
    }
    p.ti = 2 * p.ti + (q >> 1);
    p.tj = 2 * p.tj + (q & 1);
  }
  return p;
}

}  // namespace dmpt
