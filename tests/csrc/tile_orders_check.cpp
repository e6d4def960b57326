// Host-side check of which tile runs where: the small-size kernels' tile order
// (dmpt_tiles.h, small_split) and the job lists of the general products
// (build_prod_list).  Every tile of every matrix runs exactly once, whole, as the
// quarters of a 64 x 64 tile or as consecutive pieces of its K range; every entry of
// the partial sums is written or cleared exactly once and lies in the area the
// runtime reserves; packed fields do not overflow.  Exits non-zero on the first
// violation.  Usage: tile_orders_check [drop]  (drop: leave out one workgroup of
// every launch and one job of every list, which has to be noticed).
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "dmpt_lists.h"
#include "dmpt_tiles.h"

using namespace dmpt;

namespace {

bool drop = false;

bool fail(const char* what, int a, int b, int c, int d, int e) {
  std::printf("FAIL %s: %d %d %d %d %d\n", what, a, b, c, d, e);
  return false;
}

// One step launch as launch_step_small lays it out.
bool step_launch(bool fp32, int n_pad, int ts, int nz, int with_p) {
  const SmallSplit sp = small_split(fp32, n_pad, ts, nz, with_p);
  const int tri = small_tile_count(n_pad, ts), zq = 4 * (nz * tri - sp.zw), pq = with_p ? 4 * (tri - sp.pw) : 0;
  const int grid = sp.zw + zq + (with_p ? sp.pw : 0) + pq, n32 = n_pad / 32, cap = small_tile_count(n_pad, 32);
  std::vector<std::vector<int>> cover(nz + 1, std::vector<int>((size_t)n32 * n32, 0));
  std::vector<std::vector<int>> entry(nz + 1);
  std::vector<int> slots(nz + 1, 0);
  for (int b = 0; b < grid; ++b) {
    if (drop && b == grid / 2) continue;
    const bool z = b < sp.zw + zq;
    const bool quarter = z ? b >= sp.zw : b >= sp.zw + zq + sp.pw;
    const int at = z ? (quarter ? b - sp.zw : b) : quarter ? b - sp.zw - zq - sp.pw : b - sp.zw - zq;
    const int edge = quarter ? 32 : ts;
    const SmallPlace p = small_place(n_pad, edge, at, z ? sp.zw : sp.pw, quarter, nz <= 1);
    if (p.none) {
      if (b == grid - 1) return fail("the workgroup that records the decision has no tile", n_pad, ts, nz, with_p, b);
      continue;
    }
    const int m = z ? p.obs : nz;
    if (m < 0 || m > nz || (z && m == nz)) return fail("observable out of range", n_pad, ts, nz, with_p, b);
    if (p.ti < 0 || p.tj < p.ti || p.tj >= n_pad / edge) return fail("tile out of range", n_pad, ts, nz, with_p, b);
    const int w = edge / 32;
    for (int i = 0; i < w; ++i)
      for (int j = 0; j < w; ++j) ++cover[m][(size_t)(p.ti * w + i) * n32 + p.tj * w + j];
    slots[m] = p.slots;
    if (entry[m].empty()) entry[m].assign(p.slots, 0);
    if ((int)entry[m].size() != p.slots) return fail("entries of one matrix differ", n_pad, ts, nz, with_p, b);
    for (int q = 0; q < (p.next ? 2 : 1); ++q) {
      if (p.slot + q < 0 || p.slot + q >= p.slots) return fail("entry out of range", n_pad, ts, nz, with_p, b);
      ++entry[m][p.slot + q];
    }
  }
  for (int m = with_p || nz ? 0 : 1; m < nz + (with_p ? 1 : 0); ++m) {
    for (int i = 0; i < n32; ++i)
      for (int j = i; j < n32; ++j) {
        // a whole 64 x 64 diagonal tile also covers the block below the diagonal
        if (cover[m][(size_t)i * n32 + j] != 1) return fail("block not covered once", n_pad, ts, nz, m, i * n32 + j);
      }
    for (int c : entry[m])
      if (c != 1) return fail("entry not written once", n_pad, ts, nz, with_p, m);
    if (slots[m] > cap || slots[m] > meta_entries(n_pad)) return fail("more entries than reserved", n_pad, ts, nz, m, slots[m]);
  }
  if (with_p && slots[nz] != small_parts(fp32, n_pad, ts, nz)) return fail("partials and their count differ", n_pad, ts, nz, slots[nz], 0);
  return true;
}

// The tiles of one general product on the small-size kernels.
bool small_product(int n_pad, int ts, bool full) {
  const int nt = n_pad / ts, tiles = full ? nt * nt : nt * (nt + 1) / 2;
  std::vector<int> cover((size_t)nt * nt, 0), pos(tiles, 0);
  for (int b = 0; b < tiles; ++b) {
    if (drop && b == tiles / 2) continue;
    const int t = xcd_order(b, tiles);
    if (t < 0 || t >= tiles || pos[t]++) return fail("order is no permutation", n_pad, ts, full, b, t);
    int i, j;
    if (full) full_tile(t, nt, &i, &j);
    else tri_tile(t, nt, &i, &j);
    if (i < 0 || j < (full ? 0 : i) || i >= nt || j >= nt) return fail("tile out of range", n_pad, ts, full, i, j);
    ++cover[(size_t)i * nt + j];
  }
  for (int i = 0; i < nt; ++i)
    for (int j = full ? 0 : i; j < nt; ++j)
      if (cover[(size_t)i * nt + j] != 1) return fail("tile not covered once", n_pad, ts, full, i, j);
  return true;
}

bool product_list(int n_pad, bool full, int nb, int cus, bool long_k) {
  ProdList L = build_prod_list(n_pad, full, nb, cus, long_k);
  if (drop) L.jobs.pop_back();
  const int tr = n_pad / kStepTM, tc = n_pad / kStepTN;
  if (L.jobs.size() + L.split.size() > prod_list_entries(n_pad, nb)) return fail("list longer than its area", n_pad, full, nb, cus, long_k);
  std::vector<int> cover((size_t)nb * tr * tc, 0), used((size_t)nb * kMaxPieces, 0);
  auto at = [&](const ProdJob& j) { return ((size_t)((j.part >> 8) & 255) * tr + (j.tile & 0xffff)) * tc + (j.tile >> 16); };
  std::vector<int> first(cover.size(), -1), pieces(cover.size(), 0), seen(cover.size(), 0);
  for (const ProdJob& j : L.split) {
    const int k = (j.part >> 8) & 255, n = (j.part >> 4) & 15;
    if (k >= nb || (int)(j.tile & 0xffff) >= tr || (int)(j.tile >> 16) >= tc || n < 2 || n > 8) return fail("split tile out of range", n_pad, full, nb, cus, long_k);
    if (first[at(j)] >= 0) return fail("tile split twice", n_pad, full, nb, cus, long_k);
    first[at(j)] = j.part >> 16;
    pieces[at(j)] = n;
  }
  for (const ProdJob& j : L.jobs) {
    const int k = (j.part >> 8) & 255, piece = j.part & 15, n = (j.part >> 4) & 15, slot = j.part >> 16;
    if (k >= nb || (int)(j.tile & 0xffff) >= tr || (int)(j.tile >> 16) >= tc) return fail("job out of range", n_pad, full, nb, cus, long_k);
    if (n == 1) {
      if (first[at(j)] >= 0) return fail("split tile also runs whole", n_pad, full, nb, cus, long_k);
      ++cover[at(j)];
      continue;
    }
    if (first[at(j)] != slot || pieces[at(j)] != n || piece >= n) return fail("piece and split tile differ", n_pad, full, nb, cus, long_k);
    if ((size_t)(slot + piece) >= used.size() || used[slot + piece]++) return fail("slot out of range or used twice", n_pad, full, nb, cus, long_k);
    if (seen[at(j)]++ == 0) ++cover[at(j)];
    // whole groups of four stages a piece, none empty (16 columns a stage)
    const int n4 = n_pad / 64 * (long_k ? 2 : 1);
    if (n4 * piece / n >= n4 * (piece + 1) / n) return fail("empty piece", n_pad, full, nb, cus, long_k);
  }
  for (int k = 0; k < nb; ++k)
    for (int i = 0; i < tr; ++i)
      for (int j = 0; j < tc; ++j) {
        const size_t q = ((size_t)k * tr + i) * tc + j;
        if (cover[q] != (full || j >= 2 * i ? 1 : 0)) return fail("tile not covered once", n_pad, full, nb, cus, i * tc + j);
        if (first[q] >= 0 && seen[q] != pieces[q]) return fail("pieces missing", n_pad, full, nb, cus, i * tc + j);
      }
  return true;
}

}  // namespace

int main(int argc, char** argv) {
  drop = argc > 1 && !std::strcmp(argv[1], "drop");
  int launches = 0, lists = 0, caught = 0;
  auto count = [&](bool ok, int* n) {
    ++*n;
    if (drop) caught += !ok;
    return ok || drop;
  };
  for (int n_pad = 64; n_pad <= 4608; n_pad += 64)
    for (int ts : {32, 64}) {
      if (drop && n_pad < 256) continue;   // (a launch of one tile)
      for (int full = 0; full < 2; ++full)
        if (!count(small_product(n_pad, ts, full), &launches)) return 1;
      for (int nz : {0, 1, 2, 3, 4, 16})
        for (int with_p = nz ? 0 : 1; with_p < 2; ++with_p) {
          if (nz > 4 && n_pad > 2048) continue;
          for (int fp32 = 0; fp32 < 2; ++fp32)
            if (!count(step_launch(fp32, n_pad, ts, nz, with_p), &launches)) return 1;
        }
    }
  for (int n_pad = 1536; n_pad <= 9216; n_pad += 256)   // smaller ones take the small-size kernels
    for (int cus : {64, 104, 255, 256, 304})
      for (int nb = 1; nb <= 4; ++nb)
        for (int kind = 0; kind < 3; ++kind)
          if (!count(product_list(n_pad, kind == 0, nb, cus, kind == 2), &lists)) return 1;
  if (drop && caught != launches + lists) {
    std::printf("only %d of %d left-out workgroups and jobs noticed\n", caught, launches + lists);
    return 1;
  }
  std::printf("%d launches, %d lists\n", launches, lists);
  return 0;
}
