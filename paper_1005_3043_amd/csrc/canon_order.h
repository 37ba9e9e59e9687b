// Visiting order of wilson_apply's streaming kernel: blocks of L_x * hy * hz *
// L_t sites (cut short at the far edges), x fastest inside a block and the
// blocks t fastest, then z, then y.  The sites that an XCD has in flight then
// form a compact block instead of a run of planes, and most neighbours come
// from its own L2.
#pragma once

#include <cmath>

#include "common.h"

namespace mg {

// hy and hz are at most the extents, so that no product below passes the
// volume (which 32 bits hold).
struct CanonOrder {
  uint32_t L[4];
  uint32_t hy, hz;
};

// Extent h of the blocks in y and z: one time slice of a column of blocks (L_x
// h h sites of links and spinors) takes about 1.5 MB, so that the three slices
// the stencil spans fit an XCD's 4 MB L2 with what is in flight.  On 32^3 x 64:
// FP32 x 12 right-hand sides 4.60 / 3.80 / 4.15 ms with h = 2 / 4 / 8 (planes
// walked whole: 5.09 ms, 38 GB fetched), FP64 x 1 669 / 583 / 540 us.
inline CanonOrder canon_order(const int L[4], int nrhs) {
  const double e = std::sqrt(1.5e6 / ((double)L[0] * (192.0 * nrhs + 576.0)));
  const uint32_t h = e < 2.83 ? 2u : e < 5.66 ? 4u : e < 11.3 ? 8u : 16u;  // nearest power of two, as lattices come
  CanonOrder o;
  for (int mu = 0; mu < 4; ++mu) o.L[mu] = (uint32_t)L[mu];
  o.hy = h < o.L[1] ? h : o.L[1];
  o.hz = h < o.L[2] ? h : o.L[2];
  return o;
}

// Site (lexicographic) at position n of the order.
__host__ __device__ __forceinline__ uint32_t site_at(const CanonOrder &g, uint32_t n) {
  const uint32_t L0 = g.L[0], L1 = g.L[1], L2 = g.L[2], L3 = g.L[3];
  uint32_t per = L0 * L2 * L3 * g.hy;
  const uint32_t Y = n / per * g.hy, hy = g.hy < L1 - Y ? g.hy : L1 - Y;
  n -= Y * L0 * L2 * L3;
  per = L0 * hy * L3 * g.hz;
  const uint32_t Z = n / per * g.hz, hz = g.hz < L2 - Z ? g.hz : L2 - Z;
  n -= Z * L0 * hy * L3;
  const uint32_t area = L0 * hy * hz, t = n / area;  // whole time slices of the column: blocks in t need no split
  n -= t * area;
  const uint32_t z = n / (L0 * hy);
  n -= z * L0 * hy;
  const uint32_t y = n / L0;
  return n - y * L0 + L0 * ((Y + y) + L1 * ((Z + z) + L2 * t));
}

}  // namespace mg
