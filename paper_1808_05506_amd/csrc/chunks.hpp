// Chunks of sites that run across the ends of x-rows, their neighbours, and the
// order in which workgroups take them.
#pragma once

#include "dslash_common.hpp"

namespace dsl {

// A chunk is R consecutive sites of an (x, y) plane, across row ends: a chunk
// of an x-row alone left lanes idle wherever N_x is not a multiple of R (34
// sites: three chunks of 12 in three waves of 64 lanes, 71 % of the lanes; on
// 34^3 x 68 2813 us), and rows below 11 sites had no such kernel at all.  The
// z and t neighbours of a chunk are the same run of another plane, the y
// neighbours the run N_x further on (with one wrap).  The x neighbours are in
// the chunk but for its halo sites.  HN = 4, any chunk: the sites beyond its two
// ends, and the row start and end that lie outside it.  HN = 2, a chunk of one
// x-row (R divides N_x): the x neighbours of its two ends.
template <int HN>
struct FlatChunk {
  uint32_t p0;        // first in-plane site (x + N_x y)
  int n;              // live sites (<= R)
  int z, t;
  uint32_t plane;     // site index of (0, 0, z, t)
  uint32_t nx, nxy;
  uint32_t xa, xb;    // x of the first and the last live site
};

// Workgroup order: tiles of kb chunks x zb planes, and in a tile segment after
// segment of T t-steps, its planes and chunks inside (kb = chunks, zb = N_z:
// segment by segment over whole t-planes).
struct FlatMarch {
  uint32_t sb, chunks;   // sites per chunk, chunks per (x, y) plane
  uint32_t T, nseg;      // t steps per workgroup, segments
  uint32_t kb, zb;
  uint32_t grid;         // workgroups
  bool late;               // the diagonal term last (march_step_o)
};

inline FlatMarch make_flat_march(const Geom& g, uint32_t sb, uint32_t T) {
  FlatMarch m;
  const uint32_t plane = uint32_t(g.n[0]) * uint32_t(g.n[1]), nt = uint32_t(g.n[3]);
  m.sb = sb;
  m.chunks = (plane + sb - 1) / sb;
  m.T = T < 1 ? 1 : (T > nt ? nt : T);
  m.nseg = (nt + m.T - 1) / m.T;
  m.kb = m.chunks;
  m.zb = uint32_t(g.n[2]);
  m.grid = m.chunks * uint32_t(g.n[2]) * m.nseg;
  m.late = false;
  return m;
}

// Tiles of by x bz (y, z) rows; 0: segment by segment over whole t-planes.
inline void flat_march_tile(const Geom& g, FlatMarch& m, int by, int bz) {
  if (by <= 0 || bz <= 0) {
    m.kb = m.chunks;
    m.zb = uint32_t(g.n[2]);
    return;
  }
  const uint32_t k = (uint32_t(by) * uint32_t(g.n[0]) + m.sb / 2) / m.sb;
  m.kb = k < 1 ? 1 : (k > m.chunks ? m.chunks : k);
  m.zb = uint32_t(bz) > uint32_t(g.n[2]) ? uint32_t(g.n[2]) : uint32_t(bz);
}

template <int HN>
DSL_HD FlatChunk<HN> flat_chunk(const Geom& g, const FlatMarch& m, uint32_t L, uint32_t& seg) {
  const uint32_t nz = uint32_t(g.n[2]);
  const uint32_t slab = m.chunks * m.zb * m.nseg;
  const uint32_t sz = L / slab;
  L -= sz * slab;
  const uint32_t z0 = sz * m.zb, zw = nz - z0 < m.zb ? nz - z0 : m.zb;
  const uint32_t tile = m.kb * zw * m.nseg;
  const uint32_t sk = L / tile;
  L -= sk * tile;
  const uint32_t k0 = sk * m.kb, kw = m.chunks - k0 < m.kb ? m.chunks - k0 : m.kb;
  seg = L / (kw * zw);
  L -= seg * kw * zw;
  const uint32_t zz = L / kw;
  FlatChunk<HN> c;
  c.nx = uint32_t(g.n[0]);
  c.nxy = c.nx * uint32_t(g.n[1]);
  c.p0 = (k0 + L - zz * kw) * m.sb;
  c.n = int(c.nxy - c.p0 < m.sb ? c.nxy - c.p0 : m.sb);
  c.z = int(z0 + zz);
  c.t = int(seg * m.T);
  c.plane = c.nxy * (uint32_t(c.z) + nz * uint32_t(c.t));
  c.xa = c.p0 - g.dx.div(c.p0) * c.nx;
  const uint32_t pl = c.p0 + uint32_t(c.n) - 1;
  c.xb = pl - g.dx.div(pl) * c.nx;
  return c;
}

// In-plane halo site k, in LDS slot 0 (k = 0) or R + k of the own row (site i of
// the chunk is in slot i + 1): 0 before the first site, 1 behind the last one
// (HN = 2: with the row's wrap), 2 the start of the first site's row, 3 the end
// of the last site's row.  One that no lane needs repeats a site of the chunk.
// (Computed here: a select among four stored members became a load from
// scratch memory.)
template <int HN>
DSL_HD uint32_t halo_site(const FlatChunk<HN>& c, int k) {
  const uint32_t pl = c.p0 + uint32_t(c.n) - 1;
  if constexpr (HN == 2) {
    const uint32_t down = c.xa > 0 ? 1u : 1u - c.nx, up = c.xb + 1 < c.nx ? 1u : 1u - c.nx;
    return (k & 1 ? pl : c.p0) + (k & 1 ? up : 0u - down);
  }
  const uint32_t down = k == 0 ? uint32_t(c.xa > 0) : c.xa;
  const uint32_t up = k == 1 ? uint32_t(c.xb + 1 < c.nx) : c.nx - 1 - c.xb;
  return k & 1 ? pl + up : c.p0 - down;
}

// Site index of the neighbour of chunk site k in direction SGN * MU (y, z, t).
template <int MU, int SGN, int HN>
DSL_HD uint32_t flat_nbr(const Geom& g, const FlatChunk<HN>& c, uint32_t k) {
  static_assert(MU >= 1, "x neighbours come from the own row");
  if constexpr (MU == 1) {
    // HN = 2: the whole run wraps or none of it (p0 decides for the workgroup)
    const uint32_t p = HN == 2 ? c.p0 : c.p0 + k, d = HN == 2 ? k : 0;
    if constexpr (SGN > 0) return c.plane + (p + c.nx < c.nxy ? p + c.nx : p + c.nx - c.nxy) + d;
    else return c.plane + (p >= c.nx ? p - c.nx : p + c.nxy - c.nx) + d;
  } else {
    const uint32_t p = c.p0 + k;
    uint32_t q[2] = {uint32_t(c.z), uint32_t(c.t)};
    uint32_t& w = q[MU - 2];
    const uint32_t nw = uint32_t(g.n[MU]);
    w = SGN > 0 ? (w + 1 == nw ? 0 : w + 1) : (w == 0 ? nw - 1 : w - 1);
    return c.nxy * (q[0] + uint32_t(g.n[2]) * q[1]) + p;
  }
}

// Own-row slots of the x + 1 and x - 1 neighbours of chunk site i.
struct XSlots {
  int f, b;
};

template <int HN>
DSL_HD XSlots x_slots(const Geom& g, const FlatChunk<HN>& c, int R, int i) {
  if constexpr (HN == 2) return XSlots{i + 2, i};  // n = R: the ends' neighbours are in slots 0 and R + 1
  i = i < c.n ? i : c.n - 1;
  const uint32_t p = c.p0 + uint32_t(i);
  const int nx = int(c.nx), x = int(p - g.dx.div(p) * c.nx);
  XSlots s;
  if (x + 1 < nx) s.f = i + 1 < c.n ? i + 2 : R + 1;
  else s.f = i + 1 - nx >= 0 ? i + 2 - nx : R + 2;
  if (x > 0) s.b = i;  // slot 0 is the halo site before the chunk
  else s.b = i + nx - 1 < c.n ? i + nx : R + 3;
  return s;
}

}  // namespace dsl
