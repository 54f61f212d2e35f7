// Launch shape and workgroup order of the flat kernels (wilson_flat.hpp,
// staggered_flat.hip): which sites and columns a workgroup owns, and in what order the
// workgroups take them.
#pragma once

#include "launch.hpp"

namespace dsl {

// Workgroup order: tiles of zb planes x kb chunks, t sweeping inside a tile.
struct FlatOrder {
  uint32_t P, chunks;  // sites per chunk, chunks per plane
  uint32_t zb, kb;
  FastDiv groups;      // lanes per site in a workgroup
};

struct FlatSite {
  uint32_t p0, n;  // first in-plane site of the chunk, its live sites
  int z, t;
};

DSL_HD FlatSite flat_site(const Geom& g, const FlatOrder& o, uint32_t L) {
  const uint32_t nz = uint32_t(g.n[2]), nt = uint32_t(g.n[3]), nk = o.chunks;
  const uint32_t slab = nk * o.zb * nt;  // zb planes: all chunks and t
  const uint32_t sz = L / slab;
  L -= sz * slab;
  const uint32_t z0 = sz * o.zb, zw = nz - z0 < o.zb ? nz - z0 : o.zb;
  const uint32_t tile = o.kb * zw * nt;
  const uint32_t sk = L / tile;
  L -= sk * tile;
  const uint32_t k0 = sk * o.kb, kw = nk - k0 < o.kb ? nk - k0 : o.kb;
  const uint32_t per_t = kw * zw, t = L / per_t;
  L -= t * per_t;
  const uint32_t zz = L / kw, k = k0 + (L - zz * kw);
  const uint32_t plane = uint32_t(g.n[0]) * uint32_t(g.n[1]);
  FlatSite s;
  s.p0 = k * o.P;
  s.n = plane - s.p0 < o.P ? plane - s.p0 : o.P;
  s.z = int(z0 + zz);
  s.t = int(t);
  return s;
}

struct FlatShape {
  FlatOrder o;
  dim3 grid, block;
  size_t lds;
};

// Columns per lane: as many as 16 bytes hold and N_v is a multiple of; one for
// fields off a 16-byte boundary.
inline int flat_vw(int dtype, int nv, bool aligned) {
  int vw = dtype == DT_C128 || !aligned ? 1 : (dtype == DT_C64 ? 2 : 4);
  while (nv % vw) vw /= 2;
  return vw;
}

// The lanes address a plane of sites by 32-bit byte offsets.
inline bool flat_covers(const Geom& g, int dtype) {
  return uint64_t(g.n[0]) * uint64_t(g.n[1]) * 12u * uint64_t(g.nv) * dtype_bytes(dtype) < (1ull << 32);
}

// comps: spinor components of a site (12, D_S 3).
// P: at most 256 lanes and 80 KB of links (two workgroups a CU), and of those
// the one that wastes the fewest lanes on the chunk count and the last wave.
// zb x kb: whole planes whose spinors at one t take at most 1.2 MB where two fit,
// else three planes of about a third of 1.05 MB each (FP64, N_v = 12, 16^3 x 32: 220 us
// with 2 whole planes, 230 with 4 planes x 7 of 13 chunks); two planes where N_z is 4 or 5,
// with chunks that divide the plane, as three leave a tile of one or two (64 x 4 x 4 x 16,
// FP64, N_v = 24 84 us, 61 in two).  D_W in pieces of 16 bytes
// takes two workgroups a CU (79 KB of LDS asked for): more of them in flight than that
// push each other's neighbour rows out of the L2.  24^3 x 48, two, three and four a CU:
// FP64, N_v = 12, 1141, 1167 and 1368 us; C64, N_v = 26, 1287, 1445 and 1590.  With the clover
// term in C64 three are as good (12^4, N_v = 16: 32 us against 38 at two).
inline FlatShape flat_shape(const Geom& g, int comps, int word_bytes, int vw, int lw, bool clover) {
  FlatShape s{};
  const uint32_t plane = uint32_t(g.n[0]) * uint32_t(g.n[1]);
  const uint32_t groups = uint32_t(g.nv / vw), gb = groups < 256 ? groups : 256;
  const size_t site_lds = size_t(8 * lw + (clover ? 36 : 0)) * word_bytes;
  uint32_t pmax = 256 / gb;
  if (pmax > 80 * 1024 / site_lds) pmax = uint32_t(80 * 1024 / site_lds);
  if (pmax > plane) pmax = plane;
  if (pmax < 1) pmax = 1;
  uint32_t best = pmax;
  uint64_t cost = 0;
  for (uint32_t k = (plane + pmax - 1) / pmax, p; 2 * (p = (plane + k - 1) / k) >= pmax; ++k) {
    const uint64_t lanes = uint64_t(k) * ((p * gb + 63) / 64);
    if (cost == 0 || 10 * lanes < 9 * cost) {
      cost = lanes;
      best = p;
    }
    if (p == 1) break;
  }
  s.o.P = best;
  s.o.chunks = (plane + best - 1) / best;
  s.o.groups = FastDiv::make(gb);
  const double row = double(comps) * g.nv * word_bytes * best, full = row * s.o.chunks;
  if (full <= 0.6 * 1024 * 1024) {
    s.o.kb = s.o.chunks;
    s.o.zb = uint32_t(1.2 * 1024 * 1024 / full);
    if (s.o.zb > uint32_t(g.n[2])) s.o.zb = uint32_t(g.n[2]);
  } else {
    const bool two_planes = g.n[2] == 4 || g.n[2] == 5;
    s.o.zb = g.n[2] < 3 ? uint32_t(g.n[2]) : two_planes ? 2u : 3u;
    s.o.kb = uint32_t(1.05 * 1024 * 1024 / (s.o.zb * row));
    if (s.o.kb < 1) s.o.kb = 1;
    if (s.o.kb > s.o.chunks) s.o.kb = s.o.chunks;
    if (two_planes)
      for (uint32_t d = uint32_t(1.25 * 1024 * 1024 / (s.o.zb * row)); 3 * d >= 2 * s.o.kb && d > 0; --d)
        if (s.o.chunks % d == 0) {
          s.o.kb = d;
          break;
        }
  }
  // DSLASH_FLAT_ZB, DSLASH_FLAT_KB: from 1 to the whole range, which 0 and below stand
  // for too (flat_site divides by the products of these)
  const auto clamped = [](const Knob& k, uint32_t dflt, uint32_t whole) {
    if (!k.set) return dflt;
    return k.value < 1 || uint32_t(k.value) > whole ? whole : uint32_t(k.value);
  };
  s.o.zb = clamped(knobs().flat_zb, s.o.zb, uint32_t(g.n[2]));
  s.o.kb = clamped(knobs().flat_kb, s.o.kb, s.o.chunks);
  s.grid = dim3(s.o.chunks * uint32_t(g.n[2]) * uint32_t(g.n[3]), (groups + gb - 1) / gb);
  s.block = dim3(best * gb);
  s.lds = size_t(best) * site_lds;
  const bool two = comps == 12 && (word_bytes == 16 || (word_bytes == 8 && vw == 2 && !clover));
  if (two && s.lds < 79 * 1024) s.lds = 79 * 1024;
  if (s.lds < size_t(knobs().row_lds_extra.get(0))) s.lds = size_t(knobs().row_lds_extra.get(0));
  return s;
}

}  // namespace dsl
