// Launch shapes of the row-staged D_W kernels and even-odd hop: sites per chunk, halo
// sites, where the diagonal term is added, t steps.
#pragma once

#include "wilson_rows.hpp"

namespace dsl {

// A row of N_x sites is made of whole chunks of at most 16 sites (row_sites_default)
// that leave at most a tenth of the lanes idle.
inline bool whole_chunks(int nx, int nv, int wb) {
  const int r = row_sites_default(nx, nv);
  return r > 0 && nx % r == 0 && 10 * r * nv >= 9 * ((r * nv + 63) / 64) * 64 && r * nv <= 256 && halo_fits(r, nv, wb, 2);
}

// Where the march adds the diagonal term (march_step_o) in C64: first where that holds
// for each of the five block sizes, last elsewhere.  N_x alone decides, so that a
// column's bits do not depend on the block that it is in (at a fixed t-segment length);
// last costs up to 4 % and halves the error against FP64.
inline bool rows_fold(int nx) {
  for (const int nv : {4, 8, 12, 16, 24})
    if (!whole_chunks(nx, nv, 8)) return false;
  return true;
}

// Sites per chunk R and halo sites hn.  A chunk of one x-row (hn = 2) where the row is
// made of whole ones: it has the fewest halo loads and registers (16^3 x 32, N_v = 12:
// 92.5 us against 107.6 with hn = 4; BF16, N_v = 24: 129 against 164; FP32 N_v = 24 alone is
// faster with hn = 4, in the march only: 187 us against 193, 1570 against 1650 on 32^4),
// and in C64 at N_v = 4
// where a whole row leaves at most a quarter idle (28^4: 195 us against 244, 24^3 x 48 218
// against 242; 62 %, 20^4, 73.0 against 69.4).
// Elsewhere chunks across row ends (hn = 4).  N_v = 4: one wave (24^3 x 48: 242 us, 296 with
// four; BF16 126 and 154).  Other N_v: at most 256 lanes, and of those from the longest
// down to half of it the one that leaves the fewest lanes idle in the last chunk of the
// plane and the last wave (24^3 x 48: 499 us at R = 21 against 601 with rows of 12; 34^3 x
// 68: 2225 against 2813).  In the BF16 march three waves count as four: a CU holds eight, two
// workgroups of either (N_v = 24, 14x13x12x16: 47 us at R = 10 against 62 at 8, 34x18x18x24 304
// against 346; in C64 neither is always the faster).
// DSLASH_ROW_SITES overrides R (hn = 4); false: no such kernel
// (fewer than 64 lanes, or a chunk too short for its halo).  DSLASH_ROWS=2 asks
// for these kernels where a chunk of one x-row alone holds its halo.
// late: the diagonal term last (whatever hn the launch takes).
// pp: the buffer scheme (the one-row kernels: 0); two workgroups a CU need 80 KB.
inline bool rows_shape(const Geom& g, int dtype, int pp, bool any_nv, bool knob_form, int& R, int& hn,
                       bool& late) {
  const int nv = g.nv, wb = int(dtype_bytes(dtype));
  const uint32_t plane = uint32_t(g.n[0]) * uint32_t(g.n[1]);
  if (knobs().rows.get(1) == 2) {
    if (any_nv) return false;
    int r = knobs().row_sites.get(row_sites_default(g.n[0], nv));
    if (r > g.n[0]) r = g.n[0];
    if (r < 1 || r * nv > 256 || r * nv < 64 || !halo_fits(r, nv, wb, 2)) return false;
  }
  late = any_nv || (dtype == DT_C64 && !rows_fold(g.n[0]));
  hn = 4;
  if (knobs().row_sites.set) {
    R = knobs().row_sites.value;
    if (R > int(plane)) R = int(plane);
  } else {
    const int whole = row_sites_default(g.n[0], nv);
    const bool row4 = nv == 4 && dtype == DT_C64 && g.n[0] == whole && g.n[0] >= 24 && g.n[0] <= 32;
    if (!any_nv && !knob_form && (row4 || whole_chunks(g.n[0], nv, wb))) {
      R = whole;
      hn = nv > 16 && dtype == DT_C64 && pp && halo_fits(R, nv, wb, 4) ? 4 : 2;
      return true;
    }
    int rmax = nv == 4 ? 16 : 256 / nv;
    if (rmax < 1) return false;
    while (rmax > 1 && march_lds(rmax, nv, wb, pp, 4) > 76 * 1024) --rmax;
    if (uint32_t(rmax) > plane) rmax = int(plane);
    R = rmax;
    uint64_t cost = 0;
    for (uint32_t k = (plane + uint32_t(rmax) - 1) / uint32_t(rmax); nv != 4; ++k) {  // chunks per plane
      const int r = int((plane + k - 1) / k);
      if (2 * r < rmax || !halo_fits(r, nv, wb, 4)) break;
      const uint32_t waves = uint32_t((r * nv + 63) / 64);
      const uint64_t lanes = uint64_t(k) * (dtype == DT_BF16 && pp == 2 && waves == 3 ? 4 : waves);
      if (cost == 0 || 100 * lanes < 97 * cost) {
        cost = lanes;
        R = r;
      }
      if (r == 1) break;
    }
  }
  return R >= 1 && R * nv <= 256 && R * nv >= 64 && halo_fits(R, nv, wb, 4);
}

// t steps per workgroup: 8, or of the segment counts between that and 16 (FP32
// storage) steps the one whose rounds of resident workgroups (two waves per
// SIMD with two or more row buffers, three with one, and the LDS) march the
// fewest steps, where the grid is a few rounds (more than 8 steps for a single
// round only); a segment costs 0.7 of a step more (its first one stages a row
// more).  On 16^3 x 32: N_v = 12 and 16 take
// 16 steps (512 workgroups at two a CU); N_v = 4 and 8 took 44.4 and 65.6 us at
// 8 steps against 64.8 and 74.6 us at 16.  Small lattices take shorter
// segments until every SIMD has a wave.
inline int march_tsteps(const Geom& g, int R, int hn, int pp, int dtype) {
  const uint32_t nt = uint32_t(g.n[3]), cus = uint32_t(device_cus());
  const uint32_t wg_waves = uint32_t((R * g.nv + 63) / 64);
  const auto grid = [&](uint32_t nseg) { return make_flat_march(g, uint32_t(R), (nt + nseg - 1) / nseg).grid; };
  uint32_t per_cu = (pp ? 8u : 12u) / wg_waves;
  const uint32_t by_lds = uint32_t(160 * 1024 / march_lds(R, g.nv, int(dtype_bytes(dtype)), pp, hn));
  if (per_cu > by_lds) per_cu = by_lds;
  if (per_cu < 1) per_cu = 1;
  uint32_t best = (nt + 7) / 8;
  if (grid(best) <= 4 * per_cu * cus) {
    double cost = -1;
    for (uint32_t n = dtype == DT_C64 ? (nt + 15) / 16 : best; n <= 2 * best; ++n) {
      const uint32_t T = (nt + n - 1) / n;
      const double c = double((grid(n) + per_cu * cus - 1) / (per_cu * cus)) * (T + 0.7);
      if ((T <= 8 || grid(n) <= per_cu * cus) && grid(n) * wg_waves >= 4u * cus && (cost < 0 || c < cost)) {
        cost = c;
        best = n;
      }
    }
  }
  uint32_t T = (nt + best - 1) / best;
  while (T > 1 && make_flat_march(g, uint32_t(R), T).grid * wg_waves < 4u * cus) T = (T + 1) / 2;
  return int(T);
}

}  // namespace dsl
