// Which launches of D_B on stored links, and of its gradient with respect to W, take the
// kernels that stage the 27 runs (bri_runs.hpp), and in which blocks.
#pragma once

#include "launch.hpp"

namespace dsl {

// Columns per block: the width whose blocks cost least.  A lane's column in a block of
// 24, 16, 12, 10, 8, 6 and 4 costs, in C64, 63.6, 63.9, 70.4, 73.1, 68.3, 82.9 and 87.5 us (D_B,
// 16^3 x 32), in C128 (12, 8, 6, 4) 110, 114, 142 and 188; an idle one costs as much.
// (By the fewest idle columns alone N_v = 20 took five blocks of four in C128, 2.1 times as
// long; three of six at N_v = 18 cost what two of twelve do, and stage one run more.)
inline int bri_block(int dtype, int nv) {
  static const int widths64[] = {24, 16, 12, 10, 8, 6, 4}, cost64[] = {100, 100, 110, 115, 107, 130, 137};
  static const int widths128[] = {12, 8, 6, 4}, cost128[] = {100, 104, 135, 170};
  const bool wide = dtype != DT_C64;
  const int *w = wide ? widths128 : widths64, *c = wide ? cost128 : cost64;
  const int nw = wide ? 4 : 7;
  int nb = w[0];
  long best = 0;
  for (int k = 0; k < nw; ++k) {
    const long n = long((nv + w[k] - 1) / w[k]) * w[k] * c[k];
    if (best == 0 || n < best) {
      best = n;
      nb = w[k];
    }
  }
  return nb;
}

// Sites per chunk of D_B in blocks of nb columns.
constexpr int bri_sites(int dtype, int nb) {
  return dtype == DT_C64 ? (nb == 24 ? 8 : nb == 16 ? 16 : nb == 12 ? 21 : nb == 10 ? 25 : nb == 8 ? 32 : nb == 6 ? 42 : 64)
                         : (nb == 12 ? 20 : nb == 8 ? 32 : nb == 6 ? 42 : 64);
}

// Workgroups of D_B in chunks of P sites.
inline uint64_t bri_blocks(const Geom& g, int P, int nb) {
  const uint64_t plane = uint64_t(g.n[0]) * uint64_t(g.n[1]);
  return (plane + uint64_t(P) - 1) / uint64_t(P) * uint64_t(g.n[2]) * uint64_t(g.n[3]) * uint64_t((g.nv + nb - 1) / nb);
}

// C64 pairs in blocks of twelve: chunks of 16 sites (three waves, four workgroups a CU)
// where all of them are resident at once and those of 21 (three a CU) are not: 64 x 4 x 4 x 16,
// N_v = 12, 105 us against 148 (16 x 8 x 8 x 16 122 and 165).  Elsewhere 21 (32^4 6.23 ms, 6.26 in
// chunks of 16).
inline bool bri_short_chunks(const Geom& g, int nb, bool pairs) {
  const uint64_t cus = uint64_t(device_cus());
  return pairs && nb == 12 && bri_blocks(g, 16, 12) <= 4 * cus && bri_blocks(g, 21, 12) > 3 * cus;
}

// D_B: a workgroup takes its 27 runs one after the other, 75 to 120 us, so on lattices of
// a few rounds of workgroups the number of rounds decides (two a CU are resident, three of
// C64 pairs in more than four columns; of the direct kernel two in C64, one in C128 and at
// N_v = 2).  Measured, us here and by the direct kernel:
// C64: less than a wave per SIMD to the direct kernel (8^4, N_v = 12 73 and 69; 12 x 8^3, N_v =
// 4 78 and 71); N_v = 1 too (12^3 x 24 1.4 times, at the largest 0.9); one or two rounds
// there against one more here (12^3 x 16, N_v = 4 155 and 101, N_v = 9 221 and 189; 12^4, N_v = 5 151
// and 106; the same number, 14x13x12x16, N_v = 4 155 and 169).
// C128: few sites (4^4, N_v = 12 73 and 59, N_v = 4 90 and 65; from 1536 at N_v >= 5 79 and 84); N_v = 3
// and 4 unless there are fewer rounds here (16 x 8 x 8 x 16, N_v = 4 128 and 106; 12^3 x 16
// 273 and 211; 12^4 166 and 195; 16^4 387 and 602), N_v = 2 where there are more (12^3 x 16 259 and
// 168; 16^4 362 and 494).
// DSLASH_BRI_LANES: this kernel from so many (site, column) pairs on, whatever else.
inline bool brillouin_flat_pays(int dtype, const Geom& g) {
  const uint64_t pairs = uint64_t(g.vol) * uint64_t(g.nv), cus = uint64_t(device_cus());
  if (knobs().bri_lanes.set) return pairs >= uint64_t(knobs().bri_lanes.value < 0 ? 0 : knobs().bri_lanes.value);
  const int nv = g.nv, nb = bri_block(dtype, nv);
  const uint64_t here = (dtype == DT_C64 && nv % 2 == 0 && nb > 4 ? 3 : 2) * cus;
  const uint64_t there = (dtype == DT_C64 && nv != 2 ? 2 : 1) * cus;
  const dim3 direct = site_v_shape(g.vol, nv).grid;
  const uint64_t rounds =
      bri_short_chunks(g, nb, dtype == DT_C64 && nv % 2 == 0) ? 1 : (bri_blocks(g, bri_sites(dtype, nb), nb) + here - 1) / here;
  const uint64_t rounds_direct = (uint64_t(direct.x) * direct.y + there - 1) / there;
  if (dtype == DT_C64) return nv > 1 && pairs >= 256 * cus && (rounds_direct > 2 || rounds <= rounds_direct);
  if (nv >= 3 && g.vol < 6 * cus) return false;
  if (nv == 3 || nv == 4) return rounds < rounds_direct;
  return nv != 2 || rounds_direct > 2 || rounds <= rounds_direct;
}

// The gradient with respect to W: a workgroup takes its blocks of columns one after the
// other, about 150 us each in C128 and 60 in C64, so it is the lanes of one block that have
// to fill the chip.  Fewest of them, us here and by the direct kernel: C128 160 a CU (N_v = 12,
// 6^3 x 8 153 and 83, 8^4 175 and 213; N_v = 24 332 and 184, 372 and 461), below N_v = 6 384 a CU
// (N_v = 5, 16 x 8 x 8 x 16 1.16 times, 14x13x12x16 0.94; 256 at N_v = 4, 64 x 4 x 4 x 16 274 and
// 315), below N_v = 4 never; C64 224 a CU (N_v =
// 48, 6^3 x 8 175 and 121; N_v = 20, 8^4 165 and 131, 12 x 8^3 0.58 times), and 256 of all columns
// (8^4, N_v = 12 84 and 63; 12 x 8^3 97 and 125).
inline bool brillouin_wgrad_pays(int dtype, const Geom& g) {
  const uint64_t pairs = uint64_t(g.vol) * uint64_t(g.nv), cus = uint64_t(device_cus());
  if (knobs().bri_lanes.set) return pairs >= uint64_t(knobs().bri_lanes.value < 0 ? 0 : knobs().bri_lanes.value);
  const int nv = g.nv, nb = bri_block(dtype, nv);
  const uint64_t lanes = pairs / uint64_t((nv + nb - 1) / nb);
  if (dtype == DT_C64) return pairs >= 256 * cus && lanes >= 224 * cus;
  return nv >= 4 && lanes >= (nv == 4 ? 256 : nv == 5 ? 384 : 160) * cus;
}

}  // namespace dsl
