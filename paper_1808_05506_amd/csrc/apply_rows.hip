// Row-staged D_W and even-odd hop: which launches take the kernels of
// wilson_rows.hpp, and in which shape.
#include "wilson_rows.hpp"

namespace dsl {

// Sites per chunk R and halo sites hn.  A chunk of one x-row (hn = 2) where the
// fewest chunks of at most 16 sites (more where fewer than 128 lanes would
// result) divide the row and leave at most a tenth of the lanes idle: it has the
// fewest halo loads and registers (16^3 x 32, N_v = 12: 92.5 us against 107.6
// with hn = 4; FP32 N_v = 24 alone is faster with hn = 4: 184 us against 192, 951
// against 995 on 24^3 x 48).  Elsewhere chunks across row ends of at most 256 lanes (hn =
// 4), and of those from the longest down to half of it the one that leaves
// the fewest lanes idle in the last chunk of the plane and the last wave
// (24^3 x 48: 499 us at R = 21 against 601 with rows of 12; 34^3 x 68: 2225
// against 2813).  DSLASH_ROW_SITES overrides R (hn = 4); false: no such kernel
// (fewer than 64 lanes, or a chunk too short for its halo).  DSLASH_ROWS=2 asks
// for these kernels where a chunk of one x-row alone holds its halo.
// late: no such whole chunks of a row (whatever hn the launch takes).
// pp: the buffer scheme (the one-row kernels: 0); two workgroups a CU need 80 KB.
static bool rows_shape(const Geom& g, int dtype, int pp, bool any_nv, bool knob_form, int& R, int& hn,
                       bool& late) {
  const int nv = g.nv, wb = int(dtype_bytes(dtype));
  const uint32_t plane = uint32_t(g.n[0]) * uint32_t(g.n[1]);
  if (knobs().rows.get(1) == 2) {
    if (any_nv) return false;
    int r = knobs().row_sites.get(row_sites_default(g.n[0], nv));
    if (r > g.n[0]) r = g.n[0];
    if (r < 1 || r * nv > 256 || r * nv < 64 || !halo_fits(r, nv, wb, 2)) return false;
  }
  const int whole = row_sites_default(g.n[0], nv);
  late = any_nv || whole <= 0 || g.n[0] % whole != 0 || 10 * whole * nv < 9 * ((whole * nv + 63) / 64) * 64 ||
         whole * nv > 256 || !halo_fits(whole, nv, wb, 2);
  hn = 4;
  if (knobs().row_sites.set) {
    R = knobs().row_sites.value;
    if (R > int(plane)) R = int(plane);
  } else {
    R = whole;
    if (!late && !knob_form) {
      hn = nv > 16 && dtype == DT_C64 && halo_fits(R, nv, wb, 4) ? 4 : 2;
      return true;
    }
    int rmax = 256 / nv;
    if (rmax < 1) return false;
    while (rmax > 1 && march_lds(rmax, nv, wb, pp, 4) > 76 * 1024) --rmax;
    if (uint32_t(rmax) > plane) rmax = int(plane);
    R = rmax;
    uint64_t cost = 0;
    for (uint32_t k = (plane + uint32_t(rmax) - 1) / uint32_t(rmax);; ++k) {  // chunks per plane
      const int r = int((plane + k - 1) / k);
      if (2 * r < rmax || !halo_fits(r, nv, wb, 4)) break;
      const uint64_t lanes = uint64_t(k) * uint32_t((r * nv + 63) / 64);
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
static int march_tsteps(const Geom& g, int R, int hn, int pp, int dtype) {
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

// Small lattices of 16-bit storage are faster by the direct kernel, which has more
// lanes in flight: below `lanes` (site, column) pairs, unless a tuning variable or
// a fused epilogue asks for the rows.  D_W, us by rows and directly: N_v = 4, 110k
// pairs 14.3 and 7.9 (262k 15.0 against 33 before); N_v = 24, 6k 6.6 and 5.4.
// Compressed links, 49k: 7.2 and 6.4.  Even-odd hop: F16 N_v = 4, 55k 9.4 and 7.9; C64
// N_v = 12, 25k 7.2 and 6.6.
static bool rows_too_small(const Geom& g, size_t lanes, int epi) {
  const Knobs& k = knobs();
  const bool asked = k.rows.get(1) == 2 || k.row_sites.set || k.row_depth.set || k.tsteps.set || k.march_pp.set;
  return !asked && epi == EPI_STORE && size_t(g.vol) * size_t(g.nv) < size_t(k.flat_lanes.get(int(lanes * 1024)));
}

static hipError_t rows_launch(int dtype, bool any_nv, const RowsCall& c) {
  if (any_nv) return wilson_rows_c64_any(c);
  switch (dtype) {
    case DT_C64: return wilson_rows_c64(c);
    case DT_BF16: return wilson_rows_bf16(c);
    case DT_F16: return wilson_rows_f16(c);
  }
  return hipErrorNotSupported;
}

// Row-staged even-odd hop for N_v = 4, 8, 12, 16, 24 (C64, BF16, F16
// storage), with the chunk rule of the full-lattice kernels on the packed
// planes; hipErrorNotSupported otherwise (the caller then uses the direct
// kernel).  DSLASH_ROWS=0 disables it.
hipError_t launch_wilson_eo_rows(bool adj, int dtype, const EoGeom& e, int parity, const void* Uo, const void* Ui,
                                 const void* in, void* out, const void* add, double c_add, double c_hop,
                                 hipStream_t st, int epi, EpiArgs* ea) {
  if (knobs().rows.get(1) == 0) return hipErrorNotSupported;
  if (!aligned16(Uo) || !aligned16(Ui) || !aligned16(in) || !aligned16(out) || !aligned16(add))
    return hipErrorNotSupported;
  if (epi != EPI_STORE && !ea) return hipErrorNotSupported;
  EpiArgs none;
  const int nv = e.nv;
  if (nv != 4 && nv != 8 && nv != 12 && nv != 16 && nv != 24) return hipErrorNotSupported;
  const int pdims[4] = {e.nh, e.n[1], e.n[2], e.n[3]};
  const Geom g = make_geom(pdims, nv);
  if (rows_too_small(g, dtype == DT_C64 ? 32 : nv == 4 ? 96 : 64, epi)) return hipErrorNotSupported;
  RowsCall c{};
  if (!rows_shape(g, dtype, 0, false, false, c.R, c.hn, c.late)) return hipErrorNotSupported;
  c.eo = true;
  c.adj = adj;
  c.g = &g;
  c.xcd = knobs().xcd.get(1) != 0;
  c.U = Uo;
  c.Ub = Ui;
  c.in = in;
  c.add = add;
  c.out = out;
  c.parity = parity;
  c.c_add = c_add;
  c.c_hop = c_hop;
  c.st = st;
  c.epi = epi;
  c.ea = ea ? ea : &none;
  return rows_launch(dtype, false, c);
}

// Row-staged D_W with FP32 arithmetic: C64, BF16 and F16 storage at N_v = 4, 8,
// 12, 16, 24, C64 also at the other N_v up to 23.  Returns
// hipErrorNotSupported when the configuration is not covered (the caller then
// uses the flat kernel).  DSLASH_ROWS=0 disables it.
//
// DSLASH_TSTEPS: t steps per workgroup of the t-marching kernel (march_tsteps;
// 0 selects the kernel with one output row per workgroup).
// DSLASH_ROW_DEPTH: rows in flight per workgroup (default march_depth when
// marching, 2 for the one-row kernel).
// DSLASH_MARCH_PP: 0 = one row buffer, 1 = two used in turn (one barrier per
// staged row), 2 = an own-row buffer that keeps the +t row for the next step
// plus two used in turn, 3 = the same with half-spinor neighbour rows (FP32
// storage only; others fall back to 2).
// Default: FP32 storage takes 3 (full or compressed links; 2 at odd N_v), BF16
// storage 2, FP16 storage and other compressed links one buffer.
hipError_t launch_wilson_rows(bool adj, int dtype, const Geom& g, const void* U, const void* in, void* out,
                              double mass, hipStream_t st, const void* clover, bool compressed, int epi,
                              EpiArgs* ea) {
  if (knobs().rows.get(1) == 0 || dtype == DT_C128) return hipErrorNotSupported;
  if (!aligned16(U) || !aligned16(in) || !aligned16(out) || !aligned16(clover)) return hipErrorNotSupported;
  if (epi != EPI_STORE && (!ea || clover || compressed)) return hipErrorNotSupported;
  EpiArgs none;
  const int nv = g.nv;
  const bool any_nv = nv != 4 && nv != 8 && nv != 12 && nv != 16 && nv != 24;
  if (any_nv && (dtype != DT_C64 || nv < 2 || nv > 23)) return hipErrorNotSupported;
  if (nv != 12 && (clover || compressed || epi != EPI_STORE)) return hipErrorNotSupported;
  if (rows_too_small(g, compressed ? 128 : dtype == DT_C64 ? 1 : nv == 4 ? 128 : 16, epi)) return hipErrorNotSupported;
  // N_v = 12 with the clover term or a tuning variable set: hn = 4
  const bool knob_form =
      nv == 12 && (clover || knobs().tsteps.set || knobs().march_pp.set || (knobs().row_depth.set && epi == EPI_STORE));
  int pp = clover ? 0 : (dtype == DT_C64 ? (nv % 2 == 0 ? 3 : 2) : (dtype == DT_BF16 && !compressed ? 2 : 0));
  if (nv == 12 && knobs().tsteps.set) pp = 0;
  RowsCall c{};
  if (!rows_shape(g, dtype, pp, any_nv, knob_form, c.R, c.hn, c.late)) return hipErrorNotSupported;
  c.pp = pp;
  c.tsteps = knobs().tsteps.set ? knobs().tsteps.value : march_tsteps(g, c.R, c.hn, pp, dtype);
  if (nv != 12) {
    if (c.tsteps <= 0) return hipErrorNotSupported;
  } else {
    c.pp = knobs().march_pp.get(c.pp);
    if (c.pp == 3 && dtype != DT_C64) c.pp = 2;
    if (c.pp < 0 || c.pp > 3 || (compressed && c.pp != 3)) c.pp = 0;
  }
  // the clover term is fused into the one-row-per-workgroup kernel only;
  // compressed links are read by the t-marching kernel only
  if (compressed && (c.tsteps <= 0 || clover)) return hipErrorNotSupported;
  const bool march = c.tsteps > 0 && !clover;
  if (!march && epi != EPI_STORE) return hipErrorNotSupported;
  // the fused epilogues take the default depth of the buffer scheme
  const int dflt = march ? march_depth(c.pp) : 2;
  c.depth = epi != EPI_STORE ? dflt : knobs().row_depth.get(dflt);
  c.adj = adj;
  c.g = &g;
  c.xcd = knobs().xcd.get(1) != 0;
  c.U = c.Ub = U;
  c.in = in;
  c.out = out;
  c.clover = clover;
  c.compressed = compressed;
  c.mass = mass;
  c.st = st;
  c.epi = epi;
  c.ea = ea ? ea : &none;
  return rows_launch(dtype, any_nv, c);
}

}  // namespace dsl
