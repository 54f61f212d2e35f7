// Row-staged D_W and even-odd hop: which launches take the kernels of
// wilson_rows.hpp (rows_shape.hpp: in which shape).
#include "rows_shape.hpp"

namespace dsl {

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
