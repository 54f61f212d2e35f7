// Flat D_W kernels (see wilson_flat.hpp): the dispatch and the
// C64 and C128 forms.
#include "wilson_flat.hpp"

namespace dsl {

// Left to the direct kernel, which is faster there: N_v = 1 (16^3 x 32 C64 26.6
// against 66.4 us, its site is one contiguous run), and lanes of one 8- or 4-byte
// word where the links are short or few lanes share them (C64 compressed, N_v = 5,
// 22 x 20 x 13 x 21: 71.5 against 93 us; BF16, N_v = 5, 20 x 18 x 14 x 22: 59.9
// against 68; FP16, N_v = 7: 88.9 against 81.8, so from N_v = 6 on this one).
hipError_t launch_wilson_flat(bool adj, int dtype, const Geom& g, const void* U, const void* in, void* out, double mass,
                              hipStream_t st, const void* clover, bool compressed) {
  if (knobs().rows.get(1) == 0 || !flat_covers(g, dtype)) return hipErrorNotSupported;
  const int vw = flat_vw(dtype, g.nv, aligned16(in) && aligned16(out));
  const bool one_word = dtype != DT_C128 && vw == 1;
  if (g.nv == 1 || (!clover && one_word && (compressed || g.nv < 6))) return hipErrorNotSupported;
  // Few columns a site with the clover term or compressed links (21x16x17x33, us here
  // and directly): C64 clover N_v = 2 171 and 128, compressed N_v = 4 106 and 85, N_v = 8 148
  // and 161; BF16 clover N_v = 2 102 and 63, N_v = 8 138 and 102, N_v = 16 209 and 206 (F16
  // 216 and 293), compressed N_v = 8 103 and 90, N_v = 16 170 and 198.
  if (!knobs().flat_lanes.set &&
      ((clover && g.nv <= 2) || ((clover || compressed) && vw == 4 && g.nv < 16) ||
       (compressed && dtype == DT_C64 && g.nv < 8)))
    return hipErrorNotSupported;
  // Small lattices: several columns a lane and chunks of up to 256 lanes leave the
  // chip idle that the direct kernel fills.  Fewest lanes for this one, us here
  // and there: FP64 144k (N_v = 4, 110k 27.8 and 20.9; N_v = 12, 172k 30.0 and 30.3); two
  // columns 64k (BF16 N_v = 2, 27k 16.6 and 10.2, N_v = 6, 83k 16.2 and 20.7), with the
  // clover term 128k (C64 N_v = 4, 55k 22.8 and 18.1, 131k 42.4 and 45.3); compressed
  // or four columns 256k (C64 N_v = 4, 131k 30.1 and 26.9; F16 N_v = 4 with the clover
  // term, 65k 42.4 and 21.8).  One FP32 column a lane: any (N_v = 5 with the
  // clover term, 8^4 8.5 and 9.9).
  const uint32_t fewest = dtype == DT_C128 ? 144 : one_word ? 0 : (compressed || vw == 4) ? 256 : clover ? 128 : 64;
  if (size_t(g.vol) * size_t(g.nv / vw) < size_t(knobs().flat_lanes.get(int(fewest * 1024))))
    return hipErrorNotSupported;
  const FlatArgs a{U, in, clover, out, mass};
  if (dtype == DT_BF16 || dtype == DT_F16) return launch_wilson_flat16(dtype, vw, adj, g, a, compressed, st);
  // NVC: N_v known at compile time, so that the offsets of a site's components are part
  // of the load instructions (FP64, N_v = 12, 24^3 x 48: 1049 us, 1102 without; 16^3 x 32 204
  // and 215).
  if (dtype == DT_C128)
    return g.nv == 12 ? flat_forms<C128, double, 1, 12>(adj, g, a, compressed, st)
                      : flat_forms<C128, double, 1>(adj, g, a, compressed, st);
  return vw == 2 ? flat_forms<C64, float, 2>(adj, g, a, compressed, st) : flat_forms<C64, float, 1>(adj, g, a, compressed, st);
}

}  // namespace dsl
