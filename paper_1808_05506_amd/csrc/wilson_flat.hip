// Flat D_W kernels (see wilson_flat.hpp): the dispatch and the
// C64 and C128 forms.
#include "flat_rule.hpp"
#include "wilson_flat.hpp"

namespace dsl {

hipError_t launch_wilson_flat(bool adj, int dtype, const Geom& g, const void* U, const void* in, void* out, double mass,
                              hipStream_t st, const void* clover, bool compressed) {
  if (knobs().rows.get(1) == 0 || !flat_covers(g, dtype)) return hipErrorNotSupported;
  const int vw = flat_vw(dtype, g.nv, aligned16(in) && aligned16(out));
  if (!wilson_flat_pays(dtype, g, vw, clover != nullptr, compressed)) return hipErrorNotSupported;
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
