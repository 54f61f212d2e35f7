// Flat D_W kernels on the full lattice, BF16 and F16 storage (see wilson_flat.hpp).
#include "wilson_flat.hpp"

namespace dsl {

hipError_t launch_wilson_flat16(int dtype, int vw, bool adj, const Geom& g, const FlatArgs& a, bool compressed, int epi,
                                hipStream_t st, EpiArgs& ea) {
  if (dtype == DT_BF16) return flat_forms16<false, BF16>(vw, adj, g, a, compressed, epi, st, ea);
  return flat_forms16<false, F16>(vw, adj, g, a, compressed, epi, st, ea);
}

}  // namespace dsl
