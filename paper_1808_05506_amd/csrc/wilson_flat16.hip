// Flat D_W kernels, BF16 and F16 storage (see wilson_flat.hpp).
#include "wilson_flat.hpp"

namespace dsl {

hipError_t launch_wilson_flat16(int dtype, int vw, bool adj, const Geom& g, const FlatArgs& a, bool compressed,
                                hipStream_t st) {
  if (dtype == DT_BF16) return flat_forms16<BF16>(vw, adj, g, a, compressed, st);
  return flat_forms16<F16>(vw, adj, g, a, compressed, st);
}

}  // namespace dsl
