// Row-staged D_W and even-odd hop, C64 storage (half-spinor neighbour rows); see wilson_rows.hpp.
#include "wilson_rows.hpp"

namespace dsl {

hipError_t wilson_rows_c64(const RowsCall& c) { return rows_dispatch<C64, 3>(c); }

}  // namespace dsl
