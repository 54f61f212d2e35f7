// Row-staged D_W and even-odd hop, FP16 storage (one row buffer); see wilson_rows.hpp.
#include "wilson_rows.hpp"

namespace dsl {

hipError_t wilson_rows_f16(const RowsCall& c) { return rows_dispatch<F16, 0>(c); }

}  // namespace dsl
