// Row-staged D_W and even-odd hop, BF16 storage (own-row buffer); see wilson_rows.hpp.
#include "wilson_rows.hpp"

namespace dsl {

hipError_t wilson_rows_bf16(const RowsCall& c) { return rows_dispatch<BF16, 2>(c); }

}  // namespace dsl
