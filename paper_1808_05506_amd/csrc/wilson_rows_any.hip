// Row-staged D_W in C64 storage at the block sizes that wilson_rows_c64.hip does
// not take: N_v = 2 .. 23, half-spinor neighbour rows at even N_v, whole rows at
// odd ones (a 16-byte piece then holds words of two components).  Two rows in
// flight at odd N_v and N_v = 2 (its links take more registers), three at the others.
#include "wilson_rows.hpp"

namespace dsl {

hipError_t wilson_rows_c64_any(const RowsCall& c) {
#define DSL_NV(N) \
  case N: return march_call<(N) % 2 || (N) == 2 ? 2 : 3, N, C64, 9, (N) % 2 == 0 ? 3 : 2, 4>(c);
  switch (c.g->nv) {
    DSL_NV(2) DSL_NV(3) DSL_NV(5) DSL_NV(6) DSL_NV(7) DSL_NV(9) DSL_NV(10) DSL_NV(11) DSL_NV(13) DSL_NV(14)
    DSL_NV(15) DSL_NV(17) DSL_NV(18) DSL_NV(19) DSL_NV(20) DSL_NV(21) DSL_NV(22) DSL_NV(23)
  }
#undef DSL_NV
  return hipErrorNotSupported;
}

}  // namespace dsl
