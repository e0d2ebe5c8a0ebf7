// row-form stencil step kernels for element type cf
#include "hrow_impl.hpp"

namespace sparc {
template int hrow_single<cf>(sparc_ctx*, const StepArgs<cf>&, const RowCfg&, int64_t);
template int hrow_batched<cf>(sparc_ctx*, const void*, const int*, int, int64_t, const RowCfg&, int);
}  // namespace sparc
