// row-form stencil step kernels for element type double
#include "hrow_impl.hpp"

namespace sparc {
template int hrow_single<double>(sparc_ctx*, const StepArgs<double>&, const RowCfg&, int64_t);
template int hrow_batched<double>(sparc_ctx*, const void*, const int*, int, int64_t, const RowCfg&, int);
}  // namespace sparc
