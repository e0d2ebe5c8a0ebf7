// row-form stencil step kernels for element type float
#include "hrow_impl.hpp"

namespace sparc {
template int hrow_single<float>(sparc_ctx*, const StepArgs<float>&, const RowCfg&, int64_t);
template int hrow_batched<float>(sparc_ctx*, const void*, const int*, int, int64_t, const RowCfg&, int);
}  // namespace sparc
