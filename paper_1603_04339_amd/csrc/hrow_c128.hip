// row-form stencil step kernels for element type cd
#include "hrow_impl.hpp"

namespace sparc {
template int hrow_single<cd>(sparc_ctx*, const StepArgs<cd>&, const RowCfg&, int64_t);
template int hrow_batched<cd>(sparc_ctx*, const void*, const int*, int, int64_t, const RowCfg&, int);
}  // namespace sparc
