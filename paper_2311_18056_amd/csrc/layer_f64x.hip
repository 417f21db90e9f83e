// FP64 instantiations of the persistent layer kernel for closed loops and Ruiz-scaled problems.
#include "layer_impl.h"

namespace rqp {
const void* layer_fn_f64x(int nc, bool more) { return fn_for<double, true>(nc, more); }
}  // namespace rqp
