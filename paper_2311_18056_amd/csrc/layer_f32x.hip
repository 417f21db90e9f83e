// FP32 instantiations of the persistent layer kernel for closed loops and Ruiz-scaled problems.
#include "layer_impl.h"

namespace rqp {
const void* layer_fn_f32x(int nc, bool more) { return fn_for<float, true>(nc, more); }
}  // namespace rqp
