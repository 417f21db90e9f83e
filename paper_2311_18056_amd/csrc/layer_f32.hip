// FP32 instantiations of the persistent layer kernel for plain solves.
#include "layer_impl.h"

namespace rqp {
const void* layer_fn_f32(int nc, bool more) { return fn_for<float, false>(nc, more); }
}  // namespace rqp
