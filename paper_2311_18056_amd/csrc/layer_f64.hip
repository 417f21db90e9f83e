// FP64 instantiations of the persistent layer kernel for plain solves.
#include "layer_impl.h"

namespace rqp {
const void* layer_fn_f64(int nc, bool more) { return fn_for<double, false>(nc, more); }
}  // namespace rqp
