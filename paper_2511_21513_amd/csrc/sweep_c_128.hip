// Sweep C for d = 128.
#include "sweep_c_impl.h"

namespace intattn {
namespace sweepc {
template int launch<128, false>(const FwdParams &, int, hipStream_t);
} // namespace sweepc
} // namespace intattn
