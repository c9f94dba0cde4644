// Sweep C for d = 64.
#include "sweep_c_impl.h"

namespace intattn {
namespace sweepc {
template int launch<64, false>(const FwdParams &, int, hipStream_t);
} // namespace sweepc
} // namespace intattn
