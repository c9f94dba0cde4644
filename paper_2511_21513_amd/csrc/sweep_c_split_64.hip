// Sweep C for d = 64, the keys split over several workgroups.
#include "sweep_c_impl.h"

namespace intattn {
namespace sweepc {
template int launch<64, true>(const FwdParams &, int, hipStream_t);
} // namespace sweepc
} // namespace intattn
