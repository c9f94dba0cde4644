// Sweep C for d = 128, the keys split over several workgroups.
#include "sweep_c_impl.h"

namespace intattn {
namespace sweepc {
template int launch<128, true>(const FwdParams &, int, hipStream_t);
} // namespace sweepc
} // namespace intattn
