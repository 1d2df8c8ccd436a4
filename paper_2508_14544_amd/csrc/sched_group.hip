// sched_group.hip -- the workgroup kernels (W waves per instance, ROWS
// register rows each; see k_simulate_group in sim_device.hpp), compiled on
// their own.
#include "sim_device.hpp"

namespace sk {
SK_GROUP_KERNELS()
SK_GROUP_KERNELS_AMIN()
}  // namespace sk
