// sched_group.hip -- the workgroup kernels (W waves per instance, ROWS
// register rows each; see k_simulate_group in sim_device.hpp), compiled on
// their own, A_min's unless SK_SEPARATE_KERNELS leaves them to sched_group_amin.hip
// (built concurrently, with flags of its own).
#include "sim_device.hpp"

namespace sk {
SK_GROUP_KERNELS()
#ifndef SK_SEPARATE_KERNELS
SK_GROUP_KERNELS_AMIN()
#endif
}  // namespace sk
