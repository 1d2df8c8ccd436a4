// sched_group_amin.hip -- the workgroup kernels of A_min (see k_simulate_group in
// sim_device.hpp).
#include "sim_device.hpp"

namespace sk {
SK_GROUP_KERNELS_AMIN()
}  // namespace sk
