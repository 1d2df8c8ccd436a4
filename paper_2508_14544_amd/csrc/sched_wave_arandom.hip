// sched_wave_arandom.hip -- the one-wave kernels of A_random (see sim_wave.hpp).
#include "sim_wave.hpp"

namespace sk {
SK_WAVE_KERNELS(, SCHED_ARANDOM)
}  // namespace sk
