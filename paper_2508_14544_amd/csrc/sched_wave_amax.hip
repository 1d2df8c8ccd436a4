// sched_wave_amax.hip -- the one-wave kernels of A_max (see sim_wave.hpp).
#include "sim_wave.hpp"

namespace sk {
SK_WAVE_KERNELS(, SCHED_AMAX)
}  // namespace sk
