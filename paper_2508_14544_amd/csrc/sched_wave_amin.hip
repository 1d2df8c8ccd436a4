// sched_wave_amin.hip -- the one-wave kernels of A_min (see sim_wave.hpp).
#include "sim_wave.hpp"

namespace sk {
SK_WAVE_KERNELS_AMIN()
}  // namespace sk
