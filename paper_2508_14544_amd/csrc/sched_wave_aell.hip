// sched_wave_aell.hip -- the one-wave kernels of A_l (see sim_wave.hpp).
#include "sim_wave.hpp"

namespace sk {
SK_WAVE_KERNELS(, SCHED_AELL)
}  // namespace sk
