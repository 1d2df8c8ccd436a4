// sched_wave_hsf.hip -- the one-wave kernels of H-SF (see sim_wave.hpp).
#include "sim_wave.hpp"

namespace sk {
SK_WAVE_KERNELS(, SCHED_HSF)
}  // namespace sk
