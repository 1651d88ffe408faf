// Global-gather density and force kernels: FP64, one species.
#include "kernels_global.h"

namespace mdk {
template void density_of<double, true>(const Buffers&, int, int, const KernelShape&, const PotArgs&, int, int, hipStream_t);
template void force_of<double, true>(const Buffers&, int, int, const KernelShape&, const PotArgs&, int, ForceFlags, double,
                                 const md_state&, hipStream_t);
}  // namespace mdk
