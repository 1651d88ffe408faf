// Global-gather density and force kernels: mixed precision, one species.
#include "kernels_global.h"

namespace mdk {
template void density_of<float, true>(const Buffers&, int, int, const KernelShape&, const PotArgs&, int, int, hipStream_t);
template void force_of<float, true>(const Buffers&, int, int, const KernelShape&, const PotArgs&, int, ForceFlags, double,
                                 const md_state&, hipStream_t);
}  // namespace mdk
