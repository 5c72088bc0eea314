// FP32 tier of the sweep kernels: hardware reciprocal for divisions and the
// fused multiply-adds written out in the shared device functions.
#include "sweep_kernels.h"

namespace mhd {
template hipError_t launch_fluid<float>(const SweepParams<float>&, int, const LaunchTuning&, hipStream_t);
template bool sweep_uses_tiles<float>(const int[3], int, int, const LaunchTuning&);
template hipError_t launch_magnetic<float>(const SweepParams<float>&, int, const LaunchTuning&, hipStream_t);
template hipError_t launch_magfluid<float>(const SweepParams<float>&, int, const LaunchTuning&, hipStream_t);
template hipError_t launch_magmagfluid<float>(const SweepParams<float>&, int, const LaunchTuning&, hipStream_t);
template hipError_t launch_batch_op<float>(const BatchParams<float>&, int, int, int, hipStream_t);
template hipError_t launch_batch_tile_op<float>(const BatchParams<float>&, int, int, int, hipStream_t);
}  // namespace mhd
