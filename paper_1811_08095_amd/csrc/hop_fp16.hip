// The hopping kernels of FP16 storage (hop_kernel.h), a translation unit of its own
// so that the four precisions compile side by side.
#include "hop_kernel.h"

namespace odwf {
hipError_t launch_hop_fp16(const HopArgs& a, int Ns, hipStream_t st) { return launch_hop_p<SP16>(a, Ns, a.dag, st); }
}  // namespace odwf
