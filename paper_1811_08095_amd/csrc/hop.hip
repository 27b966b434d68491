// Launch geometry and dispatch of the hopping kernels (hop_kernel.h).
#include <algorithm>

#include "kernels.h"

namespace odwf {

// threads per block of the plain hop: FP64 rows are twice as long, and 8-site
// segments (128 threads at Ns = 16) fetch 20 % less and run 5 % faster at
// 64^4 x 16; in FP32 they fetch 10 % less in the same time
#ifndef ODWF_HOP_THREADS64
#define ODWF_HOP_THREADS64 128
#endif
#ifndef ODWF_HOP_THREADS32
#define ODWF_HOP_THREADS32 256
#endif

// Sites per block of a fused launch: as many as 256 threads hold, or fewer where
// that makes every block a segment of one x-row (scalar row addressing, tiled
// traversal) and leaves at most a tenth of its lanes idle.
int hop_spb(int hx, int nrhs, int Ns) {
  const int inner = nrhs * Ns;
  const int most = inner >= 256 ? 1 : 256 / inner;
  if (hx % most == 0) return most;
  for (int spb = most - 1; 2 * spb > most; spb--)
    if (hx % spb == 0 && 10 * spb * inner >= 9 * ((spb * inner + 63) & ~63)) return spb;
  return most;
}

int hop_nblocks(const Geom& g, int nrhs, int Ns) {
  const int spb = hop_spb(g.L[0] / 2, nrhs, Ns);
  return (int)((g.h + spb - 1) / spb);
}

// sites per block of a launch (plain launches, which carry no partial sums, may
// use smaller blocks: shorter x-row segments, so more of them per XCD share its L2)
int hop_launch_spb(int hx, int nrhs, int Ns, int prec, bool plain) {
  const int threads = !plain ? 256 : (prec == PREC64 ? ODWF_HOP_THREADS64 : ODWF_HOP_THREADS32);
  if (threads == 256) return hop_spb(hx, nrhs, Ns);
  const int spb = std::max(1, threads / (nrhs * Ns));
  return hx % spb == 0 ? spb : hop_spb(hx, nrhs, Ns);
}

hipError_t launch_hop_fp64(const HopArgs& a, int Ns, hipStream_t st);
hipError_t launch_hop_fp32(const HopArgs& a, int Ns, hipStream_t st);
hipError_t launch_hop_fp16(const HopArgs& a, int Ns, hipStream_t st);
hipError_t launch_hop_bf16(const HopArgs& a, int Ns, hipStream_t st);

hipError_t launch_hop(const HopArgs& a, int prec, int Ns, hipStream_t st) {
  switch (prec) {
    case PREC64: return launch_hop_fp64(a, Ns, st);
    case PREC32: return launch_hop_fp32(a, Ns, st);
    case PREC16: return launch_hop_fp16(a, Ns, st);
    case PRECB16: return launch_hop_bf16(a, Ns, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace odwf
