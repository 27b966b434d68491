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
// traversal) and leaves at most a tenth of its lanes idle.  Half of them (128
// threads) pay in FP64 and FP32 (16^4 x 16, one right-hand side, us per CG
// iteration: 432 against 459 and 238 against 254), not in 16-bit storage (210
// against 205).
int hop_spb(int hx, int nrhs, int Ns, int prec) {
  const int inner = nrhs * Ns;
  const int most = inner >= 256 ? 1 : 256 / inner;
  if (hx % most == 0) return most;
  const bool half = prec == PREC64 || prec == PREC32;
  for (int spb = most - 1; half ? 2 * spb >= most : 2 * spb > most; spb--)
    if (hx % spb == 0 && 10 * spb * inner >= 9 * ((spb * inner + 63) & ~63)) return spb;
  return most;
}

// Small launches take the four-wave kernel: 64 lanes of columns a block, up to
// 768 blocks in FP64 (512 fit the chip by LDS) and 1024 in the reduced
// precisions.  Measured in us per CG iteration, four-wave kernel against the
// other, one right-hand side: N_s = 16, 4^4 46 / 65 (FP64) and 50 / 62 (FP32);
// 8^4 (512 blocks) 68 / 85 and 63 / 73; 8^3 x 16 (1024) 100 / 90 and 65 / 75;
// 16^2 x 8^2 (2048) 173 / 129 and 108 / 92; N_s = 8, 10^4 (625) 82 / 90 and 58 / 75.
// N_s = 4, 8^2 x 16^2 (512) 77 / 111 and 67 / 81, 8 x 12 x 16^2 (768) 99 / 114 and 67 / 86.
// Three right-hand sides: N_s = 8, 6x10x6x8 (720) 81 / 87 and 58 / 72; N_s = 16,
// 8^3 x 4 (1024) 94 / 89 and 75 / 84.
bool hop_small(const Geom& g, int nrhs, int Ns, int prec) {
  if (!dense_ns(Ns) || nrhs * Ns > 64) return false;
  const int spb = 64 / (nrhs * Ns);
  return (g.h + spb - 1) / spb <= (prec == PREC64 ? 768 : 1024);
}

int hop_nblocks(const Geom& g, int nrhs, int Ns, int prec) {
  const int spb = hop_launch_spb(g, nrhs, Ns, prec, false);
  return (int)((g.h + spb - 1) / spb);
}

// sites per block of a launch (plain launches, which carry no partial sums, may
// use smaller blocks: shorter x-row segments, so more of them per XCD share its L2)
int hop_launch_spb(const Geom& g, int nrhs, int Ns, int prec, bool plain) {
  if (hop_small(g, nrhs, Ns, prec) && !(plain && prec != PREC64)) return 64 / (nrhs * Ns);
  const int hx = g.L[0] / 2;
  const int threads = !plain ? 256 : (prec == PREC64 ? ODWF_HOP_THREADS64 : ODWF_HOP_THREADS32);
  if (plain && prec == PREC16) return std::max(1, 256 / (nrhs * Ns));  // (its two paths differ in rounding)
  if (threads == 256) return hop_spb(hx, nrhs, Ns, prec);
  const int spb = std::max(1, threads / (nrhs * Ns));
  return hx % spb == 0 ? spb : hop_spb(hx, nrhs, Ns, prec);
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
