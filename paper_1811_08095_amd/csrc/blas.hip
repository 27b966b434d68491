// BLAS-1 kernels on even/odd half fields and the CG scalar finalisation.
//
// Threads map to 5D sites (j, r, s) with s fastest and a block size that is a
// multiple of nrhs * Ns, so every thread keeps one right-hand side across its
// grid-stride loop and per-right-hand-side reductions stay deterministic:
// per-block partial sums (fixed order) followed by a one-block finalisation
// that sums the partials in a fixed tree.  All accumulations are FP64.
#include "dev_common.h"
#include "kernels.h"

namespace odwf {

static inline int vec_spb(int nrhs, int Ns) {
  const int inner = nrhs * Ns;
  return inner >= 256 ? 1 : 256 / inner;
}

int vec_nblocks(long h, int nrhs, int Ns) {
  const int spb = vec_spb(nrhs, Ns);
  long nb = (h + spb - 1) / spb;
  if (nb > 2048) nb = 2048;
  return (int)nb;
}

// ---------------------------------------------------------------------------
// streaming kernels over 16-byte chunks: where no value depends on its 5D site
// as a whole (FP64 and FP32 storage have no scale) a thread takes UNROLL chunks
// a block apart, so a wave's accesses are contiguous and a thread holds few
// registers.  One lane per 5D site (12 chunks of FP64 a lane for each of x, p, r)
// spilled 500 bytes a lane at the default bounds: the FP64 CG step of 32^3 x 16 x 16
// took 1432 us (4.0 GB), the chunk form 660 us (6.1 TB/s).
// grid.y is the right-hand side; its rows (one site's chunks) lie nrhs rows apart.
// ---------------------------------------------------------------------------
constexpr int UNROLL = 4;
struct ChunkGeom {
  long n;       // chunks of one right-hand side
  FastDiv row;  // chunks of one site
  int nrhs;
  // chunk k of right-hand side r in the field
  __device__ long at(long k, int r) const {
    if (nrhs == 1) return k;
    const long j = k < (1L << 31) ? (long)row.div((uint32_t)k) : k / row.d;
    return k + (j * (nrhs - 1) + r) * row.d;
  }
};
static ChunkGeom chunk_geom(int cpb, long h, int nrhs, int Ns) {
  ChunkGeom g;
  g.row = FastDiv((uint32_t)(12 / cpb * Ns));
  g.n = h * (12 / cpb) * Ns;
  g.nrhs = nrhs;
  return g;
}
static dim3 chunk_grid(const ChunkGeom& g) { return dim3((unsigned)((g.n + 256 * UNROLL - 1) / (256 * UNROLL)), g.nrhs); }
__device__ __forceinline__ long chunk_first() { return (long)blockIdx.x * 256 * UNROLL + threadIdx.x; }

__global__ void __launch_bounds__(256) chunk_zero_kernel(uint4* v, ChunkGeom g) {
  const int r = blockIdx.y;
#pragma unroll
  for (int u = 0; u < UNROLL; u++) {
    const long k = chunk_first() + u * 256;
    if (k < g.n) v[g.at(k, r)] = make_uint4(0, 0, 0, 0);
  }
}
__global__ void __launch_bounds__(256) scale_zero_kernel(float* sc, long n) {
  const long k = (long)blockIdx.x * 256 + threadIdx.x;
  if (k < n) sc[k] = 0.f;
}

// FP64 += FP32, and the FP32 field = 0 behind it
__global__ void __launch_bounds__(256) chunk_32_to_64_kernel(uint4* src, uint4* dst, ChunkGeom g, int lg) {
  const int r = blockIdx.y;
#pragma unroll 2
  for (int u = 0; u < UNROLL; u++) {
    const long k = chunk_first() + u * 256;
    if (k >= g.n) break;
    // FP32 chunk (cg, s) of a site holds components 2 cg, 2 cg + 1: FP64 chunks (2 cg, s), (2 cg + 1, s)
    const long at = g.at(k, r);
    const long cg = at >> lg;  // row * 6 + chunk group; Ns = 2^lg
    const long d0 = at + (cg << lg);
    cpx<float> a[2];
    unpack_chunk<SP32>(src[at], a);
#pragma unroll
    for (int c = 0; c < 2; c++) {
      cpx<double> o;
      unpack_chunk<SP64>(dst[d0 + (c << lg)], &o);
      o = cadd(o, cpx<double>{(double)a[c].re, (double)a[c].im});
      dst[d0 + (c << lg)] = pack_chunk<SP64>(&o, 1.0);
    }
    src[at] = make_uint4(0, 0, 0, 0);
  }
}
__global__ void __launch_bounds__(256) chunk_64_to_32_kernel(const uint4* src, uint4* dst, const CGScal* gate,
                                                             int gate_mode, ChunkGeom g, int lg) {
  const int r = blockIdx.y;
  if (!gate_on(gate, gate_mode, r)) return;
#pragma unroll
  for (int u = 0; u < UNROLL; u++) {
    const long k = chunk_first() + u * 256;
    if (k >= g.n) break;
    const long at = g.at(k, r), s0 = at + (at >> lg << lg);
    cpx<float> b[2];
#pragma unroll
    for (int c = 0; c < 2; c++) {
      cpx<double> a;
      unpack_chunk<SP64>(src[s0 + (c << lg)], &a);
      b[c] = {(float)a.re, (float)a.im};
    }
    dst[at] = pack_chunk<SP32>(b, 1.0f);
  }
}
__global__ void __launch_bounds__(256) chunk_copy_kernel(const uint4* src, uint4* dst, const CGScal* gate, int gate_mode,
                                                         ChunkGeom g) {
  const int r = blockIdx.y;
  if (!gate_on(gate, gate_mode, r)) return;
#pragma unroll
  for (int u = 0; u < UNROLL; u++) {
    const long k = chunk_first() + u * 256;
    if (k < g.n) dst[g.at(k, r)] = src[g.at(k, r)];
  }
}

// The scalars of a CG vector step: the records as they are, or (partial != null)
// formed here from the partial |r|^2 and the records' copies, by every block for
// its right-hand side, one of them writing the record (and its host mirror).
struct StepScal {
  CGScal* scal;
  const double* partial;
  int nblocks;
  CGScal* host;  // pinned mirror, or null
};
__device__ __forceinline__ CGScal step_scal(const StepScal& a, int r, int nrhs, bool writer) {
  if (!a.partial) return a.scal[r];
  __shared__ double tmp[256];
  CGScal c = a.scal[SCAL_COPY + r];
  double v = 0.0;
  for (int b = threadIdx.x; b < a.nblocks; b += 256) v += a.partial[(long)b * nrhs + r];
  tmp[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) tmp[threadIdx.x] += tmp[threadIdx.x + w];
    __syncthreads();
  }
  fin_beta(c, tmp[0]);
  if (writer && threadIdx.x == 0) {
    a.scal[r] = c;
    if (a.host) a.host[r] = c;
  }
  return c;
}

// The solution is touched by the step alone: nontemporal, so that it displaces
// less of what the hops read next (16^4 x 16 FP32, two right-hand sides, 104.7 ->
// 101.5 ms a solve, 32^3 x 16 x 16 520 -> 510 ms; r as well: 8^4 x 16, twelve slots,
// 0.7 % slower, the others up to 0.8 % faster; FP16S 24^4 x 16 384 -> 380 ms).
__device__ __forceinline__ uint4 stream_load(const uint4* p) {
  const u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(w.x, w.y, w.z, w.w);
}
__device__ __forceinline__ void stream_store(uint4* p, const uint4 q) {
  const u32x4 w = {q.x, q.y, q.z, q.w};
  __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
}

// CG vector step:
//   x += alpha p   (for every right-hand side that iterated: alpha != 0, which
//                   includes one that converged at this iteration's beta)
//   p  = r + beta p (for the right-hand sides still active)
//   y += x, x = 0   (FP32 with y: for the right-hand sides that asked for an update)
template <class P>
__global__ void __launch_bounds__(256) chunk_cg_step_kernel(const uint4* r_, uint4* p_, uint4* x_, uint4* y_, StepScal sa,
                                                            ChunkGeom g, int lg) {
  using R = typename P::real;
  constexpr int N = P::CPB;
  const int r = blockIdx.y;
  cpx<R> p[UNROLL][N], x[UNROLL][N], rv[UNROLL][N];
  // the vectors travel while the scalars are formed (a block of a right-hand
  // side that does not iterate leaves below without using them)
  const bool idle = sa.partial ? !sa.scal[SCAL_COPY + r].active : (!sa.scal[r].active && sa.scal[r].alpha == 0.0);
  if (!idle) {
#pragma unroll
    for (int u = 0; u < UNROLL; u++) {
      const long k = chunk_first() + u * 256;
      if (k >= g.n) continue;
      const long at = g.at(k, r);
      unpack_chunk<P>(p_[at], p[u]);
      unpack_chunk<P>(stream_load(x_ + at), x[u]);
      unpack_chunk<P>(r_[at], rv[u]);
    }
  }
  const CGScal c = step_scal(sa, r, g.nrhs, blockIdx.x == 0);
  const bool act = c.active != 0;
  const bool flush = y_ && c.update;
  if (!act && c.alpha == 0.0) return;
  const R al = (R)c.alpha, beta = (R)c.beta;
#pragma unroll
  for (int u = 0; u < UNROLL; u++) {
    const long k = chunk_first() + u * 256;
    if (k >= g.n) continue;
    const long at = g.at(k, r);
#pragma unroll
    for (int q = 0; q < N; q++) {
      if (c.alpha != 0.0) x[u][q] = cadd(x[u][q], cscale(al, p[u][q]));
      if (act) p[u][q] = cadd(rv[u][q], cscale(beta, p[u][q]));
    }
    if (P::CPB == 2 && flush) {
      const long d0 = at + (at >> lg << lg);
#pragma unroll
      for (int q = 0; q < N; q++) {
        cpx<double> o;
        unpack_chunk<SP64>(y_[d0 + (q << lg)], &o);
        o = cadd(o, cpx<double>{(double)x[u][q].re, (double)x[u][q].im});
        y_[d0 + (q << lg)] = pack_chunk<SP64>(&o, 1.0);
        x[u][q] = {R(0), R(0)};
      }
    }
    if (c.alpha != 0.0) stream_store(x_ + at, pack_chunk<P>(x[u], R(1)));
    if (act) p_[at] = pack_chunk<P>(p[u], R(1));
  }
}

template <class PS, class PD>
__global__ void __launch_bounds__(256) vec_convert_kernel(const void* src, const float* src_sc, void* dst, float* dst_sc,
                                   int accumulate, long h, int nrhs, int Ns) {
  using RS = typename PS::real;
  using RD = typename PD::real;
  const int inner = nrhs * Ns;
  const int spb = blockDim.x / inner;
  const int sl = threadIdx.x / inner, lr = threadIdx.x % inner, r = lr / Ns, s = lr % Ns;
  for (long j = (long)blockIdx.x * spb + sl; j < h; j += (long)gridDim.x * spb) {
    cpx<RS> a[12];
    load_site<PS>(src, src_sc, j, r, s, nrhs, Ns, a);
    cpx<RD> b[12];
    if (accumulate) {
      load_site<PD>(dst, dst_sc, j, r, s, nrhs, Ns, b);
#pragma unroll
      for (int c = 0; c < 12; c++) b[c] = {b[c].re + (RD)a[c].re, b[c].im + (RD)a[c].im};
    } else {
#pragma unroll
      for (int c = 0; c < 12; c++) b[c] = {(RD)a[c].re, (RD)a[c].im};
    }
    store_site<PD>(dst, dst_sc, j, r, s, nrhs, Ns, b);
  }
}

// CG vector step after the scalars of the iteration are known (scaled formats;
// the others take chunk_cg_step_kernel):
//   x += alpha p   (for every right-hand side that iterated: alpha != 0, which
//                   includes one that converged at this iteration's beta)
//   p  = r + beta p (for the right-hand sides still active)
template <class P>
__global__ void __launch_bounds__(256) vec_cg_step_kernel(const void* r_, const float* r_sc, void* p_, float* p_sc, void* x_,
                                   float* x_sc, const CGScal* scal, long h, int nrhs, int Ns) {
  using R = typename P::real;
  const int inner = nrhs * Ns;
  const int spb = blockDim.x / inner;
  const int sl = threadIdx.x / inner, lr = threadIdx.x % inner, r = lr / Ns, s = lr % Ns;
  const bool act = scal[r].active != 0;
  const double alpha = scal[r].alpha;
  if (!act && alpha == 0.0) return;
  const R al = (R)alpha, beta = (R)scal[r].beta;
  for (long j = (long)blockIdx.x * spb + sl; j < h; j += (long)gridDim.x * spb) {
    cpx<R> pv[12];
    load_site<P>(p_, p_sc, j, r, s, nrhs, Ns, pv);
    if (alpha != 0.0) {
      cpx<R> xv[12];
      load_site<P, 1>(x_, x_sc, j, r, s, nrhs, Ns, xv);
#pragma unroll
      for (int c = 0; c < 12; c++) xv[c] = cadd(xv[c], cscale(al, pv[c]));
      store_site<P, 1>(x_, x_sc, j, r, s, nrhs, Ns, xv);
    }
    if (act) {
      cpx<R> rv[12];
      load_site<P>(r_, r_sc, j, r, s, nrhs, Ns, rv);
#pragma unroll
      for (int c = 0; c < 12; c++) pv[c] = cadd(rv[c], cscale(beta, pv[c]));
      store_site<P>(p_, p_sc, j, r, s, nrhs, Ns, pv);
    }
  }
}

template <class P>
__global__ void __launch_bounds__(256) vec_norm2_kernel(const void* v, const float* sc, double* partial, long h, int nrhs,
                                                        int Ns) {
  using R = typename P::real;
  __shared__ double red[1024];
  const int inner = nrhs * Ns;
  const int spb = blockDim.x / inner;
  const int sl = threadIdx.x / inner, lr = threadIdx.x % inner, r = lr / Ns, s = lr % Ns;
  double acc = 0.0;
  if (sl < spb)
    for (long j = (long)blockIdx.x * spb + sl; j < h; j += (long)gridDim.x * spb) {
      cpx<R> a[12];
      load_site<P>(v, sc, j, r, s, nrhs, Ns, a);
#pragma unroll
      for (int c = 0; c < 12; c++) acc += (double)cnorm2(a[c]);
    }
  block_reduce_rhs(sl < spb ? acc : 0.0, Ns, spb, nrhs, red, partial, blockIdx.x, threadIdx.x);
}

#define ODWF_PREC_SWITCH(prec, KERNEL, ...)                                             \
  switch (prec) {                                                                       \
    case PREC64: hipLaunchKernelGGL(KERNEL<SP64>, __VA_ARGS__); break;                  \
    case PREC32: hipLaunchKernelGGL(KERNEL<SP32>, __VA_ARGS__); break;                  \
    case PREC16: hipLaunchKernelGGL(KERNEL<SP16>, __VA_ARGS__); break;                  \
    case PRECB16: hipLaunchKernelGGL(KERNEL<SPB16>, __VA_ARGS__); break;                \
    default: return hipErrorInvalidValue;                                               \
  }

hipError_t launch_vec_zero(int prec, void* v, float* sc, long h, int nrhs, int Ns, hipStream_t st) {
  const ChunkGeom g = chunk_geom(prec == PREC64 ? 1 : prec == PREC32 ? 2 : 4, h, nrhs, Ns);
  hipLaunchKernelGGL(chunk_zero_kernel, chunk_grid(g), dim3(256), 0, st, reinterpret_cast<uint4*>(v), g);
  if (sc)
    hipLaunchKernelGGL(scale_zero_kernel, dim3((unsigned)((h * nrhs * Ns + 255) / 256)), dim3(256), 0, st, sc,
                       h * nrhs * Ns);
  return hipGetLastError();
}

template <class PS, class PD>
static hipError_t convert(const void* src, const float* src_sc, void* dst, float* dst_sc, int acc, long h, int nrhs,
                          int Ns, hipStream_t st) {
  const int block = vec_spb(nrhs, Ns) * nrhs * Ns;
  hipLaunchKernelGGL((vec_convert_kernel<PS, PD>), dim3(vec_nblocks(h, nrhs, Ns)), dim3(block), 0, st, src, src_sc, dst,
                     dst_sc, acc, h, nrhs, Ns);
  return hipGetLastError();
}

hipError_t launch_vec_convert(int prec_src, const void* src, const float* src_sc, int prec_dst,
                              void* dst, float* dst_sc, int accumulate, long h, int nrhs, int Ns,
                              hipStream_t st, const CGScal* gate, int gate_mode) {
  const uint4* s4 = reinterpret_cast<const uint4*>(src);
  uint4* d4 = reinterpret_cast<uint4*>(dst);
  if (prec_src == PREC64 && prec_dst == PREC32 && !accumulate) {
    const ChunkGeom g = chunk_geom(2, h, nrhs, Ns);
    hipLaunchKernelGGL(chunk_64_to_32_kernel, chunk_grid(g), dim3(256), 0, st, s4, d4, gate, gate_mode, g, __builtin_ctz(Ns));
    return hipGetLastError();
  }
  if (prec_src == prec_dst && (prec_src == PREC64 || prec_src == PREC32) && !accumulate) {
    const ChunkGeom g = chunk_geom(prec_src == PREC64 ? 1 : 2, h, nrhs, Ns);
    hipLaunchKernelGGL(chunk_copy_kernel, chunk_grid(g), dim3(256), 0, st, s4, d4, gate, gate_mode, g);
    return hipGetLastError();
  }
  if (gate) return hipErrorInvalidValue;  // (the scaled formats have no gated conversion)
  const int pair = prec_src * 4 + prec_dst;
  switch (pair) {
    case PREC64 * 4 + PREC16: return convert<SP64, SP16>(src, src_sc, dst, dst_sc, accumulate, h, nrhs, Ns, st);
    case PREC64 * 4 + PRECB16: return convert<SP64, SPB16>(src, src_sc, dst, dst_sc, accumulate, h, nrhs, Ns, st);
    case PREC16 * 4 + PREC64: return convert<SP16, SP64>(src, src_sc, dst, dst_sc, accumulate, h, nrhs, Ns, st);
    case PRECB16 * 4 + PREC64: return convert<SPB16, SP64>(src, src_sc, dst, dst_sc, accumulate, h, nrhs, Ns, st);
    case PREC16 * 4 + PREC16: return convert<SP16, SP16>(src, src_sc, dst, dst_sc, accumulate, h, nrhs, Ns, st);
    case PRECB16 * 4 + PRECB16: return convert<SPB16, SPB16>(src, src_sc, dst, dst_sc, accumulate, h, nrhs, Ns, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_vec_flush(void* x, void* y, long h, int nrhs, int Ns, hipStream_t st) {
  const ChunkGeom g = chunk_geom(2, h, nrhs, Ns);
  hipLaunchKernelGGL(chunk_32_to_64_kernel, chunk_grid(g), dim3(256), 0, st, reinterpret_cast<uint4*>(x),
                     reinterpret_cast<uint4*>(y), g, __builtin_ctz(Ns));
  return hipGetLastError();
}

// beta is formed inside the vector step while a block of it reads at most this
// many partial sums (two loads a thread, the scalar launch and its gap saved:
// 4-6 us of a 4^4 x 8 iteration); above, by a launch of its own (up to 2048:
// 8^4 x 16, twelve right-hand sides, 330 -> 358 us an FP64 iteration)
constexpr int STEP_BLOCKS = 512;

hipError_t launch_cg_step(int prec, const void* r, const float* r_sc, void* p, float* p_sc, void* x, float* x_sc,
                          void* y, const double* partial, int nblocks, CGScal* scal, CGScal* host, long h, int nrhs,
                          int Ns, hipStream_t st) {
  StepScal a = {scal, partial, nblocks, host};
  const bool chunks = prec == PREC64 || prec == PREC32;
  if (!chunks || nblocks > STEP_BLOCKS) {
    const hipError_t e = launch_fin(FIN_BETA, partial, nblocks, nrhs, scal, nullptr, st, 0, host);
    if (e != hipSuccess) return e;
    a.partial = nullptr;
  }
  if (chunks) {
    const ChunkGeom g = chunk_geom(prec == PREC64 ? 1 : 2, h, nrhs, Ns);
    const uint4* r4 = reinterpret_cast<const uint4*>(r);
    uint4 *p4 = reinterpret_cast<uint4*>(p), *x4 = reinterpret_cast<uint4*>(x), *y4 = reinterpret_cast<uint4*>(y);
    const int lg = __builtin_ctz(Ns);
    if (prec == PREC64) hipLaunchKernelGGL(chunk_cg_step_kernel<SP64>, chunk_grid(g), dim3(256), 0, st, r4, p4, x4, nullptr, a, g, lg);
    else hipLaunchKernelGGL(chunk_cg_step_kernel<SP32>, chunk_grid(g), dim3(256), 0, st, r4, p4, x4, y4, a, g, lg);
    return hipGetLastError();
  }
  const int block = vec_spb(nrhs, Ns) * nrhs * Ns;
  const dim3 gr(vec_nblocks(h, nrhs, Ns));
  if (prec == PREC16) hipLaunchKernelGGL(vec_cg_step_kernel<SP16>, gr, dim3(block), 0, st, r, r_sc, p, p_sc, x, x_sc, scal, h, nrhs, Ns);
  else if (prec == PRECB16) hipLaunchKernelGGL(vec_cg_step_kernel<SPB16>, gr, dim3(block), 0, st, r, r_sc, p, p_sc, x, x_sc, scal, h, nrhs, Ns);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_vec_norm2(int prec, const void* v, const float* sc, double* partial, long h,
                            int nrhs, int Ns, int* nblocks_out, hipStream_t st) {
  const int block = vec_spb(nrhs, Ns) * nrhs * Ns;
  const int nb = vec_nblocks(h, nrhs, Ns);
  if (nblocks_out) *nblocks_out = nb;
  ODWF_PREC_SWITCH(prec, vec_norm2_kernel, dim3(nb), dim3(block), 0, st, v, sc, partial, h, nrhs, Ns);
  return hipGetLastError();
}

// copy right-hand side r_src of an nrhs_src field into right-hand side r_dst
// of an nrhs_dst field (same parity, any storage precisions); src == nullptr
// writes zeros
template <class PS, class PD>
__global__ void __launch_bounds__(256) vec_copy_rhs_kernel(const void* src, const float* src_sc, int nrhs_src, int r_src,
                                    void* dst, float* dst_sc, int nrhs_dst, int r_dst, long h, int Ns) {
  using RS = typename PS::real;
  using RD = typename PD::real;
  const long n = h * Ns;
  for (long k = blockIdx.x * (long)blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x) {
    const long j = k / Ns;
    const int s = (int)(k % Ns);
    cpx<RD> b[12];
    if (src) {
      cpx<RS> a[12];
      load_site<PS>(src, src_sc, j, r_src, s, nrhs_src, Ns, a);
#pragma unroll
      for (int c = 0; c < 12; c++) b[c] = {(RD)a[c].re, (RD)a[c].im};
    } else {
#pragma unroll
      for (int c = 0; c < 12; c++) b[c] = {RD(0), RD(0)};
    }
    store_site<PD>(dst, dst_sc, j, r_dst, s, nrhs_dst, Ns, b);
  }
}

template <class PS>
static hipError_t copy_rhs_to(int prec_dst, const void* src, const float* src_sc, int ns, int rs,
                              void* dst, float* dst_sc, int nd, int rd, long h, int Ns, hipStream_t st) {
  long nb = (h * Ns + 255) / 256;
  if (nb > 8192) nb = 8192;
  const dim3 gr((unsigned)nb);
  switch (prec_dst) {
    case PREC64: hipLaunchKernelGGL((vec_copy_rhs_kernel<PS, SP64>), gr, dim3(256), 0, st, src, src_sc, ns, rs, dst, dst_sc, nd, rd, h, Ns); break;
    case PREC32: hipLaunchKernelGGL((vec_copy_rhs_kernel<PS, SP32>), gr, dim3(256), 0, st, src, src_sc, ns, rs, dst, dst_sc, nd, rd, h, Ns); break;
    case PREC16: hipLaunchKernelGGL((vec_copy_rhs_kernel<PS, SP16>), gr, dim3(256), 0, st, src, src_sc, ns, rs, dst, dst_sc, nd, rd, h, Ns); break;
    case PRECB16: hipLaunchKernelGGL((vec_copy_rhs_kernel<PS, SPB16>), gr, dim3(256), 0, st, src, src_sc, ns, rs, dst, dst_sc, nd, rd, h, Ns); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_vec_copy_rhs(int prec_src, const void* src, const float* src_sc, int nrhs_src,
                               int r_src, int prec_dst, void* dst, float* dst_sc, int nrhs_dst,
                               int r_dst, long h, int Ns, hipStream_t st) {
  switch (prec_src) {
    case PREC64: return copy_rhs_to<SP64>(prec_dst, src, src_sc, nrhs_src, r_src, dst, dst_sc, nrhs_dst, r_dst, h, Ns, st);
    case PREC32: return copy_rhs_to<SP32>(prec_dst, src, src_sc, nrhs_src, r_src, dst, dst_sc, nrhs_dst, r_dst, h, Ns, st);
    case PREC16: return copy_rhs_to<SP16>(prec_dst, src, src_sc, nrhs_src, r_src, dst, dst_sc, nrhs_dst, r_dst, h, Ns, st);
    case PRECB16: return copy_rhs_to<SPB16>(prec_dst, src, src_sc, nrhs_src, r_src, dst, dst_sc, nrhs_dst, r_dst, h, Ns, st);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// finalisation: one block of 1024 threads
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) fin_kernel(int kind, const double* partial, int nblocks, int nrhs, CGScal* scal,
                                                   double* out, int gated, CGScal* host) {
  __shared__ double tmp[1024];
  if (gated && !gate_any(scal, GATE_UPDATE, nrhs)) return;
  const double v = partial_sum(partial, nblocks, nrhs, tmp);
  if ((int)threadIdx.x >= nrhs) return;
  const int r = threadIdx.x;
  if (out) out[r] = v;
  if (!scal) return;
  CGScal c = scal[(kind == FIN_BETA ? SCAL_COPY : 0) + r];
  if (gated && !c.update) return;  // only the right-hand sides that asked for it
  const bool finite = isfinite(v);
  switch (kind) {
    case FIN_F2:
      c.f2 = v;
      break;
    case FIN_BETA:
      fin_beta(c, v);
      break;
    case FIN_INIT:
      // v = |r|^2 of a freshly computed true residual
      c.rr = v;
      c.rmax2 = v;
      c.update = 0;
      if (c.iters > c.upd_iters) {  // an update of this right-hand side's own iterate
        c.nupd += 1;
        c.upd_iters = c.iters;
      }
      if (!finite) {
        c.nan = 1;
        c.active = 0;
      } else if (v <= c.tol2 * c.f2) {
        c.converged = 1;
        c.active = 0;
      } else {
        c.converged = 0;
        c.active = c.iters < c.maxiter ? 1 : 0;
      }
      break;
    default:
      break;
  }
  scal[r] = c;
  if (host) host[r] = c;
}

// first stage of the finalisation for long partial arrays: block b sums the
// partials of blocks [b * 1024, (b + 1) * 1024) per right-hand side in a fixed
// tree and writes them to dst[b * nrhs + r]
__global__ void __launch_bounds__(256) partial_reduce_kernel(const double* partial, int nblocks, int nrhs, double* dst) {
  __shared__ double tmp[256];
  const int b0 = blockIdx.x * 1024;
  const double v = partial_sum(partial + (long)b0 * nrhs, min(1024, nblocks - b0), nrhs, tmp);
  if ((int)threadIdx.x < nrhs) dst[(long)blockIdx.x * nrhs + threadIdx.x] = v;
}

size_t partial_bytes(int nblocks, int nrhs) {
  return ((size_t)nblocks + (nblocks + 1023) / 1024 + 16) * nrhs * sizeof(double);
}

hipError_t launch_fin(int kind, const double* partial, int nblocks, int nrhs, CGScal* scal,
                      double* out, hipStream_t st, int gated, CGScal* host) {
  // one block reads up to 32768 values at 32 a thread (24576: 4.5 us, as much as
  // the first of two stages and its gap save); longer arrays take two stages
  if ((long)nblocks * nrhs > 32768) {
    // the second-stage inputs live behind the first-stage partials
    double* dst = const_cast<double*>(partial) + (size_t)nblocks * nrhs;
    const int nb2 = (nblocks + 1023) / 1024;
    hipLaunchKernelGGL(partial_reduce_kernel, dim3(nb2), dim3(256), 0, st, partial, nblocks, nrhs, dst);
    partial = dst;
    nblocks = nb2;
  }
  hipLaunchKernelGGL(fin_kernel, dim3(1), dim3(1024), 0, st, kind, partial, nblocks, nrhs, scal, out, gated, host);
  return hipGetLastError();
}

}  // namespace odwf
