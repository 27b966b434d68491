// Stand-alone fifth-dimension kernel on a half field, out = prog(in): A^{-dag} at the
// head of S_e^dag, A^{-1} of an admitted source, and for N_s = 32 the programs that the
// layout kernels apply below.  N_s = 32: sites are loaded in the lane layout
// (coalesced), transposed through LDS into columns of Ns values, transformed, and
// written back; N_s <= 16: on the matrix cores.
#include "dev_common.h"
#include "kernels.h"

namespace odwf {

template <class P, int NS>
__global__ void __launch_bounds__(256) m5_kernel(const void* in, const float* in_sc, void* out, float* out_sc, M5Prog prog,
                                                 const void* coefp, const KappaArr kappa, long h, int nrhs, int spb) {
  using R = typename P::real;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NSP = NS + 1;
  const int inner = nrhs * NS;
  const int tid = threadIdx.x;
  const int sl = tid / inner, lr = tid - sl * inner, r = lr / NS, s = lr - r * NS;
  const long j0 = (long)blockIdx.x * spb;
  const int nsb = (int)min((long)spb, h - j0);
  const bool valid = sl < nsb;
  const long j = j0 + sl;
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem);
  R* kap = reinterpret_cast<R*>(smem + (size_t)spb * nrhs * 12 * NSP * sizeof(cpx<R>));
  if (tid < nrhs) kap[tid] = (R)kappa.v[tid];

  cpx<R> v[12];
  if (valid) {
    load_site<P>(in, in_sc, j, r, s, nrhs, NS, v);
    cpx<R>* b = buf + ((size_t)(sl * nrhs + r) * 12) * NSP + s;
#pragma unroll
    for (int c = 0; c < 12; c++) b[c * NSP] = v[c];
  }
  __syncthreads();
  column_pass_lds<R, NS>(buf, nsb, nrhs, prog, reinterpret_cast<const R*>(coefp), kap, tid);
  __syncthreads();
  if (!valid) return;
  const cpx<R>* b = buf + ((size_t)(sl * nrhs + r) * 12) * NSP + s;
#pragma unroll
  for (int c = 0; c < 12; c++) v[c] = b[c * NSP];
  store_site<P>(out, out_sc, j, r, s, nrhs, NS, v);
}

// N_s <= 16: a lane's column set on the matrix cores, streaming (one load, one
// store per 5D site, no LDS for the data).  The columns (site, right-hand side)
// of a half field are consecutive, so a wave takes 64 / N_s of them.
template <class P, int NS>
__global__ void __launch_bounds__(256, 2) m5_dense_kernel(const void* in, const float* in_sc, void* out, float* out_sc,
                                                          const DenseArg dn, long ncol, int nrhs) {
  using R = typename P::real;
  __shared__ __align__(16) R mat[DENSE_IMAGE<R>];
  __shared__ __align__(16) R scr[4 * DENSE_SCRATCH<R>];
  const int s = threadIdx.x % NS;
  const long j = (long)blockIdx.x * (256 / NS) + threadIdx.x / NS;
  const bool valid = j < ncol;
  cpx<R> v[12];
#pragma unroll
  for (int c = 0; c < 12; c++) v[c] = {R(0), R(0)};
  if (valid) load_site<P>(in, in_sc, j, 0, s, 1, NS, v);
  const int r = nrhs > 1 ? (int)(j % nrhs) : 0;
  dense_stage<R>(mat, dn.tab, threadIdx.x);
  __syncthreads();
  dense_apply<NS>(v, mat, scr + (threadIdx.x >> 6) * DENSE_SCRATCH<R>, (R)dn.rho[r], (R)dn.rho[MAXRHS + r], dense_lim<R>(dn),
                  threadIdx.x);
  if (valid) store_site<P>(out, out_sc, j, 0, s, 1, NS, v);
}

struct M5Io {
  const void* in;
  const float* in_sc;
  void* out;
  float* out_sc;
};
template <class P, int NS>
static hipError_t launch_m5_t(const M5Io& f, const M5Prog& prog, const DenseArg& dn, const void* coef,
                              const KappaArr& kappa, long h, int nrhs, hipStream_t st) {
  using R = typename P::real;
  const int inner = nrhs * NS;
  if (inner > 256 || nrhs > MAXRHS) return hipErrorInvalidValue;
  if constexpr (NS <= DENSE_N) {
    if (!dn.tab) return hipErrorInvalidValue;
    const long ncol = h * nrhs;
    const dim3 grid((unsigned)((ncol * NS + 255) / 256));
    hipLaunchKernelGGL((m5_dense_kernel<P, NS>), grid, dim3(256), 0, st, f.in, f.in_sc, f.out, f.out_sc, dn, ncol, nrhs);
  } else {
    const int spb = 256 / inner;
    const int block = (spb * inner + 63) & ~63;
    const long nb = (h + spb - 1) / spb;
    const size_t sm = (size_t)spb * nrhs * 12 * (NS + 1) * sizeof(cpx<R>) + MAXRHS * sizeof(R);
    hipLaunchKernelGGL((m5_kernel<P, NS>), dim3((unsigned)nb), dim3(block), sm, st, f.in, f.in_sc, f.out, f.out_sc, prog,
                       coef, kappa, h, nrhs, spb);
  }
  return hipGetLastError();
}

template <class P>
static hipError_t launch_m5_p(const M5Io& f, const M5Prog& prog, const DenseArg& dn, const void* coef,
                              const KappaArr& kappa, long h, int nrhs, int Ns, hipStream_t st) {
  switch (Ns) {
    case 4: return launch_m5_t<P, 4>(f, prog, dn, coef, kappa, h, nrhs, st);
    case 8: return launch_m5_t<P, 8>(f, prog, dn, coef, kappa, h, nrhs, st);
    case 16: return launch_m5_t<P, 16>(f, prog, dn, coef, kappa, h, nrhs, st);
    case 32: return launch_m5_t<P, 32>(f, prog, dn, coef, kappa, h, nrhs, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_m5(int prec, const void* in, const float* in_sc, void* out, float* out_sc, const M5Prog& prog,
                     const DenseArg& dn, const void* coef, const KappaArr& kappa, long h, int nrhs, int Ns,
                     hipStream_t st) {
  const M5Io f = {in, in_sc, out, out_sc};
  switch (prec) {
    case PREC64: return launch_m5_p<SP64>(f, prog, dn, coef, kappa, h, nrhs, Ns, st);
    case PREC32: return launch_m5_p<SP32>(f, prog, dn, coef, kappa, h, nrhs, Ns, st);
    case PREC16: return launch_m5_p<SP16>(f, prog, dn, coef, kappa, h, nrhs, Ns, st);
    case PRECB16: return launch_m5_p<SPB16>(f, prog, dn, coef, kappa, h, nrhs, Ns, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace odwf
