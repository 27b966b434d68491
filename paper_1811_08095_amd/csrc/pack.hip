// Layout kernels: canonical complex128 fields <-> internal even/odd halves.
//
// Canonical spinor: [rhs][s][t][z][y][x][spin 4][colour 3] complex128.
// Canonical gauge:  [t][z][y][x][mu][3][3] complex128, U_mu(x) links x to x + mu.
// Internal half of parity p: site j = ((t * Lz + z) * Ly + y) * (Lx / 2) + x / 2
// over the sites with (x + y + z + t) mod 2 = p; spinor chunks as described in
// dev_common.h; links per output parity [j][8][...] with directions 0-3 the
// forward links U_mu(x) and 4-7 the backward links U_mu(x - mu)^dag, FP64 as 9
// complex doubles, reduced precision as rows 0 and 1 (12 floats).
#include "dev_common.h"
#include "kernels.h"

namespace odwf {

// ---------------------------------------------------------------------------
// canonical <-> both halves.  The canonical layout keeps slices far apart and a
// site's 12 components together, the halves keep a site's slices together, so
// a block transposes a tile of consecutive sites and all slices of one
// right-hand side through LDS: the canonical side moves runs of TS * 192 bytes,
// the half side 16-byte chunks over the slices.  One launch covers both
// parities (an absent half is skipped on the way in, zeros on the way out) and
// may apply a fifth-dimension operator while the tile is in registers: a
// diagonal one, or a dense program on the matrix cores (N_s <= 16).
// Bound: HBM (or the memory-side cache).  128 threads keep 12 16-byte loads in
// flight each, five blocks to a CU in FP64 (26 KB of LDS); the column padding
// keeps both sides of the transposition free of bank conflicts.  Measured
// against one lane per 5D site reading its 192 bytes on its own, one launch per
// parity and operator: 32^4 x 16 FP32, one parity in 499 us (was 688; 4.8 TB/s),
// one parity and zeros out 760 us (942 + 523; 5.3 TB/s); 12x10x14x20 x 16, three
// right-hand sides, both parities with omega in 93 us (2 x 74 + 2 x 59), out
// 114 us (2 x 97).
// ---------------------------------------------------------------------------
struct TileArgs {
  void* d[2];             // even, odd
  float* sc[2];
  const double* diag[2];  // coefficients of a diagonal operator, or null
  DenseArg dn;            // dense program (tab null: none) ...
  int dn_on;              // ... of the parities whose bit is set
  int r0, nrhs;
  int only;       // packing one parity alone: the tile is TS of its sites; else -1
  long n;         // sites: V, or V / 2
  long V;
  FastDiv dx, dy, dz;  // Lx (Lx / 2 with only >= 0), Ly, Lz
};

template <int NS>
struct Tile {
  static constexpr int T = 128;       // threads: two waves
  static constexpr int TS = T / NS;   // sites
};

// full-lattice index i, half-lattice index j and parity of site k of the launch
__device__ __forceinline__ void site_of(const TileArgs& a, uint32_t k, uint32_t& i, uint32_t& j, int& par) {
  const uint32_t row = a.dx.div(k), x = k - row * a.dx.d;
  const uint32_t zt = a.dy.div(row), y = row - zt * a.dy.d;
  const uint32_t t = a.dz.div(zt), z = zt - t * a.dz.d;
  if (a.only >= 0) {
    par = a.only;
    j = k;
    i = 2 * k + ((y + z + t + par) & 1);
  } else {
    par = (x + y + z + t) & 1;
    i = k;
    j = row * (a.dx.d >> 1) + (x >> 1);
  }
}

template <int NS, class R>
__device__ __forceinline__ void diag_apply(cpx<R> (&v)[12], const double* diag, int s) {
  const R p = (R)diag[s], m = (R)diag[NCOEF * NS + NS - 1 - s];
#pragma unroll
  for (int c = 0; c < 12; c++) v[c] = cscale(c < 6 ? p : m, v[c]);
}

// the operators of the lane's parity; every lane calls it.  scr: the wave's own
// sites of the tile, which hold nothing while their values are in registers
template <int NS, class R>
__device__ __forceinline__ void tile_program(cpx<R> (&v)[12], const TileArgs& a, int r, int par, int s, const R* mat, R* scr) {
  if constexpr (NS <= DENSE_N) {
    if (a.dn.tab) {
      cpx<R> w[12];
#pragma unroll
      for (int c = 0; c < 12; c++) w[c] = v[c];
      dense_apply<NS>(w, mat, scr, (R)a.dn.rho[r], (R)a.dn.rho[MAXRHS + r], dense_lim<R>(a.dn), threadIdx.x);
      const bool on = (a.dn_on >> par) & 1;
#pragma unroll
      for (int c = 0; c < 12; c++) {
        v[c].re = on ? w[c].re : v[c].re;
        v[c].im = on ? w[c].im : v[c].im;
      }
    }
  }
  const double* diag = par ? a.diag[1] : a.diag[0];
  if (diag) diag_apply<NS>(v, diag, s);
}

template <int NS, class R>
__device__ __forceinline__ void tile_stage(const TileArgs& a, R* mat) {
  if constexpr (NS <= DENSE_N)
    if (a.dn.tab) dense_stage<R>(mat, a.dn.tab, threadIdx.x);
}

template <int NS>
struct TileLds {
  static constexpr int COL = NS + 1;  // padded column
  static constexpr int N = Tile<NS>::TS * 12 * COL;
};
static_assert(DENSE_SCRATCH<double> <= TileLds<16>::N && DENSE_SCRATCH<float> <= TileLds<16>::N, "a wave's half tile");

typedef double dbl2 __attribute__((ext_vector_type(2)));

template <class P, int NS>
__global__ void __launch_bounds__(Tile<NS>::T, 3) pack_tile_kernel(const double2* __restrict__ canon, const TileArgs a) {
  using R = typename P::real;
  constexpr int T = Tile<NS>::T, TS = Tile<NS>::TS, COL = TileLds<NS>::COL;
  extern __shared__ __align__(16) unsigned char smem[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem);
  R* mat = reinterpret_cast<R*>(buf + TileLds<NS>::N);
  const int r = blockIdx.y, tid = threadIdx.x;
  const uint32_t k0 = blockIdx.x * TS;
  const int n = (int)min((long)TS, a.n - (long)k0);
  // one parity: its sites are every other one of a row, whose parity alternates
  // with the row; a thread's 12 components lie in at most four sites
  const dbl2* src = reinterpret_cast<const dbl2*>(canon) + (long)(a.r0 + r) * NS * a.V * 12;
  dbl2 q[12];
#pragma unroll
  for (int k = 0; k < 12; k++) {  // NS runs of TS * 12 components
    const int e = tid + k * T, sl = e / (TS * 12), rem = e % (TS * 12);
    const int sr = min(rem / 12, n - 1);
    uint32_t i = k0 + sr;
    if (a.only >= 0) {
      uint32_t jj;
      int pp;
      site_of(a, k0 + sr, i, jj, pp);
    }
    q[k] = __builtin_nontemporal_load(src + ((long)sl * a.V + i) * 12 + rem % 12);
  }
  tile_stage<NS, R>(a, mat);
#pragma unroll
  for (int k = 0; k < 12; k++) {
    const int e = tid + k * T, sl = e / (TS * 12), rem = e % (TS * 12);
    buf[rem * COL + sl] = {(R)q[k].x, (R)q[k].y};
  }
  const int site = tid / NS, s = tid % NS;
  int par;
  uint32_t i, j;
  site_of(a, k0 + min(site, n - 1), i, j, par);
  __syncthreads();
  cpx<R> v[12];
#pragma unroll
  for (int c = 0; c < 12; c++) v[c] = buf[(site * 12 + c) * COL + s];
  tile_program<NS, R>(v, a, r, par, s, mat, reinterpret_cast<R*>(buf + (tid >> 6) * (TileLds<NS>::N / 2)));
  if (site < n)
    store_site<P>(par ? a.d[1] : a.d[0], par ? a.sc[1] : a.sc[0], j, r, s, a.nrhs, NS, v);
}

template <class P, int NS>
__global__ void __launch_bounds__(Tile<NS>::T, 3) unpack_tile_kernel(double2* __restrict__ canon, const TileArgs a) {
  using R = typename P::real;
  constexpr int T = Tile<NS>::T, TS = Tile<NS>::TS, COL = TileLds<NS>::COL;
  extern __shared__ __align__(16) unsigned char smem[];
  cpx<R>* buf = reinterpret_cast<cpx<R>*>(smem);
  R* mat = reinterpret_cast<R*>(buf + TileLds<NS>::N);
  const int r = blockIdx.y, tid = threadIdx.x;
  const uint32_t i0 = blockIdx.x * TS;
  const int n = (int)min((long)TS, a.V - (long)i0);
  const int site = tid / NS, s = tid % NS;
  int par;
  uint32_t i, j;
  site_of(a, i0 + min(site, n - 1), i, j, par);
  const void* half = par ? a.d[1] : a.d[0];
  cpx<R> v[12];
#pragma unroll
  for (int c = 0; c < 12; c++) v[c] = {R(0), R(0)};
  if (half) load_site<P>(half, par ? a.sc[1] : a.sc[0], j, r, s, a.nrhs, NS, v);
  tile_stage<NS, R>(a, mat);
  __syncthreads();
  tile_program<NS, R>(v, a, r, par, s, mat, reinterpret_cast<R*>(buf + (tid >> 6) * (TileLds<NS>::N / 2)));
#pragma unroll
  for (int c = 0; c < 12; c++) buf[(site * 12 + c) * COL + s] = v[c];
  __syncthreads();
  dbl2* dst = reinterpret_cast<dbl2*>(canon) + ((long)(a.r0 + r) * NS * a.V + i0) * 12;
#pragma unroll
  for (int k = 0; k < 12; k++) {
    const int e = tid + k * T, sl = e / (TS * 12), rem = e % (TS * 12);
    if (rem < n * 12) {
      const cpx<R> z = buf[rem * COL + sl];
      const dbl2 w = {(double)z.re, (double)z.im};
      __builtin_nontemporal_store(w, dst + (long)sl * a.V * 12 + rem);
    }
  }
}

// Both parities (blockIdx.y) and both precisions in one launch: a thread takes
// one matrix entry, so that reads and writes are whole runs of 16 and 8 bytes.
// Bound: HBM, 75 MB in (twice, for the two directions) and 200 MB out at
// 16^3 x 32: 64 us, against 4 x 31 us of one launch per parity and precision with
// a lane per matrix.
struct GaugePack {
  const double2* canon;
  double2* out64[2];
  float2* out32[2];
  FastDiv dhx, dy, dz;
  uint32_t L0, L1, L2, L3, h;
};
constexpr int GS = 32;  // sites of a block

__global__ void __launch_bounds__(256) pack_gauge_kernel(const GaugePack a) {
  const uint32_t par = blockIdx.y, j0 = blockIdx.x * GS;
  double2* out64 = par ? a.out64[1] : a.out64[0];
  float2* out32 = par ? a.out32[1] : a.out32[0];
#pragma unroll
  for (int k = 0; k < GS * 72 / 256; k++) {
    const int e = threadIdx.x + 256 * k, js = e / 72, em = e - 72 * js, dir = em / 9, q = em - 9 * dir;
    const uint32_t j = j0 + js;
    if (j >= a.h) return;
    const uint32_t row = a.dhx.div(j), xh = j - row * a.dhx.d;
    const uint32_t zt = a.dy.div(row);
    uint32_t y = row - zt * a.L1, t = a.dz.div(zt), z = zt - t * a.L2;
    uint32_t x = 2 * xh + ((y + z + t + par) & 1);
    const int mu = dir & 3;
    const bool bwd = dir >= 4;  // the link of x - mu (periodic; the boundary factor is applied by the kernel), adjoint
    if (bwd) {
      if (mu == 0) x = x == 0 ? a.L0 - 1 : x - 1;
      if (mu == 1) y = y == 0 ? a.L1 - 1 : y - 1;
      if (mu == 2) z = z == 0 ? a.L2 - 1 : z - 1;
      if (mu == 3) t = t == 0 ? a.L3 - 1 : t - 1;
    }
    const long i = (((long)t * a.L2 + z) * a.L1 + y) * a.L0 + x;
    double2 v = a.canon[(i * 4 + mu) * 9 + (bwd ? (q % 3) * 3 + q / 3 : q)];
    if (bwd) v.y = -v.y;
    out64[(long)j * 72 + em] = v;
    if (q < 6) out32[(long)j * 48 + dir * 6 + q] = make_float2((float)v.x, (float)v.y);
  }
}

// boundary maps of the effective 4D operator, on canonical fields:
// embed: 5D [r][s][site][spin][colour] from 4D [r][site][spin][colour], the
//   chirality-minus spins (2, 3) into slice 0, the chirality-plus spins (0, 1)
//   into slice Ns - 1, zeros elsewhere;
// project: 4D from 5D, chirality-plus spins of slice Ns - 1 and chirality-minus
//   spins of slice 0 (the pair of slices the m_q boundary term couples)
__global__ void boundary_embed_kernel(const double2* __restrict__ q, double2* __restrict__ f, int nrhs,
                                      int Ns, long V) {
  const long n = (long)nrhs * Ns * V * 12;
  for (long k = blockIdx.x * (long)blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x) {
    const int c = (int)(k % 12);
    const long site = (k / 12) % V;
    const int s = (int)((k / (12 * V)) % Ns);
    const long r = k / (12 * V * Ns);
    const bool plus = c < 6;
    const bool take = (s == 0 && !plus) || (s == Ns - 1 && plus);
    f[k] = take ? q[(r * V + site) * 12 + c] : make_double2(0.0, 0.0);
  }
}

__global__ void boundary_project_kernel(const double2* __restrict__ f, double2* __restrict__ q, int nrhs,
                                        int Ns, long V) {
  const long n = (long)nrhs * V * 12;
  for (long k = blockIdx.x * (long)blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x) {
    const int c = (int)(k % 12);
    const long site = (k / 12) % V;
    const long r = k / (12 * V);
    const int s = c < 6 ? Ns - 1 : 0;
    q[k] = f[((r * Ns + s) * V + site) * 12 + c];
  }
}

static dim3 grid_for(long n, int block) {
  long b = (n + block - 1) / block;
  if (b > 65535L * 16) b = 65535L * 16;
  if (b < 1) b = 1;
  return dim3((unsigned)b);
}

template <class P, int NS>
static hipError_t launch_tile(bool pack, void* canon, const TileArgs& a, hipStream_t st) {
  using R = typename P::real;
  constexpr int TS = Tile<NS>::TS;
  if (a.dn.tab && NS > DENSE_N) return hipErrorInvalidValue;
  const size_t sm = TileLds<NS>::N * sizeof(cpx<R>) + (a.dn.tab ? DENSE_IMAGE<R> * sizeof(R) : 0);
  const dim3 grid((unsigned)((a.n + TS - 1) / TS), a.nrhs);
  double2* c = reinterpret_cast<double2*>(canon);
  if (pack) hipLaunchKernelGGL((pack_tile_kernel<P, NS>), grid, dim3(Tile<NS>::T), sm, st, c, a);
  else hipLaunchKernelGGL((unpack_tile_kernel<P, NS>), grid, dim3(Tile<NS>::T), sm, st, c, a);
  return hipGetLastError();
}

template <class P>
static hipError_t launch_tile_p(bool pack, void* canon, const TileArgs& a, int Ns, hipStream_t st) {
  switch (Ns) {
    case 4: return launch_tile<P, 4>(pack, canon, a, st);
    case 8: return launch_tile<P, 8>(pack, canon, a, st);
    case 16: return launch_tile<P, 16>(pack, canon, a, st);
    case 32: return launch_tile<P, 32>(pack, canon, a, st);
  }
  return hipErrorInvalidValue;
}

static hipError_t tile_any(bool pack, int prec, void* canon, int r0, const HalfIO& e, const HalfIO& o, int nrhs,
                           int Ns, const Geom& g, hipStream_t st) {
  TileArgs a;
  if (e.dn.tab && o.dn.tab && e.dn.tab != o.dn.tab) return hipErrorInvalidValue;  // one dense program a launch
  a.dn = e.dn.tab ? e.dn : o.dn;
  a.dn_on = (e.dn.tab ? 1 : 0) | (o.dn.tab ? 2 : 0);
  a.d[0] = e.d, a.d[1] = o.d;
  a.sc[0] = e.sc, a.sc[1] = o.sc;
  a.diag[0] = e.diag, a.diag[1] = o.diag;
  a.r0 = r0;
  a.nrhs = nrhs;
  a.V = g.V;
  a.only = !pack || (e.d && o.d) ? -1 : (e.d ? 0 : 1);
  a.n = a.only >= 0 ? g.h : g.V;
  a.dx = FastDiv(a.only >= 0 ? g.L[0] / 2 : g.L[0]);
  a.dy = FastDiv(g.L[1]);
  a.dz = FastDiv(g.L[2]);
  switch (prec) {
    case PREC64: return launch_tile_p<SP64>(pack, canon, a, Ns, st);
    case PREC32: return launch_tile_p<SP32>(pack, canon, a, Ns, st);
    case PREC16: return launch_tile_p<SP16>(pack, canon, a, Ns, st);
    case PRECB16: return launch_tile_p<SPB16>(pack, canon, a, Ns, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pack(int prec, const void* canon, int r0, const HalfIO& e, const HalfIO& o, int nrhs, int Ns,
                       const Geom& g, hipStream_t st) {
  return tile_any(true, prec, const_cast<void*>(canon), r0, e, o, nrhs, Ns, g, st);
}

hipError_t launch_unpack(int prec, const HalfIO& e, const HalfIO& o, void* canon, int r0, int nrhs, int Ns,
                         const Geom& g, hipStream_t st) {
  return tile_any(false, prec, canon, r0, e, o, nrhs, Ns, g, st);
}

hipError_t launch_boundary_embed(const void* q, void* f, int nrhs, int Ns, const Geom& g, hipStream_t st) {
  const long n = (long)nrhs * Ns * g.V * 12;
  hipLaunchKernelGGL(boundary_embed_kernel, grid_for(n, 256), dim3(256), 0, st,
                     reinterpret_cast<const double2*>(q), reinterpret_cast<double2*>(f), nrhs, Ns, g.V);
  return hipGetLastError();
}

hipError_t launch_boundary_project(const void* f, void* q, int nrhs, int Ns, const Geom& g, hipStream_t st) {
  const long n = (long)nrhs * g.V * 12;
  hipLaunchKernelGGL(boundary_project_kernel, grid_for(n, 256), dim3(256), 0, st,
                     reinterpret_cast<const double2*>(f), reinterpret_cast<double2*>(q), nrhs, Ns, g.V);
  return hipGetLastError();
}

hipError_t launch_pack_gauge(const void* canon, void* const out64[2], void* const out32[2], const Geom& g,
                             hipStream_t st) {
  GaugePack a;
  a.canon = reinterpret_cast<const double2*>(canon);
  for (int p = 0; p < 2; p++) {
    a.out64[p] = reinterpret_cast<double2*>(out64[p]);
    a.out32[p] = reinterpret_cast<float2*>(out32[p]);
  }
  a.dhx = FastDiv(g.L[0] / 2);
  a.dy = FastDiv(g.L[1]);
  a.dz = FastDiv(g.L[2]);
  a.L0 = g.L[0];
  a.L1 = g.L[1];
  a.L2 = g.L[2];
  a.L3 = g.L[3];
  a.h = (uint32_t)g.h;
  hipLaunchKernelGGL(pack_gauge_kernel, dim3((unsigned)((g.h + GS - 1) / GS), 2), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace odwf
