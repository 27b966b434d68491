// Fermion-force kernel: the link derivative of a hopping bilinear.
//
// For S = Re <chi, W psi> summed over the fifth dimension (W the hopping term
// of the 4D Wilson operator D_w that the optimal domain-wall operator applies
// on every slice; the HMC's fermion forces of §2 are sums of such terms with
// chi and psi built from the solutions of the normal equations), the only
// terms of S that contain the link U_mu(x) are
//     -1/2 b Re tr(U_mu(x) A) - 1/2 b Re tr(U_mu(x)^dag B),
//     A = sum_{s, spin} [(1 - gamma_mu) psi(x + mu, s)] (x) chi(x, s)^dag,
//     B = sum_{s, spin} [(1 + gamma_mu) psi(x, s)] (x) chi(x + mu, s)^dag,
// (b = bc_t on links that cross the t boundary), so S = Re tr(U_mu(x) M) + ...
// with M = -1/2 b (A + B^dag), and the force is F_mu(x) = TA(U_mu(x) M), the
// traceless anti-Hermitian part, for which dS/d eps = i tr(T F_mu(x)) when
// U_mu(x) -> exp(i eps T) U_mu(x).
//
// In the chiral basis sum_spin [(1 - s gamma) p] (x) c^dag = h_p (x) h_c^dag
// with h the same half-spinor projection of p and of c, so a lane forms each
// outer product from two 2 x 3 half spinors.
//
// chi and psi are read in the canonical layout (a slice's 12 components of
// consecutive sites are contiguous), without a packed copy.  A block takes 16
// consecutive sites, lane = (site, mu); each of its two waves walks every
// second slice, so M stays in the lane's registers and nothing is reduced
// across lanes.  Per slice a wave brings the 16 sites, their forward neighbours
// in y, z and t and the at most two x neighbours outside the block (25 KB of
// both fields) through LDS of its own: whole runs of the canonical layout on
// the way in, one 16-byte chunk a lane on the way out, slots padded so that the
// lanes meet different banks.  The next slice's chunks travel while a slice is
// used (25 loads of 16 bytes in flight a lane; three blocks a CU by LDS).  The
// waves' sums meet at the end and the lane writes (or adds to) its link's nine
// entries.  FP64 throughout.
// Bound: L2 fills (1.66 GB for 0.95 GB of fields, links and forces at 16^3 x 32 x
// 16, 4.9 TB/s) and, one after the other, the LDS passes of six waves a CU.
// 16^3 x 32 x 16: 340 us, against 2 x 418 us of one launch per parity with the
// sum over s through LDS and 278 us for the packed copies; 445 us with every x
// neighbour brought as well, two blocks a CU and rotated slots (twice the bank
// conflicts), 376 us with 2 x 2 (z, t) planes for the tiles of the walk.
#include "dev_common.h"
#include "kernels.h"

namespace odwf {

constexpr int FS = 16;               // sites of a block
constexpr int FSLOTS = 4 * FS + 2;   // own sites, y, z, t neighbours, two x neighbours
constexpr int FLOADS = (FSLOTS * 12 + 63) / 64;  // chunks a lane brings, per field and slice
// first chunk of slot q in LDS: 16 lanes (four sites by four directions) that
// read the same component of their slots meet 16 different 16-byte banks
__host__ __device__ constexpr int slot_at(int q) { return 12 * q + 2 * (q >> 2) + (q >> 4); }
constexpr int FCH = slot_at(FSLOTS - 1) + 12;    // chunks of a field

struct ForceArgs {
  const uint4* chi;      // canonical [s][site][12] complex128
  const uint4* psi;
  const void* links[2];  // FP64 links by parity, [h][8][18]
  cpx<double>* F;        // canonical [t][z][y][x][mu][3][3]
  int L[4];
  FastDiv dx, dy, dz;    // Lx, Ly, Lz
  long V;
  uint32_t unit, units;  // blocks of a unit of the walk (0: linear), units of an (x, y) plane
  uint32_t tile[3];      // units, z and t of a tile
  int Ns, bc_t, accumulate;
};

// The lane's direction as data: gamma_mu = [[0, B], [B^dag, 0]], row r of B has
// one entry f_r at column p_r.  f z for f in {+-1, +-i} is z or (im, re) with a
// sign for each part, so the lanes of all four directions run the same code:
// the parts are picked by LDS address, the signs enter as factors +-1.
struct Dir {
  int p[2];        // column p_r
  int im[2];       // f_r imaginary
  double s[2][2];  // signs of the real and imaginary part of f_r z
};
__device__ __forceinline__ Dir dir_of(int mu) {
  Dir d;
  d.p[0] = mu < 2 ? 1 : 0;  // x, y: p = (1, 0); z, t: p = (0, 1)
  d.p[1] = 1 - d.p[0];
  // f: x (-i, -i), y (-1, +1), z (-i, +i), t (+1, +1);  -i z = (im, -re), +i z = (-im, re)
  d.im[0] = d.im[1] = mu == 0 || mu == 2;
  d.s[0][0] = mu == 1 ? -1.0 : 1.0;
  d.s[0][1] = mu == 3 ? 1.0 : -1.0;
  d.s[1][0] = mu == 2 ? -1.0 : 1.0;
  d.s[1][1] = mu == 0 ? -1.0 : 1.0;
  return d;
}

// half spinor psi_up - SIG B psi_dn of (1 - SIG gamma_mu) of the spinor in slot q
template <int SIG>
__device__ __forceinline__ void slot_half(const double* slot, const Dir& d, cpx<double> (&h)[6]) {
  constexpr double S = SIG > 0 ? -1.0 : 1.0;
#pragma unroll
  for (int r = 0; r < 2; r++)
#pragma unroll
    for (int c = 0; c < 3; c++) {
      const double* up = slot + (r * 3 + c) * 2;
      const double* dn = slot + ((2 + d.p[r]) * 3 + c) * 2;
      h[r * 3 + c] = {fma(S * d.s[r][0], dn[d.im[r]], up[0]), fma(S * d.s[r][1], dn[1 - d.im[r]], up[1])};
    }
}

// M += A + B^dag of one slice for the lane's link (site at q, neighbour at n).  A
// slice's eight products an entry come first, so that the sum over slices rounds
// once a slice.
__device__ __forceinline__ void link_slice(const double* chi, const double* psi, int q, int n, const Dir& d,
                                           cpx<double> (&m)[9]) {
  cpx<double> pn[6], cq[6], pq[6], cn[6];
  slot_half<+1>(psi + n, d, pn);  // (1 - gamma_mu) psi(x + mu)
  slot_half<+1>(chi + q, d, cq);  // with chi(x)
  slot_half<-1>(psi + q, d, pq);  // (1 + gamma_mu) psi(x)
  slot_half<-1>(chi + n, d, cn);  // with chi(x + mu)
#pragma unroll
  for (int b = 0; b < 3; b++)
#pragma unroll
    for (int a = 0; a < 3; a++) {
      // sum_sigma pn[b] conj(cq[a]) + conj(pq[a]) cn[b]
      cpx<double> v = {0.0, 0.0};
#pragma unroll
      for (int sg = 0; sg < 2; sg++) {
        const cpx<double> p = pn[sg * 3 + b], c = cq[sg * 3 + a], r = pq[sg * 3 + a], t = cn[sg * 3 + b];
        v.re = sg ? fma(p.re, c.re, v.re) : p.re * c.re;
        v.re = fma(p.im, c.im, v.re);
        v.im = sg ? fma(p.im, c.re, v.im) : p.im * c.re;
        v.im = fma(-p.re, c.im, v.im);
        v.re = fma(r.re, t.re, v.re);
        v.re = fma(r.im, t.im, v.re);
        v.im = fma(-r.im, t.re, v.im);
        v.im = fma(r.re, t.im, v.im);
      }
      m[b * 3 + a] = cadd(m[b * 3 + a], v);
    }
}

// first site of this block: XCD b % 8 takes a contiguous range of the walk, and
// the walk takes the smallest runs of rows that are whole blocks (units) in
// tiles of (y, z, t), so that forward neighbours meet in its L2
__device__ __forceinline__ uint32_t force_first_site(const ForceArgs& a) {
  const uint32_t nb8 = gridDim.x >> 3, rem8 = gridDim.x & 7, xcd = blockIdx.x & 7;
  uint32_t lb = xcd * nb8 + min(xcd, rem8) + (blockIdx.x >> 3);
  if (a.unit > 0) {
    auto split = [](uint32_t& n, uint32_t d) {  // n mod d, n <- n / d
      const uint32_t q = n / d, r = n - q * d;
      n = q;
      return r;
    };
    const uint32_t in = split(lb, a.unit);
    uint32_t y = split(lb, a.tile[0]), z = split(lb, a.tile[1]), t = split(lb, a.tile[2]);
    y += split(lb, a.units / a.tile[0]) * a.tile[0];
    z += split(lb, a.L[2] / a.tile[1]) * a.tile[1];
    t += lb * a.tile[2];
    lb = ((t * a.L[2] + z) * a.units + y) * a.unit + in;
  }
  return lb * FS;
}

__global__ void __launch_bounds__(128, 2) force_kernel(const ForceArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int slot_site[FSLOTS];
  __shared__ int x_slot[FS];  // LDS position of x + 1 per site
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const uint32_t i0 = force_first_site(a);
  const int n = (int)min((long)FS, a.V - (long)i0);
  // sites of the slots
  if (tid < 4 * FS) {
    const uint32_t k = min(tid % FS, n - 1), i = i0 + k;
    const uint32_t row = a.dx.div(i), x = i - row * a.dx.d;
    const uint32_t zt = a.dy.div(row), y = row - zt * a.dy.d;
    const uint32_t t = a.dz.div(zt), z = zt - t * a.dz.d;
    const int dir = tid / FS;  // 0: the site itself
    const int yy = dir == 1 ? (y + 1 == a.L[1] ? 0 : y + 1) : y;
    const int zz = dir == 2 ? (z + 1 == a.L[2] ? 0 : z + 1) : z;
    const int tt = dir == 3 ? (t + 1 == a.L[3] ? 0 : t + 1) : t;
    slot_site[tid] = ((tt * a.L[2] + zz) * a.L[1] + yy) * a.L[0] + x;
    if (dir == 0) {
      // x + 1 lies in the block, but for the last site (its neighbour is the next
      // block's first) and for the end of a row that began before the block
      const bool wrap = (int)x + 1 == a.L[0];
      const uint32_t ix = wrap ? i - x : i + 1;
      const bool in = ix >= i0 && ix < i0 + n;
      const int extra = 4 * FS + (wrap ? 0 : 1);
      x_slot[tid] = slot_at(in ? (int)(ix - i0) : extra);
    }
    if (tid == 0) {
      // the row the block begins in, and the site behind the block (clamped:
      // where there is none, no lane uses the slot)
      slot_site[4 * FS] = i - x;
      slot_site[4 * FS + 1] = (int)min((long)i0 + n, a.V - 1);
    }
  }
  __syncthreads();
  u32x4* buf = reinterpret_cast<u32x4*>(smem) + w * 2 * FCH;
  // this lane's chunks of a slice: index within a field, and LDS position
  uint32_t off[FLOADS];
  uint16_t put[FLOADS];
#pragma unroll
  for (int k = 0; k < FLOADS; k++) {
    const int e = min(l + 64 * k, FSLOTS * 12 - 1), q = e / 12, c = e % 12;
    off[k] = (uint32_t)slot_site[q] * 12 + c;
    put[k] = (uint16_t)(slot_at(q) + c);
  }
  const int site = l >> 2, mu = l & 3;
  const int own = 2 * slot_at(site), nb = 2 * (mu == 0 ? x_slot[site] : slot_at(FS * mu + site));
  cpx<double> m[9];
#pragma unroll
  for (int k = 0; k < 9; k++) m[k] = {0.0, 0.0};
  const Dir d = dir_of(mu);
  const u32x4* chi0 = reinterpret_cast<const u32x4*>(a.chi);
  const u32x4* psi0 = reinterpret_cast<const u32x4*>(a.psi);
  u32x4 v[2][FLOADS];
  const long first = (long)min(w, a.Ns - 1) * a.V * 12;
#pragma unroll
  for (int k = 0; k < FLOADS; k++) {
    v[0][k] = chi0[first + off[k]];
    v[1][k] = psi0[first + off[k]];
  }
#pragma unroll 1
  for (int s = w; s < a.Ns; s += 2) {
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < FLOADS; k++) {  // (the clamped lanes write one value to one place)
      buf[put[k]] = v[0][k];
      buf[FCH + put[k]] = v[1][k];
    }
    wave_lds_order();
    const long next = (long)min(s + 2, a.Ns - 1) * a.V * 12;  // (the last slice again behind the end)
#pragma unroll
    for (int k = 0; k < FLOADS; k++) {
      v[0][k] = chi0[next + off[k]];
      v[1][k] = psi0[next + off[k]];
    }
    const double* lds = reinterpret_cast<const double*>(buf);
    link_slice(lds, lds + 2 * FCH, own, nb, d, m);
  }
  // the waves' sums
  __syncthreads();
  double* red = reinterpret_cast<double*>(smem);
  if (w == 1) {
#pragma unroll
    for (int k = 0; k < 9; k++) {
      red[(2 * k) * 64 + l] = m[k].re;
      red[(2 * k + 1) * 64 + l] = m[k].im;
    }
  }
  __syncthreads();
  if (w == 1 || site >= n) return;
  const uint32_t i = i0 + site;
  const uint32_t row = a.dx.div(i), x = i - row * a.dx.d;
  const uint32_t zt = a.dy.div(row), y = row - zt * a.dy.d;
  const uint32_t t = a.dz.div(zt), z = zt - t * a.dz.d;
  const double f = mu == 3 && a.bc_t < 0 && t + 1 == (uint32_t)a.L[3] ? 0.5 : -0.5;  // M = -1/2 b (A + B^dag)
#pragma unroll
  for (int k = 0; k < 9; k++) {
    m[k].re = f * (m[k].re + red[(2 * k) * 64 + l]);
    m[k].im = f * (m[k].im + red[(2 * k + 1) * 64 + l]);
  }
  // F = TA(U M)
  const uint32_t j = row * (a.dx.d >> 1) + (x >> 1);
  const uint4* up = reinterpret_cast<const uint4*>((x + y + z + t) & 1 ? a.links[1] : a.links[0]) + ((long)j * 8 + mu) * 9;
  cpx<double> U[9], X[9];
#pragma unroll
  for (int k = 0; k < 9; k++) unpack_chunk<SP64>(up[k], &U[k]);
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int c = 0; c < 3; c++) {
      cpx<double> q = cmul(U[r * 3], m[c]);
      q = cfma(U[r * 3 + 1], m[3 + c], q);
      X[r * 3 + c] = cfma(U[r * 3 + 2], m[6 + c], q);
    }
  const double imtr = (X[0].im + X[4].im + X[8].im) / 3.0;  // - tr(X - X^dag) / 6
  cpx<double>* dst = a.F + ((long)i * 4 + mu) * 9;
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int c = 0; c < 3; c++) {
      cpx<double> q = {0.5 * (X[r * 3 + c].re - X[c * 3 + r].re), 0.5 * (X[r * 3 + c].im + X[c * 3 + r].im)};
      if (r == c) q.im -= imtr;
      if (a.accumulate) q = cadd(dst[r * 3 + c], q);
      dst[r * 3 + c] = q;
    }
}

hipError_t launch_force(const void* chi, const void* psi, const void* const links[2], void* F, int Ns, int bc_t,
                        int accumulate, const Geom& g, hipStream_t st) {
  if (Ns < 1 || g.V * 12 > 0xffffffffL) return hipErrorInvalidValue;  // 32-bit chunk offsets within a slice
  ForceArgs a;
  a.chi = reinterpret_cast<const uint4*>(chi);
  a.psi = reinterpret_cast<const uint4*>(psi);
  a.links[0] = links[0];
  a.links[1] = links[1];
  a.F = reinterpret_cast<cpx<double>*>(F);
  for (int d = 0; d < 4; d++) a.L[d] = g.L[d];
  a.dx = FastDiv(g.L[0]);
  a.dy = FastDiv(g.L[1]);
  a.dz = FastDiv(g.L[2]);
  a.V = g.V;
  int rows = 1;  // of a unit
  while (g.L[0] * rows % FS) rows *= 2;
  a.unit = a.units = 0;
  if (g.L[1] % rows == 0) {
    a.unit = g.L[0] * rows / FS;
    a.units = g.L[1] / rows;
    auto tile = [](int n) { return n % 4 == 0 ? 4u : (n % 2 == 0 ? 2u : 1u); };
    a.tile[0] = rows >= 4 ? 1 : tile(a.units);
    a.tile[1] = tile(g.L[2]);
    a.tile[2] = tile(g.L[3]);
  }
  a.Ns = Ns;
  a.bc_t = bc_t;
  a.accumulate = accumulate;
  const dim3 grid((unsigned)((g.V + FS - 1) / FS));
  hipLaunchKernelGGL(force_kernel, grid, dim3(128), 4 * FCH * sizeof(uint4), st, a);
  return hipGetLastError();
}

}  // namespace odwf
