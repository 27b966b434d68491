// Host runtime: workspaces, fifth-dimension programs, kernel helpers and the
// hopping-kernel profiler.
#include "runtime.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>

namespace odwf {

static thread_local std::string g_last_error;
void set_error(const std::string& msg) { g_last_error = msg; }
const char* last_error_cstr() { return g_last_error.c_str(); }

size_t bytes_per_complex(int prec) {
  switch (prec) {
    case PREC64: return 16;
    case PREC32: return 8;
    default: return 4;
  }
}

size_t half_bytes(long h, int nrhs, int Ns, int prec) {
  return (size_t)h * nrhs * Ns * 12 * bytes_per_complex(prec);
}

size_t scale_bytes(long h, int nrhs, int Ns, int prec) {
  return (prec == PREC16 || prec == PRECB16) ? (size_t)h * nrhs * Ns * sizeof(float) : 0;
}

Workspace::~Workspace() {
  for (auto& kv : bufs)
    if (kv.second.p) (void)hipFree(kv.second.p);
}

void* Workspace::get(const std::string& name, size_t bytes) {
  if (bytes == 0) bytes = 16;
  DevBuf& b = bufs[name];
  if (b.bytes >= bytes) return b.p;
  if (b.p) {
    (void)hipDeviceSynchronize();
    (void)hipFree(b.p);
    b.p = nullptr;
    b.bytes = 0;
  }
  if (hipMalloc(&b.p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    b.p = nullptr;
    return nullptr;
  }
  b.bytes = bytes;
  return b.p;
}

HV Workspace::half(const std::string& name, long h, int nrhs, int Ns, int prec) {
  HV v;
  v.prec = prec;
  v.d = get(name, half_bytes(h, nrhs, Ns, prec));
  const size_t sb = scale_bytes(h, nrhs, Ns, prec);
  if (sb) v.sc = reinterpret_cast<float*>(get(name + ".sc", sb));
  return v;
}

size_t Workspace::total() const {
  size_t t = 0;
  for (auto& kv : bufs) t += kv.second.bytes;
  return t;
}

// ---- fifth-dimension programs -------------------------------------------------

static M5Prog mk(std::initializer_list<M5Op> ops, int dense = -1) {
  M5Prog p;
  std::memset(&p, 0, sizeof(p));
  p.n = 0;
  p.dense = dense;
  for (const M5Op& o : ops) p.op[p.n++] = o;
  return p;
}
static M5Op op(M5Type t, CoefId d, CoefId e = CF_ONE) { return M5Op{t, d, e, 0}; }

M5Prog prog_none() { return mk({}); }
// A^{-1} = (1 + L) B^{-1} omega,  B = a + c L
M5Prog prog_ainv() {
  return mk({op(M5_SCALE, CF_OMEGA), op(M5_SOLVE_LO, CF_A_INV, CF_C), op(M5_MUL_LO, CF_ONE, CF_ONE)}, DN_AINV);
}
// A^{-T} = omega B^{-T} (1 + L)^T
M5Prog prog_ainv_t() {
  return mk({op(M5_MUL_UP, CF_ONE, CF_ONE), op(M5_SOLVE_UP, CF_A_INV, CF_CSHIFT), op(M5_SCALE, CF_OMEGA)}, DN_AINV_T);
}
// A = omega^{-1} B (1 + L)^{-1}
M5Prog prog_a() {
  return mk({op(M5_SOLVE_LO, CF_ONE, CF_ONE), op(M5_MUL_LO, CF_A, CF_C), op(M5_SCALE, CF_OMEGA_INV)}, DN_A);
}
// A^T = (1 + L)^{-T} B^T omega^{-1}
M5Prog prog_a_t() {
  return mk({op(M5_SCALE, CF_OMEGA_INV), op(M5_MUL_UP, CF_A, CF_CSHIFT), op(M5_SOLVE_UP, CF_ONE, CF_ONE)}, DN_A_T);
}
M5Prog prog_omega() { return mk({op(M5_SCALE, CF_OMEGA)}); }
M5Prog prog_omega_inv() { return mk({op(M5_SCALE, CF_OMEGA_INV)}); }
M5Prog prog_1pl() { return mk({op(M5_MUL_LO, CF_ONE, CF_ONE)}, DN_1PL); }
M5Prog prog_1pl_inv() { return mk({op(M5_SOLVE_LO, CF_ONE, CF_ONE)}, DN_1PL_INV); }
M5Prog prog_1pl_t() { return mk({op(M5_MUL_UP, CF_ONE, CF_ONE)}, DN_1PL_T); }
M5Prog prog_ainv_winv() {
  return mk({op(M5_SOLVE_LO, CF_A_INV, CF_C), op(M5_MUL_LO, CF_ONE, CF_ONE)}, DN_AINV_WINV);
}
M5Prog prog_omega2() { return mk({op(M5_SCALE, CF_OMEGA2)}); }

// The dense forms, in the chirality-local order of the programs.  With L_k the
// shift (corner kappa) and e_l the last unit vector,
//     P = 1 + L = P0 + kappa e_0 e_l^T,   B = a + c L = B0 + kappa c_0 e_0 e_l^T,
//     (X0 + kappa x e_0 e_l^T)^{-1} = X0^{-1} - kappa x / (1 + kappa x e_l^T X0^{-1} e_0) X0^{-1} e_0 e_l^T X0^{-1},
// and a product of one factor and the inverse of the other collapses to one
// rank-1 term: A^{-1} = P B^{-1} omega has u = e_0 - c_0 P0 B0^{-1} e_0,
// w^T = e_l^T B0^{-1} omega, q = c_0 (B0^{-1})_{l0}; A = omega^{-1} B P^{-1} has
// u = omega^{-1} (c_0 e_0 - B0 P0^{-1} e_0), w^T = e_l^T P0^{-1}, q = (P0^{-1})_{l0}.
// P0^{-1} has entries (-1)^{i-j}, B0^{-1} follows a column at a time, and a factor is
// bidiagonal, so a product's entry is a sum of two: N^2 operations a matrix (16
// slices: 18 us in all).
void dense_tables(int Ns, double m0, const double* omega, double* tab, double q[][2]) {
  using ld = long double;
  using Mat = ld[DENSE_N][DENSE_N];
  const int N = Ns, l = Ns - 1;
  std::memset(tab, 0, sizeof(double) * NDENSE * DENSE_LEN);
  for (int chi = 0; chi < 2; chi++) {
    ld w[DENSE_N], a[DENSE_N], c[DENSE_N], u[DENSE_N], v[DENSE_N];
    Mat P0 = {}, Pi = {}, Bi = {}, m = {};
    for (int s = 0; s < N; s++) {
      w[s] = omega[chi ? N - 1 - s : s];
      a[s] = (4.0L - m0) * w[s] + 1.0L;
      c[s] = (4.0L - m0) * w[s] - 1.0L;
    }
    for (int j = 0; j < N; j++) {
      P0[j][j] = Pi[j][j] = 1.0L;
      Bi[j][j] = 1.0L / a[j];
      if (j > 0) P0[j][j - 1] = 1.0L;
      for (int i = j + 1; i < N; i++) {
        Pi[i][j] = -Pi[i - 1][j];
        Bi[i][j] = -c[i] * Bi[i - 1][j] / a[i];
      }
    }
    auto put = [&](int id, const Mat& m, const ld* u, const ld* v, ld qq, bool tr) {
      double* t = tab + (size_t)id * DENSE_LEN + chi * DENSE_CHI;
      for (int i = 0; i < N; i++) {
        const int si = chi ? l - i : i;  // local index of slice i
        for (int b = 0; b < DENSE_N; b += N) {
          for (int j = 0; j < N; j++) {
            const int sj = chi ? l - j : j;
            t[(b + i) * DENSE_N + b + j] = (double)(tr ? m[sj][si] : m[si][sj]);
          }
          t[DENSE_N * DENSE_N + b + i] = (double)(tr ? v[si] : u[si]);
          t[DENSE_N * DENSE_N + DENSE_N + b + i] = (double)(tr ? u[si] : v[si]);
        }
      }
      q[id][chi] = (double)qq;
    };
    // A^{-1}, A^{-T}, A^{-1} omega^{-1}
    for (int i = 0; i < N; i++)
      for (int j = 0; j <= i; j++) m[i][j] = (i > 0 ? Bi[i - 1][j] : 0.0L) + Bi[i][j];
    for (int s = 0; s < N; s++) {
      u[s] = (s == 0 ? 1.0L : 0.0L) - c[0] * m[s][0];
      v[s] = Bi[l][s];
    }
    put(DN_AINV_WINV, m, u, v, c[0] * Bi[l][0], false);
    for (int i = 0; i < N; i++)
      for (int s = 0; s < N; s++) m[i][s] *= w[s];
    for (int s = 0; s < N; s++) v[s] *= w[s];
    put(DN_AINV, m, u, v, c[0] * Bi[l][0], false);
    put(DN_AINV_T, m, u, v, c[0] * Bi[l][0], true);
    // A, A^T
    for (int i = 0; i < N; i++)
      for (int j = 0; j <= i; j++) m[i][j] = (i > 0 ? c[i] * Pi[i - 1][j] : 0.0L) + a[i] * Pi[i][j];
    for (int s = 0; s < N; s++) {
      u[s] = ((s == 0 ? c[0] : 0.0L) - m[s][0]) / w[s];
      v[s] = Pi[l][s];
    }
    for (int i = 0; i < N; i++)
      for (int s = 0; s < N; s++) m[i][s] /= w[i];
    put(DN_A, m, u, v, Pi[l][0], false);
    put(DN_A_T, m, u, v, Pi[l][0], true);
    // (1 + L)^{-1}, 1 + L, (1 + L)^T
    for (int s = 0; s < N; s++) u[s] = -Pi[s][0];
    put(DN_1PL_INV, Pi, u, v, Pi[l][0], false);
    for (int s = 0; s < N; s++) u[s] = s == 0, v[s] = s == l;
    put(DN_1PL, P0, u, v, 0.0L, false);
    put(DN_1PL_T, P0, u, v, 0.0L, true);
  }
}

DenseArg dense_arg(const OpCtx& c, const M5Prog& p) {
  DenseArg d;
  std::memset(&d, 0, sizeof(d));
  if (!dense_ns(c.Ns()) || p.n == 0 || p.dense < 0) return d;
  d.tab = c.S->dense + (size_t)p.dense * DENSE_LEN;
  double most = 1.0;  // of |rho| and 1, or NaN
  for (int chi = 0; chi < 2; chi++)
    for (int r = 0; r < c.nrhs; r++) {
      const double rho = c.kappa[r] / (1.0 + c.kappa[r] * c.S->dense_q[p.dense][chi]);
      d.rho[chi * MAXRHS + r] = rho;
      if (!std::isfinite(rho)) most = std::numeric_limits<double>::quiet_NaN();
      else if (std::fabs(rho) > most) most = std::fabs(rho);
    }
  const double reach = 4 * most * std::max(1.0, c.S->dense_w[p.dense]);  // (4: for the roundings)
  d.lim64 = std::numeric_limits<double>::max() / reach;
  d.lim32 = (float)(std::numeric_limits<float>::max() / reach);
  return d;
}

const double* diag_of(const OpCtx& c, const M5Prog& p) {
  if (p.n != 1 || p.op[0].type != M5_SCALE) return nullptr;
  return reinterpret_cast<const double*>(c.S->coef64) + p.op[0].d * c.Ns();
}

// ---- kernel helpers -------------------------------------------------------------

static size_t site_bytes(int prec) {
  return 12 * bytes_per_complex(prec) + ((prec == PREC16 || prec == PRECB16) ? 4 : 0);
}

// ---- block traversal of the hopping kernel -------------------------------------
// Default, when the x-rows split evenly into blocks: tiles of one x-row
// segment by 8 (4 when Ly is not a multiple of 8) by 4 rows in (y, z), t
// innermost, the eight XCDs walking a group of 4 x 2 adjacent tiles in
// lockstep (other group shapes, then contiguous XCD ranges, when the tile
// counts do not divide).  Otherwise XCD-aware contiguous block ranges.
// ODWF_TRAVERSAL ("linear", "xcd", "Ty,Tz", "Ty,Tz,Tt" or "Ty,Tz,Tt,Tx"; Tx = 0
// is the whole row) and ODWF_XCD ("contiguous", "lockstep" or "lockstep:Gy",
// Gy the tiles of a group along y) override for tuning.
static void traversal(HopArgs& a) {
  const int spb = a.spb;
  const int hx = a.L[0] / 2;
  a.xcd = 1;
  a.tile_y = a.tile_z = a.tile_t = a.tile_x = 0;
  a.xcd_gy = 4;
  int ty = a.L[1] % 8 == 0 ? 8 : 4, tz = 4, tt = 0, tx = 1, gy = 4;
  bool lockstep = true;
  const char* env = getenv("ODWF_TRAVERSAL");
  if (env) {
    if (!strcmp(env, "linear")) {
      a.xcd = 0;
      return;
    }
    if (!strcmp(env, "xcd")) return;
    const int n = sscanf(env, "%d,%d,%d,%d", &ty, &tz, &tt, &tx);
    if (n < 2) return;
    if (n < 3) tt = 0;
    if (n < 4) tx = 0;
  }
  if (const char* xe = getenv("ODWF_XCD")) {
    lockstep = !strncmp(xe, "lockstep", 8);
    if (lockstep && xe[8] == ':') gy = atoi(xe + 9);
  }
  if (ty > 0 && tz > 0 && hx % spb == 0 && a.L[1] % ty == 0 && a.L[2] % tz == 0) {
    const int nseg = hx / spb;
    a.tile_y = ty;
    a.tile_z = tz;
    if (tt > 0 && a.L[3] % tt == 0) a.tile_t = tt;
    if (tx > 0 && nseg % tx == 0) a.tile_x = tx;
    if (lockstep) {
      const int nty = a.L[1] / ty, ntz = a.L[2] / tz;
      const int pref[5] = {gy, 4, 2, 8, 1};
      for (int g : pref) {
        if ((g == 1 || g == 2 || g == 4 || g == 8) && nty % g == 0 && ntz % (8 / g) == 0) {
          a.xcd = 2;
          a.xcd_gy = g;
          break;
        }
      }
    }
  }
}

static hipError_t hop_args(const OpCtx& c, int out_par, int dag, const HV& in, const HV* out, const HopOpt& o,
                           HopArgs& a) {
  std::memset(&a, 0, sizeof(a));
  const odwf_lattice L = c.S->lat;
  a.in = in.d;
  a.in_sc = in.sc;
  a.links = c.links(out_par);
  a.out = out ? out->d : nullptr;
  a.out_sc = out ? out->sc : nullptr;
  a.xin = o.x ? o.x->d : nullptr;
  a.xin_sc = o.x ? o.x->sc : nullptr;
  a.cg_r = o.cg_r ? o.cg_r->d : nullptr;
  a.cg_r_sc = o.cg_r ? o.cg_r->sc : nullptr;
  a.cg_p = o.cg_p ? o.cg_p->d : nullptr;
  a.cg_p_sc = o.cg_p ? o.cg_p->sc : nullptr;
  a.scal = o.scal;
  a.partial = o.partial;
  a.fin_partial = o.fin_partial;
  a.fin_nblocks = hop_nblocks(L->g, c.nrhs, c.Ns(), c.prec);
  a.fin_scal = o.fin_scal;
  a.gate = o.gate;
  a.gate_mode = o.gate ? o.gate_mode : GATE_NONE;
  a.coef = c.coef();
  for (int r = 0; r < MAXRHS; r++) a.kappa[r] = r < c.nrhs ? c.kappa[r] : 0.0;
  a.prog_h = o.ph;
  a.prog_x = o.px;
  a.prog_o = o.po;
  a.c_h = o.ch;
  a.c_x = o.cx;
  a.h = (int)L->g.h;
  a.nrhs = c.nrhs;
  a.out_par = out_par;
  a.bc_t = L->bc_t;
  a.dag = dag;
  for (int d = 0; d < 4; d++) a.L[d] = L->g.L[d];
  a.dn_h = dense_arg(c, o.ph);
  a.dn_x = dense_arg(c, o.px);
  a.dn_o = dense_arg(c, o.po);
  a.diag_o = diag_of(c, o.po);
  // N_s <= 16 has kernels for dense programs, and for scalings of the result
  if (dense_ns(c.Ns()) && ((o.ph.n > 0 && !a.dn_h.tab) || (o.px.n > 0 && !a.dn_x.tab) ||
                           (o.po.n > 0 && !a.dn_o.tab && !a.diag_o)))
    return hipErrorInvalidValue;
  const int hx = a.L[0] / 2;
  a.plain = o.ph.n == 0 && o.po.n == 0 && !o.x && !o.partial && !o.fin_partial && o.ch == 1.0;
  a.spb = hop_launch_spb(L->g, c.nrhs, c.Ns(), c.prec, a.plain);
  a.small = hop_small(L->g, c.nrhs, c.Ns(), c.prec) && !(a.plain && c.prec != PREC64);
  a.nblocks = (a.h + a.spb - 1) / a.spb;
  a.rows = hx % a.spb == 0 && a.L[0] <= 256;
  traversal(a);
  a.d_hx = FastDiv(hx);
  a.d_y = FastDiv(a.L[1]);
  a.d_z = FastDiv(a.L[2]);
  if (a.tile_y > 0) {
    const int nseg = hx / a.spb, tx = a.tile_x > 0 ? a.tile_x : nseg, tl = a.tile_t > 0 ? a.tile_t : a.L[3];
    const int gy = a.xcd == 2 ? a.xcd_gy : 1, gz = a.xcd == 2 ? 8 / a.xcd_gy : 1;
    a.d_tx = FastDiv(tx);
    a.d_ty = FastDiv(a.tile_y);
    a.d_tz = FastDiv(a.tile_z);
    a.d_tl = FastDiv(tl);
    a.d_per = FastDiv(tx * a.tile_y * a.tile_z * tl);
    a.d_ny = FastDiv(a.L[1] / a.tile_y / gy);
    a.d_nz = FastDiv(a.L[2] / a.tile_z / gz);
    a.d_nx = FastDiv(nseg / tx);
  }
  return hipSuccess;
}

hipError_t hop(const OpCtx& c, int out_par, int dag, const HV& in, const HV* out, const HopOpt& o) {
  HopArgs a;
  HIPRET(hop_args(c, out_par, dag, in, out, o, a));
  const odwf_lattice L = c.S->lat;
  // launches gated to the active right-hand sides of a batch are counted with
  // the bytes of all nrhs (exact while every slot is active); launches gated to
  // pending reliable updates mostly exit at once and are not counted
  const bool prof = prof_on() && !c.noprof && (!o.gate || o.gate_mode == GATE_ACTIVE);
  if (prof) prof_begin(c.st, (c.prec & 3) * 2 + (dag ? 1 : 0));
  hipError_t e = launch_hop(a, c.prec, c.S->Ns, c.st);
  if (prof) {
    const double n5 = (double)L->g.h * c.nrhs * c.S->Ns;
    int streams = 1 + (out ? 1 : 0) + (o.x ? 1 : 0);
    if (o.cg_r) streams += 2;          // r read and written
    else if (o.cg_p) streams += 1;     // f read
    const double link_b = (double)L->g.h * 8 * (c.prec == PREC64 ? 18 * 8 : 12 * 4);
    prof_end(c.st, n5 * site_bytes(c.prec) * streams + link_b);
  }
  return e;
}

// Both output parities of an operator, out_p = hop(in_{1-p}) with x term in_p: one
// launch where the four-wave kernel takes them (D of 4^4 x 8 in FP64 25.3 -> 20.1 us a call), else two.
hipError_t hop_pair(const OpCtx& c, int dag, const HV& in_e, const HV& in_o, const HV& out_e, const HV& out_o,
                    HopOpt o) {
  const bool apart = out_e.d != in_e.d && out_e.d != in_o.d && out_o.d != in_e.d && out_o.d != in_o.d;
  o.x = &in_e;
  if (!hop_small(c.S->lat->g, c.nrhs, c.Ns(), c.prec) || !apart || o.partial || prof_on()) {
    HIPRET(hop(c, 0, dag, in_o, &out_e, o));
    o.x = &in_o;
    return hop(c, 1, dag, in_e, &out_o, o);
  }
  HopArgs a, b;
  HIPRET(hop_args(c, 0, dag, in_o, &out_e, o, a));
  o.x = &in_o;
  HIPRET(hop_args(c, 1, dag, in_e, &out_o, o, b));
  a.pair = 1;
  a.other = {b.in, b.in_sc, b.links, b.xin, b.xin_sc, b.out, b.out_sc, b.out_par};
  return launch_hop(a, c.prec, c.S->Ns, c.st);
}

hipError_t m5(const OpCtx& c, const HV& in, const HV& out, const M5Prog& p) {
  KappaArr k;
  for (int r = 0; r < MAXRHS; r++) k.v[r] = r < c.nrhs ? c.kappa[r] : 0.0;
  return launch_m5(c.prec, in.d, in.sc, out.d, out.sc, p, dense_arg(c, p), c.coef(), k, c.h(), c.nrhs, c.Ns(), c.st);
}

// a program that runs inside the layout kernels: none, a scaling, or a dense one
static bool in_tile(const OpCtx& c, const M5Prog& p) { return p.n == 0 || diag_of(c, p) || dense_ns(c.Ns()); }
static HalfIO half_io(const OpCtx& c, const HV* v, const M5Prog& p) {
  HalfIO h;
  if (!v) return h;
  h.d = v->d;
  h.sc = v->sc;
  if (in_tile(c, p)) {
    h.dn = dense_arg(c, p);
    h.diag = diag_of(c, p);
  }
  return h;
}

hipError_t pack(const OpCtx& c, const void* canon, int r0, const HV* e, const HV* o, const M5Prog& pe,
                const M5Prog& po) {
  HIPRET(launch_pack(c.prec, canon, r0, half_io(c, e, pe), half_io(c, o, po), c.nrhs, c.Ns(), c.S->lat->g, c.st));
  if (e && !in_tile(c, pe)) HIPRET(m5(c, *e, *e, pe));
  if (o && !in_tile(c, po)) HIPRET(m5(c, *o, *o, po));
  return hipSuccess;
}

hipError_t unpack(const OpCtx& c, const HV* e, const HV* o, void* canon, int r0, const M5Prog& p) {
  if (e && !in_tile(c, p)) HIPRET(m5(c, *e, *e, p));
  if (o && !in_tile(c, p)) HIPRET(m5(c, *o, *o, p));
  return launch_unpack(c.prec, half_io(c, e, p), half_io(c, o, p), canon, r0, c.nrhs, c.Ns(), c.S->lat->g, c.st);
}

// ---- profiler -------------------------------------------------------------------

struct ProfRec {
  hipEvent_t a, b;
  double bytes;
  int key;  // prec * 2 + dag
};
static std::mutex g_prof_mtx;
static bool g_prof = false;
static std::vector<ProfRec> g_recs;
static std::vector<hipEvent_t> g_pool;
static thread_local hipEvent_t g_open = nullptr;
static long long g_launches = 0;
static double g_ms = 0.0, g_bytes = 0.0;
static long long g_k_launches[8] = {0};
static double g_k_ms[8] = {0}, g_k_bytes[8] = {0};
static thread_local int g_open_key = 0;

bool prof_on() { return g_prof; }

static hipEvent_t take_event() {
  if (!g_pool.empty()) {
    hipEvent_t e = g_pool.back();
    g_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}

static void drain_locked() {
  for (ProfRec& r : g_recs) {
    float ms = 0.f;
    (void)hipEventSynchronize(r.b);
    (void)hipEventElapsedTime(&ms, r.a, r.b);
    g_ms += ms;
    g_bytes += r.bytes;
    g_launches += 1;
    g_k_ms[r.key] += ms;
    g_k_bytes[r.key] += r.bytes;
    g_k_launches[r.key] += 1;
    g_pool.push_back(r.a);
    g_pool.push_back(r.b);
  }
  g_recs.clear();
}

void prof_begin(hipStream_t st, int key) {
  std::lock_guard<std::mutex> lk(g_prof_mtx);
  if (g_recs.size() > 4096) drain_locked();
  g_open_key = key;
  g_open = take_event();
  (void)hipEventRecord(g_open, st);
}

void prof_end(hipStream_t st, double bytes) {
  std::lock_guard<std::mutex> lk(g_prof_mtx);
  hipEvent_t b = take_event();
  (void)hipEventRecord(b, st);
  g_recs.push_back(ProfRec{g_open, b, bytes, g_open_key});
  g_open = nullptr;
}

void prof_enable(int on) {
  std::lock_guard<std::mutex> lk(g_prof_mtx);
  drain_locked();
  g_prof = on != 0;
  g_launches = 0;
  g_ms = 0.0;
  g_bytes = 0.0;
  for (int k = 0; k < 8; k++) {
    g_k_launches[k] = 0;
    g_k_ms[k] = g_k_bytes[k] = 0.0;
  }
}

void prof_read(long long* launches, double* ms, double* bytes) {
  std::lock_guard<std::mutex> lk(g_prof_mtx);
  drain_locked();
  if (launches) *launches = g_launches;
  if (ms) *ms = g_ms;
  if (bytes) *bytes = g_bytes;
}

void prof_read_kernel(int prec, int dag, long long* launches, double* ms, double* bytes) {
  std::lock_guard<std::mutex> lk(g_prof_mtx);
  drain_locked();
  const int key = (prec & 3) * 2 + (dag ? 1 : 0);
  if (launches) *launches = g_k_launches[key];
  if (ms) *ms = g_k_ms[key];
  if (bytes) *bytes = g_k_bytes[key];
}

}  // namespace odwf

odwf::Workspace& odwf_solver_s::workspace(hipStream_t st) {
  auto it = ws.find(st);
  if (it != ws.end()) return *it->second;
  odwf::Workspace* w = new odwf::Workspace();
  ws[st] = w;
  return *w;
}
