// EAM density, embedding derivative, per-atom energy and forces from the
// r < rc + skin list (gather only: every atom sums its own row, no atomics),
// and the velocity-Verlet kick/drift updates.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace vc {

struct Box {
  double L0, L1, L2;
};

// The density and force passes of large systems are bound by the loads they
// have in flight.  Their gathers hit L1 and L2 (at 1.95M atoms the memory is
// read at a third of its rate), each going to lines of its own (the k-th
// neighbours of adjacent atoms are rarely adjacent: 46 line accesses per load
// of a wave with one lane per atom); fewer instructions (without the periodic
// images half of them, or a fifth by another split of the pair's work) and
// (x, y) and (z, w) in arrays of their own changed nothing, registers did.  So
// LPA lanes share an atom, in pairs that read the two halves of one entry's
// quadruple in the same load (one line access per entry instead of two) and
// exchange what the other needs; lane l of a group takes entries l, l + LPA, ...
// of the row, and the group's first lane adds the terms in entry order.  At
// 1.95M atoms (polycrystal, 15.6 entries) density 116 -> 111 us, forces with
// kick and drift 169 -> 156 with two lanes.
// Rounds whose indices are loaded together, and rounds whose gathers are in
// flight together: more of them cost registers and so waves.  (The loads are
// named: an array of them had the compiler move the next ones up, 91 registers
// instead of 74 with two lanes.)  Rounds in flight 1, 2, 4: 1.02M atoms (one
// lane, 20 steps) 4.09, 3.54, 3.35 ms; 1.95M (two lanes) 7.31, 6.87, 7.09;
// 2,000 (four lanes) 0.37, 0.39, 0.40.
template <int LPA>
constexpr int NRF = LPA == 4 ? 4 : 8 / LPA;
template <int LPA>
constexpr int NRG = 4 / LPA;

// A row's first indices, loaded beside its length (what lies beyond the length
// is not used); the rest of a longer row is loaded as the rounds reach it.
template <int LPA>
struct FirstIdx {
  int32_t j[NRF<LPA>];
};
template <int LPA>
__device__ __forceinline__ FirstIdx<LPA> first_indices(const int32_t *__restrict__ nj, int64_t n,
                                                       int64_t i, int lane) {
  static_assert(NRF<LPA> * LPA <= KMAX, "rows");
  FirstIdx<LPA> f;
#pragma unroll
  for (int u = 0; u < NRF<LPA>; ++u) f.j[u] = nj[(int64_t)(u * LPA + lane) * n + i];
  return f;
}

// lane exchange inside quads
template <int CTRL>
__device__ __forceinline__ int dpp32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
  return __hiloint2double(dpp32<CTRL>(__double2hiint(v)), dpp32<CTRL>(__double2loint(v)));
}
constexpr int SWAP = 0xB1;  // quad_perm 1 0 3 2: the other lane of the pair

// The quadruple of entry j (this lane's), the pair's lanes reading one entry
// per load; odd: this lane is the second of its pair.
struct PairLoad {
  double2 a, b;  // this lane's halves of the first and of the second lane's entry
};
template <int LPA>
__device__ __forceinline__ PairLoad pair_load(const double2 *__restrict__ p, int32_t j, bool odd) {
  if (LPA == 1) return PairLoad{p[2 * (int64_t)j], p[2 * (int64_t)j + 1]};
  const int32_t o = dpp32<SWAP>(j);
  const int64_t ja = odd ? o : j, jb = odd ? j : o;
  PairLoad l;
  l.a = p[2 * ja + odd];
  l.b = p[2 * jb + odd];
  return l;
}
template <int LPA>
__device__ __forceinline__ double4 pair_quad(const PairLoad &l, bool odd) {
  if (LPA == 1) return make_double4(l.a.x, l.a.y, l.b.x, l.b.y);
  const double sx = odd ? l.a.x : l.b.x, sy = odd ? l.a.y : l.b.y;  // what the other lane needs
  const double rx = dpp64<SWAP>(sx), ry = dpp64<SWAP>(sy);
  return odd ? make_double4(rx, ry, l.b.x, l.b.y) : make_double4(l.a.x, l.a.y, rx, ry);
}

// s (first lane of the group) += the group's terms in lane order
template <int LPA, int K = 1>
__device__ __forceinline__ void add_group(double &s, double t) {
  if (K == 1) s += t;
  if constexpr (K < LPA) {
    s += dpp64<0x100 + K>(t);  // row_shl: the term of the lane K further
    add_group<LPA, K + 1>(s, t);
  }
}

// Minimum image without branches, the number min_image returns (d - L, d + L
// or d): L with the sign of d, or zero, is subtracted.
__device__ __forceinline__ double min_image_sub(double d, double L) {
  return d - (fabs(d) > 0.5 * L ? copysign(L, d) : 0.0);
}

// Which axes a wave has to wrap.  A neighbour within `reach` of an atom at
// reach <= x <= L - reach needs no periodic image (reach <= L / 2, so the plain
// difference is the minimum image), and most waves hold only such atoms along
// y and z, many along x: 0 none, 1 x, 2 every axis.  The wraps were about half
// of the instructions of a list entry in the density pass and a third in the
// force pass.  reach: a list entry was within rc + skin when the list was
// built, and since then each atom has moved at most skin / 2, or in a box
// scaled by lam since the build at most (lam (rc + skin) - rc) / 2 from its
// scaled position, so it is within 2 lam (rc + skin) - rc; 1 A of slack; -1
// for a box too small: wrap always.
__device__ __forceinline__ int wrap_axes(const double4 &q, const Box &b, double reach) {
  if (reach < 0.0) return 2;
  const bool x = !(q.x >= reach && q.x <= b.L0 - reach);
  const bool yz = !(q.y >= reach && q.y <= b.L1 - reach && q.z >= reach && q.z <= b.L2 - reach);
  return __any(yz) ? 2 : (__any(x) ? 1 : 0);
}

static double list_reach(const vcsgc_ctx *c) {
  double lam = 1.0, lmin = c->box[0];
  for (int d = 0; d < 3; ++d) {
    lam = std::max(lam, c->box[d] / c->box_build[d]);
    lmin = std::min(lmin, c->box[d]);
  }
  const double reach = 2.0 * lam * (c->pot.rc + c->skin) - c->pot.rc + 1.0;
  return reach < 0.5 * lmin ? reach : -1.0;
}

// (x, y, z, species) of every atom, packed for the density pass
__global__ void k_pack(int64_t n, const double *__restrict__ x, const double *__restrict__ y,
                       const double *__restrict__ z, const uint8_t *__restrict__ sp,
                       double2 *ps4) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  packed_store(ps4, i, x[i], y[i], z[i], (double)sp[i]);
}

hipError_t launch_pack(vcsgc_ctx *c) {
  k_pack<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, c->x, c->y, c->z, c->sp, c->ps4);
  return hipGetLastError();
}

// The density term of a list entry, its distance r and (EN) pair energy: the
// entry's atom at qj, the row's at qi, `in` false for padding.  A skipped pair
// gives +0.0: the sums start at +0.0 and are never -0.0, so adding it changes
// nothing (the padding entries, the atom itself at r^2 = 0, have r = NaN from
// sqrt_md, which the select drops).
struct DensityTerm {
  double rho, phi;
};

template <bool TAB, bool EN, int W>
__device__ __forceinline__ DensityTerm density_term(const double4 &qj, const double4 &qi, int si,
                                                    bool in, const Box &b, const PotD &p) {
  double dx = qj.x - qi.x, dy = qj.y - qi.y, dz = qj.z - qi.z;
  if (W >= 1) dx = min_image_sub(dx, b.L0);
  if (W >= 2) {
    dy = min_image_sub(dy, b.L1);
    dz = min_image_sub(dz, b.L2);
  }
  const double r2 = (dx * dx + dy * dy) + dz * dz;
  const double r = sqrt_md(r2);
  const bool near = in && r < p.rc;
  DensityTerm t;
  if (TAB) {
    t.rho = spline_at(tab_radial(p, qj.w != 0.0 ? 1 : 0), p.nr, near ? r : 0.0, p.inv_dr, nullptr);
  } else {
    const double d = p.rc - r;
    t.rho = (qj.w != 0.0 ? p.t[1] : p.t[0]) * (d * d);
  }
  t.rho = near ? t.rho : 0.0;
  t.phi = 0.0;
  if (EN) {
    // (two atoms at one place: their pair energy is that of r = 0)
    const bool zero = in && r2 < 0x1p-767;
    const double re = near ? r : 0.0;
    const double e = pot_phi<TAB ? 1 : 0>(p, si, qj.w != 0.0 ? 1 : 0, re);
    t.phi = near || zero ? e : 0.0;
  }
  return t;
}

// rho_i = sum_{j: r < rc} f_{s_j}(r) over the row of i, in entry order
// (f_X = t_X (rc - r)^2, or the tables when TAB), and with EN also
// sum_j phi(r); the sums are the group's first lane's
template <int LPA, bool TAB, bool EN, int W>
__device__ __forceinline__ DensityTerm density_row(int64_t n, int64_t i, int m, int lane,
                                                   const FirstIdx<LPA> &j0,
                                                   const double4 &qi,
                                                   const double2 *__restrict__ ps4,
                                                   const int32_t *__restrict__ nj, const Box &b,
                                                   const PotD &p) {
  DensityTerm s = {0.0, 0.0};
  const int si = qi.w != 0.0 ? 1 : 0;
  const bool odd = lane & 1;
  int32_t jb[NRF<LPA>];
#pragma unroll
  for (int u = 0; u < NRF<LPA>; ++u) jb[u] = u * LPA + lane < m ? j0.j[u] : (int32_t)i;
  for (int k0 = 0; k0 < m; k0 += NRF<LPA> * LPA) {
    if (k0) {
#pragma unroll
      for (int u = 0; u < NRF<LPA>; ++u) {
        const int k = k0 + u * LPA + lane;
        jb[u] = k < m ? nj[(int64_t)k * n + i] : (int32_t)i;
      }
    }
#pragma unroll
    for (int g = 0; g < NRF<LPA>; g += NRG<LPA>) {
      if (k0 + g * LPA >= m) break;
      PairLoad l0, l1, l2, l3;
      l0 = pair_load<LPA>(ps4, jb[g], odd);
      if constexpr (NRG<LPA> > 1) l1 = pair_load<LPA>(ps4, jb[g + 1], odd);
      if constexpr (NRG<LPA> > 2) l2 = pair_load<LPA>(ps4, jb[g + 2], odd);
      if constexpr (NRG<LPA> > 2) l3 = pair_load<LPA>(ps4, jb[g + 3], odd);
#pragma unroll
      for (int u = 0; u < NRG<LPA>; ++u) {
        const double4 q = pair_quad<LPA>(u == 0 ? l0 : u == 1 ? l1 : u == 2 ? l2 : l3, odd);
        const bool in = k0 + (g + u) * LPA + lane < m;
        const DensityTerm t = density_term<TAB, EN, W>(q, qi, si, in, b, p);
        add_group<LPA>(s.rho, t.rho);
        if (EN) add_group<LPA>(s.phi, t.phi);
      }
    }
  }
  return s;
}

// rho_i, and (x_i, y_i, z_i, F'_i) with F'_i = F'_{s_i}(rho_i) for the force
// pass, the species in the sign of x_i (positions are not negative); EN: also
// E_i = F_{s_i}(rho_i) + 0.5 sum_j phi(r)
template <bool TAB, bool EN>
__device__ __forceinline__ void density_store(int64_t i, const double4 &qi, const DensityTerm &s,
                                              const PotD &p, double *rho, double2 *pf4, double *e) {
  const int si = qi.w != 0.0 ? 1 : 0;
  rho[i] = s.rho;
  const double f = dembed<TAB ? 1 : 0>(p, si, s.rho);
  packed_store(pf4, i, si ? -fabs(qi.x) : fabs(qi.x), qi.y, qi.z, f);
  if (EN) e[i] = embed<TAB ? 1 : 0>(p, si, s.rho) + 0.5 * s.phi;
}

// What a density pass does for the list rebuilds: take over the statistics of
// a one-kernel build, and before a drift that bins its atoms clear the bin
// counts (their readers, the last step's list build, have finished).
struct BinClear {
  int32_t *count;  // NULL: not cleared
  int64_t nbins;
  DevState *ds;  // NULL: nothing to do
};
__device__ __forceinline__ void bin_clear(const BinClear &c, int64_t i, int64_t threads) {
  if (c.count)
    for (int64_t q = i; q < c.nbins; q += threads) c.count[q] = 0;
  if (i == 0 && c.ds->pairs_new) {
    c.ds->pairs_md = c.ds->pairs_new & ~PAIRS_BUILT;
    c.ds->kmax_md = c.ds->kmax_new;
    c.ds->pairs_new = 0ull;
    c.ds->kmax_new = 0;
  }
}

template <int LPA, bool TAB, bool EN>
__global__ void __launch_bounds__(BLOCK)
    k_density_md(int64_t n, const double2 *__restrict__ ps4, const int32_t *__restrict__ nj,
                 const uint8_t *__restrict__ cnt, Box b, double reach, PotD p, double *rho,
                 double2 *pf4, double *e, BinClear bc) {
  const int64_t gid = xcd_block() * blockDim.x + threadIdx.x;
  if (bc.ds) bin_clear(bc, gid, (int64_t)gridDim.x * blockDim.x);
  const int64_t i = gid / LPA;
  const int lane = (int)(gid % LPA);
  if (i >= n) return;  // whole groups leave together
  const FirstIdx<LPA> j0 = first_indices<LPA>(nj, n, i, lane);
  const double4 qi = packed_load(ps4, i);
  const int m = cnt[i];
  const int w = wrap_axes(qi, b, reach);
  DensityTerm s;
  if (w == 0)
    s = density_row<LPA, TAB, EN, 0>(n, i, m, lane, j0, qi, ps4, nj, b, p);
  else if (w == 1)
    s = density_row<LPA, TAB, EN, 1>(n, i, m, lane, j0, qi, ps4, nj, b, p);
  else
    s = density_row<LPA, TAB, EN, 2>(n, i, m, lane, j0, qi, ps4, nj, b, p);
  if (lane == 0) density_store<TAB, EN>(i, qi, s, p, rho, pf4, e);
}

// The part of a drift that readies the next device-decided rebuild: with pos
// the moved atom goes to its search bin (count, bmax slots each; a bin with
// more atoms than slots is the list build's to report), else the counts are
// cleared for the binning kernel.
struct BinDrift {
  int32_t *count;
  int64_t nbins;
  double4 *pos;
  Grid g;
  int bmax;
};
__device__ __forceinline__ void bin_drift_clear(const BinDrift &d, int64_t i, int64_t threads) {
  if (!d.pos)
    for (int64_t q = i; q < d.nbins; q += threads) d.count[q] = 0;
}
__device__ __forceinline__ void bin_drift_add(const BinDrift &d, int64_t i, double x, double y,
                                              double z) {
  if (!d.pos) return;
  const int bin = cell_of(d.g, x, y, z);
  const int slot = atomicAdd(&d.count[bin], 1);
  if (slot < d.bmax) d.pos[(int64_t)bin * d.bmax + slot] = make_double4(x, y, z, (double)i);
}

// [v += (dt/2)(F cm) (closing the previous step) ;] v += (dt/2)(F cm);
// x = wrap(x + dt v); raise ds->rebuild[par] when an atom has moved more than
// skin/2 from its position at the last build.  Also readies the next
// device-decided rebuild: the flag of the other parity (read by the previous
// step's rebuild kernels, which have finished) is cleared, and so are the
// search bins.
struct KickDrift {
  double *x, *y, *z, *vx, *vy, *vz;
  const double *xr, *yr, *zr;  // positions at the last MD-list build
  double2 *ps4;
  double dt, half_skin2;
  int kick_first, par;
  BinDrift bins;
  DevState *ds;
  const double *nvt;  // Nose-Hoover: v = (v s1) s2 before the kick (nvt[3], nvt[4]); NULL: none
};

// The step's clearing work, by thread i of a grid of `threads`.
__device__ __forceinline__ void kick_drift_clear(const KickDrift &k, int64_t i, int64_t threads) {
  bin_drift_clear(k.bins, i, threads);
  if (i == 0) k.ds->rebuild[k.par ^ 1] = 0;
}

// Kick and drift of atom i (species s) from its force; every active lane of
// the wave takes part in the rebuild vote.
struct KickIn {
  double ux, uy, uz, xr, yr, zr;
};
__device__ __forceinline__ KickIn kick_load(const KickDrift &k, int64_t i) {
  return KickIn{k.vx[i], k.vy[i], k.vz[i], k.xr[i], k.yr[i], k.zr[i]};
}
__device__ __forceinline__ void kick_drift_atom(const KickDrift &k, const KickIn &in, int64_t i,
                                                int s, double x0, double y0, double z0, double fxi,
                                                double fyi, double fzi, const Box &b,
                                                const PotD &p) {
  const double cm = by_species(p.cm, s);
  const double hdt = 0.5 * k.dt;
  const double ax = fxi * cm, ay = fyi * cm, az = fzi * cm;
  double ux = in.ux, uy = in.uy, uz = in.uz;
  if (k.nvt) {
    const double s1 = k.nvt[3], s2 = k.nvt[4];
    ux = ux * s1;
    uy = uy * s1;
    uz = uz * s1;
    ux = ux * s2;
    uy = uy * s2;
    uz = uz * s2;
  }
  if (k.kick_first) {
    ux = ux + hdt * ax;
    uy = uy + hdt * ay;
    uz = uz + hdt * az;
  }
  ux = ux + hdt * ax;
  uy = uy + hdt * ay;
  uz = uz + hdt * az;
  k.vx[i] = ux;
  k.vy[i] = uy;
  k.vz[i] = uz;
  const double nx = wrap_box(x0 + k.dt * ux, b.L0);
  const double ny = wrap_box(y0 + k.dt * uy, b.L1);
  const double nz = wrap_box(z0 + k.dt * uz, b.L2);
  k.x[i] = nx;
  k.y[i] = ny;
  k.z[i] = nz;
  packed_store(k.ps4, i, nx, ny, nz, (double)s);
  bin_drift_add(k.bins, i, nx, ny, nz);
  const double ex = min_image(nx - in.xr, b.L0);
  const double ey = min_image(ny - in.yr, b.L1);
  const double ez = min_image(nz - in.zr, b.L2);
  const unsigned long long moved = __ballot((ex * ex + ey * ey) + ez * ez > k.half_skin2);
  if (moved && __lane_id() == __ffsll((long long)moved) - 1) atomicOr(&k.ds->rebuild[k.par], 1);
}

// The force terms of a list entry inside rc:
//   s (x_j - x_i) / r, s = phi'(r) + F'_i f'_{s_j}(r) + F'_j f'_{s_i}(r),
// with phi'(r) = eps ((-2 d)(c0 + c1 r) + c1 d^2) and f'_X(r) = (-2 t_X) d,
// d = rc - r (or the tables when TAB), and VIR: w = s r; +0.0 outside rc (the
// sums start at +0.0 and are never -0.0, so adding it changes nothing).
struct ForceRow {  // what an atom's row shares
  double x, y, z, fp;
  int s;
  double e0, e1, ti;
};

template <bool TAB>
__device__ __forceinline__ ForceRow force_row_of(const double4 &q, const PotD &p) {
  ForceRow o;
  o.x = fabs(q.x);
  o.y = q.y;
  o.z = q.z;
  o.fp = q.w;
  o.s = __double2hiint(q.x) < 0 ? 1 : 0;
  o.e0 = o.e1 = o.ti = 0.0;
  if (!TAB) {
    o.e0 = by_pair(p.eps, o.s);
    o.e1 = by_pair(p.eps, o.s + 1);
    o.ti = by_species(p.t, o.s);
  }
  return o;
}

template <bool TAB, bool VIR, int W>
__device__ __forceinline__ double4 force_term(const double4 &q, const ForceRow &o, bool in,
                                              const Box &b, const PotD &p) {
  double dx = fabs(q.x) - o.x, dy = q.y - o.y, dz = q.z - o.z;
  if (W >= 1) dx = min_image_sub(dx, b.L0);
  if (W >= 2) {
    dy = min_image_sub(dy, b.L1);
    dz = min_image_sub(dz, b.L2);
  }
  const double r = sqrt_md((dx * dx + dy * dy) + dz * dz);
  double4 f = make_double4(0.0, 0.0, 0.0, 0.0);
  // a branch: the select form evaluates the FP64 division for every list
  // entry and measured slower than this one
  if (in && r < p.rc) {
    const int sj = __double2hiint(q.x) < 0 ? 1 : 0;
    double dphi, dfj, dfi;
    if (TAB) {
      spline_at(tab_radial(p, 2 + o.s + sj), p.nr, r, p.inv_dr, &dphi);
      spline_at(tab_radial(p, sj), p.nr, r, p.inv_dr, &dfj);
      spline_at(tab_radial(p, o.s), p.nr, r, p.inv_dr, &dfi);
    } else {
      const double d = p.rc - r;
      const double eps = sj ? o.e1 : o.e0, tj = sj ? p.t[1] : p.t[0];
      dphi = eps * (-2.0 * d * (p.c0 + p.c1 * r) + p.c1 * (d * d));
      dfj = -2.0 * tj * d;
      dfi = -2.0 * o.ti * d;
    }
    const double s = dphi + o.fp * dfj + q.w * dfi;
    if (VIR) f.w = s * r;
    const double coef = div_md(s, r);
    f.x = coef * dx;
    f.y = coef * dy;
    f.z = coef * dz;
  }
  return f;
}

// F_i (and VIR: w_i = sum_j s_ij r_ij, the atom's share of the virial sum),
// summed in entry order by the group's first lane
template <int LPA, bool TAB, bool VIR, int W>
__device__ __forceinline__ double4 force_row(int64_t n, int64_t i, int m, int lane,
                                             const FirstIdx<LPA> &j0,
                                             const ForceRow &o, const double2 *__restrict__ pf4,
                                             const int32_t *__restrict__ nj, const Box &b,
                                             const PotD &p) {
  double4 f = make_double4(0.0, 0.0, 0.0, 0.0);
  const bool odd = lane & 1;
  int32_t jb[NRF<LPA>];
#pragma unroll
  for (int u = 0; u < NRF<LPA>; ++u) jb[u] = u * LPA + lane < m ? j0.j[u] : (int32_t)i;
  for (int k0 = 0; k0 < m; k0 += NRF<LPA> * LPA) {
    if (k0) {
#pragma unroll
      for (int u = 0; u < NRF<LPA>; ++u) {
        const int k = k0 + u * LPA + lane;
        jb[u] = k < m ? nj[(int64_t)k * n + i] : (int32_t)i;
      }
    }
#pragma unroll
    for (int g = 0; g < NRF<LPA>; g += NRG<LPA>) {
      if (k0 + g * LPA >= m) break;
      PairLoad l0, l1, l2, l3;
      l0 = pair_load<LPA>(pf4, jb[g], odd);
      if constexpr (NRG<LPA> > 1) l1 = pair_load<LPA>(pf4, jb[g + 1], odd);
      if constexpr (NRG<LPA> > 2) l2 = pair_load<LPA>(pf4, jb[g + 2], odd);
      if constexpr (NRG<LPA> > 2) l3 = pair_load<LPA>(pf4, jb[g + 3], odd);
#pragma unroll
      for (int u = 0; u < NRG<LPA>; ++u) {
        const double4 q = pair_quad<LPA>(u == 0 ? l0 : u == 1 ? l1 : u == 2 ? l2 : l3, odd);
        const bool in = k0 + (g + u) * LPA + lane < m;
        const double4 t = force_term<TAB, VIR, W>(q, o, in, b, p);
        add_group<LPA>(f.x, t.x);
        add_group<LPA>(f.y, t.y);
        add_group<LPA>(f.z, t.z);
        if (VIR) add_group<LPA>(f.w, t.w);
      }
    }
  }
  return f;
}

template <int LPA, bool TAB, bool VIR>
__device__ __forceinline__ double4 force_atom(int64_t n, int64_t i, int m, int lane,
                                              const FirstIdx<LPA> &j0,
                                              const double4 &qi, const ForceRow &o,
                                              const double2 *__restrict__ pf4,
                                              const int32_t *__restrict__ nj, const Box &b,
                                              double reach, const PotD &p) {
  const int w = wrap_axes(make_double4(o.x, qi.y, qi.z, 0.0), b, reach);
  if (w == 0) return force_row<LPA, TAB, VIR, 0>(n, i, m, lane, j0, o, pf4, nj, b, p);
  if (w == 1) return force_row<LPA, TAB, VIR, 1>(n, i, m, lane, j0, o, pf4, nj, b, p);
  return force_row<LPA, TAB, VIR, 2>(n, i, m, lane, j0, o, pf4, nj, b, p);
}

// KD: the forces are not stored but go straight into the next step's kick
// and drift (the positions it writes are not read by this pass, which
// gathers pf4).  TAB: tabulated potential.
template <int LPA, bool KD, bool TAB>
__global__ void __launch_bounds__(BLOCK)
    k_forces(int64_t n, const double2 *__restrict__ pf4, const int32_t *__restrict__ nj,
             const uint8_t *__restrict__ cnt, Box b, double reach, PotD p, double *fx, double *fy,
             double *fz, KickDrift kd) {
  const int64_t gid = xcd_block() * blockDim.x + threadIdx.x;
  const int64_t i = gid / LPA;
  const int lane = (int)(gid % LPA);
  if (KD) kick_drift_clear(kd, gid, (int64_t)gridDim.x * blockDim.x);
  if (i >= n) return;  // whole groups leave together
  const FirstIdx<LPA> j0 = first_indices<LPA>(nj, n, i, lane);
  const double4 qi = packed_load(pf4, i);
  const ForceRow o = force_row_of<TAB>(qi, p);
  KickIn ki;
  if (KD && LPA >= 4) ki = kick_load(kd, i);  // few waves: latency counts, not registers
  const double4 f = force_atom<LPA, TAB, false>(n, i, cnt[i], lane, j0, qi, o, pf4, nj, b, reach, p);
  if (lane) return;
  if (KD) {
    // the packed positions equal x, y, z bit for bit
    if (LPA < 4) ki = kick_load(kd, i);
    kick_drift_atom(kd, ki, i, o.s, o.x, o.y, o.z, f.x, f.y, f.z, b, p);
  } else {
    fx[i] = f.x;
    fy[i] = f.y;
    fz[i] = f.z;
  }
}

// forces and w_i = sum_j s_ij r_ij (the virial is -1/2 sum_i w_i)
template <int LPA, bool TAB>
__global__ void __launch_bounds__(BLOCK)
    k_forces_vir(int64_t n, const double2 *__restrict__ pf4, const int32_t *__restrict__ nj,
                 const uint8_t *__restrict__ cnt, Box b, double reach, PotD p, double *fx,
                 double *fy, double *fz, double *w) {
  const int64_t gid = xcd_block() * blockDim.x + threadIdx.x;
  const int64_t i = gid / LPA;
  const int lane = (int)(gid % LPA);
  if (i >= n) return;  // whole groups leave together
  const FirstIdx<LPA> j0 = first_indices<LPA>(nj, n, i, lane);
  const double4 qi = packed_load(pf4, i);
  const ForceRow o = force_row_of<TAB>(qi, p);
  const double4 f = force_atom<LPA, TAB, true>(n, i, cnt[i], lane, j0, qi, o, pf4, nj, b, reach, p);
  if (lane) return;
  fx[i] = f.x;
  fy[i] = f.y;
  fz[i] = f.z;
  w[i] = f.w;
}

// Lanes per atom.  Few atoms leave the chip idle and their time is latency: 4
// (20 NVE steps at 2,000 atoms 502 us with 1, 425 with 2, 375 with 4, 8 within
// 3% of 4 there and slower from 8,000 on; at 31,250 atoms 550, 460, 440; at
// 94,054 tabulated 1,370, 1,230, 1,285).  The tables' evaluations are worth a
// second lane at any size.  From there to about 1M atoms one lane: the
// quadruples fit the L2s and the exchange costs more than the saved line
// accesses (0.25M atoms 1,225 us with 1, 1,280 with 2; 1.02M 3,360 and 3,560);
// beyond, two for the passes of NVE and NPT steps (STEPS; 1.95M atoms 7,440 us
// with 1, 6,860 with 2), one for single passes over a lattice in its own
// order, whose neighbours do share lines (1.02M atoms, energy and forces: 141 us
// with 1, 162 with 2; 1.95M atoms in grains 272 and 298), and for the passes that
// store forces for a kernel of their own (NVT steps, the end of an NVE call).
// (Not measured between 1.02M and 1.95M atoms.)
template <bool STEPS, class F>
static void by_lanes(const vcsgc_ctx *c, F launch) {
  const std::integral_constant<int, 4> four{};
  const std::integral_constant<int, 2> two{};
  const std::integral_constant<int, 1> one{};
  const bool small = c->n <= 48 * 1024;
  if (c->pot.tab) {
    small ? launch(four, std::true_type{}) : launch(two, std::true_type{});
  } else if (small) {
    launch(four, std::false_type{});
  } else {
    if constexpr (STEPS)
      if (c->n > 1024 * 1024) return launch(two, std::false_type{});
    launch(one, std::false_type{});
  }
}

// the density pass (EN: with the atoms' energies) and the force pass for the
// context's potential form
template <bool EN, bool STEPS>
static void density_md_launch(vcsgc_ctx *c, const Box &b) {
  const double reach = list_reach(c);
  const BinClear bc = {md_binned_drift(c) ? c->bin_count : nullptr, c->nbins_total,
                       md_one_kernel_build(c) ? c->ds : nullptr};
  c->bins_clear = bc.count != nullptr;
  by_lanes<STEPS>(c, [&](auto lpa, auto tab) {
    k_density_md<lpa.value, tab.value, EN><<<grid_for(c->n * lpa.value), BLOCK, 0, c->stream>>>(
        c->n, c->ps4, c->md_j, c->md_cnt, b, reach, c->pot, c->rho_f, c->pf4, c->eatom, bc);
  });
}

template <bool KD>
static void forces_launch(vcsgc_ctx *c, const Box &b, const KickDrift &kd) {
  const double reach = list_reach(c);
  by_lanes<KD>(c, [&](auto lpa, auto tab) {
    k_forces<lpa.value, KD, tab.value><<<grid_for(c->n * lpa.value), BLOCK, 0, c->stream>>>(
        c->n, c->pf4, c->md_j, c->md_cnt, b, reach, c->pot, c->fx, c->fy, c->fz, kd);
  });
}

// the force pass alone (after a density pass at the same positions)
hipError_t launch_forces_only(vcsgc_ctx *c) {
  Box b{c->box[0], c->box[1], c->box[2]};
  const int h = tstart(c, VCSGC_KT_FORCES);
  forces_launch<false>(c, b, KickDrift{});
  tstop(c, h);
  return hipGetLastError();
}

hipError_t launch_forces(vcsgc_ctx *c) {
  Box b{c->box[0], c->box[1], c->box[2]};
  const int h = tstart(c, VCSGC_KT_DENSITY);
  density_md_launch<false, false>(c, b);
  tstop(c, h);
  return launch_forces_only(c);
}

static BinDrift bin_drift_args(vcsgc_ctx *c, bool binned) {
  c->bins_clear = false;
  const int *nb = c->reps[0].nb;
  return BinDrift{c->bin_count, c->reps[0].nbins, binned ? c->bin_pos : nullptr,
                  Grid{c->box[0], c->box[1], c->box[2], nb[0], nb[1], nb[2]}, c->bmax};
}

static KickDrift kick_drift_args(vcsgc_ctx *c, double dt, bool kick_first, int par) {
  const double hs = 0.5 * c->skin;
  KickDrift k{};
  k.x = c->x;
  k.y = c->y;
  k.z = c->z;
  k.vx = c->vx;
  k.vy = c->vy;
  k.vz = c->vz;
  k.xr = c->xr;
  k.yr = c->yr;
  k.zr = c->zr;
  k.ps4 = c->ps4;
  k.dt = dt;
  k.half_skin2 = hs * hs;
  k.kick_first = kick_first ? 1 : 0;
  k.par = par;
  k.bins = bin_drift_args(c, md_binned_drift(c));
  k.ds = c->ds;
  return k;
}

hipError_t launch_forces_kick_drift(vcsgc_ctx *c, double dt, bool kick_first, int par) {
  Box b{c->box[0], c->box[1], c->box[2]};
  int h = tstart(c, VCSGC_KT_DENSITY);
  density_md_launch<false, true>(c, b);
  tstop(c, h);
  h = tstart(c, VCSGC_KT_FORCES);
  forces_launch<true>(c, b, kick_drift_args(c, dt, kick_first, par));
  tstop(c, h);
  return hipGetLastError();
}

// One pass for the densities, F' and the energies.  (Densities, then the
// energies in a pass of their own, then the densities again for the forces:
// 197 us at 1,024,000 atoms, now 50.)
hipError_t launch_energy(vcsgc_ctx *c) {
  Box b{c->box[0], c->box[1], c->box[2]};
  int h = tstart(c, VCSGC_KT_ENERGY);
  density_md_launch<true, false>(c, b);
  tstop(c, h);
  return hipGetLastError();
}

__global__ void __launch_bounds__(BLOCK)
    k_kick_drift(int64_t n, const double *__restrict__ fx, const double *__restrict__ fy,
                 const double *__restrict__ fz, const uint8_t *__restrict__ sp, Box b, PotD p,
                 KickDrift k) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  kick_drift_clear(k, i, (int64_t)gridDim.x * blockDim.x);
  if (i >= n) return;
  kick_drift_atom(k, kick_load(k, i), i, sp[i], k.x[i], k.y[i], k.z[i], fx[i], fy[i], fz[i], b, p);
}

__global__ void k_kick(int64_t n, double *vx, double *vy, double *vz, const double *__restrict__ fx,
                       const double *__restrict__ fy, const double *__restrict__ fz,
                       const uint8_t *__restrict__ sp, PotD p, double dt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double cm = by_species(p.cm, sp[i]);
  const double hdt = 0.5 * dt;
  vx[i] = vx[i] + hdt * (fx[i] * cm);
  vy[i] = vy[i] + hdt * (fy[i] * cm);
  vz[i] = vz[i] + hdt * (fz[i] * cm);
}

hipError_t launch_kick_drift(vcsgc_ctx *c, double dt, bool kick_first, int par) {
  Box b{c->box[0], c->box[1], c->box[2]};
  int h = tstart(c, VCSGC_KT_KICKDRIFT);
  k_kick_drift<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, c->fx, c->fy, c->fz, c->sp, b,
                                                        c->pot,
                                                        kick_drift_args(c, dt, kick_first, par));
  tstop(c, h);
  return hipGetLastError();
}

hipError_t launch_kick(vcsgc_ctx *c, double dt) {
  int h = tstart(c, VCSGC_KT_KICK);
  k_kick<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, c->fx, c->fy, c->fz,
                                                  c->sp, c->pot, dt);
  tstop(c, h);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Nose-Hoover NVT.  Per step: the thermostat's half steps at the step
// boundary (one block), the scaled kick and drift, forces, the closing kick
// fused with the kinetic-energy chunk sums.  The kinetic energy that steers
// the thermostat is summed in a fixed shape: chunks of 256 atoms by halving
// strides (one block per chunk), chunk c into accumulator c mod 256, and the
// accumulators by halving strides again.
// ---------------------------------------------------------------------------
// chunk sums of m ((vx^2 + vy^2) + vz^2), after the closing half kick if KICK
template <bool KICK>
__global__ void __launch_bounds__(BLOCK)
    k_nvt_ke(int64_t n, double *vx, double *vy, double *vz, const double *__restrict__ fx,
             const double *__restrict__ fy, const double *__restrict__ fz,
             const uint8_t *__restrict__ sp, PotD p, double dt, double *part) {
  __shared__ double a[BLOCK];
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  double t = 0.0;
  if (i < n) {
    const int s = sp[i];
    double ux = vx[i], uy = vy[i], uz = vz[i];
    if (KICK) {
      const double cm = by_species(p.cm, s);
      const double hdt = 0.5 * dt;
      ux = ux + hdt * (fx[i] * cm);
      uy = uy + hdt * (fy[i] * cm);
      uz = uz + hdt * (fz[i] * cm);
      vx[i] = ux;
      vy[i] = uy;
      vz[i] = uz;
    }
    t = by_species(p.mass, s) * ((ux * ux + uy * uy) + uz * uz);
  }
  a[threadIdx.x] = t;
  __syncthreads();
  for (int h = BLOCK / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) a[threadIdx.x] = a[threadIdx.x] + a[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = a[0];
}

struct NvtPar {
  double dt, g, kT, Q;
};

// one half step (dt/2) of xi, eta and the carried kinetic energy K; returns
// the velocity factor s = (1 - xi dt/4) / (1 + xi dt/4)
__device__ __forceinline__ double nh_half(const NvtPar &q, double &K, double &xi, double &eta) {
  const double q4 = 0.25 * q.dt;
  xi = xi + q4 * ((2.0 * K - q.g * q.kT) / q.Q);
  const double a = xi * q4;
  const double s = (1.0 - a) / (1.0 + a);
  K = K * s * s;
  eta = eta + xi * (0.5 * q.dt);
  xi = xi + q4 * ((2.0 * K - q.g * q.kT) / q.Q);
  return s;
}

// K from the chunk sums; the end-of-step half (mode bit 0) and the next
// step's opening half (bit 1); nvt = (xi, eta, K, s1, s2)
__global__ void __launch_bounds__(BLOCK)
    k_nvt_thermo(int64_t nch, const double *__restrict__ part, double *nvt, NvtPar q, int mode) {
  __shared__ double a[BLOCK];
  double acc = 0.0;
  for (int64_t c = threadIdx.x; c < nch; c += BLOCK) acc = acc + part[c];
  a[threadIdx.x] = acc;
  __syncthreads();
  for (int h = BLOCK / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) a[threadIdx.x] = a[threadIdx.x] + a[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double K = 0.5 * a[0] / ACC;
    double xi = nvt[0], eta = nvt[1];
    double s1 = 1.0, s2 = 1.0;
    if (mode & 1) s1 = nh_half(q, K, xi, eta);
    if (mode & 2) s2 = nh_half(q, K, xi, eta);
    nvt[0] = xi;
    nvt[1] = eta;
    nvt[2] = K;
    nvt[3] = s1;
    nvt[4] = s2;
  }
}

// v = v s1 (the last end-of-step half of a call)
__global__ void k_nvt_scale(int64_t n, double *vx, double *vy, double *vz,
                            const double *__restrict__ nvt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double s1 = nvt[3];
  vx[i] = vx[i] * s1;
  vy[i] = vy[i] * s1;
  vz[i] = vz[i] * s1;
}

hipError_t launch_nvt_ke(vcsgc_ctx *c, double dt, bool closing_kick) {
  const unsigned nch = (unsigned)((c->n + BLOCK - 1) / BLOCK);
  int h = tstart(c, VCSGC_KT_KICK);
  if (closing_kick)
    k_nvt_ke<true><<<nch, BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, c->fx, c->fy, c->fz,
                                                 c->sp, c->pot, dt, c->nvt_part);
  else
    k_nvt_ke<false><<<nch, BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, c->fx, c->fy,
                                                  c->fz, c->sp, c->pot, dt, c->nvt_part);
  tstop(c, h);
  return hipGetLastError();
}

hipError_t launch_nvt_thermo(vcsgc_ctx *c, double dt, int mode) {
  NvtPar q;
  q.dt = dt;
  q.g = 3.0 * (double)c->n - 3.0;
  q.kT = KB * c->nvt_T;
  q.Q = q.g * q.kT * c->nvt_tau * c->nvt_tau;
  k_nvt_thermo<<<1, BLOCK, 0, c->stream>>>((c->n + BLOCK - 1) / BLOCK, c->nvt_part, c->nvt, q,
                                          mode);
  return hipGetLastError();
}

hipError_t launch_nvt_kick_drift(vcsgc_ctx *c, double dt, int par) {
  Box b{c->box[0], c->box[1], c->box[2]};
  KickDrift k = kick_drift_args(c, dt, false, par);
  k.nvt = c->nvt;
  int h = tstart(c, VCSGC_KT_KICKDRIFT);
  k_kick_drift<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, c->fx, c->fy, c->fz, c->sp, b,
                                                        c->pot, k);
  tstop(c, h);
  return hipGetLastError();
}

hipError_t launch_nvt_scale(vcsgc_ctx *c) {
  k_nvt_scale<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, c->nvt);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Conjugate-gradient relaxation: the per-atom work of the minimizer driven
// from the host (trial positions, the fixed-shape totals that steer it, the
// direction update).  Vectors of 3n doubles hold the x, y and z components
// one after the other.  Totals are taken in the fixed shape of the energy
// reduction: chunks of BLOCK atoms by halving strides, chunk c into
// accumulator c mod BLOCK, the accumulators by halving strides.
// ---------------------------------------------------------------------------
// x = wrap(x0 + a d) per component, ps4 packed alongside; raises
// ds->rebuild[0] when an atom is more than skin/2 from its position at the
// last MD-list build
__global__ void __launch_bounds__(BLOCK)
    k_cg_move(int64_t n, const double *__restrict__ x0, const double *__restrict__ d, double a,
              double *x, double *y, double *z, const uint8_t *__restrict__ sp, double2 *ps4,
              const double *__restrict__ xr, const double *__restrict__ yr,
              const double *__restrict__ zr, Box b, double half_skin2, BinDrift bins,
              DevState *ds) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  bin_drift_clear(bins, i, (int64_t)gridDim.x * BLOCK);
  bool far = false;
  if (i < n) {
    const double nx = wrap_box(x0[i] + a * d[i], b.L0);
    const double ny = wrap_box(x0[n + i] + a * d[n + i], b.L1);
    const double nz = wrap_box(x0[2 * n + i] + a * d[2 * n + i], b.L2);
    x[i] = nx;
    y[i] = ny;
    z[i] = nz;
    packed_store(ps4, i, nx, ny, nz, (double)sp[i]);
    bin_drift_add(bins, i, nx, ny, nz);
    const double ex = min_image(nx - xr[i], b.L0);
    const double ey = min_image(ny - yr[i], b.L1);
    const double ez = min_image(nz - zr[i], b.L2);
    far = (ex * ex + ey * ey) + ez * ez > half_skin2;
  }
  const unsigned long long moved = __ballot(far);
  if (moved && __lane_id() == __ffsll((long long)moved) - 1) atomicOr(&ds->rebuild[0], 1);
}

// K values per thread into the block's chunk values (halving strides; the
// last by maximum if MAX), value k of chunk c into part[k nch + c].
template <int K, bool MAX>
__device__ __forceinline__ void chunk_values(const double (&v)[K], double *part) {
  __shared__ double s[K][BLOCK];
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < K; ++k) s[k][t] = v[k];
  __syncthreads();
  for (int h = BLOCK / 2; h > 0; h >>= 1) {
    if (t < h)
#pragma unroll
      for (int k = 0; k < K; ++k)
        s[k][t] = MAX && k == K - 1 ? fmax(s[k][t], s[k][t + h]) : s[k][t] + s[k][t + h];
    __syncthreads();
  }
  if (t == 0)
#pragma unroll
    for (int k = 0; k < K; ++k) part[(int64_t)k * gridDim.x + blockIdx.x] = s[k][0];
}

// The start of a line search: the direction d = F (copy) or d = F + b d, the
// positions and forces kept for it (x0, f0), and the chunk values of F . d and
// max_i |d_i|^2; per-atom dot terms (a_x b_x + a_y b_y) + a_z b_z.
__global__ void __launch_bounds__(BLOCK)
    k_cg_start(int64_t n, const double *__restrict__ x, const double *__restrict__ y,
               const double *__restrict__ z, const double *__restrict__ fx,
               const double *__restrict__ fy, const double *__restrict__ fz, double *d, double *x0,
               double *f0, double b, int copy, double *part) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  double v[2] = {0.0, 0.0};
  if (i < n) {
    const double gx = fx[i], gy = fy[i], gz = fz[i];
    double ux = gx, uy = gy, uz = gz;
    if (!copy) {
      ux = gx + b * d[i];
      uy = gy + b * d[n + i];
      uz = gz + b * d[2 * n + i];
    }
    d[i] = ux;
    d[n + i] = uy;
    d[2 * n + i] = uz;
    x0[i] = x[i];
    x0[n + i] = y[i];
    x0[2 * n + i] = z[i];
    f0[i] = gx;
    f0[n + i] = gy;
    f0[2 * n + i] = gz;
    v[0] = (gx * ux + gy * uy) + gz * uz;
    v[1] = (ux * ux + uy * uy) + uz * uz;
  }
  chunk_values<2, true>(v, part);
}

// Chunk values of an evaluation: E, F . F and F . f0.
__global__ void __launch_bounds__(BLOCK)
    k_cg_eval(int64_t n, const double *__restrict__ e, const double *__restrict__ fx,
              const double *__restrict__ fy, const double *__restrict__ fz,
              const double *__restrict__ f0, double *part) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  double v[3] = {0.0, 0.0, 0.0};
  if (i < n) {
    const double gx = fx[i], gy = fy[i], gz = fz[i];
    v[0] = e[i];
    v[1] = (gx * gx + gy * gy) + gz * gz;
    v[2] = (gx * f0[i] + gy * f0[n + i]) + gz * f0[2 * n + i];
  }
  chunk_values<3, false>(v, part);
}

// The K totals from the chunk values (one block) into out[0..K); with ds also
// out[K]: what a device-decided rebuild overflowed (1: a bin, 2: a row), and
// out[K + 1]: whether one was due, the flag being lowered.  out is pinned host
// memory: one synchronization tells the host all it has to know about a move
// and the evaluation after it (a copy to pageable memory costs about 15 us
// more, and there were four per line search and two per NPT step: ten line
// searches at 128,000 atoms 2.2 -> 1.3 ms, 20 NPT steps at 2,000 atoms 1.55 ->
// 0.85 ms, at 0.5M 4.1 -> 3.6 ms).
template <int K, bool MAX>
__global__ void __launch_bounds__(BLOCK)
    k_totals(int64_t nch, const double *__restrict__ part, double *out, DevState *ds) {
  __shared__ double s[K][BLOCK];
  const int t = threadIdx.x;
  double v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = 0.0;
  for (int64_t c = t; c < nch; c += BLOCK) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double p = part[k * nch + c];
      v[k] = MAX && k == K - 1 ? fmax(v[k], p) : v[k] + p;
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) s[k][t] = v[k];
  __syncthreads();
  for (int h = BLOCK / 2; h > 0; h >>= 1) {
    if (t < h)
#pragma unroll
      for (int k = 0; k < K; ++k)
        s[k][t] = MAX && k == K - 1 ? fmax(s[k][t], s[k][t + h]) : s[k][t] + s[k][t + h];
    __syncthreads();
  }
  if (t == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = s[k][0];
    if (ds) {
      out[K] = (ds->bin_overflow ? 1.0 : 0.0) + (ds->overflow ? 2.0 : 0.0);
      out[K + 1] = ds->rebuild[0] ? 1.0 : 0.0;
      ds->rebuild[0] = 0;
    }
  }
}

hipError_t launch_cg_move(vcsgc_ctx *c, const double *x0, const double *d, double a) {
  Box b{c->box[0], c->box[1], c->box[2]};
  const double hs = 0.5 * c->skin;
  k_cg_move<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, x0, d, a, c->x, c->y, c->z, c->sp,
                                                     c->ps4, c->xr, c->yr, c->zr, b, hs * hs,
                                                     bin_drift_args(c, md_binned_drift(c)), c->ds);
  return hipGetLastError();
}

hipError_t launch_cg_start(vcsgc_ctx *c, double *d, double *x0, double *f0, double b, bool copy,
                           double *part, double *out) {
  const int nch = grid_for(c->n);
  k_cg_start<<<nch, BLOCK, 0, c->stream>>>(c->n, c->x, c->y, c->z, c->fx, c->fy, c->fz, d, x0, f0,
                                           b, copy ? 1 : 0, part);
  k_totals<2, true><<<1, BLOCK, 0, c->stream>>>(nch, part, out, nullptr);
  return hipGetLastError();
}

hipError_t launch_cg_eval(vcsgc_ctx *c, const double *f0, double *part, double *out) {
  const int nch = grid_for(c->n);
  k_cg_eval<<<nch, BLOCK, 0, c->stream>>>(c->n, c->eatom, c->fx, c->fy, c->fz, f0, part);
  k_totals<3, false><<<1, BLOCK, 0, c->stream>>>(nch, part, out, c->ds);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Isotropic NPT (Nose-Hoover thermostat and barostat), the per-atom parts of
// a step driven from the host: the scalings, kicks and drift of the
// splitting T(h) B(h) V(h) X(dt) [forces] V(h) B(h) T(h) (h = dt/2) take
// their factors from the host, which integrates the thermostat and barostat
// variables from the fixed-shape totals of the kinetic energy and virial.
// ---------------------------------------------------------------------------
// v = ((v f1) f2) c; v += h a; v = v c; x = wrap((x q + dt v) q) in the new
// box; ps4 packed; raises ds->rebuild[0] when some atom is farther than thr
// from its list-build position scaled to the new box (lam = L / L_build per
// axis), or always when thr <= 0
__global__ void __launch_bounds__(BLOCK)
    k_npt_kick_drift(int64_t n, double *x, double *y, double *z, double *vx, double *vy,
                     double *vz, const double *__restrict__ fx, const double *__restrict__ fy,
                     const double *__restrict__ fz, const uint8_t *__restrict__ sp, PotD p,
                     double f1, double f2, double c, double h, double dt, double q, Box b,
                     double lx, double ly, double lz, double thr,
                     const double *__restrict__ xr, const double *__restrict__ yr,
                     const double *__restrict__ zr, double2 *ps4, BinDrift bins, DevState *ds) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  bin_drift_clear(bins, i, (int64_t)gridDim.x * BLOCK);
  bool far = false;
  if (i < n) {
    const int s = sp[i];
    const double cm = by_species(p.cm, s);
    double ux = vx[i], uy = vy[i], uz = vz[i];
    ux = ux * f1;
    uy = uy * f1;
    uz = uz * f1;
    ux = ux * f2;
    uy = uy * f2;
    uz = uz * f2;
    ux = ux * c;
    uy = uy * c;
    uz = uz * c;
    ux = ux + h * (fx[i] * cm);
    uy = uy + h * (fy[i] * cm);
    uz = uz + h * (fz[i] * cm);
    ux = ux * c;
    uy = uy * c;
    uz = uz * c;
    vx[i] = ux;
    vy[i] = uy;
    vz[i] = uz;
    const double nx = wrap_box((x[i] * q + dt * ux) * q, b.L0);
    const double ny = wrap_box((y[i] * q + dt * uy) * q, b.L1);
    const double nz = wrap_box((z[i] * q + dt * uz) * q, b.L2);
    x[i] = nx;
    y[i] = ny;
    z[i] = nz;
    packed_store(ps4, i, nx, ny, nz, (double)s);
    bin_drift_add(bins, i, nx, ny, nz);
    const double ex = min_image(nx - lx * xr[i], b.L0);
    const double ey = min_image(ny - ly * yr[i], b.L1);
    const double ez = min_image(nz - lz * zr[i], b.L2);
    far = !(thr > 0.0) || (ex * ex + ey * ey) + ez * ez > thr * thr;
  }
  const unsigned long long moved = __ballot(far);
  if (moved && __lane_id() == __ffsll((long long)moved) - 1) atomicOr(&ds->rebuild[0], 1);
}

// [v = v c; v += h a; v = v c;] chunk values of m ((vx^2 + vy^2) + vz^2) and
// of w.  After a rebuild that overflowed nothing is kicked: the host rebuilds
// and repeats the evaluation.
template <bool KICK>
__global__ void __launch_bounds__(BLOCK)
    k_npt_kick_sums(int64_t n, double *vx, double *vy, double *vz,
                    const double *__restrict__ fx, const double *__restrict__ fy,
                    const double *__restrict__ fz, const uint8_t *__restrict__ sp, PotD p,
                    double c, double h, const double *__restrict__ w, double *part,
                    const DevState *ds) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (KICK && (ds->bin_overflow || ds->overflow)) return;
  double v[2] = {0.0, 0.0};
  if (i < n) {
    const int s = sp[i];
    double ux = vx[i], uy = vy[i], uz = vz[i];
    if (KICK) {
      const double cm = by_species(p.cm, s);
      ux = ux * c;
      uy = uy * c;
      uz = uz * c;
      ux = ux + h * (fx[i] * cm);
      uy = uy + h * (fy[i] * cm);
      uz = uz + h * (fz[i] * cm);
      ux = ux * c;
      uy = uy * c;
      uz = uz * c;
      vx[i] = ux;
      vy[i] = uy;
      vz[i] = uz;
    }
    v[0] = by_species(p.mass, s) * ((ux * ux + uy * uy) + uz * uz);
    v[1] = w[i];
  }
  chunk_values<2, false>(v, part);
}

// v *= s
__global__ void k_scale_v(int64_t n, double *vx, double *vy, double *vz, double s) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  vx[i] = vx[i] * s;
  vy[i] = vy[i] * s;
  vz[i] = vz[i] * s;
}

hipError_t launch_forces_virial(vcsgc_ctx *c, double *w) {
  Box b{c->box[0], c->box[1], c->box[2]};
  int h = tstart(c, VCSGC_KT_DENSITY);
  density_md_launch<false, true>(c, b);
  tstop(c, h);
  h = tstart(c, VCSGC_KT_FORCES);
  const double reach = list_reach(c);
  by_lanes<true>(c, [&](auto lpa, auto tab) {
    k_forces_vir<lpa.value, tab.value><<<grid_for(c->n * lpa.value), BLOCK, 0, c->stream>>>(
        c->n, c->pf4, c->md_j, c->md_cnt, b, reach, c->pot, c->fx, c->fy, c->fz, w);
  });
  tstop(c, h);
  return hipGetLastError();
}

hipError_t launch_npt_kick_drift(vcsgc_ctx *c, double f1, double f2, double cv, double h,
                                 double dt, double q, const double lam[3], double thr,
                                 bool binned) {
  Box b{c->box[0], c->box[1], c->box[2]};
  int t = tstart(c, VCSGC_KT_KICKDRIFT);
  k_npt_kick_drift<<<grid_for(c->n), BLOCK, 0, c->stream>>>(
      c->n, c->x, c->y, c->z, c->vx, c->vy, c->vz, c->fx, c->fy, c->fz, c->sp, c->pot, f1, f2,
      cv, h, dt, q, b, lam[0], lam[1], lam[2], thr, c->xr, c->yr, c->zr, c->ps4,
      bin_drift_args(c, binned), c->ds);
  tstop(c, t);
  return hipGetLastError();
}

hipError_t launch_npt_sums(vcsgc_ctx *c, bool kick, double cv, double h, const double *w,
                           double *part, double *out) {
  const int nch = grid_for(c->n);
  int t = tstart(c, VCSGC_KT_KICK);
  if (kick)
    k_npt_kick_sums<true><<<nch, BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, c->fx, c->fy,
                                                        c->fz, c->sp, c->pot, cv, h, w, part, c->ds);
  else
    k_npt_kick_sums<false><<<nch, BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, c->fx,
                                                         c->fy, c->fz, c->sp, c->pot, cv, h, w,
                                                         part, c->ds);
  k_totals<2, false><<<1, BLOCK, 0, c->stream>>>(nch, part, out, c->ds);
  tstop(c, t);
  return hipGetLastError();
}

hipError_t launch_scale_v(vcsgc_ctx *c, double s) {
  k_scale_v<<<grid_for(c->n), BLOCK, 0, c->stream>>>(c->n, c->vx, c->vy, c->vz, s);
  return hipGetLastError();
}

}  // namespace vc
