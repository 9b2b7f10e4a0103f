// C ABI: context lifecycle, argument validation, scratch management and the
// host side of the sweep / EAM / MD calls.  See include/vcsgc.h.
#include <cmath>
#include <cstdio>
#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "common.hpp"

namespace {

std::string g_create_error;

template <typename T>
hipError_t dalloc(T **p, size_t count) {
  *p = nullptr;
  if (count == 0) count = 1;
  return hipMalloc((void **)p, sizeof(T) * count);
}

void free_all(vcsgc_ctx *c) {
  void *ptrs[] = {c->bin_count,  c->bin_atoms,  c->cell_count, c->cell_start, c->cell_atoms,
                  c->cell_fill,  c->mc_j,       c->mc_r,
                  c->mc_cnt,     c->md_j,       c->md_cnt,    c->xr,   c->yr,
                  c->zr,         c->rho,        c->rho_f,      c->eatom, c->red,
                  c->rec,        c->ds,         c->ps4,        c->pf4,       c->part,
                  c->d_rs,       c->d_wg_rep,   c->d_j,        c->d_r,
                  c->d_cnt,      c->scan_tmp,   c->snap,       c->bin_pos,
                  c->md_rows,    c->sites,      c->site_lnu,
                  c->u_site,     c->u_j,        c->u_rho,      c->u_v,
                  c->stage_lnug, c->m_sites,   c->m_lnu,      c->m_lnu2,     c->m_lnug,   c->m_rec,
                  c->m_part,     c->s_rec,      c->s_part,     c->nvt,        c->nvt_part,
                  c->tab_coef,   c->cg,         c->npt_part,   c->g_start,    c->g_list,
                  c->g_cum,      c->g_cnt,      c->big_lnu,    c->big_site};
  for (void *p : ptrs)
    if (p) (void)hipFree(p);
  if (c->h_pin) (void)hipHostFree(c->h_pin);
  if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
  if (c->graph) (void)hipGraphDestroy(c->graph);
  vc::free_stage_graph(c);
  vc::free_pipe_graph(c);
}

vcsgc_status fail(vcsgc_ctx *c, vcsgc_status st, const std::string &msg) {
  if (c) {
    c->err = msg;
    if (st == VCSGC_E_DEVICE) c->sticky = true;
  } else {
    g_create_error = msg;
  }
  return st;
}

vcsgc_status dev_fail(vcsgc_ctx *c, hipError_t e, const char *where) {
  std::string m = std::string(where) + ": " + hipGetErrorString(e);
  return fail(c, VCSGC_E_DEVICE, m);
}

#define VC_CHECK(ctx, expr, where)                      \
  do {                                                  \
    hipError_t _e = (expr);                             \
    if (_e != hipSuccess) return dev_fail(ctx, _e, where); \
  } while (0)

bool is_fin(double v) { return std::isfinite(v); }

vc::DevState read_state(vcsgc_ctx *c, hipError_t *e) {
  vc::DevState h;
  std::memset(&h, 0, sizeof(h));
  // through the pinned copy when there is one (a pageable copy is staged)
  vc::DevState *dst = c->h_state ? c->h_state : &h;
  *e = hipMemcpyAsync(dst, c->ds, sizeof(h), hipMemcpyDeviceToHost, c->stream);
  if (*e == hipSuccess) *e = hipStreamSynchronize(c->stream);
  if (*e == hipSuccess && dst != &h) h = *dst;
  return h;
}

// Grow the search bins after an overflow (capacity doubles).
vcsgc_status grow_bins(vcsgc_ctx *c) {
  if (c->bmax >= 1024) return fail(c, VCSGC_E_OVERFLOW, "more than 1024 atoms in a search bin");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  (void)hipFree(c->bin_atoms);
  (void)hipFree(c->bin_pos);
  c->bin_atoms = nullptr;
  c->bin_pos = nullptr;
  c->bmax *= 2;
  VC_CHECK(c, dalloc(&c->bin_atoms, (size_t)c->nbins_total * c->bmax), "allocation");
  if (c->reps.size() == 1)
    VC_CHECK(c, dalloc(&c->bin_pos, (size_t)c->nbins_total * c->bmax), "allocation");
  int zero = 0;
  VC_CHECK(c, hipMemcpyAsync(&c->ds->bin_overflow, &zero, sizeof(int), hipMemcpyHostToDevice,
                             c->stream),
           "reset");
  return VCSGC_OK;
}

// Rebuild cells + the r < rc list + the density cache; checks row overflow.
vcsgc_status refresh_mc(vcsgc_ctx *c) {
  for (;;) {
    for (const RepHost &r : c->reps) {
      VC_CHECK(c, vc::launch_bin_cells(c, r), "binning");
      VC_CHECK(c, vc::launch_bin_search(c, r), "binning");
      VC_CHECK(c, vc::launch_build_mc_list(c, r), "neighbour list");
      if (c->desc) VC_CHECK(c, vc::launch_build_desc_list(c, r), "descriptor list");
    }
    VC_CHECK(c, vc::launch_mc_row_stats(c), "neighbour list");
    VC_CHECK(c, vc::launch_density_mc(c), "density");
    hipError_t e;
    vc::DevState h = read_state(c, &e);
    if (e != hipSuccess) return dev_fail(c, e, "neighbour list");
    if (h.bin_overflow) {
      vcsgc_status st = grow_bins(c);
      if (st) return st;
      continue;
    }
    if (h.overflow)
      return fail(c, VCSGC_E_OVERFLOW, "a site has more than 32 neighbours within rc");
    c->kmax_used = h.kmax_used;
    c->mc_stats_stale = false;
    c->mc_valid = true;
    return VCSGC_OK;
  }
}

// After MD the r < rc + skin list is valid for the current positions and
// rho_f holds the current densities: the cells are re-binned, the r < rc rows
// are filtered out of the MD rows and the density cache is a copy of rho_f
// (both bitwise what a fresh build gives).  No row can overflow here.
vcsgc_status refresh_mc_from_md(vcsgc_ctx *c) {
  VC_CHECK(c, vc::launch_bin_cells(c, c->reps[0]), "binning");
  VC_CHECK(c, vc::launch_mc_from_md(c), "neighbour list");
  c->mc_stats_stale = true;  // taken when asked for (vcsgc_get_info)
  VC_CHECK(c, hipMemcpyAsync(c->rho, c->rho_f, sizeof(double) * c->n, hipMemcpyDeviceToDevice,
                             c->stream),
           "density");
  c->mc_valid = true;
  return VCSGC_OK;
}

vcsgc_status ensure_mc(vcsgc_ctx *c) {
  if (c->mc_valid) return VCSGC_OK;
  if (c->rho_f_fresh && c->md_valid && !c->desc && c->reps.size() == 1)
    return refresh_mc_from_md(c);
  return refresh_mc(c);
}

vcsgc_status refresh_md(vcsgc_ctx *c) {
  for (;;) {
    VC_CHECK(c, vc::launch_bin_search(c, c->reps[0]), "binning");
    VC_CHECK(c, vc::launch_build_md_list(c), "neighbour list (MD)");
    hipError_t e;
    vc::DevState h = read_state(c, &e);
    if (e != hipSuccess) return dev_fail(c, e, "neighbour list (MD)");
    if (h.bin_overflow) {
      vcsgc_status st = grow_bins(c);
      if (st) return st;
      continue;
    }
    if (h.overflow)
      return fail(c, VCSGC_E_OVERFLOW, "a site has more than 32 neighbours within rc + skin");
    c->md_valid = true;
    c->md_rebuilds += 1;
    for (int d = 0; d < 3; ++d) c->box_build[d] = c->box[d];
    return VCSGC_OK;
  }
}

// The persistent sweep's graph is built again by the next call.
void drop_graph(vcsgc_ctx *c) {
  if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
  c->graph_exec = nullptr;
}

// Workgroups of the persistent sweep.  A replica whose densities and species
// (nine bytes per atom) fit the LDS of one workgroup runs in one: its stages
// then need no device barrier.  The others get trial groups for
// PERSIST_SPEC / trials_per_group stages of their active cells per batch (at
// least one workgroup, a multiple of 8 starting at a multiple of 8 from 8 on,
// so that their shares can be laid out XCD by XCD).  Workgroups that wait for
// each other must all be resident (one per CU: eight waves of more than 128
// registers): first fewer stages are tried per batch, then trials_per_group
// doubles.  Where the LDS of the largest resident replica and of the largest
// share of cells do not go together, the bound of residence is lowered.
// One system whose groups make just one stage at a time has a whole grid, not
// only the groups of that stage (152 to 248 of 256 workgroups): its batches of
// several stages are then made in full passes.  At rest 2.45M sites 844 -> 592 us
// a sweep, 3.46M 973 -> 788, 1.02M with 27 colours 445 -> 322.  Where more than
// 0.3 of the stages are accepted a batch seldom has a second one and fewer
// workgroups meet sooner, so the rest of the grid leaves (G_busy; 2.45M at 27%
// 1,781 us with 152, 1,779 with 256, at 82% 2,407 and 2,783).
// More replicas than CUs get one workgroup each: none of them waits, so the
// grid may be any size and the rest follows as workgroups end.  A share of
// cells whose draws of one stage the LDS does not hold (some 7,900 cells, two
// million active cells on 256 workgroups) has them in memory.
constexpr int PERSIST_SPEC = 8;
constexpr int64_t PERSIST_MAX = ((int64_t)1 << 28) - 1;  // active cells, by the packed counts
constexpr int64_t PERSIST_WG = 8 * 255;                  // and workgroups of a replica, at most
// replicas of a batch, per CU (vcsgc_create_batch states the limit)
constexpr int REPLICAS_PER_CU = 4, REPLICAS_PER_CU_TAB = 3;

vcsgc_status assign_workgroups(vcsgc_ctx *c) {
  int dev_cu = 0, lds_cu = 0, per_cu = 0;
  VC_CHECK(c, hipDeviceGetAttribute(&dev_cu, hipDeviceAttributeMultiprocessorCount, c->device),
           "device query");
  VC_CHECK(c, hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                                    c->device),
           "device query");
  const int R = (int)c->reps.size();
  const bool tab = c->pot.tab != 0;
  if (R > dev_cu * (tab ? REPLICAS_PER_CU_TAB : REPLICAS_PER_CU))
    return fail(c, VCSGC_E_INVALID_ARG, "more replicas than co-resident workgroups");
  for (const RepHost &r : c->reps)
    if (r.ncpc > PERSIST_MAX)
      return fail(c, VCSGC_E_INVALID_ARG, "too many cells for the persistent sweep");
  // LDS of a workgroup with the static part and some slack left out
  const size_t room = (size_t)lds_cu - 1024;
  VC_CHECK(c, vc::persist_max_blocks(&per_cu, tab, false, room), "occupancy query");
  const int64_t cap0 = (int64_t)dev_cu * per_cu;  // workgroups of the least LDS
  const bool single = R > cap0;                   // one workgroup per replica
  // (the pipeline strategies' parameter is the stages of their kernels' batch)
  int tpg = c->strategy >= 2 || c->trials_per_group < 1 ? 1 : c->trials_per_group;
  std::vector<int> want(R), order(R);
  std::vector<char> res(R);
  const size_t bounds[] = {room, (size_t)lds_cu / 2 - 1024, 0};
  for (;; tpg *= 2) {  // (one workgroup per replica fits in the end)
    for (int spec = PERSIST_SPEC; spec >= 1; --spec) {
      for (const size_t bound : bounds) {
        int64_t total = 0, chunk = 1, nres = 0;
        int busy = 1;
        for (int k = 0; k < R; ++k) {
          const RepHost &r = c->reps[k];
          res[k] = vc::persist_lds_need(r.ncpc, r.n, nullptr) <= bound;
          const int64_t per = (int64_t)vc::persist_groups() * tpg;
          int64_t g = res[k] || single ? 1 : (spec * r.ncpc + per - 1) / per;
          if (g < 1) g = 1;
          if (g >= 8) g = std::min<int64_t>((g + 7) / 8 * 8, PERSIST_WG);
          busy = (int)g;  // (of the last replica: used for a single one)
          if (R == 1 && spec == 1 && tpg == 1 && g >= 8)
            g = std::max(g, std::min(cap0 / 8 * 8, PERSIST_WG));
          want[k] = (int)g;
          total += g;
          chunk = std::max<int64_t>(chunk, (r.ncpc + busy - 1) / busy);
          if (res[k]) nres = std::max<int64_t>(nres, r.n);
        }
        const bool waits = total > R;
        if (waits && total > cap0) break;  // a lower bound only adds workgroups
        int ndraw = 0;
        size_t lds = vc::persist_lds_need(chunk, nres, &ndraw);
        const bool big = vc::persist_lds_need(chunk, 0, nullptr) > room;
        if (big) lds = vc::persist_lds_need(0, nres, &ndraw);
        if (lds > room) continue;
        int by_regs = per_cu;
        if (big)
          VC_CHECK(c, vc::persist_max_blocks(&by_regs, tab, true, room), "occupancy query");
        const int by_lds = std::max(1, (int)(lds_cu / (lds + 2048)));
        if (waits && total > (int64_t)dev_cu * std::min(by_regs, by_lds)) break;
        // large replicas first (aligned; of one workgroup each, by atoms, so
        // that none of the long ones starts last), then the single-digit ones
        for (int k = 0; k < R; ++k) order[k] = k;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
          return single ? c->reps[a].n > c->reps[b].n : (want[a] >= 8) > (want[b] >= 8);
        });
        std::vector<int32_t> map((size_t)total);
        int g0 = 0;
        for (int k : order) {
          c->reps[k].g0 = g0;
          c->reps[k].G = c->reps[k].G_busy = want[k];
          c->reps[k].res = res[k] != 0;
          for (int q = 0; q < want[k]; ++q) map[g0 + q] = k;
          g0 += want[k];
        }
        if (R == 1) c->reps[0].G_busy = busy;
        if (c->d_wg_rep) (void)hipFree(c->d_wg_rep);
        c->d_wg_rep = nullptr;
        VC_CHECK(c, dalloc(&c->d_wg_rep, (size_t)total), "allocation");
        VC_CHECK(c, hipMemcpy(c->d_wg_rep, map.data(), sizeof(int32_t) * total,
                              hipMemcpyHostToDevice),
                 "copy");
        c->grid_total = (int)total;
        if (c->strategy < 2) c->trials_per_group = tpg;
        c->persist_lds = lds;
        c->persist_ndraw = ndraw;
        c->persist_waits = waits;
        drop_graph(c);
        if (c->big_lnu) (void)hipFree(c->big_lnu);
        if (c->big_site) (void)hipFree(c->big_site);
        c->big_lnu = nullptr;
        c->big_site = nullptr;
        if (big) {
          const RepHost &z = c->reps.back();
          VC_CHECK(c, dalloc(&c->big_lnu, (size_t)(z.roff + z.ncpc)), "allocation");
          VC_CHECK(c, dalloc(&c->big_site, (size_t)(z.roff + z.ncpc)), "allocation");
        }
        return VCSGC_OK;
      }
    }
  }
}

vcsgc_status check_ctx(vcsgc_ctx *c) {
  if (!c) return VCSGC_E_INVALID_ARG;
  if (c->sticky) return VCSGC_E_STATE;
  (void)hipSetDevice(c->device);
  return VCSGC_OK;
}

}  // namespace

namespace vc {

int tstart(vcsgc_ctx *c, int cls) {
  if (!(c->tmask & (1u << cls))) return -1;
  if (c->kt_seen[cls]++ % c->t_every != 0) return -1;
  // timing-only events: no system-scope fence when recorded (the stream is
  // synchronized before the times are read)
  hipEvent_t ev[2];
  for (int k = 0; k < 2; ++k) {
    if (!c->ev_pool.empty()) {
      ev[k] = c->ev_pool.back();
      c->ev_pool.pop_back();
    } else if (hipEventCreateWithFlags(&ev[k], hipEventDisableSystemFence) != hipSuccess) {
      if (k == 1) c->ev_pool.push_back(ev[0]);
      return -1;
    }
  }
  if (hipEventRecord(ev[0], c->stream) != hipSuccess) {
    c->ev_pool.push_back(ev[0]);
    c->ev_pool.push_back(ev[1]);
    return -1;
  }
  c->ev_pending.push_back({cls, ev[0], ev[1]});
  return (int)c->ev_pending.size() - 1;
}

void tstop(vcsgc_ctx *c, int h) {
  if (h < 0) return;
  (void)hipEventRecord(c->ev_pending[h].b, c->stream);
}

}  // namespace vc

namespace {

// fold pending event pairs into the per-class totals (synchronizes)
hipError_t drain_timers(vcsgc_ctx *c) {
  if (c->ev_pending.empty()) return hipSuccess;
  hipError_t e = hipStreamSynchronize(c->stream);
  for (auto &p : c->ev_pending) {
    float ms = 0.f;
    if (e == hipSuccess && hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
      c->kt_ms[p.cls] += ms;
      c->kt_n[p.cls] += 1;
    }
    c->ev_pool.push_back(p.a);
    c->ev_pool.push_back(p.b);
  }
  c->ev_pending.clear();
  return e;
}

}  // namespace

extern "C" {

vcsgc_status vcsgc_kernel_timing_sampled(vcsgc_ctx *c, uint32_t mask, int32_t every) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (every < 1) return fail(c, VCSGC_E_INVALID_ARG, "every must be >= 1");
  VC_CHECK(c, drain_timers(c), "timing");
  c->tmask = mask & ((1u << VCSGC_KT_CLASSES) - 1);
  c->t_every = every;
  for (int k = 0; k < VCSGC_KT_CLASSES; ++k) {
    c->kt_ms[k] = 0.0;
    c->kt_n[k] = 0;
    c->kt_seen[k] = 0;
  }
  return VCSGC_OK;
}

vcsgc_status vcsgc_kernel_timing(vcsgc_ctx *c, uint32_t mask) {
  return vcsgc_kernel_timing_sampled(c, mask, 1);
}

vcsgc_status vcsgc_get_kernel_timing(vcsgc_ctx *c, vcsgc_ktimes *out) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!out) return fail(c, VCSGC_E_INVALID_ARG, "null output");
  VC_CHECK(c, drain_timers(c), "timing");
  for (int k = 0; k < VCSGC_KT_CLASSES; ++k) {
    out->total_ms[k] = c->kt_ms[k];
    out->count[k] = c->kt_n[k];
    out->launches[k] = c->kt_seen[k];
  }
  return VCSGC_OK;
}

}  // extern "C"

namespace {

// Coefficients (a0, a1, a2, a3) per interval of the cubic Hermite
// interpolant through y[0 .. n-1] at unit-spaced knots, knot slopes by
// central differences and one-sided at the two ends (the interpolation
// vcsgc_eam_table defines).
void hermite_coeffs(int32_t n, const double *y, double *c) {
  for (int32_t k = 0; k + 1 < n; ++k) {
    const double m0 = k == 0 ? y[1] - y[0] : 0.5 * (y[k + 1] - y[k - 1]);
    const double m1 = k + 2 == n ? y[n - 1] - y[n - 2] : 0.5 * (y[k + 2] - y[k]);
    const double d = y[k + 1] - y[k];
    double *a = c + 4 * (int64_t)k;
    a[0] = y[k];
    a[1] = m0;
    a[2] = (3.0 * d - 2.0 * m0) - m1;
    a[3] = (m0 + m1) - 2.0 * d;
  }
}

// Shared by vcsgc_create (one replica) and vcsgc_create_batch.
vcsgc_status create_impl(const vcsgc_system *sys, int R, const int64_t *rep_atoms,
                         const double *rep_box, hipStream_t stream, vcsgc_ctx **out) {
  if (!sys || !out) return fail(nullptr, VCSGC_E_INVALID_ARG, "null argument");
  const vcsgc_eam_fs &P = sys->pot;
  if (sys->n_atoms < 2 || sys->n_atoms > (int64_t)0x7fffffff)
    return fail(nullptr, VCSGC_E_INVALID_ARG, "n_atoms must be in [2, 2^31)");
  if (!sys->x || !sys->y || !sys->z || !sys->species)
    return fail(nullptr, VCSGC_E_INVALID_ARG, "positions and species are required");
  const vcsgc_eam_table *T = sys->table;
  if (T) {
    if (T->nr < 2 || T->nrho < 2 || !(T->dr > 0.0) || !(T->drho > 0.0) || !is_fin(T->dr) ||
        !is_fin(T->drho) || !(T->rc > 0.0) || !is_fin(T->rc) ||
        T->rc > (double)(T->nr - 1) * T->dr)
      return fail(nullptr, VCSGC_E_INVALID_ARG,
                  "table needs nr, nrho >= 2, dr, drho > 0 and 0 < rc <= (nr - 1) dr");
    const double *arrs[] = {T->f[0], T->f[1], T->phi[0], T->phi[1], T->phi[2], T->F[0], T->F[1]};
    for (int k = 0; k < 7; ++k) {
      if (!arrs[k]) return fail(nullptr, VCSGC_E_INVALID_ARG, "missing table");
      const int32_t nk = k < 5 ? T->nr : T->nrho;
      for (int32_t q = 0; q < nk; ++q)
        if (!is_fin(arrs[k][q])) return fail(nullptr, VCSGC_E_INVALID_ARG, "non-finite table value");
    }
  } else {
    const double pv[] = {P.rc, P.c0, P.c1, P.eps_aa, P.eps_ab, P.eps_bb,
                         P.t_a, P.t_b, P.a_a, P.a_b};
    for (double v : pv)
      if (!is_fin(v)) return fail(nullptr, VCSGC_E_INVALID_ARG, "non-finite potential parameter");
  }
  const double rc = T ? T->rc : P.rc;
  if (!(rc > 0.0)) return fail(nullptr, VCSGC_E_INVALID_ARG, "rc must be positive");
  if (!(sys->skin >= 0.0) || !is_fin(sys->skin) || sys->skin > rc)
    return fail(nullptr, VCSGC_E_INVALID_ARG, "skin must be in [0, rc]");
  const bool has_v = sys->vx || sys->vy || sys->vz;
  if (has_v && !(sys->vx && sys->vy && sys->vz))
    return fail(nullptr, VCSGC_E_INVALID_ARG, "velocities must be all set or all NULL");
  const bool has_f = sys->fx || sys->fy || sys->fz;
  if (has_f && !(sys->fx && sys->fy && sys->fz))
    return fail(nullptr, VCSGC_E_INVALID_ARG, "forces must be all set or all NULL");
  if (has_v && (!(P.mass_a > 0.0) || !(P.mass_b > 0.0) || !is_fin(P.mass_a) || !is_fin(P.mass_b)))
    return fail(nullptr, VCSGC_E_INVALID_ARG, "masses must be positive with velocities");
  const double r_dep = sys->r_dep == 0.0 ? 2.0 * rc : sys->r_dep;
  if (!(r_dep >= 2.0 * rc) || !is_fin(r_dep))
    return fail(nullptr, VCSGC_E_INVALID_ARG, "r_dep must be >= 2 rc");
  const int per = (sys->flags & VCSGC_FLAG_COLOURS27) ? 3 : 2, ncol = per * per * per;
  const double ge = sys->grow_edge;
  if (!is_fin(ge) || ge < 0.0) return fail(nullptr, VCSGC_E_INVALID_ARG, "grow_edge must be >= 0");
  const bool grown = ge > 0.0;
  if (grown && (R != 1 || per != 2))
    return fail(nullptr, VCSGC_E_INVALID_ARG,
                "grown domains need a single system and the eight-colour scheme");

  std::vector<RepHost> reps((size_t)R);
  int64_t aoff = 0, coff = 0, boff = 0, roff = 0;
  for (int k = 0; k < R; ++k) {
    RepHost &r = reps[k];
    r.n = rep_atoms[k];
    if (r.n < 2) return fail(nullptr, VCSGC_E_INVALID_ARG, "every replica needs >= 2 atoms");
    r.aoff = aoff;
    for (int d = 0; d < 3; ++d) {
      r.box[d] = rep_box[3 * k + d];
      if (!(r.box[d] > 0.0) || !is_fin(r.box[d]))
        return fail(nullptr, VCSGC_E_INVALID_ARG, "box edges must be positive and finite");
      if (grown) {
        r.nc[d] = (int)std::floor(r.box[d] / std::max(ge, 2.0 * r_dep));
        if (r.nc[d] < 1)
          return fail(nullptr, VCSGC_E_BOX_TOO_SMALL,
                      "box must hold one cell of edge max(grow_edge, 2 r_dep) in every dimension");
      } else {
        r.nc[d] = per * (int)std::floor(r.box[d] / ((double)per * (r_dep / (double)(per - 1))));
        if (r.nc[d] < per)
          return fail(nullptr, VCSGC_E_BOX_TOO_SMALL,
                      per == 2 ? "box must hold two cells of edge r_dep in every dimension"
                               : "box must hold three cells of edge r_dep / 2 in every dimension");
      }
      const double bin_edge = (sys->flags & VCSGC_FLAG_DESCRIPTOR)
                                  ? std::max(rc + sys->skin, vc::DESC_CUT)
                                  : rc + sys->skin;
      r.nb[d] = (int)std::floor(r.box[d] / bin_edge);
      if (r.nb[d] < 2)
        return fail(nullptr, VCSGC_E_BOX_TOO_SMALL, "box too small for the neighbour search");
    }
    r.ncells = (int64_t)r.nc[0] * r.nc[1] * r.nc[2];
    r.coff = coff;
    r.cso = coff + k;
    r.S = (grown ? 1 : (int64_t)ncol) * ((r.n + r.ncells - 1) / r.ncells);
    r.ncpc = grown ? r.ncells : r.ncells / ncol;
    r.roff = roff;
    r.nbins = (int64_t)r.nb[0] * r.nb[1] * r.nb[2];
    r.boff = boff;
    aoff += r.n;
    coff += r.ncells;
    boff += r.nbins;
    roff += r.ncpc;
  }
  if (aoff != sys->n_atoms)
    return fail(nullptr, VCSGC_E_INVALID_ARG, "replica sizes must add up to n_atoms");

  vcsgc_ctx *c = new vcsgc_ctx();
  (void)hipGetDevice(&c->device);
  c->stream = stream;
  c->n = sys->n_atoms;
  c->reps = reps;
  const RepHost &r0 = reps[0];
  for (int d = 0; d < 3; ++d) {
    c->box[d] = r0.box[d];
    c->nc[d] = r0.nc[d];
    c->nb[d] = r0.nb[d];
  }
  c->ncells = r0.ncells;
  c->per = per;
  c->ncol = ncol;
  c->S = r0.S;
  c->nbins = r0.nbins;
  c->nbins_total = boff;
  c->x = sys->x;
  c->y = sys->y;
  c->z = sys->z;
  c->vx = sys->vx;
  c->vy = sys->vy;
  c->vz = sys->vz;
  c->fx = sys->fx;
  c->fy = sys->fy;
  c->fz = sys->fz;
  c->sp = sys->species;
  c->skin = sys->skin;
  c->r_dep = r_dep;
  vc::PotD &p = c->pot;
  p.rc = rc;
  p.c0 = P.c0;
  p.c1 = P.c1;
  p.eps[0] = P.eps_aa;
  p.eps[1] = P.eps_ab;
  p.eps[2] = P.eps_bb;
  p.t[0] = P.t_a;
  p.t[1] = P.t_b;
  p.A[0] = P.a_a;
  p.A[1] = P.a_b;
  p.mass[0] = P.mass_a;
  p.mass[1] = P.mass_b;
  p.cm[0] = P.mass_a > 0.0 ? vc::ACC / P.mass_a : 0.0;
  p.cm[1] = P.mass_b > 0.0 ? vc::ACC / P.mass_b : 0.0;
  c->bmax = 16;
  c->strategy = 0;
  c->grown = grown;
  c->grow_edge = ge;
  c->desc = (sys->flags & VCSGC_FLAG_DESCRIPTOR) != 0;
  c->bin_edge = c->desc ? std::max(rc + sys->skin, vc::DESC_CUT) : rc + sys->skin;
  for (int d = 0; d < 3; ++d) {
    c->nb_max[d] = r0.nb[d];
    c->box_build[d] = r0.box[d];
  }
  if (T) {
    // the interpolants' coefficients: f_A, f_B, phi_AA, phi_AB, phi_BB, then F_A, F_B
    const int64_t nir = T->nr - 1, nid = T->nrho - 1;
    std::vector<double> co((size_t)(4 * (5 * nir + 2 * nid)));
    const double *arrs[] = {T->f[0], T->f[1], T->phi[0], T->phi[1], T->phi[2], T->F[0], T->F[1]};
    size_t o = 0;
    for (int k = 0; k < 7; ++k) {
      const int32_t nk = k < 5 ? T->nr : T->nrho;
      hermite_coeffs(nk, arrs[k], co.data() + o);
      o += (size_t)4 * (nk - 1);
    }
    hipError_t e1 = dalloc(&c->tab_coef, co.size());
    if (e1 == hipSuccess)
      e1 = hipMemcpy(c->tab_coef, co.data(), sizeof(double) * co.size(), hipMemcpyHostToDevice);
    if (e1 != hipSuccess) {
      free_all(c);
      delete c;
      return fail(nullptr, VCSGC_E_OUT_OF_MEMORY, "table upload");
    }
    p.tab = 1;
    p.nr = T->nr;
    p.nrho = T->nrho;
    p.inv_dr = 1.0 / T->dr;
    p.inv_drho = 1.0 / T->drho;
    p.tc = c->tab_coef;
  }

  const int64_t n = c->n, K = vc::KMAX;
  const bool single = R == 1;
  hipError_t e = hipSuccess;
  auto A = [&](hipError_t rr) {
    if (e == hipSuccess) e = rr;
  };
  A(dalloc(&c->bin_count, boff));
  A(dalloc(&c->bin_atoms, boff * c->bmax));
  if (single) {
    A(dalloc(&c->bin_pos, boff * c->bmax));
    A(dalloc(&c->sites, reps[0].S * reps[0].ncpc));
    A(dalloc(&c->site_lnu, reps[0].S * reps[0].ncpc));
    A(dalloc(&c->stage_lnug, reps[0].S));
    // fused stage pipeline: two sweeps of site tables, two stages of records
    // and trial-block sums
    const int64_t S1 = reps[0].S, nc1 = reps[0].ncpc;
    A(dalloc(&c->m_sites, 2 * S1 * nc1));
    A(dalloc(&c->m_lnu, 2 * S1 * nc1));
    A(dalloc(&c->m_lnu2, 2 * S1 * nc1));
    A(dalloc(&c->m_lnug, 2 * S1));
    A(dalloc(&c->m_rec, 2 * nc1));
    A(dalloc(&c->m_part, 2 * vc::NPART * (int64_t)vc::grid_for(nc1 * 16)));
    A(dalloc(&c->s_rec, 2 * vc::SPEC_MAX * nc1));
    A(dalloc(&c->s_part, 2 * vc::SPEC_MAX * 3 * (int64_t)vc::grid_for(nc1 * 16)));
  }
  A(dalloc(&c->cell_count, coff));
  A(dalloc(&c->cell_start, coff + R));
  A(dalloc(&c->cell_fill, coff));
  A(dalloc(&c->cell_atoms, n));
  {
    int64_t mx = 1;
    for (const RepHost &r : c->reps)
      mx = std::max<int64_t>(mx, (std::max({r.ncells, r.nbins, grown ? 8 * r.ncells : 0}) +
                                  vc::SCAN_CHUNK - 1) / vc::SCAN_CHUNK);
    A(dalloc(&c->scan_tmp, mx));
  }
  if (grown) {
    A(dalloc(&c->g_start, 8 * c->ncells + 1));
    A(dalloc(&c->g_cnt, 8 * c->ncells));
    A(dalloc(&c->g_list, 8 * n));
    A(dalloc(&c->g_cum, 8 * n));
  }
  A(dalloc(&c->mc_j, K * n));
  A(dalloc(&c->mc_r, K * n));
  A(dalloc(&c->mc_cnt, n));
  if (single) {
    A(dalloc(&c->md_j, K * n));
    A(dalloc(&c->md_rows, K * n));
    A(dalloc(&c->md_cnt, n));
    A(dalloc(&c->xr, n));
    A(dalloc(&c->yr, n));
    A(dalloc(&c->zr, n));
    A(dalloc(&c->ps4, 2 * n));
    A(dalloc(&c->pf4, 2 * n));
    A(dalloc(&c->rho_f, n));
    A(dalloc(&c->eatom, n));
    A(dalloc(&c->nvt, 8));
    A(dalloc(&c->nvt_part, (n + vc::BLOCK - 1) / vc::BLOCK));
  }
  if (c->desc) {
    A(dalloc(&c->d_j, K * n));
    A(dalloc(&c->d_r, K * n));
    A(dalloc(&c->d_cnt, n));
  }
  A(dalloc(&c->rho, n));
  A(dalloc(&c->red, (n + vc::BLOCK - 1) / vc::BLOCK + 8));
  A(dalloc(&c->rec, roff));
  A(dalloc(&c->ds, 1));
  A(dalloc((unsigned char **)&c->d_rs, vc::repstate_size() * R));
  {  // the pinned buffers in one allocation (0.1 ms each)
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t n_rs = up(vc::repstate_size() * R), n_reps = up(vc::repd_size() * R),
                 n_st = up(sizeof(vc::DevState));
    if (e == hipSuccess)
      e = hipHostMalloc((void **)&c->h_pin, n_rs + n_reps + n_st + 256, hipHostMallocDefault);
    if (e == hipSuccess) {
      c->h_rs = c->h_pin;
      c->h_reps = c->h_pin + n_rs;
      c->h_state = (vc::DevState *)(c->h_pin + n_rs + n_reps);
      c->h_tot = (double *)(c->h_pin + n_rs + n_reps + n_st);
    }
  }
  if (e != hipSuccess) {
    free_all(c);
    delete c;
    (void)hipGetLastError();
    return fail(nullptr, e == hipErrorOutOfMemory ? VCSGC_E_OUT_OF_MEMORY : VCSGC_E_DEVICE,
                std::string("allocation: ") + hipGetErrorString(e));
  }
  auto bail = [&](vcsgc_status st) {
    g_create_error = c->err;
    (void)hipStreamSynchronize(c->stream);
    free_all(c);
    delete c;
    return st;
  };
  vcsgc_status st = assign_workgroups(c);
  if (st) return bail(st);
  // trial-kernel partial sums
  const int64_t npart_stage = (r0.ncpc * 16 + vc::BLOCK - 1) / vc::BLOCK + 1;
  c->npart = npart_stage;
  if ((e = dalloc(&c->part, vc::NPART * c->npart)) != hipSuccess)
    return bail(dev_fail(c, e, "allocation"));
  if ((e = hipMemsetAsync(c->ds, 0, sizeof(vc::DevState), c->stream)) != hipSuccess)
    return bail(dev_fail(c, e, "init"));
  // MD rows hold valid indices beyond their lengths too (empty until built)
  if (c->md_j &&
      ((e = hipMemsetAsync(c->md_j, 0, sizeof(int32_t) * vc::KMAX * n, c->stream)) != hipSuccess ||
       (e = hipMemsetAsync(c->md_rows, 0, sizeof(int32_t) * vc::KMAX * n, c->stream)) != hipSuccess ||
       (e = hipMemsetAsync(c->md_cnt, 0, sizeof(uint8_t) * n, c->stream)) != hipSuccess))
    return bail(dev_fail(c, e, "init"));
  for (const RepHost &r : c->reps) {
    if ((e = vc::launch_validate(c, r)) != hipSuccess) return bail(dev_fail(c, e, "validate"));
  }
  {
    hipError_t e2;
    vc::DevState h = read_state(c, &e2);
    if (e2 != hipSuccess) return bail(dev_fail(c, e2, "validate"));
    if (h.bad_input)
      return bail(fail(c, VCSGC_E_INVALID_ARG,
                       "positions must lie in [0, L) and species in {0, 1}"));
  }
  if ((e = vc::persist_count(c)) != hipSuccess) return bail(dev_fail(c, e, "count"));
  if (grown) {  // the batched pipeline, three stages per batch
    c->strategy = 3;
    c->trials_per_group = 3;
  }
  st = refresh_mc(c);
  if (st != VCSGC_OK) return bail(st);
  *out = c;
  return VCSGC_OK;
}

}  // namespace

extern "C" {

vcsgc_status vcsgc_create(const vcsgc_system *sys, hipStream_t stream, vcsgc_ctx **out) {
  if (!sys || !out) return fail(nullptr, VCSGC_E_INVALID_ARG, "null argument");
  const int64_t n = sys->n_atoms;
  return create_impl(sys, 1, &n, sys->box, stream, out);
}

vcsgc_status vcsgc_create_batch(const vcsgc_system *sys, int32_t n_rep, const int64_t *rep_atoms,
                                const double *rep_box, hipStream_t stream, vcsgc_ctx **out) {
  if (!sys || !out || n_rep < 1 || !rep_atoms || !rep_box)
    return fail(nullptr, VCSGC_E_INVALID_ARG, "null argument or n_rep < 1");
  return create_impl(sys, n_rep, rep_atoms, rep_box, stream, out);
}

vcsgc_status vcsgc_destroy(vcsgc_ctx *c) {
  if (!c) return VCSGC_OK;
  (void)hipSetDevice(c->device);
  (void)hipStreamSynchronize(c->stream);
  for (auto &p : c->ev_pending) {
    c->ev_pool.push_back(p.a);
    c->ev_pool.push_back(p.b);
  }
  for (hipEvent_t ev : c->ev_pool) (void)hipEventDestroy(ev);
  free_all(c);
  delete c;
  return VCSGC_OK;
}

const char *vcsgc_last_error(const vcsgc_ctx *c) {
  return c ? c->err.c_str() : g_create_error.c_str();
}

}  // extern "C"

namespace {

bool valid_params(double dmu0, double kappa, double cbar, double T) {
  return is_fin(dmu0) && is_fin(kappa) && kappa >= 0.0 && is_fin(cbar) && cbar >= 0.0 &&
         cbar <= 1.0 && is_fin(T) && T > 0.0;
}

// Sweeps of a single system with kernels per stage or batch of stages.
vcsgc_status sweep_stages(vcsgc_ctx *c, double dmu0, double kappa, double cbar, double T,
                          int64_t n_sweeps, uint64_t seed, vcsgc_stats *out) {
  VC_CHECK(c, vc::persist_sync_nb_to_stage(c), "sweep");
  c->h_state_final = false;
  VC_CHECK(c, vc::launch_sweeps(c, dmu0, kappa, cbar, T, n_sweeps, seed), "sweep");
  // the pipelines end with the device state read and n_B synchronized
  const bool have = c->h_state_final;
  c->h_state_final = false;
  if (!have) VC_CHECK(c, vc::persist_sync_nb_from_stage(c), "sweep");
  c->w += (uint64_t)n_sweeps;
  if (have && c->h_state->stages)
    c->m_stage_acc = (double)c->h_state->stage_acc / (double)c->h_state->stages;
  if (out) {
    hipError_t e = hipSuccess;
    vc::DevState h = have ? *c->h_state : read_state(c, &e);
    if (e != hipSuccess) return dev_fail(c, e, "sweep");
    out->trials = (int64_t)h.trials;
    out->local_accepts = (int64_t)h.local_acc;
    out->stages = (int64_t)h.stages;
    out->stage_accepts = (int64_t)h.stage_acc;
    out->flips = (int64_t)h.flips;
    out->near_ties = (int64_t)h.near_ties;
    out->n_final = h.n_b_cur;
    out->sum_n = h.sum_n;
    out->sum_n2 = h.sum_n2;
    out->stage1_pass = (int64_t)h.stage1_pass;
  }
  return VCSGC_OK;
}

// Sweeps of every replica with per-replica parameters; stats may be NULL.
vcsgc_status sweep_impl(vcsgc_ctx *c, const double *dmu0, const double *kappa, const double *cbar,
                        const double *T, int64_t n_sweeps, uint64_t seed, vcsgc_stats *out) {
  const int R = (int)c->reps.size();
  if (n_sweeps < 0) return fail(c, VCSGC_E_INVALID_ARG, "n_sweeps must be >= 0");
  for (int k = 0; k < R; ++k)
    if (!valid_params(dmu0[k], kappa[k], cbar[k], T[k]))
      return fail(c, VCSGC_E_INVALID_ARG,
                  "need finite dmu0, kappa >= 0, cbar in [0,1], T > 0 for every replica");
  if (R == 1)  // the box may have changed under the barostat
    for (int d = 0; d < 3; ++d)
      if (c->box[d] / (double)c->nc[d] <
          (c->grown ? 2.0 * c->r_dep : c->r_dep / (double)(c->per - 1)))
        return fail(c, VCSGC_E_BOX_TOO_SMALL,
                    "the box has shrunk below the sweep's cell grid (edge < r_dep)");
  {
    vcsgc_status st = ensure_mc(c);
    if (st) return st;
  }
  c->last_seed = seed;
  if (n_sweeps > 0) c->rho_f_fresh = false;
  if (c->local_steps > 1 && (c->da_mode || c->smp_cap > 0))
    return fail(c, VCSGC_E_INVALID_ARG,
                "delayed acceptance and the sample log need one trial per cell per stage");
  // The training-sample log, local chains, grown domains and delayed
  // acceptance other than with the network run with kernels per stage or batch
  // of stages, and so do the network's where its stages are logged or timed,
  // where the dU row is not part of the descriptor list (rc > 4.41 A), or
  // beyond about 6M sites (8.2M sites: 11.9 ms either way; 4.2M 3.1 ms
  // persistent, 6.3 ms with 16 stages per kernel); and so do the
  // pipeline strategies where their stages are logged or timed, or where a
  // workgroup of the persistent sweep would hold more active cells than
  // trial groups.  Below that (about 4M sites) the persistent sweep is the
  // faster form of the same chain: a batch of stages costs it one device
  // barrier and one round of gathers (6 - 12 us) instead of a kernel with its
  // launch, site table and row reads one after the other (10 - 12 us), and it
  // fits the length of its batches to the acceptance.  Per stage, persistent
  // against the best of 3, 8 and 16 stages per kernel: 250,000 sites at 28%
  // accepted stages 2.6 / 4.5 us, 0.5M at 24% 2.9 / 4.6, 2M at 23% 4.8 / 7.5,
  // 1M at 0% 1.1 / 1.2, 4M at 0% 3.5 / 3.5, 8M at 0% 7.2 / 6.3.
  // Tabulated potentials: where the last call accepted next to nothing, the
  // stages are bound by the tables' gathers, for which the pipeline has more
  // waves; it is the faster one with long batches, or where the persistent
  // sweep's workgroups hold most of their groups in one stage.  At 0%, 16
  // stages per kernel against persistent: 128,000 sites 335 / 383 us a sweep,
  // 0.25M 266 / 340, 1.02M 477 / 589, with 27 colours 153 / 174, 195 / 212,
  // 450 / 823 (4 stages 594); but with 8 per kernel 438 / 383, 378 / 340,
  // 596 / 589, and at 10% accepted 838 / 770 (54,000 sites).
  // The analytic form at rest with more than 13/16 of the groups in one stage:
  // 16 stages per kernel against persistent 3.72M sites 771 / 831 us a sweep, with
  // 27 colours 1.77M 452 / 489, 4.0M 932 / 934; with fewer cells 3.46M 834 / 788,
  // 2.45M 641 / 592; with 8 per kernel 3.72M 876, 1.77M 501.
  const int64_t cells = c->reps[0].ncpc;
  const int64_t groups = (int64_t)c->reps[0].G * vc::persist_groups();
  const int batch = c->trials_per_group;
  const bool quiet = c->strategy == 3 && c->m_stage_acc >= 0.0 &&
                     (c->pot.tab ? c->m_stage_acc < 0.02 && (batch > 8 || 2 * cells > groups)
                                 : c->m_stage_acc < 0.01 && batch > 8 && 16 * cells > 13 * groups);
  const bool logged = c->tlog || c->slog || c->dalog;
  const unsigned stage_timers =
      1u << VCSGC_KT_STAGE | 1u << VCSGC_KT_TRIAL | 1u << VCSGC_KT_COMMIT;
  // (the network's dU row is the r < rc part of the descriptor list)
  bool da = n_sweeps > 0 && c->da_mode == 1 && c->smp_cap == 0 && !c->grown && !logged &&
            !(c->tmask & stage_timers) && c->pot.rc <= vc::DESC_CUT;
  if (da) {
    VC_CHECK(c, vc::persist_da_grid(c), "occupancy query");
    da = c->da_wg > 0;
  }
  const bool per_stage =
      (c->da_mode && !da) || c->smp_cap > 0 || c->local_steps > 1 || c->grown ||
      (!da && c->strategy >= 2 &&
       (n_sweeps == 0 || quiet || logged || (c->tmask & (1u << VCSGC_KT_STAGE)) || cells > groups));
  if (per_stage && R == 1)
    return sweep_stages(c, dmu0[0], kappa[0], cbar[0], T[0], n_sweeps, seed, out);
  // A replica whose workgroups did not all start has not changed: it is tried
  // again, or, where the call need not be persistent, run with kernels per
  // stage.
  int err = 0;
  vcsgc_stats one;
  vcsgc_stats *const got = out ? out : R == 1 ? &one : nullptr;
  std::vector<char> todo((size_t)R, 1);
  for (uint64_t polls = 0;;) {
    vc::persist_stage_params(c, dmu0, kappa, cbar, T, n_sweeps, todo.data(), seed, da);
    if (n_sweeps > 0) {
      int h = vc::tstart(c, VCSGC_KT_PERSIST);
      if (da)
        VC_CHECK(c, vc::launch_persistent_da(c), "persistent sweep");
      else
        VC_CHECK(c, vc::launch_persistent(c, n_sweeps, c->strategy != 1), "persistent sweep");
      vc::tstop(c, h);
    }
    // the error words are read after every call, with or without statistics:
    // a workgroup that left a timed-out wait may have committed part of a stage
    VC_CHECK(c, vc::persist_read_stats(c, got, todo.data(), &err, n_sweeps > 0, da), "sweep");
    if (!(err & vc::PERSIST_NOT_STARTED)) break;
    if (R == 1 && (da || c->strategy >= 2))
      return sweep_stages(c, dmu0[0], kappa[0], cbar[0], T[0], n_sweeps, seed, out);
    polls += std::min(c->spin_limit, vc::ENTRY_LIMIT);  // (at least one)
    if (polls >= c->spin_limit || (err & vc::PERSIST_TIMEOUT)) break;
  }
  c->w += (uint64_t)n_sweeps;
  if (R == 1 && got->stages && !err)
    c->m_stage_acc = (double)got->stage_accepts / (double)got->stages;
  if (err) {
    c->sticky = true;
    return fail(c, VCSGC_E_BARRIER_TIMEOUT, "persistent sweep: a barrier wait exceeded its limit");
  }
  return VCSGC_OK;
}

}  // namespace

extern "C" {

vcsgc_status vcsgc_sweep(vcsgc_ctx *c, double dmu0, double kappa, double cbar, double T_K,
                         int64_t n_sweeps, uint64_t seed, vcsgc_stats *out) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1) return fail(c, VCSGC_E_INVALID_ARG, "batch context: use vcsgc_sweep_batch");
  return sweep_impl(c, &dmu0, &kappa, &cbar, &T_K, n_sweeps, seed, out);
}

vcsgc_status vcsgc_sweep_batch(vcsgc_ctx *c, const double *dmu0, const double *kappa,
                               const double *cbar, const double *T, int64_t n_sweeps,
                               uint64_t seed, vcsgc_stats *out) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!dmu0 || !kappa || !cbar || !T) return fail(c, VCSGC_E_INVALID_ARG, "null parameter array");
  return sweep_impl(c, dmu0, kappa, cbar, T, n_sweeps, seed, out);
}

vcsgc_status vcsgc_set_wait_limit(vcsgc_ctx *c, uint32_t polls) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (polls < 1) return fail(c, VCSGC_E_INVALID_ARG, "polls must be >= 1");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  c->spin_limit = polls;
  drop_graph(c);  // its kernel node holds the old limit
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_tuning(vcsgc_ctx *c, int32_t strategy, int32_t trials_per_group) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (strategy < 0 || strategy > 3 || trials_per_group < 1 || trials_per_group > 64)
    return fail(c, VCSGC_E_INVALID_ARG, "strategy in {0,1,2,3}, trials_per_group in [1,64]");
  if (strategy == 3 && trials_per_group > vc::SPEC_MAX)
    return fail(c, VCSGC_E_INVALID_ARG, "stages per batch in [1,16]");
  if (strategy >= 2 && c->reps.size() != 1)
    return fail(c, VCSGC_E_INVALID_ARG, "per-stage launches need a single-system context");
  if (strategy < 2 && c->grown)
    return fail(c, VCSGC_E_INVALID_ARG, "grown domains run on the pipeline strategies (2, 3)");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  const bool same = trials_per_group == c->trials_per_group && strategy / 2 == c->strategy / 2;
  c->strategy = strategy;
  c->trials_per_group = trials_per_group;
  if (!same) {
    st = assign_workgroups(c);
    if (st) return st;
  }
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_local_steps(vcsgc_ctx *c, int32_t k) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1) return fail(c, VCSGC_E_INVALID_ARG, "local chains need a single system");
  if (k < 1 || k > 64) return fail(c, VCSGC_E_INVALID_ARG, "local chain length in [1, 64]");
  if (k == c->local_steps) return VCSGC_OK;
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  vc::free_stage_graph(c);  // its nodes hold the old buffers
  void *old[] = {c->sites, c->site_lnu, c->stage_lnug, c->u_site, c->u_j, c->u_rho, c->u_v};
  for (void *p : old)
    if (p) (void)hipFree(p);
  c->sites = c->u_site = c->u_j = nullptr;
  c->site_lnu = c->stage_lnug = c->u_rho = c->u_v = nullptr;
  c->local_steps = k;
  const int64_t ncpc = vc::active_cells(c), K = k;
  const int64_t tab = vc::stages_per_sweep(c) * ncpc * K;
  VC_CHECK(c, dalloc(&c->sites, tab), "allocation");
  VC_CHECK(c, dalloc(&c->site_lnu, tab), "allocation");
  VC_CHECK(c, dalloc(&c->stage_lnug, vc::stages_per_sweep(c)), "allocation");
  if (K > 1) {
    VC_CHECK(c, dalloc(&c->u_site, ncpc * K), "allocation");
    VC_CHECK(c, dalloc(&c->u_j, ncpc * K * vc::KMAX), "allocation");
    VC_CHECK(c, dalloc(&c->u_rho, ncpc * K * vc::KMAX), "allocation");
    VC_CHECK(c, dalloc(&c->u_v, ncpc * K * 3), "allocation");
  }
  return VCSGC_OK;
}

vcsgc_status vcsgc_get_tuning(vcsgc_ctx *c, int32_t *strategy, int32_t *trials_per_group,
                              int32_t *workgroups) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (strategy) *strategy = c->strategy;
  if (trials_per_group) *trials_per_group = c->trials_per_group;
  if (workgroups) *workgroups = c->grid_total;
  return VCSGC_OK;
}

vcsgc_status eam_energy_forces(vcsgc_ctx *c, double *energy_eV, int want_forces) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1) return fail(c, VCSGC_E_INVALID_ARG, "not available on a batch context");
  if (want_forces && !c->fx)
    return fail(c, VCSGC_E_INVALID_ARG, "forces requested but the system has no force arrays");
  if (!c->md_valid) {
    st = refresh_md(c);
    if (st) return st;
  }
  VC_CHECK(c, vc::launch_pack(c), "pack");
  VC_CHECK(c, vc::launch_energy(c), "energy");
  if (want_forces) VC_CHECK(c, vc::launch_forces_only(c), "forces");
  c->rho_f_fresh = true;
  if (energy_eV) {
    VC_CHECK(c, vc::launch_reduce_sum(c, c->eatom, c->n, c->h_tot), "reduce");
    VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
    *energy_eV = c->h_tot[0];
  }
  return VCSGC_OK;
}

}  // extern "C"

namespace {

// Steps with the rebuild decision taken on the host after every drift
// (handles bin growth); used when the device path cannot be.
vcsgc_status md_steps_host(vcsgc_ctx *c, double dt_fs, int64_t n_steps) {
  VC_CHECK(c, vc::launch_pack(c), "pack");
  VC_CHECK(c, vc::launch_forces(c), "forces");
  for (int64_t k = 0; k < n_steps; ++k) {
    // the closing half-kick of step k-1 is fused into the opening one of step k
    VC_CHECK(c, vc::launch_kick_drift(c, dt_fs, k > 0, 0), "kick-drift");
    int flag = 0;
    VC_CHECK(c, hipMemcpyAsync(&flag, &c->ds->rebuild[0], sizeof(int), hipMemcpyDeviceToHost,
                               c->stream),
             "copy");
    VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
    if (flag) {
      VC_CHECK(c, hipMemsetAsync(&c->ds->rebuild[0], 0, sizeof(int), c->stream), "reset");
      vcsgc_status st = refresh_md(c);
      if (st) return st;
    }
    VC_CHECK(c, vc::launch_forces(c), "forces");
  }
  if (n_steps > 0) VC_CHECK(c, vc::launch_kick(c, dt_fs), "kick");
  return VCSGC_OK;
}

// Steps with the rebuild decided on the device (no host round trip per step).
// State at entry is kept; if a bin or a row overflowed on the way, it is
// restored and the steps are redone on the host-decided path.
vcsgc_status md_steps_device(vcsgc_ctx *c, double dt_fs, int64_t n_steps) {
  const size_t nb = sizeof(double) * (size_t)c->n;
  if (!c->snap) VC_CHECK(c, dalloc(&c->snap, 6 * (size_t)c->n), "allocation");
  double *state[6] = {c->x, c->y, c->z, c->vx, c->vy, c->vz};
  for (int k = 0; k < 6; ++k)
    VC_CHECK(c, hipMemcpyAsync(c->snap + k * c->n, state[k], nb, hipMemcpyDeviceToDevice,
                               c->stream),
             "snapshot");
  VC_CHECK(c, hipMemsetAsync(&c->ds->md_rebuilds, 0, sizeof(unsigned long long), c->stream),
           "reset");
  VC_CHECK(c, hipMemsetAsync(c->ds->rebuild, 0, 2 * sizeof(int), c->stream), "reset");
  VC_CHECK(c, vc::launch_pack(c), "pack");
  // step k uses the rebuild flag of parity k & 1 (its drift clears the
  // other); its kick and drift run inside the force pass before it, and
  // the last force pass stores the forces for the closing half kick
  VC_CHECK(c, vc::launch_forces_kick_drift(c, dt_fs, false, 0), "forces");
  for (int64_t k = 0; k < n_steps; ++k) {
    VC_CHECK(c, vc::launch_md_rebuild_cond(c, (int)(k & 1), vc::md_binned_drift(c)), "neighbour list (MD)");
    if (k + 1 < n_steps)
      VC_CHECK(c, vc::launch_forces_kick_drift(c, dt_fs, true, (int)((k + 1) & 1)), "forces");
    else
      VC_CHECK(c, vc::launch_forces(c), "forces");
  }
  VC_CHECK(c, vc::launch_kick(c, dt_fs), "kick");
  hipError_t e;
  vc::DevState h = read_state(c, &e);
  if (e != hipSuccess) return dev_fail(c, e, "MD");
  c->md_rebuilds += (int64_t)h.md_rebuilds;
  if (!h.bin_overflow && !h.overflow) return VCSGC_OK;
  for (int k = 0; k < 6; ++k)
    VC_CHECK(c, hipMemcpyAsync(state[k], c->snap + k * c->n, nb, hipMemcpyDeviceToDevice,
                               c->stream),
             "restore");
  const int zero[2] = {0, 0};
  VC_CHECK(c, hipMemcpyAsync(&c->ds->overflow, zero, 2 * sizeof(int), hipMemcpyHostToDevice,
                             c->stream),
           "reset");
  VC_CHECK(c, hipMemsetAsync(c->ds->rebuild, 0, 2 * sizeof(int), c->stream), "reset");
  if (h.bin_overflow) {
    vcsgc_status st = grow_bins(c);
    if (st) return st;
  }
  vcsgc_status st = refresh_md(c);
  if (st) return st;
  return md_steps_host(c, dt_fs, n_steps);
}

// Nose-Hoover NVT steps: per step the thermostat's half steps at the step
// boundary, the scaled kick and drift, the rebuild decision (on the device
// when the search bins allow it, else read by the host), forces, and the
// closing kick with the kinetic-energy chunk sums.  On a bin or row overflow
// of a device-decided rebuild the call's entry state (positions,
// velocities, xi, eta) is restored and the steps are redone with host
// decisions.
vcsgc_status md_nvt_steps(vcsgc_ctx *c, double dt_fs, int64_t n_steps, bool dev) {
  const size_t nb = sizeof(double) * (size_t)c->n;
  double *state[6] = {c->x, c->y, c->z, c->vx, c->vy, c->vz};
  if (dev) {
    if (!c->snap) VC_CHECK(c, dalloc(&c->snap, 6 * (size_t)c->n), "allocation");
    for (int k = 0; k < 6; ++k)
      VC_CHECK(c, hipMemcpyAsync(c->snap + k * c->n, state[k], nb, hipMemcpyDeviceToDevice,
                                 c->stream),
               "snapshot");
    VC_CHECK(c, hipMemcpyAsync(c->nvt + 5, c->nvt, 2 * sizeof(double), hipMemcpyDeviceToDevice,
                               c->stream),
             "snapshot");
    VC_CHECK(c, hipMemsetAsync(&c->ds->md_rebuilds, 0, sizeof(unsigned long long), c->stream),
             "reset");
  }
  VC_CHECK(c, hipMemsetAsync(c->ds->rebuild, 0, 2 * sizeof(int), c->stream), "reset");
  VC_CHECK(c, vc::launch_pack(c), "pack");
  VC_CHECK(c, vc::launch_forces(c), "forces");
  if (n_steps > 0) {  // a call of no steps leaves xi and eta
    VC_CHECK(c, vc::launch_nvt_ke(c, dt_fs, false), "thermostat");
    VC_CHECK(c, vc::launch_nvt_thermo(c, dt_fs, 2), "thermostat");
  }
  for (int64_t k = 0; k < n_steps; ++k) {
    const int par = dev ? (int)(k & 1) : 0;
    VC_CHECK(c, vc::launch_nvt_kick_drift(c, dt_fs, par), "kick-drift");
    if (dev) {
      VC_CHECK(c, vc::launch_md_rebuild_cond(c, par, vc::md_binned_drift(c)), "neighbour list (MD)");
    } else {
      int flag = 0;
      VC_CHECK(c, hipMemcpyAsync(&flag, &c->ds->rebuild[0], sizeof(int), hipMemcpyDeviceToHost,
                                 c->stream),
               "copy");
      VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
      if (flag) {
        VC_CHECK(c, hipMemsetAsync(&c->ds->rebuild[0], 0, sizeof(int), c->stream), "reset");
        vcsgc_status st = refresh_md(c);
        if (st) return st;
      }
    }
    VC_CHECK(c, vc::launch_forces(c), "forces");
    VC_CHECK(c, vc::launch_nvt_ke(c, dt_fs, true), "thermostat");
    VC_CHECK(c, vc::launch_nvt_thermo(c, dt_fs, k + 1 < n_steps ? 3 : 1), "thermostat");
  }
  if (n_steps > 0) VC_CHECK(c, vc::launch_nvt_scale(c), "thermostat");
  if (!dev) return VCSGC_OK;
  hipError_t e;
  vc::DevState h = read_state(c, &e);
  if (e != hipSuccess) return dev_fail(c, e, "MD");
  c->md_rebuilds += (int64_t)h.md_rebuilds;
  if (!h.bin_overflow && !h.overflow) return VCSGC_OK;
  for (int k = 0; k < 6; ++k)
    VC_CHECK(c, hipMemcpyAsync(state[k], c->snap + k * c->n, nb, hipMemcpyDeviceToDevice,
                               c->stream),
             "restore");
  VC_CHECK(c, hipMemcpyAsync(c->nvt, c->nvt + 5, 2 * sizeof(double), hipMemcpyDeviceToDevice,
                             c->stream),
           "restore");
  const int zero[2] = {0, 0};
  VC_CHECK(c, hipMemcpyAsync(&c->ds->overflow, zero, 2 * sizeof(int), hipMemcpyHostToDevice,
                             c->stream),
           "reset");
  if (h.bin_overflow) {
    vcsgc_status st = grow_bins(c);
    if (st) return st;
  }
  vcsgc_status st = refresh_md(c);
  if (st) return st;
  return md_nvt_steps(c, dt_fs, n_steps, false);
}

// After a device-decided rebuild that overflowed (code of k_totals): the bins
// grow if it was a bin, and the list is rebuilt on the host's decisions.
vcsgc_status rebuild_after_overflow(vcsgc_ctx *c, int code) {
  const int zero[2] = {0, 0};
  VC_CHECK(c, hipMemcpyAsync(&c->ds->overflow, zero, 2 * sizeof(int), hipMemcpyHostToDevice,
                             c->stream),
           "reset");
  if (code & 1) {
    vcsgc_status st = grow_bins(c);
    if (st) return st;
  }
  return refresh_md(c);
}

// the host's part of a list rebuild decision: the flag of the last move
vcsgc_status rebuild_if_due(vcsgc_ctx *c) {
  int flag = 0;
  VC_CHECK(c, hipMemcpyAsync(&flag, &c->ds->rebuild[0], sizeof(int), hipMemcpyDeviceToHost,
                             c->stream),
           "copy");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  if (!flag) return VCSGC_OK;
  VC_CHECK(c, hipMemsetAsync(&c->ds->rebuild[0], 0, sizeof(int), c->stream), "reset");
  return refresh_md(c);
}

// a device-decided rebuild has been taken: the list is of the current box
void rebuilt_on_device(vcsgc_ctx *c) {
  c->md_rebuilds += 1;
  for (int d = 0; d < 3; ++d) c->box_build[d] = c->box[d];
}

// Energy, forces, F . F and F . f0 (fixed-shape totals into t[0..2]) at the
// current positions; after a move the MD list is rebuilt first when it raised
// ds->rebuild[0].  One host round trip (a relaxation's iteration took four,
// with the decision, the energy and the totals each in one).
vcsgc_status cg_eval(vcsgc_ctx *c, bool after_move, const double *f0, double t[3]) {
  double *part = c->cg + 9 * c->n;
  const double *h = c->h_tot;
  const bool dev = after_move && vc::md_rebuild_on_device(c);
  if (after_move && !dev) {
    vcsgc_status st = rebuild_if_due(c);
    if (st) return st;
  }
  if (dev)
    VC_CHECK(c, vc::launch_md_rebuild_cond(c, 0, vc::md_binned_drift(c)), "neighbour list (MD)");
  for (;;) {
    VC_CHECK(c, vc::launch_energy(c), "energy");
    VC_CHECK(c, vc::launch_forces_only(c), "forces");
    VC_CHECK(c, vc::launch_cg_eval(c, f0, part, c->h_tot), "relaxation");
    VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
    for (int k = 0; k < 3; ++k) t[k] = h[k];
    if (dev && h[3] != 0.0) {
      vcsgc_status st = rebuild_after_overflow(c, (int)h[3]);
      if (st) return st;
      continue;
    }
    if (dev && h[4] != 0.0) rebuilt_on_device(c);
    return VCSGC_OK;
  }
}

// A line search's start (launch_cg_start): F . d and max |d_i|^2 into t.
vcsgc_status cg_start(vcsgc_ctx *c, double b, bool copy, double t[2]) {
  const int64_t n = c->n;
  VC_CHECK(c, vc::launch_cg_start(c, c->cg, c->cg + 3 * n, c->cg + 6 * n, b, copy, c->cg + 9 * n,
                                  c->h_tot),
           "relaxation");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  t[0] = c->h_tot[0];
  t[1] = c->h_tot[1];
  return VCSGC_OK;
}

// New box edges L (single-system context): the search bins are re-gridded
// to floor(L / bin_edge) per axis, at most the grid of creation (whose
// arrays hold it).  False if an axis would hold fewer than two bins.
bool set_box(vcsgc_ctx *c, const double L[3]) {
  int nb[3];
  for (int d = 0; d < 3; ++d) {
    nb[d] = std::min(c->nb_max[d], (int)std::floor(L[d] / c->bin_edge));
    if (nb[d] < 2) return false;
  }
  RepHost &r = c->reps[0];
  for (int d = 0; d < 3; ++d) {
    c->box[d] = r.box[d] = L[d];
    c->nb[d] = r.nb[d] = nb[d];
  }
  c->nbins = r.nbins = (int64_t)nb[0] * nb[1] * nb[2];
  return true;
}

// the thermostat's half step with the barostat momentum (as in the NPT
// splitting documented at vcsgc_set_barostat); returns the velocity factor
double npt_thermo(double h, double g1kT, double Q, double W, double &K, double &pe, double &xi,
                  double &eta) {
  const double q = 0.5 * h;
  xi = xi + q * ((2.0 * K + pe * pe / W - g1kT) / Q);
  const double a = xi * q;
  const double s = (1.0 - a) / (1.0 + a);
  K = K * s * s;
  pe = pe * s;
  eta = eta + xi * h;
  xi = xi + q * ((2.0 * K + pe * pe / W - g1kT) / Q);
  return s;
}

// Forces with the virial terms at the current positions, the closing kick
// (if kick), and the totals: *K (eV) and *vir (eV).
// dev: a device-decided rebuild comes first (binned: of atoms the drift has
// binned).
vcsgc_status npt_forces_sums(vcsgc_ctx *c, bool kick, bool dev, bool binned, double cv, double h,
                             double *K, double *vir) {
  const double *t = c->h_tot;
  if (dev) VC_CHECK(c, vc::launch_md_rebuild_cond(c, 0, binned), "neighbour list (MD)");
  for (;;) {
    VC_CHECK(c, vc::launch_forces_virial(c, c->eatom), "forces");
    VC_CHECK(c, vc::launch_npt_sums(c, kick, cv, h, c->eatom, c->npt_part, c->h_tot), "barostat");
    VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
    if (dev && t[2] != 0.0) {  // nothing was kicked
      vcsgc_status st = rebuild_after_overflow(c, (int)t[2]);
      if (st) return st;
      continue;
    }
    if (dev && t[3] != 0.0) rebuilt_on_device(c);
    *K = 0.5 * t[0] / vc::ACC;
    *vir = -0.5 * t[1];
    return VCSGC_OK;
  }
}

// Nose-Hoover NPT steps, driven from the host (the box changes every step;
// its edges are kernel arguments), one round trip per step: the MD list is
// rebuilt on the device's decision (on the host's where the search bins do
// not allow it), and the flags come with the totals.  c->eatom holds the
// per-atom virial terms.
vcsgc_status md_npt_steps(vcsgc_ctx *c, double dt, int64_t n_steps) {
  const int64_t n = c->n;
  if (!c->npt_part)
    VC_CHECK(c, dalloc(&c->npt_part, 2 * (size_t)((n + vc::BLOCK - 1) / vc::BLOCK) + 8),
             "allocation");
  double th[2];
  VC_CHECK(c, hipMemcpyAsync(th, c->nvt, sizeof(th), hipMemcpyDeviceToHost, c->stream), "copy");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  double xi = th[0], eta = th[1], pe = c->npt_pe;
  const double h = 0.5 * dt;
  const double g = 3.0 * (double)n - 3.0;
  const double g1kT = (g + 1.0) * (vc::KB * c->nvt_T);
  const double Q = g1kT * c->nvt_tau * c->nvt_tau;
  const double W = g1kT * c->npt_tau * c->npt_tau;
  const double rc = c->pot.rc, reach = c->pot.rc + c->skin;
  VC_CHECK(c, hipMemsetAsync(&c->ds->rebuild[0], 0, sizeof(int), c->stream), "reset");
  VC_CHECK(c, vc::launch_pack(c), "pack");
  double K = 0.0, vir = 0.0;
  vcsgc_status st = npt_forces_sums(c, false, false, false, 1.0, h, &K, &vir);
  if (st) return st;
  double s_pend = 1.0;
  // writes the thermostat and barostat state back (the velocities take the
  // pending end-of-step factor)
  auto finish = [&](double xi_, double eta_, double pe_) -> vcsgc_status {
    VC_CHECK(c, vc::launch_scale_v(c, s_pend), "barostat");
    th[0] = xi_;
    th[1] = eta_;
    VC_CHECK(c, hipMemcpyAsync(c->nvt, th, sizeof(th), hipMemcpyHostToDevice, c->stream), "copy");
    VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
    c->npt_pe = pe_;
    c->npt_vir = vir;
    return VCSGC_OK;
  };
  for (int64_t k = 0; k < n_steps; ++k) {
    const double xi0 = xi, eta0 = eta, pe0 = pe;
    const double s = npt_thermo(h, g1kT, Q, W, K, pe, xi, eta);
    double V = c->box[0] * c->box[1] * c->box[2];
    double P = (2.0 * K + vir) / (3.0 * V);
    pe = pe + h * (3.0 * V * (P - c->npt_p) + (3.0 / g) * (2.0 * K));
    const double ve = pe / W;
    const double cv = std::exp(-(1.0 + 3.0 / g) * ve * (0.5 * h));
    const double q = std::exp(ve * h);
    const double L[3] = {c->box[0] * q * q, c->box[1] * q * q, c->box[2] * q * q};
    if (!set_box(c, L)) {  // the state of the last complete step is kept
      if ((st = finish(xi0, eta0, pe0))) return st;
      return fail(c, VCSGC_E_BOX_TOO_SMALL, "the box has shrunk below two search bins");
    }
    double lam[3], lmin = 1e300;
    for (int d = 0; d < 3; ++d) {
      lam[d] = L[d] / c->box_build[d];
      lmin = std::min(lmin, lam[d]);
    }
    const double thr = 0.5 * (lmin * reach - rc);
    // (the grid of search bins may have changed with the box)
    const bool dev = vc::md_rebuild_on_device(c), binned = c->bins_clear && vc::md_binned_drift(c);
    VC_CHECK(c, vc::launch_npt_kick_drift(c, s_pend, s, cv, h, dt, q, lam, thr, binned),
             "kick-drift");
    if (!dev && (st = rebuild_if_due(c))) return st;
    if ((st = npt_forces_sums(c, true, dev, binned, cv, h, &K, &vir))) return st;
    V = c->box[0] * c->box[1] * c->box[2];
    P = (2.0 * K + vir) / (3.0 * V);
    pe = pe + h * (3.0 * V * (P - c->npt_p) + (3.0 / g) * (2.0 * K));
    s_pend = npt_thermo(h, g1kT, Q, W, K, pe, xi, eta);
  }
  return finish(xi, eta, pe);
}

}  // namespace

extern "C" {

vcsgc_status vcsgc_set_thermostat(vcsgc_ctx *c, double T_K, double tau_fs, double xi,
                                  double eta) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1 || !c->nvt)
    return fail(c, VCSGC_E_INVALID_ARG, "the thermostat needs a single-system MD context");
  if (!is_fin(T_K) || T_K < 0.0 || !(tau_fs > 0.0) || !is_fin(xi) || !is_fin(eta))
    return fail(c, VCSGC_E_INVALID_ARG, "need T >= 0, tau > 0 and finite xi, eta");
  const double h[2] = {xi, eta};
  VC_CHECK(c, hipMemcpyAsync(c->nvt, h, sizeof(h), hipMemcpyHostToDevice, c->stream), "copy");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  c->nvt_T = T_K;
  c->nvt_tau = tau_fs;
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_barostat(vcsgc_ctx *c, double p_ext, double tau_p_fs, double pe) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1 || !c->nvt)
    return fail(c, VCSGC_E_INVALID_ARG, "the barostat needs a single-system MD context");
  if (!is_fin(p_ext) || !is_fin(tau_p_fs) || tau_p_fs < 0.0 || !is_fin(pe))
    return fail(c, VCSGC_E_INVALID_ARG, "need finite p_ext and pe and tau_p >= 0");
  c->npt_p = p_ext;
  c->npt_tau = tau_p_fs;
  c->npt_pe = pe;
  return VCSGC_OK;
}

vcsgc_status vcsgc_get_barostat(vcsgc_ctx *c, double *pe, double *box, double *virial) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (pe) *pe = c->npt_pe;
  if (box)
    for (int d = 0; d < 3; ++d) box[d] = c->box[d];
  if (virial) *virial = c->npt_vir;
  return VCSGC_OK;
}

vcsgc_status vcsgc_get_thermostat(vcsgc_ctx *c, double *xi, double *eta) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!c->nvt) return fail(c, VCSGC_E_INVALID_ARG, "not an MD context");
  double h[2];
  VC_CHECK(c, hipMemcpyAsync(h, c->nvt, sizeof(h), hipMemcpyDeviceToHost, c->stream), "copy");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  if (xi) *xi = h[0];
  if (eta) *eta = h[1];
  return VCSGC_OK;
}

vcsgc_status vcsgc_minimize(vcsgc_ctx *c, const vcsgc_cg_params *prm, vcsgc_cg_result *res) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1) return fail(c, VCSGC_E_INVALID_ARG, "not available on a batch context");
  if (!prm || !c->fx)
    return fail(c, VCSGC_E_INVALID_ARG, "relaxation needs parameters and force arrays");
  const double lmin = std::min({c->box[0], c->box[1], c->box[2]});
  if (prm->max_iter < 0 || prm->max_eval < 0 || !is_fin(prm->etol) || !is_fin(prm->ftol) ||
      prm->ftol < 0.0 || !is_fin(prm->dmax) || !(prm->dmax > 0.0) || !(prm->dmax < 0.5 * lmin))
    return fail(c, VCSGC_E_INVALID_ARG,
                "need max_iter, max_eval >= 0, finite etol, ftol >= 0, 0 < dmax < L/2");
  const int64_t n = c->n;
  if (!c->cg) VC_CHECK(c, dalloc(&c->cg, 9 * (size_t)n + 3 * (size_t)((n + vc::BLOCK - 1) / vc::BLOCK) + 8),
                       "allocation");
  double *d = c->cg, *x0 = c->cg + 3 * n, *f0 = c->cg + 6 * n;
  c->rho_f_fresh = false;
  if (!c->md_valid) {
    st = refresh_md(c);
    if (st) return st;
  }
  VC_CHECK(c, hipMemsetAsync(&c->ds->rebuild[0], 0, sizeof(int), c->stream), "reset");
  VC_CHECK(c, vc::launch_pack(c), "pack");
  double e[3], t[2];
  st = cg_eval(c, false, f0, e);  // (F . f0 means nothing yet)
  if (st) return st;
  double E = e[0], gg = e[1], b = 0.0, dE_prev = 0.0;
  int64_t it = 0, ev = 0;
  int32_t reason = 0;
  bool moved = false;
  for (;;) {
    if (std::sqrt(gg) <= prm->ftol) {
      reason = VCSGC_CG_FORCE;
      break;
    }
    if (it >= prm->max_iter) {
      reason = VCSGC_CG_ITER;
      break;
    }
    if (ev >= prm->max_eval) {
      reason = VCSGC_CG_EVAL;
      break;
    }
    // d = F, or F + b d
    if ((st = cg_start(c, b, it == 0, t))) return st;
    double sl = t[0], dm2 = t[1];
    if (!(sl > 0.0)) {  // not a descent direction: restart along the force
      if ((st = cg_start(c, 0.0, true, t))) return st;
      sl = t[0];
      dm2 = t[1];
    }
    double a = prm->dmax / std::sqrt(dm2);
    if (it > 0) {
      const double a1 = 2.0 * dE_prev / sl;
      if (a1 < a) a = a1;
    }
    double Et = 0.0;
    bool accepted = false;
    for (int k = 0; k < VCSGC_CG_TRIALS; ++k) {
      VC_CHECK(c, vc::launch_cg_move(c, x0, d, a), "relaxation");
      moved = true;
      if ((st = cg_eval(c, true, f0, e))) return st;
      Et = e[0];
      ev += 1;
      if (Et <= E - VCSGC_CG_C1 * a * sl && Et < E) {
        accepted = true;
        break;
      }
      a = a * 0.5;
    }
    if (!accepted) {  // back to the line search's start (forces recomputed there)
      VC_CHECK(c, vc::launch_cg_move(c, x0, d, 0.0), "relaxation");
      if ((st = cg_eval(c, true, f0, e))) return st;
      reason = VCSGC_CG_LINESEARCH;
      break;
    }
    const double g_new = e[1], g_mix = e[2];
    b = (g_new - g_mix) / gg;
    if (!(b > 0.0)) b = 0.0;
    const double dE = E - Et;
    dE_prev = dE;
    E = Et;
    gg = g_new;
    it += 1;
    if (dE <= prm->etol * std::fabs(E)) {
      reason = VCSGC_CG_ENERGY;
      break;
    }
  }
  if (moved) c->mc_valid = false;
  c->rho_f_fresh = true;  // the last evaluation ran at the final positions
  if (res) {
    res->iterations = it;
    res->evaluations = ev;
    res->energy = E;
    res->fnorm = std::sqrt(gg);
    res->reason = reason;
  }
  return VCSGC_OK;
}

vcsgc_status md_verlet_step(vcsgc_ctx *c, double dt_fs, int64_t n_steps) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1) return fail(c, VCSGC_E_INVALID_ARG, "not available on a batch context");
  if (!c->vx || !c->fx)
    return fail(c, VCSGC_E_INVALID_ARG, "MD needs velocity and force arrays");
  if (!is_fin(dt_fs) || !(dt_fs > 0.0) || n_steps < 0)
    return fail(c, VCSGC_E_INVALID_ARG, "need dt > 0 and n_steps >= 0");
  c->rho_f_fresh = false;
  if (!c->md_valid) {
    st = refresh_md(c);
    if (st) return st;
  }
  if (c->npt_tau > 0.0 && !(c->nvt_T > 0.0))
    return fail(c, VCSGC_E_INVALID_ARG, "the barostat needs the thermostat (vcsgc_set_thermostat)");
  if (n_steps > 0) c->mc_valid = false;
  if (c->npt_tau > 0.0)
    st = md_npt_steps(c, dt_fs, n_steps);
  else if (c->nvt_T > 0.0)
    st = md_nvt_steps(c, dt_fs, n_steps, vc::md_rebuild_on_device(c));
  else
    st = (n_steps > 0 && vc::md_rebuild_on_device(c)) ? md_steps_device(c, dt_fs, n_steps)
                                                      : md_steps_host(c, dt_fs, n_steps);
  if (st) return st;
  c->rho_f_fresh = true;  // the last force pass ran at the final positions
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_log(vcsgc_ctx *c, double *tlog, int64_t tcap, double *slog, int64_t scap) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if ((tlog && tcap < 0) || (slog && scap < 0))
    return fail(c, VCSGC_E_INVALID_ARG, "negative log capacity");
  c->tlog = tlog;
  c->tcap = tlog ? tcap : 0;
  c->slog = slog;
  c->scap = slog ? scap : 0;
  const unsigned long long zero[2] = {0, 0};
  VC_CHECK(c, hipMemcpyAsync(&c->ds->tlog_n, zero, 2 * sizeof(unsigned long long),
                             hipMemcpyHostToDevice, c->stream),
           "log reset");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  drop_graph(c);  // its kernel node holds the old buffers and capacities
  return VCSGC_OK;
}

vcsgc_status vcsgc_log_counts(vcsgc_ctx *c, int64_t *n_trials, int64_t *n_stages) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  hipError_t e;
  vc::DevState h = read_state(c, &e);
  if (e != hipSuccess) return dev_fail(c, e, "log counts");
  if (n_trials) *n_trials = (int64_t)h.tlog_n;
  if (n_stages) *n_stages = (int64_t)h.slog_n;
  return VCSGC_OK;
}

vcsgc_status vcsgc_get_state(vcsgc_ctx *c, vcsgc_state *out) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!out) return fail(c, VCSGC_E_INVALID_ARG, "null output");
  int64_t n_b = 0;
  VC_CHECK(c, vc::persist_read_nb(c, &n_b), "state");
  out->sweeps_done = c->w;
  out->n_b = n_b;
  out->seed = c->last_seed;
  if (out->rho_dev) {
    st = ensure_mc(c);
    if (st) return st;
    VC_CHECK(c, hipMemcpyAsync(out->rho_dev, c->rho, sizeof(double) * c->n,
                               hipMemcpyDeviceToDevice, c->stream),
             "state");
    VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  }
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_state(vcsgc_ctx *c, const vcsgc_state *in) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!in) return fail(c, VCSGC_E_INVALID_ARG, "null input");
  c->w = in->sweeps_done;
  c->last_seed = in->seed;
  VC_CHECK(c, vc::persist_count(c), "state");  // n_B recounted from the species
  c->mc_valid = false;  // species may have been restored: fresh density cache
  c->rho_f_fresh = false;
  if (in->rho_dev) {
    // lists for the current positions (with a fresh cache), then the saved cache
    st = refresh_mc(c);
    if (st) return st;
    VC_CHECK(c, hipMemcpyAsync(c->rho, in->rho_dev, sizeof(double) * c->n,
                               hipMemcpyDeviceToDevice, c->stream),
             "state");
  }
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  return VCSGC_OK;
}

vcsgc_status vcsgc_copy_rho(vcsgc_ctx *c, double *rho_dev) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!rho_dev) return fail(c, VCSGC_E_INVALID_ARG, "null output");
  st = ensure_mc(c);
  if (st) return st;
  VC_CHECK(c, hipMemcpyAsync(rho_dev, c->rho, sizeof(double) * c->n, hipMemcpyDeviceToDevice,
                             c->stream),
           "copy");
  return VCSGC_OK;
}

vcsgc_status vcsgc_atom_energies(vcsgc_ctx *c, double *e_dev) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (c->reps.size() != 1) return fail(c, VCSGC_E_INVALID_ARG, "not available on a batch context");
  if (!e_dev) return fail(c, VCSGC_E_INVALID_ARG, "null output");
  if (!c->md_valid) {
    st = refresh_md(c);
    if (st) return st;
  }
  VC_CHECK(c, vc::launch_pack(c), "pack");
  VC_CHECK(c, vc::launch_energy(c), "energy");
  c->rho_f_fresh = true;
  VC_CHECK(c, hipMemcpyAsync(e_dev, c->eatom, sizeof(double) * c->n, hipMemcpyDeviceToDevice,
                             c->stream),
           "copy");
  return VCSGC_OK;
}

vcsgc_status vcsgc_get_info(vcsgc_ctx *c, vcsgc_info *out) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!out) return fail(c, VCSGC_E_INVALID_ARG, "null output");
  for (int d = 0; d < 3; ++d) out->n_cells[d] = c->nc[d];
  out->stages_per_sweep = c->reps.size() == 1 ? vc::stages_per_sweep(c) : c->S;
  out->kmax = vc::KMAX;
  if (c->mc_valid && c->mc_stats_stale) {
    VC_CHECK(c, vc::launch_mc_row_stats(c), "neighbour list");
    c->mc_stats_stale = false;
  }
  hipError_t e;
  vc::DevState h = read_state(c, &e);
  if (e != hipSuccess) return dev_fail(c, e, "info");
  out->mc_kmax_used = c->mc_valid ? h.kmax_used : 0;
  out->mc_pairs = c->mc_valid ? (int64_t)h.pairs_mc : 0;
  out->md_pairs = c->md_valid ? (int64_t)h.pairs_md : 0;
  out->md_rebuilds = c->md_rebuilds;
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_sample_log(vcsgc_ctx *c, double *desc_dev, double *dE_dev, int64_t cap,
                                  int64_t stride) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (desc_dev && (!c->desc || !dE_dev || cap < 0 || stride < 1))
    return fail(c, VCSGC_E_INVALID_ARG,
                "sample log needs VCSGC_FLAG_DESCRIPTOR, both buffers, cap >= 0, stride >= 1");
  if (desc_dev && c->reps.size() != 1)
    return fail(c, VCSGC_E_INVALID_ARG, "sample log needs a single-system context");
  c->smp_desc = desc_dev;
  c->smp_de = desc_dev ? dE_dev : nullptr;
  c->smp_cap = desc_dev ? cap : 0;
  c->smp_stride = stride < 1 ? 1 : stride;
  const unsigned long long zero = 0;
  VC_CHECK(c, hipMemcpyAsync(&c->ds->smp_n, &zero, sizeof(zero), hipMemcpyHostToDevice, c->stream),
           "reset");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  return VCSGC_OK;
}

vcsgc_status vcsgc_sample_count(vcsgc_ctx *c, int64_t *n_logged) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!n_logged) return fail(c, VCSGC_E_INVALID_ARG, "null output");
  hipError_t e;
  vc::DevState h = read_state(c, &e);
  if (e != hipSuccess) return dev_fail(c, e, "sample count");
  *n_logged = (int64_t)h.smp_n;
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_surrogate(vcsgc_ctx *c, const vcsgc_mlp *m, int32_t mode) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (mode < 0 || mode > 3) return fail(c, VCSGC_E_INVALID_ARG, "mode must be in [0, 3]");
  if (mode != 0 && c->reps.size() != 1)
    return fail(c, VCSGC_E_INVALID_ARG, "delayed acceptance needs a single-system context");
  if (mode == 1) {
    if (!m) return fail(c, VCSGC_E_NO_SURROGATE, "mode 1 needs a network");
    if (!c->desc) return fail(c, VCSGC_E_INVALID_ARG, "mode 1 needs VCSGC_FLAG_DESCRIPTOR");
    if (c->r_dep < vc::DESC_CUT + c->pot.rc)
      return fail(c, VCSGC_E_INVALID_ARG, "mode 1 needs r_dep >= 4.41 + rc");
  }
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  c->mlp = mode == 1 ? m : nullptr;
  c->da_mode = mode;
  return VCSGC_OK;
}

vcsgc_status vcsgc_set_surrogate_log(vcsgc_ctx *c, double *log_dev, int64_t cap) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (log_dev && cap < 0) return fail(c, VCSGC_E_INVALID_ARG, "negative capacity");
  c->dalog = log_dev;
  c->dacap = log_dev ? cap : 0;
  const unsigned long long zero = 0;
  VC_CHECK(c, hipMemcpyAsync(&c->ds->dalog_n, &zero, sizeof(zero), hipMemcpyHostToDevice,
                             c->stream),
           "reset");
  VC_CHECK(c, hipStreamSynchronize(c->stream), "sync");
  return VCSGC_OK;
}

vcsgc_status vcsgc_descriptors(vcsgc_ctx *c, const int32_t *sites_dev, int64_t n, int32_t flip,
                               double *out_dev) {
  vcsgc_status st = check_ctx(c);
  if (st) return st;
  if (!c->desc) return fail(c, VCSGC_E_INVALID_ARG, "needs VCSGC_FLAG_DESCRIPTOR");
  if (n < 0 || (n > 0 && (!sites_dev || !out_dev))) return fail(c, VCSGC_E_INVALID_ARG, "bad arguments");
  st = ensure_mc(c);
  if (st) return st;
  VC_CHECK(c, vc::launch_descriptors(c, sites_dev, n, flip, out_dev), "descriptors");
  return VCSGC_OK;
}

vcsgc_status vcsgc_selftest_sqrt(const double *in_dev, double *out_dev, int64_t n,
                                 hipStream_t stream) {
  if (n < 0 || (n > 0 && (!in_dev || !out_dev))) return VCSGC_E_INVALID_ARG;
  hipError_t e = vc::launch_sqrt(in_dev, out_dev, n, stream);
  return e == hipSuccess ? VCSGC_OK : VCSGC_E_DEVICE;
}

vcsgc_status vcsgc_selftest_md_math(const double *a_dev, const double *b_dev, double *sqrt_dev,
                                    double *div_dev, int64_t n, hipStream_t stream) {
  if (n < 0 || (n > 0 && (!a_dev || !b_dev || !sqrt_dev || !div_dev)))
    return VCSGC_E_INVALID_ARG;
  hipError_t e = vc::launch_md_math(a_dev, b_dev, sqrt_dev, div_dev, n, stream);
  return e == hipSuccess ? VCSGC_OK : VCSGC_E_DEVICE;
}

}  // extern "C"
