// Persistent parallel VC-SGC sweep for a batch of independent replicas
// (a single system is a batch of one), one launch for all sweeps of a call,
// a cooperative one where workgroups wait for each other.
//
// Replica r owns workgroups [g0, g0 + G) of the grid, each a contiguous share
// of the replica's active cells.  A stage whose global test fails changes
// nothing, so a batch of consecutive stages of a sweep is tried at once on the
// state as it is, one group of PTL lanes per trial:
//   1. every group makes its trials (the arithmetic of the per-stage kernels):
//      local factor of Eq. trans_vcsgc_par1; the workgroup's counts per stage
//      (accepts with dn = +1 and -1) are summed in LDS;
//   2. replicas of several workgroups: each adds its counts, packed with an
//      arrival, to one device word per stage and polls until every workgroup
//      has arrived (one round trip is the barrier and the reduction);
//   3. every workgroup evaluates the stages' global factors of
//      Eq. trans_vcsgc_par2 (identical decisions) up to the first accepted
//      stage; the trials of later stages are dropped;
//   4. an accepted stage is committed by the groups that hold its trials
//      (species, density cache, velocity rescaling), and a second barrier
//      makes it visible before the next batch.
// The chain is the one-stage-at-a-time chain, stage for stage.
//
// What bounds it: the latency of a batch (6 - 12 us), not bytes or
// arithmetic.  Shader cycles of a batch at 128,000 sites with 53% accepted stages,
// 16,900: the trials' dependent chain 4,000, the barrier of the counts 4,100, the
// commit 440 and its barrier 4,000, the next rows and the LDS barrier before
// them 2,250, the draws that are due 1,200, the decision 950.  With few accepted
// stages the trials of more of them: 6,700 of 17,900 (2.5%; 11 stages per
// batch); at 1.95M sites 25,000 of 45,500 (2%), with the network 18,700 of 34,800.
// Therefore:
//   - sites, ln u and ln u_g are drawn ahead into LDS rings by waves that
//     would otherwise wait (two Philox blocks, a logarithm and two dependent
//     loads per trial);
//   - the rows of the next batch are read before the decision of this one;
//   - a batch holds as many stages as the groups try in one pass, and twice
//     as many after each rejected batch, so that with few accepted stages its
//     fixed cost is shared by more of them.  (It is never shorter than a pass: with
//     60% accepted stages 128,000 sites try 8 stages to decide 1.6.)
//   - a replica whose densities and species fit the LDS runs in one workgroup
//     that keeps them there (RES) and needs no device barrier;
//   - 8 lanes per trial, two entries' chains side by side in a lane (16 lanes
//     per trial doubled the instructions a SIMD issues per batch).
// Measured (calls included; before: one stage per two release/acquire
// barriers of the device scope, every draw on the path): a sweep of 2,000
// rigid sites 11.2 -> 0.20 ms; of 128,000 thermal sites 4.3 -> 1.35 ms near
// equilibrium (0.42 ms from a random start, where few stages are accepted);
// two sweeps of 64 replicas of 2,000 to 250,000 sites 21.8 -> 5.5 ms.
//
// The densities and species of replicas of several workgroups are read and
// written with relaxed device-scope atomics, which bypass the caches that are
// not shared between XCDs; everything else the loop reads from memory is
// constant during the call.  A workgroup waits for its own stores (vmcnt)
// before it arrives at a barrier.  Barrier waits are bounded: a wait that
// exceeds the spin limit sets the replica's error flag and the workgroup
// leaves the kernel, so the launch always drains.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "mlp_device.hpp"

namespace vc {

constexpr int PTL = 8;                // lanes per trial
constexpr int PH = KMAX / PTL;        // row entries per lane
constexpr int PBLOCK = 512;           // threads of a workgroup
constexpr int PGROUPS = PBLOCK / PTL; // trials per workgroup pass
constexpr int PDMAX = 32;             // stages per batch, at most
constexpr int PDG = 16;               // the same with several workgroups
constexpr int PWIN = 256;             // stages whose counters are drawn ahead (a power of two)
constexpr int PDRAW = 1024;           // trials drawn ahead (twice that without a resident replica)
// Rings over the batches of a call: the counts in LDS and the words in memory.
// The batch number runs modulo a multiple of both (a 32-bit counter left the
// LDS ring's order when it wrapped: 2^32 mod 3 = 1, so after 2^32 batches of one
// call a batch added to counts that had not been cleared).
constexpr int PCW = 3, PWORDS = 4, PRINGS = 12;
static_assert(PRINGS % PCW == 0 && PRINGS % PWORDS == 0, "batch rings");
static_assert(8 * PDG == 128 && 2 * PDMAX <= PBLOCK && PDMAX <= 64, "a wave holds a batch's words");

struct RepD {
  int64_t n, aoff;
  int n0, n1, n2;
  int per, ncol;  // colour period per axis, colours
  int64_t cso, ncpc, roff, S;
  double beta, dmu0, kN, ncbar;
  uint64_t seed, key1;
  int g0, G;
  int res;  // one workgroup with the state in LDS
  int64_t n_sweeps, w0;
};

// Packed counts of a stage: accepts with dn = +1 (bits 0-27), with dn = -1
// (28-55), arrivals at one row of words (56-63).  A replica has fewer than 2^31
// cells, so fewer than 2^28 are active, and at most 8 * 255 workgroups (the
// arrivals are read per row; the sum of the rows may carry out at the top).
constexpr int PK_BITS = 28;
constexpr unsigned long long PK_MASK = (1ull << PK_BITS) - 1;
// A workgroup's counts of a stage with delayed acceptance: trials, trials that
// pass the network, near ties (a workgroup's share of cells is its LDS ring's
// at most, far below 2^21)
constexpr int DA_BITS = 21;
constexpr unsigned long long DA_MASK = (1ull << DA_BITS) - 1;

struct alignas(128) RepState {
  // words of the batches' stages, a ring of four batches: the words of batch
  // b + 2 are cleared by a workgroup that has seen all of them arrive at
  // batch b - 1 (so none still polls b - 2) and before it arrives at b.
  // Workgroup q adds to row q mod 8, a 128-byte line: the adds to one line are
  // served one after the other (216 workgroups on one line took 8 us a batch)
  unsigned long long word[PWORDS][8][PDG];
  // commit barrier: 64-bit arrival counters, one line per row of workgroups
  // (they grow by the row's workgroups per accepted stage and are zeroed only
  // once per call)
  struct alignas(128) Bar {
    unsigned long long n;
  } bar[8];
  // workgroups that have started; the top bit: given up
  struct alignas(128) Entry {
    unsigned long long n;
  } entry;
  alignas(128) long long n_b;  // n_B at the start of the next call
  unsigned long long trials, stage1, local_acc, stages, stage_acc, flips, near_ties;
  double sum_n, sum_n2;
  int err;  // PERSIST_TIMEOUT, PERSIST_NOT_STARTED
  long long n_final;
};
constexpr unsigned long long ENTRY_GIVEN_UP = 1ull << 63;

struct PersistArgs {
  const RepD *reps;
  RepState *rs;
  const int32_t *wg_rep;
  const int32_t *cstart, *catoms, *nj;
  const double *nr;  // r of each r < rc entry
  const uint8_t *cnt;
  uint8_t *sp;
  double *rho;
  double *vx, *vy, *vz;
  PotD p;
  double *tlog;
  int64_t tcap;
  double *slog;
  int64_t scap;
  unsigned long long *log_n;  // [2]: trial and stage records written
  unsigned int spin_limit, entry_limit;  // polls of a barrier, and for the start
  int ndraw;  // trials drawn ahead (LDS entries)
  // BIG: the drawn trials and records of one stage, per active cell of the replicas
  double *big_lnu;
  int32_t *big_site, *big_rec;
};

// delayed acceptance with the network: its parameters and the r < 4.41 A list
// (sorted rows, of which the r < rc entries are the dU row)
struct PersistArgsDa : PersistArgs {
  MlpDev md;
  const int32_t *dj;
  const double *dr;
  const uint8_t *dcnt;
};

// dynamic LDS of a workgroup: the groups' terms, the drawn trials and ln u_g,
// counts, and the state of a resident replica of nres atoms
struct PLds {
  double2 *terms;           // [PGROUPS][KMAX]
  double *lnu, *lnug;       // [ndraw], [PWIN]: ln u of trials, ln u_g of stages
  unsigned long long *cw;   // [PCW][PDMAX][2]: packed accepts; trials | ties << 32
  unsigned long long *tot;  // [PDMAX]
  double *rho;              // [nres]
  int32_t *site, *rec;      // [ndraw] each
  uint8_t *col;             // [PWIN] colours of stages
  uint8_t *sp;              // [nres]
  double *lnu2;             // [ndraw]: ln u of the second stage (delayed acceptance)
  struct DaLds *da;
};

static size_t persist_lds_bytes(int64_t ndraw, int64_t nres) {
  return sizeof(double2) * PGROUPS * KMAX + sizeof(double) * (ndraw + PWIN) +
         sizeof(unsigned long long) * (2 * PCW + 1) * PDMAX + sizeof(double) * nres +
         2 * sizeof(int32_t) * ndraw + PWIN + nres;
}

__device__ __forceinline__ PLds persist_lds(unsigned char *base, int ndraw, int64_t nres) {
  PLds l;
  l.terms = (double2 *)base;
  l.lnu = (double *)(l.terms + PGROUPS * KMAX);
  l.lnug = l.lnu + ndraw;
  l.cw = (unsigned long long *)(l.lnug + PWIN);
  l.tot = l.cw + 2 * PCW * PDMAX;
  l.rho = (double *)(l.tot + PDMAX);
  l.site = (int32_t *)(l.rho + nres);
  l.rec = l.site + ndraw;
  l.col = (uint8_t *)(l.rec + ndraw);
  l.sp = l.col + PWIN;
  return l;
}

__device__ __forceinline__ int64_t p_colour_cell(const RepD &r, int colour, uint32_t t) {
  const uint32_t P = (uint32_t)r.per;
  const uint32_t hx = (uint32_t)r.n0 / P, hy = (uint32_t)r.n1 / P;
  const uint32_t q = t / hx, ia = t - q * hx, ic = q / hy, ib = q - ic * hy;
  const uint32_t k = (uint32_t)colour, k1 = k / P;
  const int64_t cx = (int64_t)(P * ia + (k - k1 * P)), cy = (int64_t)(P * ib + (k1 % P)),
                cz = (int64_t)(P * ic + k1 / P);
  return cx + (int64_t)r.n0 * (cy + (int64_t)r.n1 * cz);
}

// this wave's vector-memory stores have been performed
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// What a lane holds of a site's row: entries lane + h PTL (inside the
// KMAX-entry row; entries beyond the row length are not dereferenced), and
// the densities the trial read for them.
struct PRow {
  int32_t j[PH];
  double r[PH], rj[PH];
  int m;
};

__device__ __forceinline__ void p_row(const int32_t *nj, const double *nr, const uint8_t *cnt,
                                      int64_t i, int lane, PRow &v) {
  v.m = cnt[i];
#pragma unroll
  for (int h = 0; h < PH; ++h) {
    const int64_t e = i * KMAX + lane + h * PTL;
    v.j[h] = nj[e];
    v.r[h] = nr[e];
  }
}

// Species and densities of a replica: in LDS (RES), or in memory through
// device-scope atomics.
template <bool RES>
struct PState {
  const PersistArgs &a;
  const PLds &l;
  int64_t aoff;
  __device__ __forceinline__ int sp(int64_t i) const {
    if (RES) return l.sp[i - aoff];
    return __hip_atomic_load(a.sp + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ double rho(int64_t i) const {
    if (RES) return l.rho[i - aoff];
    return __hip_atomic_load(a.rho + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void set_sp(int64_t i, int s) const {
    if (RES)
      l.sp[i - aoff] = (uint8_t)s;
    else
      __hip_atomic_store(a.sp + i, (uint8_t)s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void set_rho(int64_t i, double v) const {
    if (RES)
      l.rho[i - aoff] = v;
    else
      __hip_atomic_store(a.rho + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// F_X(rho) of the trial without a branch for the densities that sqrt_md
// serves; `slow` is raised for others (0 among them)
template <int F>
__device__ __forceinline__ double p_embed(const PotD &p, int s, double rho, bool &slow) {
  if (F == 1) return embed<1>(p, s, rho);
  const bool in = rho > 0x1p-700 && rho < 0x1p1000;
  slow = slow || !in;
  return -by_species(p.A, s) * sqrt_md(in ? rho : 1.0);
}

// transmutation energy change by the PTL lanes of a group (in-order sums of
// the terms the lanes leave in the group's LDS slots; a group is 8 lanes of
// one wave, whose LDS accesses are performed in order); s: the site's species.
// One wave per SIMD works on a stage here, so the chains of a lane's entries
// are laid side by side: two entries at a time without a branch (unused ones
// read the site itself and leave +0.0), the second two only where some row of
// the wave has more than 16 entries.
template <int F, bool RES>
__device__ __forceinline__ double p_delta_u(const PState<RES> &st, int64_t i, int lane, PRow &v,
                                            double2 *grp, int &s) {
  const PotD &p = st.a.p;
  s = st.sp(i);
  const double ri = st.rho(i);
  const bool more = __any(v.m > 2 * PTL);
  int sj[PH];
#pragma unroll
  for (int h0 = 0; h0 < PH; h0 += 2) {
    if (h0 && !more) break;
#pragma unroll
    for (int h = h0; h < h0 + 2; ++h) {
      const int64_t j = lane + h * PTL < v.m ? (int64_t)v.j[h] : i;
      sj[h] = st.sp(j);
      v.rj[h] = st.rho(j);
    }
  }
  bool slow = false;
  const double own_new = p_embed<F>(p, 1 - s, ri, slow), own_old = p_embed<F>(p, s, ri, slow);
#pragma unroll
  for (int h0 = 0; h0 < PH; h0 += 2) {
    if (h0 && !more) {
      grp[lane + h0 * PTL] = grp[lane + (h0 + 1) * PTL] = make_double2(0.0, 0.0);
      continue;
    }
    double tp[2], te[2];
    bool odd = false;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int h = h0 + q;
      const bool in = lane + h * PTL < v.m;
      const double r = in ? v.r[h] : p.rc;
      bool sl = false;
      const double shift = flip_rho_shift<F>(p, s, r);
      const double a = flip_pair_term<F>(p, s, sj[h], r);
      const double b = p_embed<F>(p, sj[h], v.rj[h] + shift, sl) -
                       p_embed<F>(p, sj[h], v.rj[h], sl);
      tp[q] = in ? a : 0.0;
      te[q] = in ? b : 0.0;
      odd = odd || (in && sl);
    }
    if (F == 0 && odd) {  // a density outside sqrt_md's range: the general form
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (lane + (h0 + q) * PTL < v.m)
          te[q] = flip_embed_term<0>(p, sj[h0 + q], v.rj[h0 + q],
                                     flip_rho_shift<0>(p, s, v.r[h0 + q]));
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) grp[lane + (h0 + q) * PTL] = make_double2(tp[q], te[q]);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double pair, emb;
  sum_flip_terms(grp, v.m, pair, emb);
  const double own = F == 0 && slow ? flip_own_term<0>(p, s, ri) : own_new - own_old;
  return own + pair + emb;
}

// the flip of site i (species s0) by its group: densities of the row's
// neighbours (rj as the trial read them: nothing was committed since; DA: the
// row reaches beyond rc), species, velocity
template <int F, bool RES, bool DA>
__device__ __forceinline__ void p_commit(const PState<RES> &st, int64_t i, int lane, int s0,
                                         const PRow &v) {
  const PersistArgs &a = st.a;
#pragma unroll
  for (int h = 0; h < PH; ++h)
    if (lane + h * PTL < v.m && (!DA || v.r[h] < a.p.rc))
      st.set_rho(v.j[h], v.rj[h] + flip_rho_shift<F>(a.p, s0, v.r[h]));
  if (lane == 0) {
    st.set_sp(i, 1 - s0);
    if (a.vx) {
      const double f = sqrt(by_species(a.p.mass, s0) / by_species(a.p.mass, 1 - s0));
      a.vx[i] = a.vx[i] * f;
      a.vy[i] = a.vy[i] * f;
      a.vz[i] = a.vz[i] * f;
    }
  }
}

// ---- delayed acceptance: the trials of a wave's eight groups ----------------
// The two-stage test of the per-stage kernels, in the batches of this sweep:
// a kernel per batch took 14.5 us, and two of them per accepted stage.  128,000
// sites: 2.3 ms at 4 and 1.4 ms at 16 stages per kernel, now 0.69 ms (9%
// accepted stages); 5.3 -> 3.2 ms (62%); 2,000 sites 6.7 -> 0.69, 1.02M sites
// 2.0 -> 0.97, 4.2M 6.3 -> 3.1 ms.
// The 16 descriptor rows (current and flipped environment of eight sites) are
// the rows of one MFMA tile, so a wave evaluates its own trials from the
// weights in LDS, without meeting the workgroup's other waves.
constexpr int DKP = MLP_KP + 8, DHP = MLP_H + 8;  // padded rows: no 16-way bank conflicts
constexpr int PWAVES = PBLOCK / 64;
struct DaWave {
  // an entry's densities before and after the flip, its pair and embedding
  // terms (zeros outside rc), and per entry 1 + shell (0: none)
  double q[64 / PTL][KMAX][4];
  uint8_t code[64 / PTL][KMAX];
};
struct DaHidden {  // in the place of the terms, once they are summed
  __bf16 h1[16 * DHP], h2[16 * DHP];
};
static_assert(sizeof(DaHidden) <= sizeof(DaWave), "hidden layers in the terms' place");
struct DaLds {
  DaWave wave[PWAVES];
  __bf16 zs[PWAVES][16 * DKP];
  __bf16 w1[MLP_H * DKP], w2[MLP_H * DHP];
  float b1[MLP_H], b2[MLP_H], w3[MLP_H];
  float mu[MLP_IN], sd[MLP_IN];
};

// dynamic LDS with delayed acceptance
static size_t persist_lds_bytes_da(int64_t ndraw) {
  return sizeof(DaLds) + sizeof(double) * (2 * ndraw + PWIN) +
         sizeof(unsigned long long) * (2 * PCW + 1) * PDMAX + 2 * sizeof(int32_t) * ndraw + PWIN;
}
__device__ __forceinline__ PLds persist_lds_da(unsigned char *base, int ndraw) {
  PLds l;
  l.da = (DaLds *)base;
  l.lnu = (double *)(base + sizeof(DaLds));
  l.lnu2 = l.lnu + ndraw;
  l.lnug = l.lnu2 + ndraw;
  l.cw = (unsigned long long *)(l.lnug + PWIN);
  l.tot = l.cw + 2 * PCW * PDMAX;
  l.site = (int32_t *)(l.tot + PDMAX);
  l.rec = l.site + ndraw;
  l.col = (uint8_t *)(l.rec + ndraw);
  l.terms = nullptr;
  l.rho = nullptr;
  l.sp = nullptr;
  return l;
}

__device__ __forceinline__ void da_weights(const MlpDev &m, DaLds &d, int tid) {
  for (int e = tid; e < MLP_H * MLP_KP; e += PBLOCK)
    d.w1[(e / MLP_KP) * DKP + e % MLP_KP] = m.w1[e];
  for (int e = tid; e < MLP_H * MLP_H; e += PBLOCK) d.w2[(e / MLP_H) * DHP + e % MLP_H] = m.w2[e];
  for (int e = tid; e < MLP_H; e += PBLOCK) {
    d.b1[e] = m.b1[e];
    d.b2[e] = m.b2[e];
    d.w3[e] = m.w3[e];
  }
  for (int e = tid; e < MLP_IN; e += PBLOCK) {
    d.mu[e] = m.mu[e];
    d.sd[e] = m.sd[e];
  }
}

__device__ __forceinline__ void wave_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ bf16x8 da_frag(const __bf16 *p) { return *(const bf16x8 *)p; }

// Network values of the wave's 16 rows of z: lane L < 16 returns row L's
// normalized output (the products and sums of mlp_block16f).
__device__ __forceinline__ float da_network(const MlpDev &m, const DaLds &d, const __bf16 *z,
                                            DaHidden &h) {
  const int wl = threadIdx.x & 63, r = wl & 15, kb = (wl >> 4) * 8;
  {
    const bf16x8 a = da_frag(z + r * DKP + kb);
#pragma unroll
    for (int t = 0; t < MLP_H / 16; ++t) {
      const int n = 16 * t + r;
      floatx4 c = {0.f, 0.f, 0.f, 0.f};
      c = mfma16(a, da_frag(d.w1 + n * DKP + kb), c);
      const float b = d.b1[n];
#pragma unroll
      for (int q = 0; q < 4; ++q) h.h1[((wl >> 4) * 4 + q) * DHP + n] = to_bf16(silu(c[q] + b));
    }
  }
  wave_lds();
  {
    const bf16x8 a0 = da_frag(h.h1 + r * DHP + kb), a1 = da_frag(h.h1 + r * DHP + 32 + kb);
#pragma unroll
    for (int t = 0; t < MLP_H / 16; ++t) {
      const int n = 16 * t + r;
      floatx4 c = {0.f, 0.f, 0.f, 0.f};
      c = mfma16(a0, da_frag(d.w2 + n * DHP + kb), c);
      c = mfma16(a1, da_frag(d.w2 + n * DHP + 32 + kb), c);
      const float b = d.b2[n];
#pragma unroll
      for (int q = 0; q < 4; ++q) h.h2[((wl >> 4) * 4 + q) * DHP + n] = to_bf16(silu(c[q] + b));
    }
  }
  wave_lds();
  float y = 0.0f;
  if (wl < 16) {
    y = m.b3[0];
    for (int k = 0; k < MLP_H; k += 8) {
      const bf16x8 v = da_frag(h.h2 + wl * DHP + k);
#pragma unroll
      for (int u = 0; u < 8; ++u) y += d.w3[k + u] * (float)v[u];
    }
  }
  wave_lds();
  return y;
}

// Exact dU of site i and the network's forward and reverse values, by all
// lanes of a wave (groups without a site: has = false, i any atom).  Lane c of
// a group sums one column of its entries in order (c < 3: densities of shell
// c, c < 6: the densities after the flip, 6: pair terms, 7: embedding terms);
// an entry of another shell adds +0.0 (the sums are never -0.0).
template <int F>
__device__ __forceinline__ double da_trial(const PState<false> &st, const PersistArgsDa &a,
                                           DaLds &d, bool has, int64_t i, int lane, PRow &v,
                                           int &s, double &ef, double &er) {
  const PotD &p = st.a.p;
  const int wl = threadIdx.x & 63, g = wl / PTL;
  DaWave &w = d.wave[threadIdx.x >> 6];
  __bf16 *z = d.zs[threadIdx.x >> 6];
  s = st.sp(i);
  const double ri = st.rho(i);
  const int m = has ? v.m : 0;
  int sj[PH];
#pragma unroll
  for (int h = 0; h < PH; ++h) {
    const int64_t j = lane + h * PTL < m ? (int64_t)v.j[h] : i;
    sj[h] = st.sp(j);
    v.rj[h] = st.rho(j);
  }
  // numbers of neighbours per shell (8 bits each) and of B among them
  unsigned int cnt = 0, cb = 0;
#pragma unroll
  for (int h = 0; h < PH; ++h) {
    const int k = lane + h * PTL;
    double rj = 0.0, rjf = 0.0, tp = 0.0, te = 0.0;
    int code = 0;
    if (k < m) {
      const double r = v.r[h];
      code = r < 2.68 ? 1 : (r < 3.46 ? 2 : (r < DESC_CUT ? 3 : 0));
      rj = v.rj[h];
      rjf = rj;
      if (r < p.rc) {
        const double delta = flip_rho_shift<F>(p, s, r);
        rjf = rj + delta;
        tp = flip_pair_term<F>(p, s, sj[h], r);
        te = flip_embed_term<F>(p, sj[h], rj, delta);
      }
      const unsigned int one = code ? 1u << (8 * (code - 1)) : 0u;
      cnt += one;
      cb += sj[h] ? one : 0u;
    }
    w.code[g][k] = (uint8_t)code;
    *(double4 *)w.q[g][k] = make_double4(rj, rjf, tp, te);
  }
  const double own = flip_own_term<F>(p, s, ri);
#pragma unroll
  for (int o = 1; o < PTL; o <<= 1) {
    cnt += __shfl_xor(cnt, o);
    cb += __shfl_xor(cb, o);
  }
  wave_lds();
  const int col = lane < 6 ? lane / 3 : lane - 4, shell = lane % 3;
  const int want = lane < 6 ? shell + 1 : -1;
  double sum = 0.0;
#pragma unroll
  for (int k0 = 0; k0 < KMAX; k0 += 8) {
    if (!__any(k0 < m)) break;
    const unsigned long long cd = *(const unsigned long long *)&w.code[g][k0];
    double t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = w.q[g][k0 + u][col];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int ck = (int)((cd >> (8 * u)) & 255u);
      sum += want < 0 || ck == want ? t[u] : 0.0;
    }
  }
  const double pair = __shfl(sum, 6, PTL), emb = __shfl(sum, 7, PTL);
  // descriptors: species, B per shell, neighbours per shell, mean densities
  {
    const int cs = (int)((cnt >> (8 * shell)) & 255u), bs = (int)((cb >> (8 * shell)) & 255u);
    const double mean = cs > 0 ? sum / (double)cs : 0.0;
    auto input = [&](int k, double x) {
      return to_bf16((float)((x - (double)d.mu[k]) / (double)d.sd[k]));
    };
    __bf16 *zf = z + g * DKP, *zr = z + (8 + g) * DKP;
    // lanes 0-5: a count for both rows, and the mean of one of them
    const int kc = lane < 6 ? 1 + lane : 0;
    const double xc = lane < 3 ? (double)bs : lane < 6 ? (double)cs
                                                       : (double)(lane == 6 ? s : 1 - s);
    const __bf16 vc = input(kc, xc);
    if (lane != 7) zf[kc] = vc;
    if (lane != 6) zr[kc] = vc;
    if (lane < 6) (lane < 3 ? zf : zr)[7 + shell] = input(7 + shell, mean);
    for (int k = MLP_IN / 2 + lane; k < MLP_KP / 2; k += PTL) {
      ((unsigned int *)zf)[k] = 0u;
      ((unsigned int *)zr)[k] = 0u;
    }
  }
  wave_lds();
  const float y = da_network(a.md, d, z, *(DaHidden *)&w);
  ef = (double)(__shfl(y, g) * a.md.out_sd + a.md.out_mu);
  er = (double)(__shfl(y, 8 + g) * a.md.out_sd + a.md.out_mu);
  return own + pair + emb;
}

// The start of a replica's workgroups.  Another process's grid on the same
// device can keep some of them from it for as long as it waits for workgroups that
// these keep out.  So each counts itself in, and one that has polled `limit`
// times for the rest gives up unless all have come: one compare-and-swap
// decides it for all of them, before anything is committed or logged.  (A limit of
// 0 gives up outright.)
__device__ __forceinline__ void p_arrive(RepState *st) {
  __hip_atomic_fetch_add(&st->entry.n, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool p_entered(RepState *st, unsigned long long G, unsigned int limit) {
  unsigned int it = 0;
  while (limit > 0) {
    unsigned long long v =
        __hip_atomic_load(&st->entry.n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v == G) return true;
    if (v & ENTRY_GIVEN_UP) return false;
    if (++it <= limit)
      __builtin_amdgcn_s_sleep(1);
    else if (__hip_atomic_compare_exchange_strong(&st->entry.n, &v, v | ENTRY_GIVEN_UP,
                                                  __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT))
      break;  // (else another one has arrived or given up)
  }
  __hip_atomic_fetch_or(&st->err, PERSIST_NOT_STARTED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return false;
}

// Draws ahead of the trials.  Stage counters: the colour and ln u_g of stages
// [s_lo, s_hi) into the ring of PWIN slots; trials: the site drawn from each
// own cell and ln u of its local test for stages [s_lo, s_hi) (counters drawn
// before) into the ring of `win` rows of `chunk` entries.  By threads t of nt.
__device__ __forceinline__ void p_draw_stages(const RepD &r, const PLds &l, uint64_t w,
                                              uint32_t s_lo, uint32_t s_hi, int t, int nt) {
  for (uint32_t s = s_lo + t; s < s_hi; s += nt) {
    const U4 g = philox(r.seed, r.key1, w, (uint64_t)s, 0, 0);
    l.col[s & (PWIN - 1)] = (uint8_t)stage_colour(g.v[0], r.ncol);
    l.lnug[s & (PWIN - 1)] = log(unit_open(g.v[1]));
  }
}

template <bool DA>
__device__ __forceinline__ void p_draw_trials(const RepD &r, const PLds &l, const int32_t *cstart,
                                              const int32_t *catoms, uint64_t w, uint32_t s_lo,
                                              uint32_t s_hi, int64_t t_lo, int own, int chunk,
                                              int win, int t, int nt) {
  const unsigned n = (s_hi - s_lo) * (unsigned)own;
  for (unsigned e = (unsigned)t; e < n; e += (unsigned)nt) {
    const unsigned k = e / (unsigned)own, c = e - k * (unsigned)own;
    const uint32_t s = s_lo + k;
    const int64_t cell = p_colour_cell(r, l.col[s & (PWIN - 1)], (uint32_t)(t_lo + c));
    const int32_t c0 = cstart[cell];
    const uint32_t m = (uint32_t)(cstart[cell + 1] - c0);
    int32_t site = -1;
    double lnu = 0.0, lnu2 = 0.0;
    if (m > 0) {
      const U4 rr = philox(r.seed, r.key1, w, (uint64_t)s, (uint64_t)cell, 1);
      site = catoms[c0 + draw_index(rr.v[0], m)];
      lnu = log(unit_open(rr.v[1]));
      if (DA) lnu2 = log(unit_open(rr.v[2]));
    }
    const int slot = (int)(s % (uint32_t)win) * chunk + (int)c;
    l.site[slot] = site;
    l.lnu[slot] = lnu;
    if (DA) l.lnu2[slot] = lnu2;
  }
}

// the sweeps of one replica by one of its workgroups; BIG: the share of cells is
// more than the LDS can draw a stage of (one stage per batch, LOG), the draws are
// in memory, and the block's barriers order memory too
template <int F, bool RES, bool LOG, bool DA, bool BIG>
__device__ __forceinline__ void sweep_replica(
    const typename std::conditional<DA, PersistArgsDa, PersistArgs>::type &a, const RepD &r,
    RepState *st, const PLds &lds, int *flag) {
  static_assert(!DA || (!RES && !LOG), "delayed acceptance");
  static_assert(!BIG || LOG, "one stage per batch");
  auto sync = [] {
    if constexpr (BIG)
      __syncthreads();
    else
      block_sync_lds();
  };
  auto row_of = [&](int64_t i, PRow &v) {
    if constexpr (DA)
      p_row(a.dj, a.dr, a.dcnt, i, threadIdx.x % PTL, v);
    else
      p_row(a.nj, a.nr, a.cnt, i, threadIdx.x % PTL, v);
  };
  const int tid = threadIdx.x, lane = tid % PTL, grp = tid / PTL, wl = tid & 63;
  const int q = (int)blockIdx.x - r.g0;  // rank inside the replica
  if (q >= r.G) return;                  // (not needed by this call)
  // contiguous share of the active cells; consecutive shares on one XCD
  // (workgroup ids advance round-robin over the 8 XCDs)
  int qc = q;
  if ((r.G & 7) == 0 && (r.g0 & 7) == 0) qc = (q & 7) * (r.G >> 3) + (q >> 3);
  const int chunk = (int)((r.ncpc + r.G - 1) / r.G);
  const int64_t t_lo = (int64_t)qc * chunk;
  const int64_t t_hi = t_lo + chunk < r.ncpc ? t_lo + chunk : r.ncpc;
  const int own = t_hi > t_lo ? (int)(t_hi - t_lo) : 0;
  const int32_t *cstart = a.cstart + r.cso;
  const int32_t *catoms = a.catoms + r.aoff;
  PLds l = lds;
  if constexpr (BIG) {
    l.lnu = a.big_lnu + r.roff + t_lo;
    l.site = a.big_site + r.roff + t_lo;
    l.rec = a.big_rec + r.roff + t_lo;
  }
  const PState<RES> state{a, l, r.aoff};
  // stages of drawn trials
  const int win = BIG ? 1 : a.ndraw / chunk < PWIN ? a.ndraw / chunk : PWIN;
  const int wave = tid >> 6;
  // Stages per batch: as many as the trial groups make in one pass, doubled
  // (more passes) while whole batches are rejected, so that a batch's fixed
  // cost is shared by more stages where few are accepted; one with logs on
  // (dropped trials would be logged).  Twice a batch has to be drawn ahead.
  const int fit = LOG || chunk > PGROUPS ? 1 : PGROUPS / chunk;
  const int cap = LOG ? 1 : max(1, min(RES || r.G == 1 ? PDMAX : PDG, win / 4));
  const int span0 = min(fit, cap);
  int span = span0;
  const uint32_t S = (uint32_t)r.S;  // below 2^31 for n < 2^31
  long long nb = st->n_b;
  // per lane k of every wave: counts of the stages k of the batches; replica
  // totals in the first workgroup
  unsigned long long n_trial = 0, n_tie = 0, n_acc = 0, n_stage = 0, n_sacc = 0, n_flip = 0;
  unsigned long long n_pass = 0;  // trials that pass the network's stage
  double sum_n = 0.0, sum_n2 = 0.0;
  unsigned long long ncom = 0;
  unsigned int batch = 0;
  bool entered = RES || r.G == 1;
  if (!entered && tid == 0) p_arrive(st);
  if (RES)
    for (int64_t i = tid; i < r.n; i += PBLOCK) {
      l.rho[i] = a.rho[r.aoff + i];
      l.sp[i] = a.sp[r.aoff + i];
    }
  for (int e = tid; e < 2 * PCW * PDMAX; e += PBLOCK) l.cw[e] = 0;
  if constexpr (DA) da_weights(a.md, *l.da, tid);
  __syncthreads();

  for (int64_t sw = 0; sw < r.n_sweeps; ++sw) {
    const uint64_t w = (uint64_t)(r.w0 + sw);
    uint32_t hs = 0, hd = 0;  // stages whose counters / trials are drawn
    bool have = false;        // the batch's rows are in `row`
    PRow row;
    row.m = 0;
    for (uint32_t s0 = 0; s0 < S; batch = batch + 1 == PRINGS ? 0 : batch + 1) {
      const int len = S - s0 < (uint32_t)span ? (int)(S - s0) : span;
      const bool one_pass = len * own <= PGROUPS;
      unsigned long long *cw = l.cw + 2 * PDMAX * (batch % PCW);
      if (s0 + len > hd) {  // the trials of this batch (and a few more) are due now
        sync();   // the last batch's readers of the rings are done
        const uint32_t ts = min(s0 + 4 * len, S);
        if (hs < ts) {
          p_draw_stages(r, l, w, hs, ts, tid, PBLOCK);
          hs = ts;
        }
        sync();
        const uint32_t to = min(min(s0 + 3 * len, s0 + win), S);
        p_draw_trials<DA>(r, l, cstart, catoms, w, hd, to, t_lo, own, chunk, win, tid, PBLOCK);
        hd = to;
        if (!entered && tid == 0)  // the call's first draws are made
          *flag = !p_entered(st, (unsigned long long)r.G, a.entry_limit);
        sync();
        if (!entered) {
          if (*flag) return;
          entered = true;
          sync();  // (the flag has been read)
        }
      }
      // what the waves draw while the others work or wait: about a batch of
      // trials and of stage counters, kept clear of the slots of the last batch
      const uint32_t td = max(hd, min(hd + 2 * len, min(s0 + win - cap, hs)));
      const uint32_t ts = max(hs, min(hs + 4 * len, min(s0 + PWIN - 2 * PDMAX, S)));
      auto draw_ahead = [&](int first) {
        if (wave == PBLOCK / 64 - 1)
          p_draw_stages(r, l, w, hs, ts, wl, 64);
        else if (wave >= first)
          p_draw_trials<DA>(r, l, cstart, catoms, w, hd, td, t_lo, own, chunk, win, tid - 64 * first,
                        PBLOCK - 64 - 64 * first);
      };
      // ---- trials: p = k own + c, stage s0 + k and cell t_lo + c
      int my_s = 0;         // one pass: the species of an accepted trial's site
      int32_t my_i = -1;    // and the site
      if constexpr (DA) {
        // whole waves: the lanes of one network evaluation
        for (int pw = grp & ~(64 / PTL - 1); pw < len * own; pw += PGROUPS) {
          const int p = pw + grp % (64 / PTL), k = p < len * own ? p / own : 0;
          const int e = (int)((s0 + k) % (uint32_t)win) * chunk + (p - k * own);
          const int32_t i = p < len * own ? l.site[e] : -1;
          int32_t rec = -1;
          const bool has = i >= 0;
          if (__any(has)) {
            if (has && (!have || p != grp)) row_of(i, row);
            int s;
            double ef, er;
            const double du = da_trial<F>(state, a, *l.da, has, has ? (int64_t)i : r.aoff, lane,
                                          row, s, ef, er);
            if (has) {
              const int dn = 1 - 2 * s;
              const double lnu1 = l.lnu[e], lnu2 = l.lnu2[e];
              const double x1 = r.beta * (ef + r.dmu0 * (double)dn);
              const bool pass1 = lnu1 < -x1;
              bool ok = false;
              double margin = lnu1 + x1;
              if (pass1) {
                const double sr = er - r.dmu0 * (double)dn;
                const double xl = r.beta * (du + r.dmu0 * (double)dn);
                const double xr = -(r.beta * sr);
                const double l2 = (-xl + (xr < 0.0 ? xr : 0.0)) - (-x1 < 0.0 ? -x1 : 0.0);
                ok = lnu2 < l2;
                margin = lnu2 - l2;
              }
              if (lane == 0) {
                if (ok) atomicAdd(&cw[2 * k], dn > 0 ? 1ull : 1ull << PK_BITS);
                atomicAdd(&cw[2 * k + 1], 1ull | (pass1 ? 1ull << DA_BITS : 0ull) |
                                              (fabs(margin) < TIE ? 1ull << (2 * DA_BITS) : 0ull));
              }
              if (ok) {
                rec = i;
                my_i = i;
                my_s = s;
              }
            }
          }
          if (!one_pass && lane == 0 && p < len * own) l.rec[p] = rec;
        }
      } else
      for (int p = grp; p < len * own; p += PGROUPS) {
        const int k = p / own;
        const int e = (int)((s0 + k) % (uint32_t)win) * chunk + (p - k * own);
        const int32_t i = l.site[e];
        int32_t rec = -1;
        if (i >= 0) {
          if (!have || p != grp) row_of(i, row);
          int s;
          const double du = p_delta_u<F, RES>(state, i, lane, row, l.terms + grp * KMAX, s);
          const double lnu = l.lnu[e];
          const int dn = 1 - 2 * s;
          const double xl = r.beta * (du + r.dmu0 * (double)dn);
          const double margin = lnu + xl;
          const bool ok = lnu < -xl;  // the same on every lane of the group
          if (lane == 0) {
            if (ok) atomicAdd(&cw[2 * k], dn > 0 ? 1ull : 1ull << PK_BITS);
            atomicAdd(&cw[2 * k + 1], 1ull | (fabs(margin) < TIE ? 1ull << 32 : 0ull));
            if (LOG && a.tlog) {
              const unsigned long long idx = atomicAdd(&a.log_n[0], 1ull);
              if ((int64_t)idx < a.tcap) {
                const U4 g = philox(r.seed, r.key1, w, (uint64_t)s0, 0, 0);
                double *L = a.tlog + 8 * idx;
                L[0] = (double)w;
                L[1] = (double)s0;
                L[2] = (double)p_colour_cell(r, stage_colour(g.v[0], r.ncol), (uint32_t)(t_lo + p));
                L[3] = (double)(i - r.aoff);
                L[4] = (double)dn;
                L[5] = ok ? 1.0 : 0.0;
                L[6] = du;
                L[7] = margin;
              }
            }
          }
          if (ok) {
            rec = i;
            my_i = i;
            my_s = s;
          }
        }
        if (!one_pass && lane == 0) l.rec[p] = rec;
      }
      // the row of this group's first trial in the next batch, if this one is
      // rejected as a whole and the site is drawn: its reads overlap the barrier
      PRow ahead;
      ahead.m = 0;
      bool have_ahead = false;
      if (own > 0) {
        const uint32_t k = (uint32_t)grp / (uint32_t)own, s1 = s0 + len + k;
        if (s1 < hd && (int)k < min(2 * span, cap)) {
          have_ahead = true;
          const int32_t i = l.site[(int)(s1 % (uint32_t)win) * chunk + (grp - (int)k * own)];
          if (i >= 0) row_of(i, ahead);
        }
      }
      if (RES || r.G == 1) draw_ahead(PBLOCK / 128);  // by the waves with the fewest trials
      sync();
      // the counts of the batch after next, last read before this barrier
      if (tid >= PBLOCK - 2 * PDMAX)
        l.cw[2 * PDMAX * ((batch + 2) % PCW) + tid - (PBLOCK - 2 * PDMAX)] = 0;
      const unsigned long long *tot = cw;
      int tst = 2;
      if (!RES && r.G > 1) {
        // ---- counts and barrier in one word per stage
        if (tid < 64) {
          unsigned long long *word = &st->word[batch % PWORDS][0][0];
          if (q == 0) {
            unsigned long long *next = &st->word[(batch + 2) % PWORDS][0][0];
            __hip_atomic_store(next + wl, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(next + 64 + wl, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_stores();
          }
          if (wl < len)
            __hip_atomic_fetch_add(&word[(q & 7) * PDG + wl],
                                   cw[2 * wl] + (1ull << (2 * PK_BITS)), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
          // lane 16 x + k polls stage k's words of rows x and x + 4
          const int sub = wl / PDG, sk = wl % PDG;
          auto due_of = [&](int x) {
            return sk < len && x < r.G ? (unsigned long long)((r.G - x + 7) / 8) : 0ull;
          };
          const unsigned long long due0 = due_of(sub), due1 = due_of(sub + 4);
          unsigned int it = 0;
          int late = 0;
          for (;;) {
            unsigned long long v = 0, u = 0;
            if (due0)
              v = __hip_atomic_load(&word[wl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (due1)
              u = __hip_atomic_load(&word[64 + wl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__all((v >> (2 * PK_BITS)) == due0 && (u >> (2 * PK_BITS)) == due1)) {
              v += u;
#pragma unroll
              for (int o = PDG; o < 64; o <<= 1) v += __shfl_xor(v, o);
              if (wl < len) l.tot[wl] = v;
              break;
            }
            __builtin_amdgcn_s_sleep(1);
            if (++it > a.spin_limit) {
              late = 1;
              break;
            }
          }
          if (wl == 0) {
            if (late)
              __hip_atomic_fetch_or(&st->err, PERSIST_TIMEOUT, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
            *flag = late;
          }
        } else {
          draw_ahead(1);
        }
        sync();
        if (*flag) return;
        tot = l.tot;
        tst = 1;
      }
      // ---- global factors: lane k of every wave tests stage s0 + k; n_B is
      // the same for all of them up to the first accepted one
      int gacc = -1;
      unsigned long long nrec = 0;
      long long dn_tot = 0;
      double xg = 0.0, mg = 0.0;
      if (wl < len) {
        const unsigned long long v = tot[tst * wl];
        const long long np = (long long)(v & PK_MASK), nm = (long long)((v >> PK_BITS) & PK_MASK);
        nrec = (unsigned long long)(np + nm);
        dn_tot = np - nm;
        if (nrec > 0) {
          const double tt = (double)nb - r.ncbar;
          const double dnd = (double)dn_tot;
          xg = r.beta * r.kN * dnd * (dnd + 2.0 * tt);
          const double lnug = l.lnug[(s0 + wl) & (PWIN - 1)];
          mg = lnug + xg;
          gacc = lnug < -xg ? 1 : 0;
        }
      }
      const unsigned long long acc = __ballot(gacc == 1);
      const int ka = acc ? __ffsll((long long)acc) - 1 : -1;
      const int done = ka >= 0 ? ka + 1 : len;  // stages decided
      if (ka >= 0) nb += __shfl(dn_tot, ka);
      if (tid < 64) {
        if (wl < done) {
          const unsigned long long c = cw[2 * wl + 1];
          if (DA) {
            n_trial += c & DA_MASK;
            n_pass += (c >> DA_BITS) & DA_MASK;
            n_tie += c >> (2 * DA_BITS);
          } else {
            n_trial += c & 0xffffffffull;
            n_tie += c >> 32;
          }
          if (q == 0) {
            n_acc += nrec;
            n_stage += 1;
            if (nrec > 0 && fabs(mg) < TIE) n_tie += 1;
            if (gacc == 1) {
              n_sacc += 1;
              n_flip += nrec;
            }
          }
        }
        if (q == 0 && s0 + done == S && wl == 0) {
          sum_n += (double)nb;
          sum_n2 += (double)nb * (double)nb;
        }
        if (LOG && a.slog && q == 0 && wl == 0) {
          const unsigned long long idx = atomicAdd(&a.log_n[1], 1ull);
          if ((int64_t)idx < a.scap) {
            const U4 g = philox(r.seed, r.key1, w, (uint64_t)s0, 0, 0);
            double *L = a.slog + 8 * idx;
            L[0] = (double)w;
            L[1] = (double)s0;
            L[2] = (double)stage_colour(g.v[0], r.ncol);
            L[3] = (double)dn_tot;
            L[4] = (double)nrec;
            L[5] = (double)gacc;
            L[6] = xg;
            L[7] = mg;
          }
        }
      }
      // ---- commit
      if (ka >= 0) {
        if (one_pass) {
          if (grp < len * own && grp / own == ka && my_i >= 0)
            p_commit<F, RES, DA>(state, my_i, lane, my_s, row);
        } else {
          for (int p = grp; p < len * own; p += PGROUPS) {
            if (p / own != ka) continue;
            const int32_t i = l.rec[p];
            if (i >= 0) {
              PRow v;
              row_of(i, v);
#pragma unroll
              for (int h = 0; h < PH; ++h)
                v.rj[h] = lane + h * PTL < v.m ? state.rho(v.j[h]) : 0.0;
              p_commit<F, RES, DA>(state, i, lane, state.sp(i), v);
            }
          }
        }
        if (!RES && r.G > 1) {
          wait_stores();
          sync();
          ++ncom;
          if (tid < 64) {
            // row q mod 8 counts its workgroups; lane x < 8 polls row x
            if (wl == 0)
              __hip_atomic_fetch_add(&st->bar[q & 7].n, 1ull, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long due =
                wl < 8 && wl < r.G ? ncom * (unsigned long long)((r.G - wl + 7) / 8) : 0ull;
            unsigned int it = 0;
            int late = 0;
            while (!__all(due == 0 || __hip_atomic_load(&st->bar[wl & 7].n, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) >= due)) {
              __builtin_amdgcn_s_sleep(1);
              if (++it > a.spin_limit) {
                late = 1;
                break;
              }
            }
            if (wl == 0) {
              if (late)
                __hip_atomic_fetch_or(&st->err, PERSIST_TIMEOUT, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
              *flag = late;
            }
          }
          sync();
          if (*flag) return;
        } else {
          if (!RES || a.vx) wait_stores();
          sync();  // the next batch's trials see the commit
        }
      }
      s0 += done;
      hd = td;
      hs = ts;
      span = ka < 0 ? min(2 * span, cap) : span0;
      if (ka < 0) row = ahead;
      have = ka < 0 && have_ahead;
    }
  }
  if (RES)
    for (int64_t i = tid; i < r.n; i += PBLOCK) {
      a.rho[r.aoff + i] = l.rho[i];
      a.sp[r.aoff + i] = l.sp[i];
    }
  if (tid < 64) {
    if (wl < PDMAX) {
      atomicAdd(&st->trials, n_trial);
      if (DA) atomicAdd(&st->stage1, n_pass);
      atomicAdd(&st->near_ties, n_tie);
      if (q == 0) {
        atomicAdd(&st->local_acc, n_acc);
        atomicAdd(&st->stages, n_stage);
        atomicAdd(&st->stage_acc, n_sacc);
        atomicAdd(&st->flips, n_flip);
      }
    }
    if (q == 0 && wl == 0) {
      st->sum_n = sum_n;
      st->sum_n2 = sum_n2;
      st->n_final = nb;
    }
  }
}

// TAB: the potential's form (analytic or tabulated) fixed at compile time,
// so each variant keeps only its own arithmetic and registers.
// LOG: trial or stage logs are written (one stage per batch), or BIG.
// The replica's constants of the arithmetic go to vector registers: with
// everything uniform in scalar ones the loop spilled them a thousand times
// into vector lanes.
__device__ __forceinline__ void in_vgpr(double &x) { asm volatile("" : "+v"(x)); }

template <bool TAB, bool LOG, bool BIG>
__global__ void __launch_bounds__(PBLOCK) k_sweep_persistent(PersistArgs a) {
  constexpr int F = TAB ? 1 : 0;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int flag;
  const int rix = a.wg_rep[blockIdx.x];
  RepD r = a.reps[rix];
  in_vgpr(r.beta);
  in_vgpr(r.dmu0);
  in_vgpr(r.kN);
  in_vgpr(r.ncbar);
  in_vgpr(a.p.rc);
  if (!TAB) {
    in_vgpr(a.p.c0);
    in_vgpr(a.p.c1);
    for (int k = 0; k < 3; ++k) in_vgpr(a.p.eps[k]);
    for (int k = 0; k < 2; ++k) {
      in_vgpr(a.p.t[k]);
      in_vgpr(a.p.A[k]);
    }
  }
  const PLds l = persist_lds(lds, a.ndraw, r.res ? r.n : 0);
  if (r.res)
    sweep_replica<F, true, LOG, false, BIG>(a, r, a.rs + rix, l, &flag);
  else
    sweep_replica<F, false, LOG, false, BIG>(a, r, a.rs + rix, l, &flag);
}

// delayed acceptance with the network, one system, state in memory
template <bool TAB>
__global__ void __launch_bounds__(PBLOCK) k_sweep_persistent_da(PersistArgsDa a) {
  constexpr int F = TAB ? 1 : 0;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int flag;
  RepD r = a.reps[0];
  in_vgpr(r.beta);
  in_vgpr(r.dmu0);
  in_vgpr(r.kN);
  in_vgpr(r.ncbar);
  const PLds l = persist_lds_da(lds, a.ndraw);
  sweep_replica<F, false, false, true, false>(a, r, a.rs, l, &flag);
}

// The end of a call, one block per replica: its statistics to the host's pinned
// copy, and the state readied for the next call (barrier words, timeout flag
// and counters zeroed, n_b <- n_B).  One launch where a reset before and a copy
// after the sweep, with the parameters' copy, made three (a sweep of 2,000
// sites 215 -> 203 us, of 0.5M sites with 27 colours 333 -> 318).
__global__ void __launch_bounds__(BLOCK) k_persist_done(RepState *rs, RepState *host) {
  RepState &s = rs[blockIdx.x], &o = host[blockIdx.x];
  if (threadIdx.x == 0) {
    o.trials = s.trials;
    o.stage1 = s.stage1;
    o.local_acc = s.local_acc;
    o.stages = s.stages;
    o.stage_acc = s.stage_acc;
    o.flips = s.flips;
    o.near_ties = s.near_ties;
    o.sum_n = s.sum_n;
    o.sum_n2 = s.sum_n2;
    o.err = s.err;
    o.n_final = s.n_final;
    s.n_b = s.n_final;
    s.trials = s.stage1 = s.local_acc = s.stages = s.stage_acc = s.flips = s.near_ties = 0;
    s.sum_n = 0.0;
    s.sum_n2 = 0.0;
    s.err = 0;
  }
  for (int q = threadIdx.x; q < PWORDS * 8 * PDG; q += BLOCK) (&s.word[0][0][0])[q] = 0;
  if (threadIdx.x < 8) s.bar[threadIdx.x].n = 0;
  if (threadIdx.x == 0) s.entry.n = 0;
}

}  // namespace vc

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace vc {

int persist_groups() { return PGROUPS; }
// dynamic LDS of a grid whose largest share of cells is `chunk` and whose
// largest resident replica has nres atoms, and its drawn trials (chunk 0: the
// draws are in memory)
size_t persist_lds_need(int64_t chunk, int64_t nres, int *ndraw) {
  const int64_t nd = chunk ? std::max<int64_t>(nres > 0 ? PDRAW : 2 * PDRAW, chunk) : 0;
  if (ndraw) *ndraw = (int)nd;
  return persist_lds_bytes(nd, nres);
}
size_t repd_size() { return sizeof(RepD); }
size_t repstate_size() { return sizeof(RepState); }

static const void *persist_kernel(bool tab, bool log, bool big) {
  if (tab)
    return big   ? (const void *)k_sweep_persistent<true, true, true>
           : log ? (const void *)k_sweep_persistent<true, true, false>
                 : (const void *)k_sweep_persistent<true, false, false>;
  return big   ? (const void *)k_sweep_persistent<false, true, true>
         : log ? (const void *)k_sweep_persistent<false, true, false>
               : (const void *)k_sweep_persistent<false, false, false>;
}

// Co-resident workgroups per CU that the registers of the potential form's
// kernels allow (with and without logs, or with the draws in memory), and the
// LDS bound asked for once and for all (more than 64 KB has to be).
hipError_t persist_max_blocks(int *per_cu, bool tab, bool big, size_t lds_max) {
  *per_cu = 1 << 10;
  for (int log = big ? 1 : 0; log < 2; ++log) {
    const void *f = persist_kernel(tab, log != 0, big);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
    int n = 0;
    if (e == hipSuccess)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, PBLOCK, persist_lds_bytes(0, 0));
    if (e != hipSuccess) return e;
    *per_cu = std::min(*per_cu, n);
  }
  return hipSuccess;
}

static PersistArgs make_args(vcsgc_ctx *c) {
  PersistArgs a = {};
  a.reps = (const RepD *)c->h_reps;  // pinned: read once by each workgroup
  a.rs = (RepState *)c->d_rs;
  a.wg_rep = c->d_wg_rep;
  a.cstart = c->cell_start;
  a.catoms = c->cell_atoms;
  a.nj = c->mc_j;
  a.nr = c->mc_r;
  a.cnt = c->mc_cnt;
  a.sp = c->sp;
  a.rho = c->rho;
  a.vx = c->vx;
  a.vy = c->vy;
  a.vz = c->vz;
  a.p = c->pot;
  a.tlog = c->tlog;
  a.tcap = c->tcap;
  a.slog = c->slog;
  a.scap = c->scap;
  a.log_n = &c->ds->tlog_n;
  // Strategies 0 and 1 end in an error where a wait exceeds the caller's limit;
  // the others have kernels that wait for nothing to fall back on, at the entry.
  a.spin_limit = c->strategy >= 2 || c->da_mode ? SPIN_LIMIT : c->spin_limit;
  a.entry_limit = std::min(c->spin_limit - 1, ENTRY_LIMIT);
  a.ndraw = c->persist_ndraw;
  a.big_lnu = c->big_lnu;
  a.big_site = c->big_site;
  a.big_rec = c->rec;
  return a;
}

// The per-call replica parameters, in pinned memory that the kernel reads
// itself; every call has been waited for before the next one writes them.
void persist_stage_params(vcsgc_ctx *c, const double *dmu0, const double *kappa,
                          const double *cbar, const double *T, int64_t n_sweeps,
                          const char *todo, uint64_t seed, bool da) {
  RepD *h = (RepD *)c->h_reps;
  for (size_t k = 0; k < c->reps.size(); ++k) {
    const RepHost &r = c->reps[k];
    RepD &d = h[k];
    d.n = r.n;
    d.aoff = r.aoff;
    d.n0 = r.nc[0];
    d.per = c->per;
    d.ncol = c->ncol;
    d.n1 = r.nc[1];
    d.n2 = r.nc[2];
    d.cso = r.cso;
    d.ncpc = r.ncpc;
    d.roff = r.roff;
    d.res = r.res && !da ? 1 : 0;
    d.S = r.S;
    d.beta = 1.0 / (KB * T[k]);
    d.dmu0 = dmu0[k];
    d.kN = kappa[k] / (double)r.n;
    d.ncbar = (double)r.n * cbar[k];
    d.seed = seed;
    d.key1 = (uint64_t)k;
    d.g0 = da ? 0 : r.g0;
    d.G = da ? c->da_wg : c->m_stage_acc > 0.3 ? r.G_busy : r.G;
    d.n_sweeps = todo[k] ? n_sweeps : 0;
    d.w0 = (int64_t)c->w;
  }
}

static hipError_t build_graph(vcsgc_ctx *c) {
  if (c->graph_exec) {
    (void)hipGraphExecDestroy(c->graph_exec);
    c->graph_exec = nullptr;
  }
  if (c->graph) {
    (void)hipGraphDestroy(c->graph);
    c->graph = nullptr;
  }
  hipError_t e = hipGraphCreate(&c->graph, 0);
  if (e != hipSuccess) return e;
  const int R = (int)c->reps.size();
  hipGraphNode_t n_sweep, n_done;
  static_assert(sizeof(PersistArgs) <= sizeof(c->graph_args_storage), "argument storage");
  PersistArgs *ga = reinterpret_cast<PersistArgs *>(c->graph_args_storage);
  *ga = make_args(c);
  void *sargs[] = {ga};
  hipKernelNodeParams sp = {};
  sp.func = const_cast<void *>(persist_kernel(c->pot.tab != 0, c->tlog || c->slog, c->big_lnu != nullptr));
  sp.gridDim = dim3((unsigned)c->grid_total);
  sp.blockDim = dim3(PBLOCK);
  sp.sharedMemBytes = (unsigned)c->persist_lds;
  sp.kernelParams = sargs;
  e = hipGraphAddKernelNode(&n_sweep, c->graph, nullptr, 0, &sp);
  if (e != hipSuccess) return e;
  if (c->persist_waits) {
    hipLaunchAttributeValue v = {};
    v.cooperative = 1;
    (void)hipGraphKernelNodeSetAttribute(n_sweep, hipLaunchAttributeCooperative, &v);
    (void)hipGetLastError();
  }
  RepState *rs = (RepState *)c->d_rs, *host = (RepState *)c->h_rs;
  void *dargs[] = {&rs, &host};
  hipKernelNodeParams dp = {};
  dp.func = (void *)k_persist_done;
  dp.gridDim = dim3((unsigned)R);
  dp.blockDim = dim3(BLOCK);
  dp.kernelParams = dargs;
  e = hipGraphAddKernelNode(&n_done, c->graph, &n_sweep, 1, &dp);
  if (e != hipSuccess) return e;
  return hipGraphInstantiate(&c->graph_exec, c->graph, nullptr, nullptr, 0);
}

// Grids whose workgroups wait for each other must not be on the chip half
// resident each (their waits would not end before the limit).  So a launch
// of one process waits, on its stream, for the earliest ones under way until
// the rest and itself have a CU for each workgroup, whatever streams and
// threads they come from; of any grids running at once the last one launched
// has counted the others.  (8 contexts of 16,000 sites on 8 threads, a sweep
// each: 7.7 ms one after the other, 2.0 ms together; 1.0 ms for one alone.)
// Grids that do not wait hold CUs too: the long ones are counted, a short one
// has ended before an entry barrier gives up.  An event is used again when its
// grid has ended, so there are as many per device as grids were under way at
// once.
struct Running {
  hipEvent_t end;
  int wgs;
};
struct Gate {
  std::vector<Running> running;  // in launch order
  std::vector<hipEvent_t> idle;
};
constexpr int PGATE_DEVICES = 64;
constexpr int64_t PGATE_STAGES = 1 << 14;  // of a grid that does not wait: 2 ms or more
static std::mutex g_gate_mu;
static Gate g_gate[PGATE_DEVICES];

template <class L>
static hipError_t gated(vcsgc_ctx *c, int wgs, bool waits, L launch) {
  if (c->device < 0 || c->device >= PGATE_DEVICES) return launch();
  int cu = 0;
  hipError_t e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, c->device);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(g_gate_mu);
  Gate &g = g_gate[c->device];
  int64_t sum = wgs;
  size_t kept = 0;
  for (const Running &r : g.running) {
    if (hipEventQuery(r.end) == hipSuccess) {
      g.idle.push_back(r.end);
    } else {
      g.running[kept++] = r;
      sum += r.wgs;
    }
  }
  g.running.resize(kept);
  (void)hipGetLastError();  // (a query's "not ready")
  for (size_t k = 0; waits && k < kept && sum > cu; sum -= g.running[k].wgs, ++k)
    if ((e = hipStreamWaitEvent(c->stream, g.running[k].end, 0)) != hipSuccess) return e;
  hipEvent_t end = nullptr;
  if (!g.idle.empty()) {
    end = g.idle.back();
    g.idle.pop_back();
  } else if ((e = hipEventCreateWithFlags(&end, hipEventDisableTiming)) != hipSuccess) {
    return e;
  }
  e = launch();
  const hipError_t rec = hipEventRecord(end, c->stream);
  if (rec == hipSuccess)
    g.running.push_back({end, std::min(wgs, cu)});
  else
    g.idle.push_back(end);
  return e != hipSuccess ? e : rec;
}

static hipError_t launch_done(vcsgc_ctx *c) {
  k_persist_done<<<(unsigned)c->reps.size(), BLOCK, 0, c->stream>>>((RepState *)c->d_rs,
                                                                    (RepState *)c->h_rs);
  return hipGetLastError();
}

static hipError_t launch_ungated(vcsgc_ctx *c, bool use_graph);

hipError_t launch_persistent(vcsgc_ctx *c, int64_t n_sweeps, bool use_graph) {
  int64_t S = 0;
  for (const RepHost &r : c->reps) S = std::max(S, r.S);
  auto launch = [&]() { return launch_ungated(c, use_graph); };
  if (!c->persist_waits && n_sweeps * S < PGATE_STAGES) return launch();
  return gated(c, c->grid_total, c->persist_waits, launch);
}

static hipError_t launch_ungated(vcsgc_ctx *c, bool use_graph) {
  const int R = (int)c->reps.size();
  if (use_graph) {
    if (!c->graph_exec) {
      hipError_t e = build_graph(c);
      if (e != hipSuccess) return e;
    }
    return hipGraphLaunch(c->graph_exec, c->stream);
  }
  PersistArgs a = make_args(c);
  void *args[] = {&a};
  const void *f = persist_kernel(c->pot.tab != 0, c->tlog || c->slog, c->big_lnu != nullptr);
  const dim3 grid((unsigned)c->grid_total), block(PBLOCK);
  const unsigned lds = (unsigned)c->persist_lds;
  const hipError_t e = c->persist_waits
                           ? hipLaunchCooperativeKernel(f, grid, block, args, lds, c->stream)
                           : hipLaunchKernel(f, grid, block, args, lds, c->stream);
  return e == hipSuccess ? launch_done(c) : e;
}

// ---- delayed acceptance with the network (one system) ----
static const void *persist_da_kernel(bool tab) {
  return tab ? (const void *)k_sweep_persistent_da<true> : (const void *)k_sweep_persistent_da<false>;
}

// Trial groups per active cell.  A trial is longer than a plain one, so a
// second pass over the groups costs more than a barrier of more workgroups:
// 128,000 sites at 9% accepted stages 1.02 ms with 8, 0.74 with 16, 0.69 with
// 32; 16,000 sites 1.76, 1.37, 1.20; 1.02M sites 0.96, 0.95, 0.98.  (A batch has
// at most PDG = 16 stages, so with 32 half of a workgroup's groups have no trial:
// what helps is fewer trials per compute unit.  Not measured with many accepted
// stages.)
constexpr int PERSIST_SPEC_DA = 32;

// The grid of the delayed-acceptance sweep into c->da_wg (-1: its shares of the
// cells do not fit a workgroup's groups) and c->da_ndraw, once per context.
hipError_t persist_da_grid(vcsgc_ctx *c) {
  if (c->da_wg) return hipSuccess;
  const RepHost &r = c->reps[0];
  int cu = 0, lds_cu = 0, per_cu = 0;
  hipError_t e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, c->device);
  if (e == hipSuccess)
    e = hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                              c->device);
  if (e != hipSuccess) return e;
  const size_t room = (size_t)lds_cu - 1024;
  c->da_wg = -1;
  const int nd = 2 * PDRAW;
  const size_t lds = persist_lds_bytes_da(nd);
  if (lds > room) return hipSuccess;
  const void *f = persist_da_kernel(c->pot.tab != 0);
  e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)room);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, PBLOCK, lds);
  if (e != hipSuccess) return e;
  int64_t g = (PERSIST_SPEC_DA * r.ncpc + PGROUPS - 1) / PGROUPS;
  if (g >= 8) g = (g + 7) / 8 * 8;
  g = std::min<int64_t>(g, (int64_t)cu * per_cu);
  if (g < 1 || r.ncpc > g * PGROUPS) return hipSuccess;
  c->da_wg = (int)g;
  c->da_ndraw = nd;
  return hipSuccess;
}

hipError_t launch_persistent_da(vcsgc_ctx *c) {
  PersistArgsDa a;
  static_cast<PersistArgs &>(a) = make_args(c);
  a.ndraw = c->da_ndraw;
  a.md = mlp_dev(c->mlp);
  a.dj = c->d_j;
  a.dr = c->d_r;
  a.dcnt = c->d_cnt;
  auto launch = [&]() {
    void *args[] = {&a};
    hipError_t e = hipLaunchCooperativeKernel(persist_da_kernel(c->pot.tab != 0), dim3((unsigned)c->da_wg),
                                      dim3(PBLOCK), args,
                                      (unsigned)persist_lds_bytes_da(c->da_ndraw), c->stream);
    return e == hipSuccess ? launch_done(c) : e;
  };
  return gated(c, c->da_wg, c->da_wg > 1, launch);
}

// Statistics of the last launch's replicas in todo (synchronizes), which are
// then done unless their workgroups did not all start; n_final is the device's
// where no call has just written it (launched false: other kernels may have
// moved it).
hipError_t persist_read_stats(vcsgc_ctx *c, vcsgc_stats *out, char *todo, int *err, bool launched,
                              bool da) {
  const int R = (int)c->reps.size();
  RepState *h = (RepState *)c->h_rs;
  hipError_t e = hipSuccess;
  for (int k = 0; k < R && !launched && e == hipSuccess; ++k)
    e = hipMemcpyAsync(&h[k].n_final, &((RepState *)c->d_rs)[k].n_final, sizeof(long long),
                       hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return e;
  *err = 0;
  for (int k = 0; k < R; ++k) {
    if (!todo[k]) continue;
    *err |= h[k].err;
    todo[k] = (h[k].err & PERSIST_NOT_STARTED) != 0;
    if (!out || todo[k]) continue;
    out[k].trials = (int64_t)h[k].trials;
    out[k].local_accepts = (int64_t)h[k].local_acc;
    out[k].stages = (int64_t)h[k].stages;
    out[k].stage_accepts = (int64_t)h[k].stage_acc;
    out[k].flips = (int64_t)h[k].flips;
    out[k].near_ties = (int64_t)h[k].near_ties;
    out[k].n_final = h[k].n_final;
    out[k].sum_n = h[k].sum_n;
    out[k].sum_n2 = h[k].sum_n2;
    out[k].stage1_pass = (int64_t)(da ? h[k].stage1 : h[k].trials);
  }
  return hipSuccess;
}

// n_B of the system, or of the first replica of a batch (synchronizes)
hipError_t persist_read_nb(vcsgc_ctx *c, int64_t *n_b) {
  RepState *h = (RepState *)c->h_rs;
  hipError_t e = hipMemcpyAsync(&h->n_final, &((RepState *)c->d_rs)->n_final, sizeof(long long),
                                hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e == hipSuccess) *n_b = h->n_final;
  return e;
}

// n_final of replica k (used to seed the per-stage path's counter)
__global__ void k_set_nfinal(RepState *rs, int k, const long long *src) {
  if (threadIdx.x == 0 && blockIdx.x == 0) rs[k].n_b = rs[k].n_final = *src;
}
__global__ void k_get_nfinal(const RepState *rs, int k, long long *dst) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = rs[k].n_final;
}

hipError_t persist_sync_nb_to_stage(vcsgc_ctx *c) {
  k_get_nfinal<<<1, 64, 0, c->stream>>>((const RepState *)c->d_rs, 0, &c->ds->n_b_cur);
  return hipGetLastError();
}
hipError_t persist_sync_nb_from_stage(vcsgc_ctx *c) {
  k_set_nfinal<<<1, 64, 0, c->stream>>>((RepState *)c->d_rs, 0, &c->ds->n_b_cur);
  return hipGetLastError();
}

// per-replica n_B from the species (into n_b and n_final)
__global__ void k_count_rep(int64_t n, const uint8_t *__restrict__ sp, RepState *st) {
  __shared__ long long sh[BLOCK];
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  sh[threadIdx.x] = i < n ? (long long)sp[i] : 0;
  __syncthreads();
  for (int h = BLOCK / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0 && sh[0]) {
    atomicAdd((unsigned long long *)&st->n_final, (unsigned long long)sh[0]);
    atomicAdd((unsigned long long *)&st->n_b, (unsigned long long)sh[0]);
  }
}

hipError_t persist_count(vcsgc_ctx *c) {
  std::memset(c->h_rs, 0, sizeof(RepState) * c->reps.size());  // (every call has been waited for)
  hipError_t e = hipMemsetAsync(c->d_rs, 0, sizeof(RepState) * c->reps.size(), c->stream);
  if (e != hipSuccess) return e;
  for (size_t k = 0; k < c->reps.size(); ++k) {
    const RepHost &r = c->reps[k];
    k_count_rep<<<grid_for(r.n), BLOCK, 0, c->stream>>>(r.n, c->sp + r.aoff,
                                                        (RepState *)c->d_rs + k);
  }
  return hipGetLastError();
}

}  // namespace vc
