// Hand-written HIP kernels of the multislice Leiden path (gfx950, wave64, no MFMA: every
// step is a scan, a gather or a hash update, bounded by HBM bandwidth).
//
// Units are supra-nodes at level 0 and super-nodes at later levels.  Several independent
// solves can share one launch as a disjoint union: each unit knows its solve (coefficients,
// priority seed, local id offset) and its slices are global slice ids, so nothing here
// ever compares quantities of two different solves.
#pragma once
#include <type_traits>
#include <math.h>

#include "device.hpp"

namespace mslm {

typedef __int128 i128;

// Barrier for one workgroup that also makes global writes of every wave visible to the
// others: release before the barrier, and drop possibly stale vector-L1 lines after it
// (Sigma-table atomics are performed in L2).
__device__ inline void block_sync_global() {
  __threadfence();
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// ------------------------------------------------------------------ per-solve constants
struct SolveDev {
  const int64_t *p, *q, *pb, *a, *b;   // gamma = p/q, omega = a/b (reduced), pb = p*b
  const uint64_t *seedmix;             // mix64(seed)
  const int64_t *uoff;                 // first unit of the solve at the current level
  const int32_t *sfirst;               // first global slice of the solve
  const int64_t *S;                    // per global slice: 2m_s, or 1 for an empty slice
  // doubles of the multi-slice estimates: values are scaled by L, the least common multiple of the
  // solve's S when it is below 2^53 (else 1).  rS: per global slice a -> a * L / S; scale: per solve
  // L, then from index J on the bound below which a scaled value is exact (2^53, or 0 when L is not
  // used)
  const SliceRecip *rS;
  const double *scale;
  int J;
  int64_t *fallbacks;                  // exact-comparison counter per solve
  // per solve: the smallest mark of a near-tie that a kernel without the big-integer path could
  // not settle (kRedoUnset: none).  Refinement marks 0; a window of colours marks the unit's
  // colour, so that only the colours whose decisions count ask for a repeat
  int32_t *redo;
  // during local-moving sweeps: solves that take no part in the sweep (stopped, or not being
  // taken again); their units are not decided (their moves would not be applied); else nullptr
  const uint8_t *frozen;
  // a sweep replayed from a HIP graph reads the base of its fresh labels here (its launches
  // were captured once); nullptr: the base passed to the kernel
  const uint32_t *fresh;
  int32_t mark = 0;                    // what a near-tie writes into redo
  // sweeps that keep track of units at rest (Rest), else nullptr; the counters they are measured
  // against: per Sigma slice the degree moved, then from index nsl on per solve the degree moved
  // over the slices' totals in units of 2^-32, summed over the slices
  struct Rest *rest = nullptr;
  int64_t *ctr = nullptr;
  int nsl = 0;
};
constexpr int kRedoByte = 0x7f;
constexpr int32_t kRedoUnset = 0x7f7f7f7f;   // four equal bytes: set by a byte fill

// A unit at rest.  A unit that stays is compared with its best target by q*W - p*b*sum_s k_s y_s/S_s,
// and of this only the y (Sigma values) change while none of its neighbours moves: a target's y_s
// falls and the own community's rises by at most the slice-s degree that moves anywhere.  So with
// `slack` between staying and the best target the unit goes on staying while
// 2 p b k dM <= slack, dM the degree moved in its slice since (or, spanning several slices,
// 2 p b max_s(k_s) sum_s dM_s / S_s <= slack); targets that were pruned by q*W alone stay below the
// best of that time.  That holds while the counter is below `limit`; a neighbour's move sets it to
// 0.  Skipping such units changes no decision.
//
// A counter stays below 2^64: a sweep moves a unit at most once, so per sweep a slice's counter
// grows by at most its total (below 2^31) and a solve's by at most 2^32 per snapshot, or per copy
// under the CPM (S = 1), and 1 per profile entry for rounding up; snapshots, copies and entries are
// each no more than the units of level 0, and those times the sweeps stay below 2^32.
struct Rest {
  uint64_t limit;
  int32_t ctr;    // the counter: the unit's Sigma slice, or nsl + solve
  int32_t pad;
};
__device__ inline bool at_rest(const SolveDev &sd, int64_t v) {
  if (!sd.rest) return false;
  const Rest r = sd.rest[v];
  return (uint64_t)sd.ctr[r.ctr] < r.limit;
}

__device__ inline uint32_t fresh_of(const SolveDev &sd, uint32_t fresh_base) {
  return sd.fresh ? *sd.fresh : fresh_base;
}

// ------------------------------------------------------------------ level views
// Level 0: the supra-CSR of Eq. 3 with raw weights; an entry whose column lies outside the
// unit's slice is a coupling entry of raw weight c_sr and scaled weight a * c_sr (absent when
// a == 0).
struct View0 {
  static constexpr bool kLevel0 = true;
  const int64_t *rp;
  const int32_t *col;
  const int32_t *w;        // raw weight per entry (intra w, coupling c_sr), or nullptr: all 1
  // degree in the null model of the unit's solve: the intra degree k_i^s (Eq. 6), or the
  // scaled supra-degree b*k_i^s + a*(coupling entries of the unit) (the global null model)
  const int32_t *k;
  const int32_t *uslice;   // global slice of each unit
  const int64_t *sstart;   // [slices + 1] first unit of each global slice
  const int32_t *usolve;   // solve of each unit
  // Sigma slice of each global slice (nullptr: the slice itself); a solve under the global
  // null model maps all its slices to one Sigma slice
  const int32_t *pmap;
  const int32_t *rev;      // per entry (u, x): offset of (x, u) within x's row
  int64_t N1 = 0;          // one solve: nodes per slice (slice and solve follow from the id)
  double invN1 = 0.0;      // 1 / N1
  struct Row {
    int64_t lo, hi, slo, shi, a, b;
  };
  // slice of unit v: v / N1 for one solve (a double estimate corrected by one step either
  // way, exact for every v < 2^32), else the stored slice
  __device__ int slice_of(int64_t v) const {
    if (N1 == 0) return uslice[v];
    int64_t q = (int64_t)((double)v * invN1);
    if (q * N1 > v) q--;
    else if ((q + 1) * N1 <= v) q++;
    return (int)q;
  }
  __device__ int solve_of(int64_t v) const { return N1 ? 0 : usolve[v]; }
  __device__ Row row(int64_t v, const SolveDev &sd) const {
    const int gs = slice_of(v);
    const int j = solve_of(v);
    const int64_t slo = N1 ? (int64_t)gs * N1 : sstart[gs];
    const int64_t shi = N1 ? slo + N1 : sstart[gs + 1];
    return Row{rp[v], rp[v + 1], slo, shi, sd.a[j], sd.b[j]};
  }
  __device__ int64_t wt(const Row &r, int64_t e, int32_t x) const {
    return (x >= r.slo && x < r.shi ? r.b : r.a) * (w ? (int64_t)w[e] : 1);
  }
  // whether an entry of this column has weight (raw weights are never 0, omega may be)
  __device__ bool live(const Row &r, int32_t x) const {
    return (x >= r.slo && x < r.shi ? r.b : r.a) != 0;
  }
  // neighbour of entry e and its scaled weight
  __device__ int64_t nbr(const Row &r, int64_t e, int64_t &ww) const {
    const int32_t x = col[e];
    ww = wt(r, e, x);
    return x;
  }
  __device__ int64_t orig(int64_t v) const { return v; }
  __device__ uint32_t lab_at(const uint32_t *comm, int64_t, int64_t x) const { return comm[x]; }
  __device__ int plen(int64_t v) const { return k[v] > 0 ? 1 : 0; }
  __device__ void pent(int64_t v, int, int &gs, int64_t &kk) const {
    gs = slice_of(v);
    if (pmap) gs = pmap[gs];
    kk = k[v];
  }
  __device__ int64_t degree(int64_t v) const { return rp[v + 1] - rp[v]; }
};

// Level 0 in colour-batch order, for the local-moving sweeps: the level's units are stored in
// the order of their colour batches (colour, degree bin, id), so a batch is one contiguous
// range of positions whose rows, degrees, slices and labels are read in sequence; only the
// neighbours' labels and the Sigma probes stay random.  Entries hold neighbour positions,
// with bit 31 set on the coupling entries (scaled weight a); labels and priorities keep the
// unit ids (orig), so every decision is the one the id-ordered level makes.
struct ViewP {
  static constexpr bool kLevel0 = true;
  const int64_t *rp;       // [n+1] rows by position
  const int32_t *col;      // neighbour position | coupling << 31
  const int32_t *w;        // raw intra weight per entry, or nullptr for unit weights
  const int32_t *k;        // null-model degree by position (View0::k)
  const int32_t *slice;    // Sigma slice by position
  const int32_t *solve;    // solve by position, or nullptr (one solve)
  const int32_t *uid;      // unit id by position
  // per entry, the neighbour's current label (kept up to date by the moves: a moved unit
  // writes its new label into the entries that point at it, found through prev), so the
  // decisions read labels in entry order instead of gathering them; nullptr: gather
  uint32_t *elab;
  const int32_t *prev;     // per entry (i, x): index of the entry (x, i)
  int64_t nnz;             // entries (host use)
  struct Row {
    int64_t lo, hi, a, b;
  };
  __device__ int solve_of(int64_t i) const { return solve ? solve[i] : 0; }
  __device__ Row row(int64_t i, const SolveDev &sd) const {
    const int j = solve_of(i);
    return Row{rp[i], rp[i + 1], sd.a[j], sd.b[j]};
  }
  __device__ int64_t nbr(const Row &r, int64_t e, int64_t &ww) const {
    const int32_t raw = col[e];
    ww = (raw < 0 ? r.a : r.b) * (w ? (int64_t)w[e] : 1);
    return raw & 0x7fffffff;
  }
  __device__ int64_t orig(int64_t i) const { return uid[i]; }
  __device__ int64_t unit_at(const int32_t *, int64_t pos) const { return pos; }
  __device__ uint32_t lab_at(const uint32_t *comm, int64_t e, int64_t x) const {
    return elab ? elab[e] : comm[x];
  }
  __device__ int plen(int64_t i) const { return k[i] > 0 ? 1 : 0; }
  __device__ void pent(int64_t i, int, int &gs, int64_t &kk) const {
    gs = slice[i];
    kk = k[i];
  }
  __device__ int64_t degree(int64_t i) const { return rp[i + 1] - rp[i]; }
};

// Aggregated levels: scaled int64 weights, per-unit slice profiles (global slice, degree).
struct ViewK {
  static constexpr bool kLevel0 = false;
  const int64_t *rp;
  const int32_t *col;
  const int64_t *w;
  const int64_t *pp;
  const int32_t *ps;
  const int32_t *pk;
  const int32_t *usolve;
  struct Row {
    int64_t lo, hi;
  };
  __device__ Row row(int64_t v, const SolveDev &) const { return Row{rp[v], rp[v + 1]}; }
  __device__ int64_t wt(const Row &, int64_t e, int32_t) const { return w[e]; }
  __device__ bool live(const Row &, int32_t) const { return true; }   // aggregated: always > 0
  __device__ int64_t nbr(const Row &, int64_t e, int64_t &ww) const {
    ww = w[e];
    return col[e];
  }
  __device__ int64_t orig(int64_t v) const { return v; }
  __device__ int64_t unit_at(const int32_t *units, int64_t pos) const { return units[pos]; }
  __device__ uint32_t lab_at(const uint32_t *comm, int64_t, int64_t x) const { return comm[x]; }
  __device__ int solve_of(int64_t v) const { return usolve[v]; }
  __device__ int plen(int64_t v) const { return (int)(pp[v + 1] - pp[v]); }
  __device__ void pent(int64_t v, int j, int &gs, int64_t &kk) const {
    gs = ps[pp[v] + j];
    kk = pk[pp[v] + j];
  }
  __device__ int64_t degree(int64_t v) const { return rp[v + 1] - rp[v]; }
};

// ------------------------------------------------------------------ gains
// Targets: a community label, the empty community (label kNone, gain 0), or "stay" (the
// unit's own community without itself).  The value compared for unit v and target X is
//     q*W_X - p*b * sum_s k_{v,s} * y_{X,s} / S_s
// (W_X the scaled edge weight from v to X, y_{X,s} the slice-s degree of X), which orders
// targets exactly as the change of Q in Eq. 6 does (a positive multiple of it).
enum { kTarget = 0, kEmpty = 1, kStay = 2 };

struct UnitCtx {
  int64_t v;
  int j;
  uint32_t D;
  int m;          // profile length
  int gs0;        // first profile slice
  int64_t k0;     // first profile degree
  int64_t p, q, pb, S0;
  double scale, lim;   // of the multi-slice estimates (SolveDev)
  mutable bool tied = false;   // this lane met a near-tie that it could not settle
};

template <class V>
__device__ inline UnitCtx unit_ctx(const V &g, const SolveDev &sd, int64_t v, uint32_t D) {
  UnitCtx u;
  u.v = v;
  u.j = g.solve_of(v);
  u.D = D;
  u.m = g.plen(v);
  u.gs0 = 0;
  u.k0 = 0;
  if (u.m > 0) g.pent(v, 0, u.gs0, u.k0);
  u.p = sd.p[u.j];
  u.q = sd.q[u.j];
  u.pb = sd.pb[u.j];
  u.S0 = u.m > 0 ? sd.S[u.gs0] : 1;
  u.scale = sd.scale[u.j];
  u.lim = sd.scale[sd.J + u.j];
  return u;
}

// Record how long unit v (decided `out`, one thread) stays at rest; kmax: its largest profile
// degree when it spans several slices.  Rounded down by 2^-30, far above the rounding of the
// doubles involved.  tied: a comparison of the unit was left to the exact kernels, so its best
// target may not be the best ("the heavier one" of a near-tie is no order: over several targets it
// leads any number of steps down); such a unit is not at rest.
__device__ inline void settle(const SolveDev &sd, const UnitCtx &u, uint32_t out, double slack,
                              double kmax, bool tied) {
  if (!sd.rest) return;
  Rest r{0, 0, 0};
  if (out == kNone && slack >= 0.0 && !tied) {
    const bool one = u.m <= 1;
    r.ctr = one ? (u.m ? u.gs0 : 0) : sd.nsl + u.j;
    const double den = 2.0 * (double)u.pb * (one ? (double)u.k0 : kmax);
    if (den == 0.0) {
      r.limit = ~0ull;
    } else {
      const double room = slack / den * (one ? 1.0 : 0x1p32) * (1.0 - 0x1p-30);
      const uint64_t now = (uint64_t)sd.ctr[r.ctr], left = ~0ull - now - 1;
      const uint64_t more = (uint64_t)(room < 0x1p61 ? room : 0x1p61);
      r.limit = now + 1 + (more < left ? more : left);
    }
  }
  sd.rest[u.v] = r;
}

__device__ inline int64_t target_y(const SliceTable &tab, int gs, int64_t k, uint32_t lab, int kind) {
  if (kind == kEmpty) return 0;
  int64_t y = tab_get(tab, gs, lab);
  return kind == kStay ? y - k : y;
}

// Level 0: one slice per unit; exact in int64 under the checked head-room precondition.
struct Score0 {
  int64_t g;
  uint32_t lab;
};

struct Policy0 {
  typedef Score0 Score;
  template <class V>
  __device__ static Score make(const V &, const UnitCtx &u, const SolveDev &, const SliceTable &tab,
                               uint32_t lab, int64_t W, int kind) {
    Score s;
    s.lab = kind == kEmpty ? kNone : lab;
    if (u.m == 0) {
      s.g = u.q * W;
    } else {
      int64_t y = target_y(tab, u.gs0, u.k0, lab, kind);
      s.g = u.q * u.S0 * W - u.pb * (u.k0 * y);
    }
    return s;
  }
  template <class V>
  __device__ static int cmp(const V &, const UnitCtx &, const SolveDev &, const SliceTable &,
                            const Score &a, const Score &b) {
    return a.g < b.g ? -1 : (a.g > b.g ? 1 : 0);
  }
  // the null term is never negative, so q*S*W bounds a target's value from above; a target
  // whose bound is strictly below the best value so far can neither win nor tie
  __device__ static bool prunable(const UnitCtx &u, int64_t W, const Score &best) {
    int64_t ub = u.m == 0 ? u.q * W : u.q * u.S0 * W;
    return ub < best.g;
  }
  __device__ static Score shfl(const Score &s, int m) {
    Score o;
    o.g = shfl_xor64(s.g, m);
    o.lab = shfl_xor32(s.lab, m);
    return o;
  }
  // how far staying is ahead of the best target (never above the true difference by more than
  // rounding, which settle() allows for)
  __device__ static double slack(const UnitCtx &, const Score &stay, const Score &best) {
    return (double)(stay.g - best.g);
  }
  // the score of staying when the Sigma of the unit's own community is already known
  __device__ static Score stay_from(const UnitCtx &u, uint32_t D, int64_t W, int64_t yD) {
    Score s;
    s.lab = D;
    s.g = u.m == 0 ? u.q * W : u.q * u.S0 * W - u.pb * (u.k0 * (yD - u.k0));
    return s;
  }
};

// Aggregated levels: int128 when the unit lies in one slice, otherwise a double estimate
// with a rigorous error bound and an exact big-integer evaluation when the estimates of
// two targets are too close to order.
struct ScoreK {
  i128 ex;
  double ap, er;
  int64_t W;
  uint32_t lab;
  int kind;   // kTarget / kEmpty / kStay; +4 when the value has no null term (it is q*W)
};

template <class V>
__device__ __noinline__ int exact_big(const V &g, const UnitCtx &u, const SolveDev &sd,
                                      const SliceTable &tab, uint32_t la, int ka, int64_t Wa,
                                      uint32_t lb, int kb, int64_t Wb) {
  atomicAdd(reinterpret_cast<unsigned long long *>(sd.fallbacks + u.j), 1ull);
  ExactAcc acc;
  acc.init();
  for (int jj = 0; jj < u.m; jj++) {
    int gs;
    int64_t k;
    g.pent(u.v, jj, gs, k);
    int64_t ya = target_y(tab, gs, k, la, ka);
    int64_t yb = target_y(tab, gs, k, lb, kb);
    acc.term(k * (ya - yb), sd.S[gs]);
  }
  return acc.sign(u.q, Wa - Wb, u.pb);
}

// Exact order of two targets whose estimates cannot be told apart.  Equal per-slice terms
// (the usual case: both targets hold the same Sigma in every slice of the unit) are settled
// here, inline; only a genuine near-tie calls the out-of-line big-integer evaluation (a call
// spills the caller's registers, so it must stay off the common path).
template <class V>
__device__ inline int exact_cmp(const V &g, const UnitCtx &u, const SolveDev &sd,
                                const SliceTable &tab, uint32_t la, int ka, int64_t Wa,
                                uint32_t lb, int kb, int64_t Wb) {
  bool same = true;
  for (int jj = 0; jj < u.m && same; jj++) {
    int gs;
    int64_t k;
    g.pent(u.v, jj, gs, k);
    same = target_y(tab, gs, k, la, ka) == target_y(tab, gs, k, lb, kb);
  }
  if (same) return Wa > Wb ? 1 : (Wa < Wb ? -1 : 0);
  return exact_big(g, u, sd, tab, la, ka, Wa, lb, kb, Wb);
}

// The same order for the sweeps that run without the big-integer path (it needs per-lane
// scratch memory, which slows every launch of a kernel that contains it): equal per-slice
// terms are settled here as well; a genuine near-tie raises its solve's redo flag and gets a
// provisional answer, and the host takes that solve's sweep again with the exact kernels.
template <class V>
__device__ inline int exact_cmp_flag(const V &g, const UnitCtx &u, const SolveDev &sd,
                                     const SliceTable &tab, uint32_t la, int ka, int64_t Wa,
                                     uint32_t lb, int kb, int64_t Wb) {
  bool same = true;
  for (int jj = 0; jj < u.m && same; jj++) {
    int gs;
    int64_t k;
    g.pent(u.v, jj, gs, k);
    same = target_y(tab, gs, k, la, ka) == target_y(tab, gs, k, lb, kb);
  }
  if (!same) {
    atomicMin(sd.redo + u.j, sd.mark);
    u.tied = true;
  }
  return Wa > Wb ? 1 : (Wa < Wb ? -1 : 0);
}

// Exact: near-ties go to the big-integer evaluation; otherwise they raise the redo flag.
template <bool Exact>
struct PolicyKT {
  typedef ScoreK Score;
  template <class V>
  __device__ static Score make(const V &g, const UnitCtx &u, const SolveDev &sd,
                               const SliceTable &tab, uint32_t lab, int64_t W, int kind) {
    Score s;
    s.lab = kind == kEmpty ? kNone : lab;
    s.kind = kind;
    s.W = W;
    s.ex = 0;
    s.ap = 0;
    s.er = 0;
    if (u.m <= 1) {
      i128 val = (i128)u.q * W;
      if (u.m == 1) {
        int64_t y = target_y(tab, u.gs0, u.k0, lab, kind);
        val = val * u.S0 - (i128)u.pb * (i128)(u.k0 * y);
      }
      s.ex = val;
    } else if (kind == kEmpty) {
      // every null term of the empty community is 0: the value is q*W, no slice to visit
      finish(u, W, 0.0, 0.0, s);
    } else {
      double acc = 0.0, mag = 0.0;
      for (int jj = 0; jj < u.m; jj++) {
        int gs;
        int64_t k;
        g.pent(u.v, jj, gs, k);
        int64_t y = target_y(tab, gs, k, lab, kind);
        double t = sd.rS[gs].of((double)(k * y));
        acc += t;
        mag += fabs(t);
      }
      finish(u, W, acc, mag, s);
    }
    return s;
  }
  // estimate and error bound from the summed null terms (any summation order).  With the solve's
  // common denominator every operand and partial sum is an integer, and no larger than `all`:
  // below 2^53 nothing was rounded.
  __device__ static void finish(const UnitCtx &u, int64_t W, double acc, double mag, Score &s) {
    const double qw = (double)u.q * (double)W * u.scale;
    const double all = fabs(qw) + (double)u.pb * mag;
    s.ap = qw - (double)u.pb * acc;
    s.er = all < u.lim ? 0.0 : (double)(u.m + 8) * 0x1p-50 * all;
    if (mag == 0.0 || u.pb == 0) s.kind |= 4;
  }
  template <class V>
  __device__ static int cmp(const V &g, const UnitCtx &u, const SolveDev &sd, const SliceTable &tab,
                            const Score &a, const Score &b) {
    if (u.m <= 1) return a.ex < b.ex ? -1 : (a.ex > b.ex ? 1 : 0);
    if (a.lab == b.lab && a.kind == b.kind && a.W == b.W) return 0;   // the same target
    if ((a.kind & 4) && (b.kind & 4)) return a.W < b.W ? -1 : (a.W > b.W ? 1 : 0);   // both q*W
    double d = a.ap - b.ap;
    if (fabs(d) > 2.0 * (a.er + b.er)) return d > 0 ? 1 : -1;
    if (a.er + b.er == 0.0) return 0;   // both exact
    if constexpr (Exact)
      return exact_cmp(g, u, sd, tab, a.lab, a.kind & 3, a.W, b.lab, b.kind & 3, b.W);
    else
      return exact_cmp_flag(g, u, sd, tab, a.lab, a.kind & 3, a.W, b.lab, b.kind & 3, b.W);
  }
  __device__ static double slack(const UnitCtx &u, const Score &stay, const Score &best) {
    if (u.m <= 1) return (double)(stay.ex - best.ex);
    return ((stay.ap - stay.er) - (best.ap + best.er)) / u.scale;
  }
  __device__ static bool prunable(const UnitCtx &u, int64_t W, const Score &best) {
    if (u.m <= 1) {
      i128 ub = (i128)u.q * W * (u.m ? u.S0 : 1);
      return ub < best.ex;
    }
    // q*W rounded up versus a rigorous lower bound of the best value
    double ub = (double)u.q * (double)W * u.scale * (1.0 + 0x1p-48);
    return ub < best.ap - best.er;
  }
  __device__ static Score shfl(const Score &s, int m) {
    Score o;
    uint64_t lo = (uint64_t)s.ex, hi = (uint64_t)(s.ex >> 64);
    lo = (uint64_t)shfl_xor64((int64_t)lo, m);
    hi = (uint64_t)shfl_xor64((int64_t)hi, m);
    o.ex = (i128)(((unsigned __int128)hi << 64) | lo);
    o.ap = __shfl_xor(s.ap, m, 64);
    o.er = __shfl_xor(s.er, m, 64);
    o.W = shfl_xor64(s.W, m);
    o.lab = shfl_xor32(s.lab, m);
    o.kind = __shfl_xor(s.kind, m, 64);
    return o;
  }
};
using PolicyK = PolicyKT<true>;
using PolicyKF = PolicyKT<false>;
// policies of units spanning several slices (cooperative evaluation applies to them)
template <class P>
struct IsMulti : std::false_type {};
template <bool E>
struct IsMulti<PolicyKT<E>> : std::true_type {};
// policies whose near-ties are left to the exact kernels
template <class P>
struct LeavesTies : std::false_type {};
template <>
struct LeavesTies<PolicyKF> : std::true_type {};

// Aggregated levels, units in at most one slice: the same int128 value as PolicyK's
// single-slice case without the multi-slice machinery (far fewer registers).
struct Score1 {
  i128 ex;
  uint32_t lab;
};
struct PolicyK1 {
  typedef Score1 Score;
  template <class V>
  __device__ static Score make(const V &, const UnitCtx &u, const SolveDev &,
                               const SliceTable &tab, uint32_t lab, int64_t W, int kind) {
    Score s;
    s.lab = kind == kEmpty ? kNone : lab;
    i128 val = (i128)u.q * W;
    if (u.m == 1) {
      int64_t y = target_y(tab, u.gs0, u.k0, lab, kind);
      val = val * u.S0 - (i128)u.pb * (i128)(u.k0 * y);
    }
    s.ex = val;
    return s;
  }
  template <class V>
  __device__ static int cmp(const V &, const UnitCtx &, const SolveDev &, const SliceTable &,
                            const Score &a, const Score &b) {
    return a.ex < b.ex ? -1 : (a.ex > b.ex ? 1 : 0);
  }
  __device__ static double slack(const UnitCtx &, const Score &stay, const Score &best) {
    return (double)(stay.ex - best.ex);
  }
  __device__ static bool prunable(const UnitCtx &u, int64_t W, const Score &best) {
    i128 ub = (i128)u.q * W * (u.m ? u.S0 : 1);
    return ub < best.ex;
  }
  __device__ static Score shfl(const Score &s, int m) {
    Score o;
    uint64_t lo = (uint64_t)s.ex, hi = (uint64_t)(s.ex >> 64);
    lo = (uint64_t)shfl_xor64((int64_t)lo, m);
    hi = (uint64_t)shfl_xor64((int64_t)hi, m);
    o.ex = (i128)(((unsigned __int128)hi << 64) | lo);
    o.lab = shfl_xor32(s.lab, m);
    return o;
  }
};

// largest profile degree of a unit spanning several slices (one thread)
template <class V>
__device__ inline double profile_max(const V &g, const UnitCtx &u) {
  int64_t best = u.k0;
  for (int jj = 1; jj < u.m; jj++) {
    int gs;
    int64_t k;
    g.pent(u.v, jj, gs, k);
    best = k > best ? k : best;
  }
  return (double)best;
}

template <class P, class V>
__device__ inline bool better(const V &g, const UnitCtx &u, const SolveDev &sd, const SliceTable &tab,
                              const typename P::Score &a, const typename P::Score &b) {
  int c = P::cmp(g, u, sd, tab, a, b);
  return c > 0 || (c == 0 && a.lab < b.lab);
}

template <class P, class V>
__device__ inline typename P::Score wave_best(const V &g, const UnitCtx &u, const SolveDev &sd,
                                              const SliceTable &tab, typename P::Score s) {
  for (int m = 32; m >= 1; m >>= 1) {
    typename P::Score o = P::shfl(s, m);
    if (better<P>(g, u, sd, tab, o, s)) s = o;
  }
  return s;
}

// ------------------------------------------------------------------ accumulation tables
// LDS accumulation table with the list of its occupied slots (L holds at most the number of
// distinct keys: the unit's degree bound for its bin, and never more than the table size).
struct LdsTab {
  uint32_t *K;
  int64_t *V;
  int lg;
  uint16_t *L;
  int *n;
  __device__ int size() const { return 1 << lg; }
  __device__ void add(uint32_t lab, int64_t w) const { lds_add_listed(K, V, lg, lab, w, L, n); }
  __device__ int64_t get(uint32_t lab) const { return lds_get(K, V, lg, lab); }
  __device__ int count() const { return *(volatile int *)n; }
  __device__ int slot(int i) const { return L[i]; }
  __device__ void reset(int rank) const {
    if (rank == 0) *n = 0;
  }
};
struct GTab {
  uint32_t *K;
  int64_t *V;
  int lg;
  __device__ int size() const { return 1 << lg; }
  __device__ void add(uint32_t lab, int64_t w) const {
    gtab_add(K, V, (1u << lg) - 1, 32 - lg, lab, w);
  }
  __device__ int64_t get(uint32_t lab) const {
    return gtab_get(K, V, (1u << lg) - 1, 32 - lg, lab);
  }
  __device__ int count() const { return 1 << lg; }
  __device__ int slot(int i) const { return i; }
  __device__ void reset(int) const {}
};

// The thread's index for one work item.  Kernels that loop over items take it anew for each: the
// compiler would keep what follows from it, lane positions and LDS addresses of every bin's code, in
// registers across the loop.  That cost the window kernels 64 registers and 15 spilled (k_win_lm0,
// now 52), 124 (k_win_multi at level 0, now 71) and 211 (k_win_all of aggregated levels, now 157);
// the 32 level-0 sweeps of 64M units took 1225 ms with it, 1030 without.
__device__ inline int item_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Group = the threads cooperating on one unit: one wave, or a whole block.
struct WaveGrp {
  __device__ int rank() const { return item_thread() & 63; }
  __device__ int size() const { return 64; }
  __device__ void sync() const { wave_sync(); }
  __device__ bool any(bool x) const { return __any(x); }
};
struct BlockGrp {
  __device__ int rank() const { return item_thread(); }
  __device__ int size() const { return blockDim.x; }
  __device__ void sync() const { __syncthreads(); }
  __device__ bool any(bool x) const { return __syncthreads_or(x); }
};
// A block whose accumulation table lives in global memory: its barriers must also make the
// plain stores and atomics of every wave visible to the others.
struct BlockGrpG {
  __device__ int rank() const { return threadIdx.x; }
  __device__ int size() const { return blockDim.x; }
  __device__ void sync() const { block_sync_global(); }
};

// Reduce a score over the group; every thread gets the result.
template <class P, class V>
__device__ inline typename P::Score group_best(WaveGrp, const V &g, const UnitCtx &u,
                                               const SolveDev &sd, const SliceTable &tab,
                                               typename P::Score s, typename P::Score *) {
  return wave_best<P>(g, u, sd, tab, s);
}
template <class P, class V>
__device__ inline typename P::Score group_best(BlockGrp grp, const V &g, const UnitCtx &u,
                                               const SolveDev &sd, const SliceTable &tab,
                                               typename P::Score s, typename P::Score *red) {
  s = wave_best<P>(g, u, sd, tab, s);
  int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wv] = s;
  grp.sync();
  typename P::Score b = red[0];
  for (int i = 1; i < nw; i++)
    if (better<P>(g, u, sd, tab, red[i], b)) b = red[i];
  grp.sync();
  return b;
}

template <class P, class V>
__device__ inline typename P::Score group_best(BlockGrpG, const V &g, const UnitCtx &u,
                                               const SolveDev &sd, const SliceTable &tab,
                                               typename P::Score s, typename P::Score *red) {
  return group_best<P>(BlockGrp(), g, u, sd, tab, s, red);   // LDS only
}

// heaviest entry of the accumulation table over the group (ties to the lower label), skipping
// one excluded label; kNone when there is none
template <class Grp, class Tab>
__device__ inline void group_heaviest(Grp grp, const Tab &tab, uint32_t skip, const uint8_t *ok,
                                      int64_t &W, uint32_t &lab, int64_t *sred, uint32_t *lred) {
  const int r = grp.rank(), gsz = grp.size();
  W = -1;
  lab = kNone;
  const int nc = tab.count();
  for (int i = r; i < nc; i += gsz) {
    const int h = tab.slot(i);
    uint32_t key = tab.K[h];
    if (key == 0 || key - 1 == skip) continue;
    if (ok && !ok[key - 1]) continue;
    int64_t w = tab.V[h];
    if (w > W || (w == W && key - 1 < lab)) {
      W = w;
      lab = key - 1;
    }
  }
  for (int m = 32; m >= 1; m >>= 1) {
    int64_t w2 = shfl_xor64(W, m);
    uint32_t l2 = shfl_xor32(lab, m);
    if (w2 > W || (w2 == W && l2 < lab)) {
      W = w2;
      lab = l2;
    }
  }
  if (gsz > 64) {
    const int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) {
      sred[wv] = W;
      lred[wv] = lab;
    }
    grp.sync();
    for (int i = 0; i < nw; i++)
      if (sred[i] > W || (sred[i] == W && lred[i] < lab)) {
        W = sred[i];
        lab = lred[i];
      }
    grp.sync();
  }
}

// ------------------------------------------------------------------ cooperative evaluation
// Units spanning many slices: the lanes of an aligned subgroup of mp = 2^ceil(log2 m) lanes
// hold one profile slice each (slice, degree, S and that slice's Sigma sub-table, loaded
// once per unit), so one candidate costs one independent lookup per lane and a butterfly
// sum instead of m dependent lookups in one lane.
constexpr int kCoopMinM = 4;
__host__ __device__ inline int coop_width(int m) {
  int mp = 4;
  while (mp < m) mp <<= 1;
  return mp;
}

struct CoopLane {
  int mp;          // subgroup width
  int j;           // this lane's slice index within the profile (valid when j < m)
  bool valid;
  int64_t k;       // unit degree in that slice
  SliceRecip r;    // that slice's denominator
  const uint64_t *sub;
  uint32_t mask;
  int shift;
};

template <class V>
__device__ inline CoopLane coop_lane(const V &g, const UnitCtx &u, const SolveDev &sd,
                                     const SliceTable &tab, int rank) {
  CoopLane c;
  c.mp = coop_width(u.m);
  c.j = rank & (c.mp - 1);
  c.valid = c.j < u.m;
  c.k = 0;
  c.r = SliceRecip{0.0, 0.0};
  c.sub = tab.slots;
  c.mask = 0;
  c.shift = 32;
  if (c.valid) {
    int gs;
    g.pent(u.v, c.j, gs, c.k);
    c.r = sd.rS[gs];
    c.shift = tab.shift[gs];
    c.mask = 0xffffffffu >> c.shift;
    c.sub = tab.slots + tab.base[gs];
  }
  return c;
}

// This lane's slice Sigma of U targets (the raw table value, 0 when absent or when the lane
// holds no slice); the U first probes are issued together so that their latencies overlap.
template <int U>
__device__ inline void coop_lookup(const CoopLane &c, const uint32_t *lab, const bool *ok,
                                   int64_t *y) {
  uint64_t e[U];
  uint32_t h[U];
  for (int k = 0; k < U; k++) {
    const bool on = c.valid && ok[k];
    h[k] = on ? fib_hash(lab[k], c.shift) : 0u;
    e[k] = on ? c.sub[h[k]] : 0ull;
  }
  for (int k = 0; k < U; k++) {
    int64_t yy = 0;
    if (c.valid && ok[k]) {
      const uint32_t key = lab[k] + 1;
      for (;;) {
        const uint32_t kk = (uint32_t)e[k];
        if (kk == key) {
          yy = (int32_t)(e[k] >> 32);
          break;
        }
        if (kk == 0) break;
        h[k] = (h[k] + 1) & c.mask;
        e[k] = c.sub[h[k]];
      }
    }
    y[k] = yy;
  }
}

// Score of one target from this lane's Sigma y of it, identical on every lane of the subgroup.
__device__ inline ScoreK coop_score(const UnitCtx &u, const CoopLane &c, uint32_t lab, int64_t W,
                                    int64_t y, int kind) {
  ScoreK s;
  s.lab = kind == kEmpty ? kNone : lab;
  s.kind = kind;
  s.W = W;
  s.ex = 0;
  double t = 0.0;
  if (c.valid && kind != kEmpty) {
    if (kind == kStay) y -= c.k;
    t = c.r.of((double)(c.k * y));
  }
  double acc = t, mag = fabs(t);
  for (int o = 1; o < c.mp; o <<= 1) {
    acc += __shfl_xor(acc, o, 64);
    mag += __shfl_xor(mag, o, 64);
  }
  s.ap = 0;
  s.er = 0;
  PolicyK::finish(u, W, acc, mag, s);
  return s;
}

__device__ inline ScoreK coop_make(const UnitCtx &u, const CoopLane &c, uint32_t lab, int64_t W,
                                   int kind) {
  const bool ok = kind != kEmpty;
  int64_t y = 0;
  coop_lookup<1>(c, &lab, &ok, &y);
  return coop_score(u, c, lab, W, y, kind);
}

// Candidates evaluated per subgroup turn (their Sigma lookups in flight together).
constexpr int kCoopBatch = 4;

// ------------------------------------------------------------------ local moving
// One unit: accumulate neighbour-community weights in the table, evaluate every candidate
// community (strictly better gain wins, ties to the lower label, the empty community has
// gain 0 and label +inf), and decide a move only when it beats staying strictly.
// Counters of the decision kernels (filled only when counting is requested), kLmWords per colour of
// the level: [0] units decided, [1] entries scanned, [2] candidate communities evaluated in the
// present window, from 4 on the most of each in the sweep's earlier windows.  When a colour's
// decisions count, k_win_apply adds the most that one window decided of it to the level's total:
// what was decided ahead in vain is not the schedule's work, and a unit that was decided ahead and
// is still at rest when its colour's turn comes is.
constexpr int kLmWords = 8;
struct LmCounters {
  unsigned long long *c;
  __device__ LmCounters of(int colour) const {
    return LmCounters{c ? c + kLmWords * colour : nullptr};
  }
};

template <class P, class Grp, class Tab, class V>
__device__ inline uint32_t lm_unit_coop(Grp grp, Tab tab, const V &g, const SolveDev &sd,
                                        const UnitCtx &u, const SliceTable &sig,
                                        uint32_t fresh_base, typename P::Score *red,
                                        LmCounters pc, typename P::Score best, int64_t hW,
                                        uint32_t hL) {
  const int r = grp.rank(), gsz = grp.size();
  const CoopLane c = coop_lane(g, u, sd, sig, r);
  const int sub = r / c.mp, nsub = gsz / c.mp;
  int ncand = 0;
  if (hL != kNone) {
    ScoreK s = coop_make(u, c, hL, hW, kTarget);
    if (better<P>(g, u, sd, sig, s, best)) best = s;
    ncand = r == 0;
  }
  // subgroups take table slots kCoopBatch at a time; every lane runs the same turns
  const int nc = tab.count();
  for (int i0 = 0; i0 < nc; i0 += nsub * kCoopBatch) {
    uint32_t lab[kCoopBatch];
    int64_t W[kCoopBatch], y[kCoopBatch];
    bool ok[kCoopBatch];
    for (int k = 0; k < kCoopBatch; k++) {
      const int i = i0 + k * nsub + sub;
      const int h = i < nc ? tab.slot(i) : 0;
      const uint32_t key = i < nc ? tab.K[h] : 0u;
      lab[k] = key - 1;
      ok[k] = key != 0 && key - 1 != u.D && key - 1 != hL;
      W[k] = ok[k] ? tab.V[h] : 0;
      ok[k] = ok[k] && !P::prunable(u, W[k], best);
    }
    coop_lookup<kCoopBatch>(c, lab, ok, y);
    for (int k = 0; k < kCoopBatch; k++) {
      if (!ok[k]) continue;
      ncand += c.j == 0;
      ScoreK s = coop_score(u, c, lab[k], W[k], y[k], kTarget);
      if (better<P>(g, u, sd, sig, s, best)) best = s;
    }
  }
  if (pc.c) {
    if (ncand) atomicAdd(pc.c + 2, (unsigned long long)ncand);
    if (r == 0) {
      atomicAdd(pc.c + 0, 1ull);
      atomicAdd(pc.c + 1, (unsigned long long)g.degree(u.v));
    }
  }
  best = group_best<P>(grp, g, u, sd, sig, best, red);
  const int64_t wD = tab.get(u.D);
  const ScoreK stay = coop_make(u, c, u.D, wD, kStay);
  uint32_t out = kNone;
  if (P::cmp(g, u, sd, sig, best, stay) > 0)
    out = best.lab == kNone ? fresh_of(sd, fresh_base) + (uint32_t)g.orig(u.v) : best.lab;
  if (sd.rest) {
    double kmax = (double)c.k;
    for (int o = 1; o < c.mp; o <<= 1) kmax = fmax(kmax, __shfl_xor(kmax, o, 64));
    const bool tied = LeavesTies<P>::value && grp.any(u.tied);
    if (r == 0) settle(sd, u, out, P::slack(u, stay, best), kmax, tied);
  }
  grp.sync();
  return out;
}

template <class P, class V, class Grp, class Tab>
__device__ inline uint32_t lm_unit(Grp grp, Tab tab, const V &g, const SolveDev &sd, int64_t v,
                                   const uint32_t *comm, const SliceTable &sig, uint32_t fresh_base,
                                   typename P::Score *red, LmCounters pc, int64_t *sredW = nullptr,
                                   uint32_t *sredL = nullptr) {
  const int r = grp.rank(), gsz = grp.size();
  if (sd.frozen && sd.frozen[g.solve_of(v)]) return kNone;   // its solve is out of this sweep
  if (at_rest(sd, v)) return kNone;
  for (int i = r; i < tab.size(); i += gsz) {
    tab.K[i] = 0;
    tab.V[i] = 0;
  }
  tab.reset(r);
  grp.sync();
  const uint32_t D = comm[v];
  typename V::Row row = g.row(v, sd);
  // kGather entries per lane at a time: their column and label loads go out together
  constexpr int kGather = 4;
  for (int64_t e0 = row.lo + r; e0 < row.hi; e0 += (int64_t)kGather * gsz) {
    int64_t w[kGather];
    uint32_t lab[kGather];
#pragma unroll
    for (int t = 0; t < kGather; t++) {
      const int64_t e = e0 + (int64_t)t * gsz;
      w[t] = 0;
      int64_t x = 0;
      if (e < row.hi) x = g.nbr(row, e, w[t]);
      lab[t] = w[t] != 0 ? g.lab_at(comm, e, x) : kNone;
    }
#pragma unroll
    for (int t = 0; t < kGather; t++)
      if (lab[t] != kNone) tab.add(lab[t], w[t]);
  }
  grp.sync();
  UnitCtx u = unit_ctx(g, sd, v, D);
  typename P::Score best = P::make(g, u, sd, sig, kNone, 0, kEmpty);
  // the heaviest candidate first: its value is a strong bound for pruning the others
  int64_t hW;
  uint32_t hL;
  group_heaviest(grp, tab, D, (const uint8_t *)nullptr, hW, hL, sredW, sredL);
  if constexpr (!V::kLevel0 && IsMulti<P>::value) {
    if (u.m >= kCoopMinM)
      return lm_unit_coop<P>(grp, tab, g, sd, u, sig, fresh_base, red, pc, best, hW, hL);
  }
  int ncand = 0;
  if (hL != kNone) {
    typename P::Score s = P::make(g, u, sd, sig, hL, hW, kTarget);
    if (better<P>(g, u, sd, sig, s, best)) best = s;
    ncand = r == 0;
  }
  const int nc = tab.count();
  for (int i = r; i < nc; i += gsz) {
    const int h = tab.slot(i);
    uint32_t key = tab.K[h];
    if (key == 0 || key - 1 == D || key - 1 == hL) continue;
    if (P::prunable(u, tab.V[h], best)) continue;
    ncand++;
    typename P::Score s = P::make(g, u, sd, sig, key - 1, tab.V[h], kTarget);
    if (better<P>(g, u, sd, sig, s, best)) best = s;
  }
  if (pc.c) {
    if (ncand) atomicAdd(pc.c + 2, (unsigned long long)ncand);
    if (r == 0) {
      atomicAdd(pc.c + 0, 1ull);
      atomicAdd(pc.c + 1, (unsigned long long)(row.hi - row.lo));
    }
  }
  best = group_best<P>(grp, g, u, sd, sig, best, red);
  int64_t wD = tab.get(D);
  typename P::Score stay = P::make(g, u, sd, sig, D, wD, kStay);
  uint32_t out = kNone;
  if (P::cmp(g, u, sd, sig, best, stay) > 0)
    out = best.lab == kNone ? fresh_of(sd, fresh_base) + (uint32_t)g.orig(v) : best.lab;
  if (sd.rest) {
    const bool tied = LeavesTies<P>::value && grp.any(u.tied);
    if (r == 0) settle(sd, u, out, P::slack(u, stay, best), profile_max(g, u), tied);
  }
  grp.sync();
  return out;
}

constexpr int kWaveLg = 9;        // 512-slot LDS table per wave: units of degree <= 256
constexpr int kBlockLg = 13;      // 8192-slot LDS table per block: degree <= 4096
constexpr int kSmallBlockLg = 11; // 2048-slot LDS table per 256-thread block: degree <= 1024
constexpr int kWaveMaxDeg = 256;
constexpr int kSmallBlockMaxDeg = 1024;
constexpr int kBlockMaxDeg = 4096;

// Degree bins of the decision kernels: 0..3 lane groups of 4/8/16/32 lanes per unit (one
// adjacency entry per lane, equal labels merged in an LDS table), 4 a wave with an LDS
// table, 5 a block with an LDS table, 6 a block with a global-memory table.
constexpr int kNumBins = 8;
constexpr int kBinWaveLast = 4;          // bins 0..4 fit a wave's table
constexpr int kBinGtab = kNumBins - 1;   // global-memory tables
// Colour batches are bucketed by (colour, slot): slots 0..7 are the degree bins; at aggregated
// levels units in at most one slice use slots 8..15 and the lean single-slice decision.
constexpr int kBatchShift = 4;
constexpr int kBatchSlots = 1 << kBatchShift;
__host__ __device__ inline uint32_t degree_bin(int64_t d) {
  return d <= 4 ? 0u : d <= 8 ? 1u : d <= 16 ? 2u : d <= 32 ? 3u
       : d <= kWaveMaxDeg ? 4u : d <= kSmallBlockMaxDeg ? 5u : d <= kBlockMaxDeg ? 6u : 7u;
}
// Bin of a unit of degree d in m slices: by degree; a unit in kCoopMinM or more slices is
// evaluated cooperatively by a wave, or by a block when its (candidate x slice) work exceeds
// 64 turns of a wave.  A bin never receives a degree above its table's capacity
// (bin_fits checks that on the host before the first solve).
__host__ __device__ inline uint32_t bin_of(int64_t d, int m) {
  if (m < kCoopMinM) return degree_bin(d);
  if (d > kBlockMaxDeg) return 7u;
  if (d <= kWaveMaxDeg && d * coop_width(m) <= 64 * 64) return 4u;
  return d <= kSmallBlockMaxDeg ? 5u : 6u;
}
__host__ __device__ inline bool bin_fits(int64_t d, uint32_t bin) {
  const int64_t cap[kNumBins] = {4, 8, 16, 32, kWaveMaxDeg, kSmallBlockMaxDeg, kBlockMaxDeg,
                                 INT64_MAX};
  return bin < (uint32_t)kNumBins && d <= cap[bin];
}
__device__ inline uint32_t unit_bin(const View0 &g, int64_t v) { return degree_bin(g.degree(v)); }
__device__ inline uint32_t unit_bin(const ViewK &g, int64_t v) {
  return bin_of(g.degree(v), g.plen(v));
}
__device__ inline uint32_t batch_slot(const View0 &g, int64_t v) { return unit_bin(g, v); }
__device__ inline uint32_t batch_slot(const ViewK &g, int64_t v) {
  return unit_bin(g, v) + (g.plen(v) <= 1 ? (uint32_t)kNumBins : 0u);
}

// Where a decision goes: the target of its position and, when it is a move, the smallest moving
// colour of the window (the stored value only falls, so a look before the atomic drops nearly
// all of them).
struct Emit {
  uint32_t *target;
  int32_t *first_move;
  int32_t colour;
  __device__ void put(int64_t pos, uint32_t out) const {
    target[pos] = out;
    if (out != kNone &&
        __hip_atomic_load(first_move, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > colour)
      atomicMin(first_move, colour);
  }
};

// Units of degree <= G: G lanes per unit, one adjacency entry per lane; the group merges
// equal community labels in a 2G-slot LDS table per group (the lane that claims a label's slot
// leads it), every leader evaluates its community, and the group reduces to the best.  lk/lv:
// the block's LDS, 128 slots per wave.
template <class P, class V, int G>
__device__ inline void lm_group_block(const V &g, const SolveDev &sd, const int32_t *units,
                                      int64_t pos, int count, const uint32_t *comm,
                                      const SliceTable &sig, const Emit &em, uint32_t fresh_base,
                                      LmCounters pc, uint32_t *lk, int64_t *lv) {
  const int tid = item_thread(), lane = tid & 63;
  const int gl = lane & (G - 1);
  const int gbase = lane & ~(G - 1);
  const int idx = tid / G;
  if (idx >= count) return;   // whole groups leave together; shuffles stay inside a group
  const int64_t v = g.unit_at(units, pos + idx);
  if ((sd.frozen && sd.frozen[g.solve_of(v)]) || at_rest(sd, v)) {   // nothing to decide
    if (gl == 0) em.target[pos + idx] = kNone;
    return;
  }
  const uint32_t D = comm[v];
  typename V::Row row = g.row(v, sd);
  UnitCtx u = unit_ctx(g, sd, v, D);
  // level 0: the lookup of the own community's Sigma goes out with the neighbour gathers
  int64_t yD = 0;
  if constexpr (std::is_same<P, Policy0>::value)
    if (gl == 0 && u.m > 0) yD = tab_get(sig, u.gs0, D);
  const int64_t e = row.lo + gl;
  uint32_t c = kNone;
  int64_t w = 0;
  if (e < row.hi) {
    const int64_t x = g.nbr(row, e, w);
    if (w != 0) c = g.lab_at(comm, e, x);
  }
  int64_t wsum = 0, wD = 0;
  bool leader = false;
  {
    constexpr int kSlots = 2 * G;
    uint32_t *sk = lk + (tid >> 6) * 128 + (gbase / G) * kSlots;
    unsigned long long *sv =
        reinterpret_cast<unsigned long long *>(lv) + (tid >> 6) * 128 + (gbase / G) * kSlots;
    sk[gl] = 0u;
    sk[gl + G] = 0u;
    sv[gl] = 0ull;
    sv[gl + G] = 0ull;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the clears land before the claims
    int h = -1;
    if (c != kNone) {
      const uint32_t key = c + 1;
      uint32_t hh = (c * 2654435769u) >> (32 - __builtin_ctz(kSlots));
      for (;;) {
        const uint32_t prev = atomicCAS(sk + hh, 0u, key);
        if (prev == 0u || prev == key) {
          leader = prev == 0u;
          break;
        }
        hh = (hh + 1) & (kSlots - 1);
      }
      h = (int)hh;
      atomicAdd(sv + hh, (unsigned long long)w);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);
    if (leader) wsum = (int64_t)sv[h];
    if (gl == 0) {   // the own community's weight
      const uint32_t key = D + 1;
      uint32_t hh = (D * 2654435769u) >> (32 - __builtin_ctz(kSlots));
      for (int probes = 0; probes < kSlots; probes++) {
        const uint32_t k = sk[hh];
        if (k == key) {
          wD = (int64_t)sv[hh];
          break;
        }
        if (k == 0u) break;
        hh = (hh + 1) & (kSlots - 1);
      }
    }
  }
  typename P::Score best = P::make(g, u, sd, sig, kNone, 0, kEmpty);
  const bool cand = leader && c != D;
  if (cand) {
    typename P::Score s = P::make(g, u, sd, sig, c, wsum, kTarget);
    if (better<P>(g, u, sd, sig, s, best)) best = s;
  }
  const uint64_t gmask = (G == 64 ? ~0ull : ((1ull << G) - 1)) << gbase;
  for (int m = G / 2; m >= 1; m >>= 1) {
    typename P::Score o = P::shfl(best, m);
    if (better<P>(g, u, sd, sig, o, best)) best = o;
  }
  const bool tied = LeavesTies<P>::value && (__ballot(u.tied) & gmask) != 0;
  if (pc.c) {
    unsigned long long nc = __popcll(__ballot(cand) & gmask);
    if (gl == 0) {
      atomicAdd(pc.c + 0, 1ull);
      atomicAdd(pc.c + 1, (unsigned long long)(row.hi - row.lo));
      if (nc) atomicAdd(pc.c + 2, nc);
    }
  }
  if (gl == 0) {
    typename P::Score stay;
    if constexpr (std::is_same<P, Policy0>::value) stay = Policy0::stay_from(u, D, wD, yD);
    else stay = P::make(g, u, sd, sig, D, wD, kStay);
    uint32_t out = kNone;
    if (P::cmp(g, u, sd, sig, best, stay) > 0)
      out = best.lab == kNone ? fresh_of(sd, fresh_base) + (uint32_t)g.orig(v) : best.lab;
    em.put(pos + idx, out);
    if (sd.rest) settle(sd, u, out, P::slack(u, stay, best), profile_max(g, u), tied || u.tied);
  }
}

// One slice's Sigma sub-table, resolved once per unit (the probes of the unit's own community
// and of its candidates all go to it).
struct SubTab {
  const uint64_t *sub;
  int sh;
  __device__ void open(const SliceTable &t, int s) {
    sh = t.shift[s];
    sub = t.slots + t.base[s];
  }
  // first probe: its slot and entry (issued for several units before any is resolved)
  __device__ uint64_t first(uint32_t label, uint32_t &h) const {
    h = fib_hash(label, sh);
    return sub[h];
  }
  // the value of `label` from its first probe, continuing the linear probe when needed
  __device__ int64_t resolve(uint32_t label, uint32_t h, uint64_t e) const {
    const uint32_t key = label + 1, mask = 0xffffffffu >> sh;
    for (;;) {
      const uint32_t k = (uint32_t)e;
      if (k == key) return (int32_t)(e >> 32);
      if (k == 0) return 0;
      h = (h + 1) & mask;
      e = sub[h];
    }
  }
};

// Level 0 in colour-batch order, units of degree <= G, Policy0.  Each group of G lanes decides
// U units in lockstep (their dependent loads in flight together; one unit measured fastest, at
// 8 waves per SIMD); a batch segment is a range of positions, so a unit's position is computed,
// not loaded.  Equal neighbour labels are merged in a small LDS table per group (a claim, an
// add, a read) rather than by G rounds of shuffles.  Entry weights travel as 32-bit raw values
// (coupling entries flagged in bit 31) and are scaled once per candidate:
// W = b * (raw intra weight) + a * (coupling entries).  Every decision equals
// lm_group_block's with Policy0: the same candidates and values (the best under the same total
// order).
template <int G, int U, bool kOne, bool kCopy>
__device__ inline void lm0_lockstep(const ViewP &g, const SolveDev &sd, int64_t first,
                                    int count, const uint32_t *comm, const SliceTable &sig,
                                    const Emit &em, uint32_t fresh_base, LmCounters pc,
                                    uint32_t *lm0_keys, unsigned long long *lm0_vals) {
  constexpr int kGroups = 256 / G;
  const int tid = item_thread(), lane = tid & 63;
  const int gl = lane & (G - 1);
  const int gbase = lane & ~(G - 1);
  const int base = tid / G;
  if (base >= count) return;   // whole groups leave together
  int64_t pos[U];
  bool live[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int i = base + u * kGroups;
    live[u] = i < count;
    pos[u] = first + (live[u] ? i : 0);
  }
  // unit headers
  uint32_t D[U];
  int64_t lo[U], hi[U];
  int32_t kv[U], gs[U], js[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int64_t v = pos[u];
    D[u] = comm[v];
    lo[u] = g.rp[v];
    hi[u] = live[u] ? g.rp[v + 1] : lo[u];
    kv[u] = g.k[v];
    gs[u] = g.slice[v];
    js[u] = kOne ? 0 : g.solve_of(v);   // one solve: its constants are uniform
    if ((sd.frozen && sd.frozen[js[u]]) || at_rest(sd, v)) {   // nothing to decide
      if (live[u] && gl == 0) em.target[pos[u]] = kNone;
      live[u] = false;
      hi[u] = lo[u];
    }
  }
  // entries and each unit's Sigma sub-table
  // entries: column (coupling flag), weight and, with kCopy, the neighbour's label from the
  // label copy, all read in entry order
  int32_t cr[U], deg[U];
  uint32_t val[U], c[U];
  SubTab tb[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int64_t e = lo[u] + gl;
    const bool has = e < hi[u];
    deg[u] = (int32_t)(hi[u] - lo[u]);
    cr[u] = has ? g.col[e] : 0x7fffffff;
    c[u] = (kCopy && has) ? g.elab[e] : kNone;
    const uint32_t w = (has && g.w) ? (uint32_t)g.w[e] : 1u;
    tb[u].open(sig, gs[u]);
    val[u] = !has ? 0u : (cr[u] < 0 ? 0x80000000u | w : w);
  }
  // a coupling entry of zero weight is no entry; the own community's first probe
  uint32_t hD[U];
  uint64_t eD[U];
  int64_t a[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    a[u] = sd.a[js[u]];
    const bool ent = val[u] != 0u && (cr[u] >= 0 || a[u] != 0);
    if (!ent) c[u] = kNone;
    else if (!kCopy) c[u] = comm[cr[u] & 0x7fffffff];   // gathered
    if (gl == 0 && kv[u] > 0) eD[u] = tb[u].first(D[u], hD[u]);
  }
  // equal labels merged inside the group in a small LDS table per (group, unit): each entry
  // adds its raw weight (low half) or coupling multiplier (high half) to its label's slot; the
  // lane that claims a slot leads that label.  Three LDS steps instead of G shuffle rounds.
  constexpr int kSlots = 2 * G;   // load at most one half
  uint32_t *sk = lm0_keys + (tid >> 6) * (U * 128) + (gbase / G) * kSlots;
  unsigned long long *sv = lm0_vals + (tid >> 6) * (U * 128) + (gbase / G) * kSlots;
#pragma unroll
  for (int u = 0; u < U; u++) {
    sk[u * 128 + gl] = 0u;
    sk[u * 128 + gl + G] = 0u;
    sv[u * 128 + gl] = 0ull;
    sv[u * 128 + gl + G] = 0ull;
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the clears land before the claims
  bool lead[U];
  int slot[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    lead[u] = false;
    slot[u] = -1;
    if (c[u] != kNone) {
      const uint32_t key = c[u] + 1;
      uint32_t h = (c[u] * 2654435769u) >> (32 - __builtin_ctz(kSlots));
      for (;;) {
        const uint32_t prev = atomicCAS(sk + u * 128 + h, 0u, key);
        if (prev == 0u || prev == key) {
          lead[u] = prev == 0u;
          break;
        }
        h = (h + 1) & (kSlots - 1);
      }
      slot[u] = (int)h;
      const unsigned long long add =
          (unsigned long long)(val[u] & 0x7fffffffu) << ((val[u] >> 31) ? 32 : 0);
      atomicAdd(sv + u * 128 + h, add);
    }
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_s_waitcnt(0xc07f);
  uint32_t wr[U], wrD[U];
  int nc[U], ncD[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    wr[u] = 0;
    nc[u] = 0;
    wrD[u] = 0;
    ncD[u] = 0;
    if (lead[u]) {
      const unsigned long long t = sv[u * 128 + slot[u]];
      wr[u] = (uint32_t)t;
      nc[u] = (int)(t >> 32);
    }
    if (gl == 0) {   // the own community's weight
      const uint32_t key = D[u] + 1;
      uint32_t h = (D[u] * 2654435769u) >> (32 - __builtin_ctz(kSlots));
      for (int probes = 0; probes < kSlots; probes++) {
        const uint32_t k = sk[u * 128 + h];
        if (k == key) {
          const unsigned long long t = sv[u * 128 + h];
          wrD[u] = (uint32_t)t;
          ncD[u] = (int)(t >> 32);
          break;
        }
        if (k == 0u) break;
        h = (h + 1) & (kSlots - 1);
      }
    }
  }
  // candidates' first probes, all units together
  bool cand[U];
  uint32_t hc[U];
  uint64_t ec[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    cand[u] = lead[u] && c[u] != D[u];
    if (cand[u] && kv[u] > 0) ec[u] = tb[u].first(c[u], hc[u]);
  }
  // values, the group's best, the decision
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int j = js[u];
    const int64_t p = sd.p[j], q = sd.q[j], pb = sd.pb[j], b = sd.b[j];
    const int64_t k0 = kv[u];
    const int64_t S0 = k0 > 0 ? sd.S[gs[u]] : 1;
    Score0 best;
    best.g = 0;
    best.lab = kNone;
    if (cand[u]) {
      const int64_t W = b * (int64_t)wr[u] + a[u] * nc[u];
      Score0 s;
      s.lab = c[u];
      s.g = k0 > 0 ? q * S0 * W - pb * (k0 * tb[u].resolve(c[u], hc[u], ec[u])) : q * W;
      if (s.g > best.g || (s.g == best.g && s.lab < best.lab)) best = s;
    }
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) {
      Score0 o;
      o.g = shfl_xor64(best.g, m);
      o.lab = (uint32_t)__shfl_xor((int)best.lab, m, 64);
      if (o.g > best.g || (o.g == best.g && o.lab < best.lab)) best = o;
    }
    if (pc.c) {
      const unsigned long long nk =
          __popcll(__ballot(cand[u] && live[u]) &
                   (((G == 64) ? ~0ull : ((1ull << G) - 1)) << gbase));
      if (gl == 0 && live[u]) {
        atomicAdd(pc.c + 0, 1ull);
        atomicAdd(pc.c + 1, (unsigned long long)deg[u]);
        if (nk) atomicAdd(pc.c + 2, nk);
      }
    }
    if (gl == 0 && live[u]) {
      const int64_t wD = b * (int64_t)wrD[u] + a[u] * ncD[u];
      int64_t stay;
      if (k0 > 0) {
        const int64_t yD = tb[u].resolve(D[u], hD[u], eD[u]);
        stay = q * S0 * wD - pb * (k0 * (yD - k0));
      } else {
        stay = q * wD;
      }
      uint32_t out = kNone;
      if (best.g > stay)
        out = best.lab == kNone ? fresh_of(sd, fresh_base) + (uint32_t)g.uid[pos[u]] : best.lab;
      em.put(pos[u], out);
      if (sd.rest) {
        UnitCtx uc;
        uc.v = pos[u];
        uc.j = j;
        uc.m = k0 > 0 ? 1 : 0;
        uc.gs0 = gs[u];
        uc.k0 = k0;
        uc.pb = pb;
        settle(sd, uc, out, (double)(stay - best.g), 0.0, false);
      }
    }
    (void)p;
  }
}

// ------------------------------------------------------------------ colour windows
// A sweep visits the colours one after another: the units of a colour decide together, their
// moves are applied, the next colour follows.  Past a level's first sweeps most colours move
// nothing (1215 of 8158 aggregated-level batches of a 3.2M-copy solve, 68 of 1082 of a warm
// start), so a window of consecutive colours is decided at once from the state before it.  The
// decisions of the colours up to and including the first one that moves are those of the
// colour-by-colour sweep (nothing moved before them); that colour's moves are applied and the
// next window starts behind it, so every move is the one the sweep makes.  The window is kept
// on the device: decision kernels read it, the apply kernel writes the next one, and the host
// queues pairs of both without waiting; a pair that comes after the last colour does nothing.
//
// Work is cut into items of one block each, listed per kernel family in colour order.
enum { kFamAll, kFamGroup1, kFamGroup, kFamMulti1, kFamMulti, kFamBlock, kFamHub, kFams };

struct WinItem {
  int32_t pos, count;   // positions [pos, pos + count) of the colour order
  int32_t slot;         // batch slot (class and degree bin) the block's code follows
  int32_t colour;
};
struct WinSeg {         // one (colour, slot) run of units, cut into items of `per` units
  int32_t item0, items, pos, count, per, slot, colour, pad;
};
struct WinState {
  int32_t c0, c1;       // the window; empty once every colour has been visited
  int32_t budget;       // blocks of work the next window may hold
  int32_t windows;      // windows decided in this sweep
  int32_t t;            // the sweep
};
struct WinLevel {
  const WinItem *items;
  const int32_t *ip;    // [kFams][ncol + 1] first item of each colour
  const int32_t *cost;  // [ncol + 1] blocks of work before each colour
  const int32_t *cptr;  // [ncol + 1] first position of each colour
  int32_t *moved_at;    // [ncol] last sweep in which the colour moved
  WinState *st;         // [3] ring: pair r uses r % 3
  int32_t *first_move;  // [3] smallest moving colour of the pair's window
  int32_t *near_tie;    // [3][J] smallest colour of each solve with an unsettled near-tie
  int32_t ncol, floor, J;
  int32_t hubs_last;    // no colour with a hub is decided behind one that will probably move
};
constexpr int32_t kNoColour = 0x7fffffff;
constexpr int kXcds = 8;   // MI355X: eight accelerator complex dies, each with its own L2

__global__ __launch_bounds__(256) void k_win_items(const WinSeg *segs, WinItem *items) {
  const WinSeg s = segs[blockIdx.x];
  for (int i = threadIdx.x; i < s.items; i += blockDim.x) {
    const int left = s.count - i * s.per;
    items[s.item0 + i] = WinItem{s.pos + i * s.per, left < s.per ? left : s.per, s.slot, s.colour};
  }
}

// Items of a family in pair r's window, in the order that gives each XCD a contiguous eighth of
// them (blocks are dealt to the XCDs round-robin): units are in id order inside a batch, so an
// XCD's L2 sees the labels and Sigma sub-tables of a few slices.
struct WinRange {
  int i0, n, per;
  __device__ WinRange(const WinLevel &L, int fam, int r) {
    const WinState s = L.st[r];
    const int32_t *ip = L.ip + fam * (L.ncol + 1);
    i0 = s.c0 < s.c1 ? ip[s.c0] : 0;
    n = s.c0 < s.c1 ? ip[s.c1] - i0 : 0;
    per = (n + kXcds - 1) / kXcds;
  }
  __device__ int turns() const { return per * kXcds; }
  // item of turn k, -1 when the turn has none
  __device__ int item(int k) const {
    const int i = (k % kXcds) * per + k / kXcds;
    return i < n ? i0 + i : -1;
  }
};

// Window from colour c0 on (one wave): as many colours as the budget holds, at least one, up to
// and including the next colour that moved in the last sweep (it will probably move again, and
// what lies behind it would be decided twice); below `floor` blocks the chip is not full and
// deciding further ahead costs nothing, except for hubs, whose kernels take their time by
// themselves: one hub of 8000 entries in the last of 14 colours was decided five times a sweep.
// At level 0 (hubs_last) such colours wait until nothing before them will probably move; aggregated
// levels have hubs in many colours, and the windows that this adds cost as much as it saves (a solve
// of 250k units 62.8 -> 64.5 ms).
__device__ inline int win_end(const WinLevel &L, int t, int c0, int budget) {
  const int lane = threadIdx.x & 63;
  const int lim = budget > L.floor ? budget : L.floor;
  const int32_t *hubs = L.ip + kFamHub * (L.ncol + 1);
  int c1 = c0;
  const int base = c0 < L.ncol ? L.cost[c0] : 0;
  bool moves = false;   // a colour before c1 will probably move
  while (c1 < L.ncol) {
    const int c = c1 + lane;
    const int cost = c < L.ncol ? L.cost[c + 1] - base : 0;
    const uint64_t likely = __ballot(c < L.ncol && (t == 0 || L.moved_at[c] >= t - 1));
    const bool behind = moves || (likely & ((1ull << lane) - 1));
    moves = moves || likely;
    const bool wait = L.hubs_last && behind && c < L.ncol && hubs[c + 1] > hubs[c];
    const bool in = c < L.ncol && (c == c0 || (cost <= lim && !wait));
    const bool stop = in && cost > L.floor && L.moved_at[c] >= t - 1;
    const uint64_t out = ~__ballot(in), stops = __ballot(stop);
    const int n_in = out ? __builtin_ctzll(out) : 64;
    const int n_stop = stops ? __builtin_ctzll(stops) + 1 : 64;
    const int take = n_in < n_stop ? n_in : n_stop;
    c1 += take;
    if (take < 64) break;
  }
  return c1;
}

constexpr int32_t kWinUnbounded = 1 << 28;

// Start of sweep t (one block): first window, cleared counters.  The first sweep of a level
// starts with a narrow window; later ones are led by what moved in the sweep before.
__global__ __launch_bounds__(256) void k_win_begin(WinLevel L, int t, uint32_t *moved,
                                                   int32_t *redo, int *flag) {
  for (int i = threadIdx.x; i < L.J; i += blockDim.x) {
    moved[i] = 0;
    redo[i] = kRedoUnset;
    if (L.near_tie)
      for (int k = 0; k < 3; k++) L.near_tie[k * L.J + i] = kNoColour;
  }
  if (threadIdx.x == 0) *flag = 0;
  if (threadIdx.x < 3) L.first_move[threadIdx.x] = kNoColour;
  if (threadIdx.x < 64) {
    const int budget = t == 0 ? L.floor : kWinUnbounded;
    const int c1 = win_end(L, t, 0, budget);
    if (threadIdx.x == 0) L.st[0] = WinState{0, c1, budget, 0, t};
  }
}

// One block's share of a unit bin: lane groups, waves (a table of 512 slots each), or the whole
// block with a table of 2^11 slots (bin 5) or 2^LG (bin 6).
template <class P, int LG, class V>
__device__ inline void win_item(const V &g, const SolveDev &sd, const int32_t *units,
                                const WinItem &it, const uint32_t *comm, const SliceTable &sig,
                                const Emit &em, uint32_t fresh_base, LmCounters pc, uint32_t *sk,
                                int64_t *sv, uint16_t *sl, int *sn, typename P::Score *red,
                                int64_t *hw, uint32_t *hl) {
  switch (it.slot % kNumBins) {
    case 0:
      lm_group_block<P, V, 4>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base, pc, sk, sv);
      break;
    case 1:
      lm_group_block<P, V, 8>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base, pc, sk, sv);
      break;
    case 2:
      lm_group_block<P, V, 16>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base, pc, sk,
                               sv);
      break;
    case 3:
      lm_group_block<P, V, 32>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base, pc, sk,
                               sv);
      break;
    case 4: {
      const int tid = item_thread(), wv = tid >> 6;
      if (wv >= it.count) break;
      // a unit of at most 64 entries in fewer than kCoopMinM slices: the wave as one lane group
      // (entries one per lane, labels merged in this wave's LDS region)
      const int64_t v = g.unit_at(units, it.pos + wv);
      if (g.degree(v) <= 64 && g.plen(v) < kCoopMinM) {
        // lm_group_block addresses 128 slots per wave from the pointer it gets: shift it so
        // that this wave lands on its own 512-slot wave table, which no other wave touches
        lm_group_block<P, V, 64>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base, pc,
                                 sk + (wv << kWaveLg) - wv * 128, sv + (wv << kWaveLg) - wv * 128);
        break;
      }
      LdsTab tab{sk + (wv << kWaveLg), sv + (wv << kWaveLg), kWaveLg, sl + wv * kWaveMaxDeg,
                 sn + wv};
      const uint32_t out = lm_unit<P>(WaveGrp(), tab, g, sd, v, comm, sig, fresh_base,
                                      (typename P::Score *)nullptr, pc);
      if ((tid & 63) == 0) em.put(it.pos + wv, out);
      break;
    }
    default: {
      LdsTab tab{sk, sv, it.slot % kNumBins == 5 ? kSmallBlockLg : LG, sl, sn};
      const uint32_t out = lm_unit<P>(BlockGrp(), tab, g, sd, g.unit_at(units, it.pos), comm, sig,
                                      fresh_base, red, pc, hw, hl);
      if (threadIdx.x == 0) em.put(it.pos, out);
    }
  }
}

// Waves per SIMD that the registers must allow (the exact policy needs scratch anyway); see
// item_thread for what they come to.
template <class P>
constexpr int kWinWaves = std::is_same<P, PolicyK>::value ? 1 : IsMulti<P>::value ? 3 : 4;

// Bins 4 and 5 of a window's large colours, one class of units.
template <class P, class V>
__global__ __launch_bounds__(256, kWinWaves<P>) void k_win_multi(V g, SolveDev sd, WinLevel L, int fam, int r,
                                                   const int32_t *units, const uint32_t *comm,
                                                   SliceTable sig, uint32_t *target,
                                                   uint32_t fresh_base, LmCounters pc) {
  __shared__ uint32_t sk[1 << kSmallBlockLg];        // 4 wave tables of 512, or one of 2048
  __shared__ int64_t sv[1 << kSmallBlockLg];
  __shared__ uint16_t sl[kSmallBlockMaxDeg];         // 4 lists of 256, or one of 1024
  __shared__ int sn[4];
  __shared__ typename P::Score red[4];
  __shared__ int64_t hw[4];
  __shared__ uint32_t hl[4];
  const WinRange w(L, fam, r);
  if (sd.redo) sd.redo = L.near_tie + r * L.J;
  for (int k = blockIdx.x; k < w.turns(); k += gridDim.x) {
    const int i = w.item(k);
    if (i < 0) continue;
    const WinItem it = L.items[i];
    const Emit em{target, L.first_move + r, it.colour};
    sd.mark = it.colour;
    win_item<P, kSmallBlockLg>(g, sd, units, it, comm, sig, em, fresh_base, pc.of(it.colour), sk, sv,
                               sl, sn, red, hw, hl);
    __syncthreads();   // the next item lays its tables over this one's
  }
}

// Every bin below the hubs of a window of small colours (but for the block bin where make_windows
// keeps that apart), in one launch: such windows are bound by latency, and one launch over both
// classes (units of class 1, slots from kNumBins on, by P1, the others by P) takes the place of up to
// five in a row.  LG: the rows fill at most half the table; small tables let more blocks share a CU.
// Blocks of 512 threads cost the exact policy's levels a quarter (57k units: 67.5 ms against 53.7)
// and gained a tenth or less elsewhere.
template <class P, class P1, class V, int LG>
__global__ __launch_bounds__(256) void k_win_all(V g, SolveDev sd, WinLevel L, int r,
                                                         const int32_t *units,
                                                         const uint32_t *comm, SliceTable sig,
                                                         uint32_t *target, uint32_t fresh_base,
                                                         LmCounters pc) {
  static_assert(LG >= 11, "a wave table of 512 slots for each wave");
  constexpr int kWaves = 4;
  __shared__ uint32_t sk[1 << LG];
  __shared__ int64_t sv[1 << LG];
  __shared__ uint16_t sl[1 << (LG - 1)];
  __shared__ int sn[kWaves];
  __shared__ typename P::Score red[kWaves];
  __shared__ typename P1::Score red1[kWaves];
  __shared__ int64_t hw[kWaves];
  __shared__ uint32_t hl[kWaves];
  const WinRange w(L, kFamAll, r);
  if (sd.redo) sd.redo = L.near_tie + r * L.J;
  for (int k = blockIdx.x; k < w.turns(); k += gridDim.x) {
    const int i = w.item(k);
    if (i < 0) continue;
    const WinItem it = L.items[i];
    const Emit em{target, L.first_move + r, it.colour};
    sd.mark = it.colour;
    if (!std::is_same<P, P1>::value && it.slot >= kNumBins)
      win_item<P1, LG>(g, sd, units, it, comm, sig, em, fresh_base, pc.of(it.colour), sk, sv, sl, sn,
                       red1, hw, hl);
    else
      win_item<P, LG>(g, sd, units, it, comm, sig, em, fresh_base, pc.of(it.colour), sk, sv, sl, sn,
                      red, hw, hl);
    __syncthreads();   // the next item lays its tables over this one's
  }
}

// Bins 0..3 alone: little LDS, so large batches run at the occupancy the group code's registers
// allow, where the fused kernel's tables would hold it lower.
template <class P, class V>
__global__ __launch_bounds__(256, IsMulti<P>::value ? 1 : 8) void k_win_groups(V g, SolveDev sd, WinLevel L, int fam, int r,
                                                    const int32_t *units, const uint32_t *comm,
                                                    SliceTable sig, uint32_t *target,
                                                    uint32_t fresh_base, LmCounters pc) {
  __shared__ uint32_t lk[4 * 128];
  __shared__ int64_t lv[4 * 128];
  const WinRange w(L, fam, r);
  if (sd.redo) sd.redo = L.near_tie + r * L.J;
  for (int k = blockIdx.x; k < w.turns(); k += gridDim.x) {
    const int i = w.item(k);
    if (i < 0) continue;
    const WinItem it = L.items[i];
    const Emit em{target, L.first_move + r, it.colour};
    sd.mark = it.colour;
    switch (it.slot % kNumBins) {
      case 0:
        lm_group_block<P, V, 4>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base,
                                 pc.of(it.colour), lk, lv);
        break;
      case 1:
        lm_group_block<P, V, 8>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base,
                                 pc.of(it.colour), lk, lv);
        break;
      case 2:
        lm_group_block<P, V, 16>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base,
                                 pc.of(it.colour), lk, lv);
        break;
      default:
        lm_group_block<P, V, 32>(g, sd, units, it.pos, it.count, comm, sig, em, fresh_base,
                                 pc.of(it.colour), lk, lv);
    }
  }
}

// Bins 0..3 of level 0 in position order (lm0_lockstep).  kOne: a single solve; kCopy:
// neighbour labels from the label copy.
template <int U, bool kOne, bool kCopy>
__global__ __launch_bounds__(256, 8) void k_win_lm0(ViewP g, SolveDev sd, WinLevel L, int r,
                                                 const uint32_t *comm, SliceTable sig,
                                                 uint32_t *target, uint32_t fresh_base,
                                                 LmCounters pc) {
  __shared__ uint32_t keys[4 * U * 128];
  __shared__ unsigned long long vals[4 * U * 128];
  const WinRange w(L, kFamGroup, r);
  for (int k = blockIdx.x; k < w.turns(); k += gridDim.x) {
    const int i = w.item(k);
    if (i < 0) continue;
    const WinItem it = L.items[i];
    const Emit em{target, L.first_move + r, it.colour};
    switch (it.slot) {
      case 0:
        lm0_lockstep<4, U, kOne, kCopy>(g, sd, it.pos, it.count, comm, sig, em, fresh_base,
                                        pc.of(it.colour), keys, vals);
        break;
      case 1:
        lm0_lockstep<8, U, kOne, kCopy>(g, sd, it.pos, it.count, comm, sig, em, fresh_base,
                                        pc.of(it.colour), keys, vals);
        break;
      case 2:
        lm0_lockstep<16, U, kOne, kCopy>(g, sd, it.pos, it.count, comm, sig, em, fresh_base,
                                        pc.of(it.colour), keys, vals);
        break;
      default:
        lm0_lockstep<32, U, kOne, kCopy>(g, sd, it.pos, it.count, comm, sig, em, fresh_base,
                                        pc.of(it.colour), keys, vals);
    }
  }
}

// Bin 6: one block per unit, a table for up to kBlockMaxDeg distinct labels.  The multi-slice
// policy needs more than the 128 registers per lane that 1024-thread blocks allow.
template <class P>
constexpr int kBlockThreads = IsMulti<P>::value ? 512 : 1024;

template <class P, class V, int NT>
__global__ __launch_bounds__(NT) void k_win_block(V g, SolveDev sd, WinLevel L, int r,
                                                  const int32_t *units, const uint32_t *comm,
                                                  SliceTable sig, uint32_t *target,
                                                  uint32_t fresh_base, LmCounters pc) {
  __shared__ uint32_t sk[1 << kBlockLg];
  __shared__ int64_t sv[1 << kBlockLg];
  __shared__ uint16_t sl[kBlockMaxDeg];
  __shared__ int sn;
  __shared__ typename P::Score red[NT / 64];
  __shared__ int64_t hw[NT / 64];
  __shared__ uint32_t hl[NT / 64];
  LdsTab tab{sk, sv, kBlockLg, sl, &sn};
  const WinRange w(L, kFamBlock, r);
  if (sd.redo) sd.redo = L.near_tie + r * L.J;
  for (int k = blockIdx.x; k < w.turns(); k += gridDim.x) {
    const int i = w.item(k);
    if (i < 0) continue;
    const WinItem it = L.items[i];
    sd.mark = it.colour;
    const uint32_t out = lm_unit<P>(BlockGrp(), tab, g, sd, g.unit_at(units, it.pos), comm, sig,
                                    fresh_base, red, pc.of(it.colour), hw, hl);
    if (threadIdx.x == 0) Emit{target, L.first_move + r, it.colour}.put(it.pos, out);
    __syncthreads();
  }
}

// ------------------------------------------------------------------ hub units
// Units above the block bins are spread over kHubBlocks blocks each (grid = kHubBlocks x
// window's hubs): the blocks clear, fill and scan disjoint parts of the unit's global table, each
// scan keeps its best candidate, and one wave per unit reduces those with the same total
// order (value, then label) and compares with staying.  The result equals one group's.
constexpr int kHubBlocks = 16;

template <class V>
__global__ __launch_bounds__(256) void k_hub_clear(V g, SolveDev sd, WinLevel L, int r,
                                                   const int32_t *units,
                                                   const int64_t *goff, const int32_t *glg,
                                                   uint32_t *gk, int64_t *gv) {
  const WinRange w(L, kFamHub, r);
  for (int y = blockIdx.y; y < w.n; y += gridDim.y) {
    const int64_t v = g.unit_at(units, L.items[w.i0 + y].pos);
    if (at_rest(sd, v)) continue;
    const int64_t size = 1ll << glg[v], base = goff[v];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < size;
         i += (int64_t)gridDim.x * blockDim.x) {
      gk[base + i] = 0;
      gv[base + i] = 0;
    }
  }
}

// A hub's entries mostly fall into few communities, so adding each one to the global table
// would queue thousands of atomics on the same words: each block first sums its share of the
// entries in an LDS table of at most kHubLdsKeys keys (entries of further keys go straight to
// the global table), then adds each LDS key's sum to the global table once.
constexpr int kHubLdsLg = 11;
constexpr int kHubLdsKeys = 1 << (kHubLdsLg - 1);

template <class V>
__global__ __launch_bounds__(256) void k_hub_accum(V g, SolveDev sd, WinLevel L, int r,
                                                   const int32_t *units, const uint32_t *comm,
                                                   const int64_t *goff, const int32_t *glg,
                                                   uint32_t *gk, int64_t *gv, LmCounters pc) {
  __shared__ uint32_t sk[1 << kHubLdsLg];
  __shared__ int64_t sv[1 << kHubLdsLg];
  __shared__ int s_claimed;
  const WinRange win(L, kFamHub, r);
  for (int y = blockIdx.y; y < win.n; y += gridDim.y) {
    const int64_t v = g.unit_at(units, L.items[win.i0 + y].pos);
    if ((sd.frozen && sd.frozen[g.solve_of(v)]) || at_rest(sd, v)) continue;   // nothing to decide
    GTab tab{gk + goff[v], gv + goff[v], glg[v]};
    typename V::Row row = g.row(v, sd);
    for (int i = threadIdx.x; i < (1 << kHubLdsLg); i += blockDim.x) {
      sk[i] = 0;
      sv[i] = 0;
    }
    if (threadIdx.x == 0) s_claimed = 0;
    __syncthreads();
    constexpr uint32_t mask = (1u << kHubLdsLg) - 1;
    for (int64_t e = row.lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < row.hi;
         e += (int64_t)gridDim.x * blockDim.x) {
      int64_t w;
      const int64_t x = g.nbr(row, e, w);
      if (w == 0) continue;
      const uint32_t lab = g.lab_at(comm, e, x), key = lab + 1;
      uint32_t h = fib_hash(lab, 32 - kHubLdsLg);
      bool done = false;
      // at most kHubLdsKeys slots are ever claimed, so an empty slot is always reached
      for (;;) {
        const uint32_t k = sk[h];
        if (k == key) {
          atomicAdd(reinterpret_cast<unsigned long long *>(&sv[h]), (unsigned long long)w);
          done = true;
          break;
        }
        if (k == 0) {
          if (atomicAdd(&s_claimed, 1) >= kHubLdsKeys) break;   // LDS table closed to new keys
          const uint32_t prev = atomicCAS(&sk[h], 0u, key);
          if (prev == 0 || prev == key) {
            atomicAdd(reinterpret_cast<unsigned long long *>(&sv[h]), (unsigned long long)w);
            done = true;
            break;
          }
        }
        h = (h + 1) & mask;
      }
      if (!done) tab.add(lab, w);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < (1 << kHubLdsLg); i += blockDim.x)
      if (sk[i] != 0) tab.add(sk[i] - 1, sv[i]);
    if (pc.c && blockIdx.x == 0 && threadIdx.x == 0) {
      unsigned long long *c = pc.of(L.items[win.i0 + y].colour).c;
      atomicAdd(c + 0, 1ull);
      atomicAdd(c + 1, (unsigned long long)(row.hi - row.lo));
    }
    __syncthreads();   // the tables are reused for the next hub
  }
}

constexpr int kHubWin = 2048;   // table slots compacted at a time by a hub evaluation block

template <class P, class V>
__global__ __launch_bounds__(256) void k_hub_eval(V g, SolveDev sd, WinLevel L, int r,
                                                  const int32_t *units, const uint32_t *comm,
                                                  SliceTable sig, const int64_t *goff,
                                                  const int32_t *glg, const uint32_t *gk,
                                                  const int64_t *gv, typename P::Score *part,
                                                  LmCounters pc) {
  __shared__ typename P::Score red[4];
  __shared__ int32_t wl[kHubWin];
  __shared__ int wn;
  const WinRange win(L, kFamHub, r);
  const int32_t hub0 = L.ip[kFamHub * (L.ncol + 1)];
  if (sd.redo) sd.redo = L.near_tie + r * L.J;
  for (int y = blockIdx.y; y < win.n; y += gridDim.y) {
    const WinItem it = L.items[win.i0 + y];
    const int64_t v = g.unit_at(units, it.pos);
    if ((sd.frozen && sd.frozen[g.solve_of(v)]) || at_rest(sd, v)) continue;
    sd.mark = it.colour;
    const uint32_t D = comm[v];
    const uint32_t *K = gk + goff[v];
    const int64_t *Wt = gv + goff[v];
    const int64_t size = 1ll << glg[v];
    const int64_t span = (size + gridDim.x - 1) / gridDim.x;
    const int64_t s0 = (int64_t)blockIdx.x * span, s1 = s0 + span < size ? s0 + span : size;
    const UnitCtx u = unit_ctx(g, sd, v, D);
    typename P::Score best = P::make(g, u, sd, sig, kNone, 0, kEmpty);
    int ncand = 0;
    bool coop = false;
    if constexpr (!V::kLevel0 && IsMulti<P>::value) coop = u.m >= kCoopMinM;
    if (coop) {
      if constexpr (!V::kLevel0 && IsMulti<P>::value) {
        // the block's span of the table is mostly empty slots: each window of kHubWin slots is
        // first compacted into an LDS list of its candidates, and only those take coop turns
        const CoopLane c = coop_lane(g, u, sd, sig, threadIdx.x);
        const int sub = threadIdx.x / c.mp, nsub = blockDim.x / c.mp;
        for (int64_t w0 = s0; w0 < s1; w0 += kHubWin) {
          const int64_t w1 = w0 + kHubWin < s1 ? w0 + kHubWin : s1;
          if (threadIdx.x == 0) wn = 0;
          __syncthreads();
          for (int64_t i = w0 + threadIdx.x; i < w1; i += blockDim.x) {
            const uint32_t key = K[i];
            if (key != 0 && key - 1 != D) wl[atomicAdd(&wn, 1)] = (int32_t)(i - w0);
          }
          __syncthreads();
          const int nw = wn;
          for (int i0 = 0; i0 < nw; i0 += nsub * kCoopBatch) {
            uint32_t lab[kCoopBatch];
            int64_t W[kCoopBatch], y2[kCoopBatch];
            bool ok[kCoopBatch];
            for (int k = 0; k < kCoopBatch; k++) {
              const int ii = i0 + k * nsub + sub;
              const int64_t i = ii < nw ? w0 + wl[ii] : -1;
              const uint32_t key = i >= 0 ? K[i] : 0u;
              lab[k] = key - 1;
              ok[k] = key != 0;
              W[k] = ok[k] ? Wt[i] : 0;
              ok[k] = ok[k] && !P::prunable(u, W[k], best);
            }
            coop_lookup<kCoopBatch>(c, lab, ok, y2);
            for (int k = 0; k < kCoopBatch; k++) {
              if (!ok[k]) continue;
              ncand += c.j == 0;
              ScoreK sc = coop_score(u, c, lab[k], W[k], y2[k], kTarget);
              if (better<P>(g, u, sd, sig, sc, best)) best = sc;
            }
          }
          __syncthreads();   // the list is rewritten by the next window
        }
      }
    } else {
      for (int64_t i = s0 + threadIdx.x; i < s1; i += blockDim.x) {
        const uint32_t key = K[i];
        if (key == 0 || key - 1 == D) continue;
        const int64_t W = Wt[i];
        if (P::prunable(u, W, best)) continue;
        ncand++;
        typename P::Score sc = P::make(g, u, sd, sig, key - 1, W, kTarget);
        if (better<P>(g, u, sd, sig, sc, best)) best = sc;
      }
    }
    if (pc.c && ncand) atomicAdd(pc.of(it.colour).c + 2, (unsigned long long)ncand);
    best = group_best<P>(BlockGrp(), g, u, sd, sig, best, red);
    if (threadIdx.x == 0) part[(int64_t)(win.i0 + y - hub0) * gridDim.x + blockIdx.x] = best;
  }
}

template <class P, class V>
__global__ __launch_bounds__(64) void k_hub_final(V g, SolveDev sd, WinLevel L, int r,
                                                  const int32_t *units, const uint32_t *comm,
                                                  SliceTable sig, const int64_t *goff,
                                                  const int32_t *glg, const uint32_t *gk,
                                                  const int64_t *gv,
                                                  const typename P::Score *part, int nparts,
                                                  uint32_t *target, uint32_t fresh_base) {
  const WinRange win(L, kFamHub, r);
  const int32_t hub0 = L.ip[kFamHub * (L.ncol + 1)];
  if (sd.redo) sd.redo = L.near_tie + r * L.J;
  const int lane = threadIdx.x & 63;
  for (int y = blockIdx.x; y < win.n; y += gridDim.x) {
    const WinItem it = L.items[win.i0 + y];
    const int64_t v = g.unit_at(units, it.pos);
    if ((sd.frozen && sd.frozen[g.solve_of(v)]) || at_rest(sd, v)) {
      if (lane == 0) target[it.pos] = kNone;
      continue;
    }
    sd.mark = it.colour;
    const uint32_t D = comm[v];
    const UnitCtx u = unit_ctx(g, sd, v, D);
    typename P::Score best = P::make(g, u, sd, sig, kNone, 0, kEmpty);
    if (lane < nparts) best = part[(int64_t)(win.i0 + y - hub0) * nparts + lane];
    best = wave_best<P>(g, u, sd, sig, best);
    GTab tab{const_cast<uint32_t *>(gk) + goff[v], const_cast<int64_t *>(gv) + goff[v], glg[v]};
    const int64_t wD = tab.get(D);
    typename P::Score stay;
    bool coop = false;
    if constexpr (!V::kLevel0 && IsMulti<P>::value) coop = u.m >= kCoopMinM;
    if (coop) {
      if constexpr (!V::kLevel0 && IsMulti<P>::value)
        stay = coop_make(u, coop_lane(g, u, sd, sig, lane), D, wD, kStay);
    } else {
      stay = P::make(g, u, sd, sig, D, wD, kStay);
    }
    if (lane == 0) {
      uint32_t out = kNone;
      if (P::cmp(g, u, sd, sig, best, stay) > 0)
        out = best.lab == kNone ? fresh_of(sd, fresh_base) + (uint32_t)g.orig(v) : best.lab;
      Emit{target, L.first_move + r, it.colour}.put(it.pos, out);
      // the near-ties of the blocks that scanned the table are not known here
      const bool tied = LeavesTies<P>::value && u.m > 1;
      if (sd.rest)
        settle(sd, u, out, P::slack(u, stay, best), tied ? 0.0 : profile_max(g, u), tied);
    }
  }
}

// Apply the moves of pair r's window (those of its first moving colour): new label, Sigma delta
// for every profile slice, the label copy of level 0, the neighbours no longer at rest; and set up
// the next window.  Few units take a wave each, its lanes over the profile slices (up to 64, two
// Sigma atomics each) and the row; many units take a thread each, the long rows of the movers a
// wave.  Near-ties of the colours whose decisions count ask for a repeat of their solve's sweep.
template <class V>
__device__ inline void apply_sigma(const V &g, const SolveDev &sd, const SliceTable &sig, int64_t v,
                                   uint32_t D, uint32_t C, int jj, int64_t &share) {
  int gs;
  int64_t k;
  g.pent(v, jj, gs, k);
  tab_add(sig, gs, D, -(int32_t)k);
  tab_add(sig, gs, C, (int32_t)k);
  if (sd.rest) {
    atomicAdd(reinterpret_cast<unsigned long long *>(sd.ctr + gs), (unsigned long long)k);
    if (!V::kLevel0) share += (int64_t)((((uint64_t)k << 32) + sd.S[gs] - 1) / (uint64_t)sd.S[gs]);
  }
}
// entry e of a moved unit: its neighbour is not at rest any more, and reads the new label C
template <class V>
__device__ inline void apply_entry(const V &g, const SolveDev &sd, int64_t e, uint32_t C) {
  if (sd.rest) sd.rest[g.col[e] & 0x7fffffff].limit = 0;
  if constexpr (std::is_same<V, ViewP>::value) {
    if (g.elab) g.elab[g.prev[e]] = C;
  }
}

template <class V>
__global__ __launch_bounds__(256) void k_win_apply(V g, SolveDev sd, WinLevel L, int r,
                                                   const int32_t *units, const uint32_t *target,
                                                   uint32_t *comm, SliceTable sig,
                                                   uint32_t *moved, LmCounters pc,
                                                   unsigned long long *total) {
  __shared__ uint32_t s_moves;
  const WinState s = L.st[r];
  const int f = L.first_move[r];
  const bool live = s.c0 < s.c1, dirty = live && f < s.c1;
  if (blockIdx.x == 0) {
    if (threadIdx.x < 64) {
      const int next = (r + 1) % 3;
      const int c0 = !live ? s.c0 : dirty ? f + 1 : s.c1;
      int budget = s.budget;
      const int t = s.t;
      if (dirty && L.moved_at[f] < t - 1) {   // an unforeseen move: look less far ahead
        const int used = L.cost[c0] - L.cost[s.c0];
        budget = used > L.floor ? used : L.floor;
      } else if (live && !dirty && budget < kWinUnbounded) {
        budget *= 4;
      }
      const int c1 = win_end(L, t, c0, budget);
      if (threadIdx.x == 0) {
        if (dirty) L.moved_at[f] = t;
        L.st[next] = WinState{c0, c1, budget, s.windows + (live ? 1 : 0), t};
        L.first_move[(r + 2) % 3] = kNoColour;
      }
    }
    if (pc.c && live)
      for (int i = 4 * s.c0 + threadIdx.x; i < 4 * s.c1; i += blockDim.x) {
        unsigned long long *now = pc.of(i / 4).c + i % 4, *most = now + 4;
        const unsigned long long m = *now > *most ? *now : *most;
        const bool counts = i / 4 <= f;
        if (counts && m) atomicAdd(total + i % 4, m);
        *now = 0;
        *most = counts ? 0 : m;
      }
    if (L.near_tie)
      for (int j = threadIdx.x; j < L.J; j += blockDim.x) {
        const int c = L.near_tie[r * L.J + j];
        if (live && c < s.c1 && c <= f) sd.redo[j] = 0;
        L.near_tie[((r + 2) % 3) * L.J + j] = kNoColour;
      }
  }
  if (!dirty) return;
  const int lo = L.cptr[f], hi = L.cptr[f + 1];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int waves = gridDim.x * 4;
  bool rows = sd.rest != nullptr;   // moved units' rows are visited
  if constexpr (std::is_same<V, ViewP>::value) rows = rows || g.elab;
  if (hi - lo <= 2 * waves) {
    for (int i = lo + blockIdx.x * 4 + wv; i < hi; i += waves) {
      const uint32_t C = target[i];
      if (C == kNone) continue;
      const int64_t v = g.unit_at(units, i);
      const uint32_t D = comm[v];
      const int m = g.plen(v);
      const int j = g.solve_of(v);
      int64_t share = 0;
      for (int jj = lane; jj < m; jj += 64) apply_sigma(g, sd, sig, v, D, C, jj, share);
      if (!V::kLevel0 && sd.rest) share = wave_sum64(share);
      if (rows)
        for (int64_t e = g.rp[v] + lane; e < g.rp[v + 1]; e += 64) apply_entry(g, sd, e, C);
      if (lane == 0) {
        comm[v] = C;
        atomicAdd(moved + j, 1u);
        if (!V::kLevel0 && sd.rest)
          atomicAdd(reinterpret_cast<unsigned long long *>(sd.ctr + sd.nsl + j),
                    (unsigned long long)share);
      }
    }
    return;
  }
  if (threadIdx.x == 0) s_moves = 0;
  __syncthreads();
  uint32_t mine = 0;
  for (int i0 = lo + (blockIdx.x * 4 + wv) * 64; i0 < hi; i0 += waves * 64) {
    const int i = i0 + lane;
    const uint32_t C = i < hi ? target[i] : kNone;
    const bool mv = C != kNone;
    int64_t v = 0, share = 0;
    int j = 0;
    if (mv) {
      v = g.unit_at(units, i);
      j = g.solve_of(v);
      const uint32_t D = comm[v];
      const int m = g.plen(v);
      for (int jj = 0; jj < m; jj++) apply_sigma(g, sd, sig, v, D, C, jj, share);
      comm[v] = C;
      mine++;
    }
    if (L.J > 1) wave_count(moved, j, mv);
    if (!V::kLevel0 && sd.rest) wave_add64(sd.ctr + sd.nsl, j, share);
    if (rows) {
      int64_t e0 = 0, e1 = 0;
      if (mv) {
        e0 = g.rp[v];
        e1 = g.rp[v + 1];
      }
      const bool wide = e1 - e0 > 16;
      if (!wide)
        for (int64_t e = e0; e < e1; e++) apply_entry(g, sd, e, C);
      for (uint64_t b = __ballot(wide); b; b &= b - 1) {
        const int l = __builtin_ctzll(b);
        const int64_t a0 = __shfl(e0, l, 64), a1 = __shfl(e1, l, 64);
        const uint32_t c = (uint32_t)__shfl((int)C, l, 64);
        for (int64_t e = a0 + lane; e < a1; e += 64) apply_entry(g, sd, e, c);
      }
    }
  }
  if (L.J == 1) {
    if (mine) atomicAdd(&s_moves, mine);
    __syncthreads();
    if (threadIdx.x == 0 && s_moves) atomicAdd(moved, s_moves);
  }
}

// Profile entries per global slice (how many units of a level can hold a key in the slice's
// Sigma sub-table): an LDS histogram per block when the slices fit, else global atomics.
constexpr int kSliceHistMax = 4096;
__global__ void k_profile_slice_count(const int32_t *ps, int64_t ne, int nslices, int64_t *cnt) {
  __shared__ uint32_t h[kSliceHistMax];
  const bool lds = nslices <= kSliceHistMax;
  if (lds)
    for (int i = threadIdx.x; i < nslices; i += blockDim.x) h[i] = 0;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ne;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (lds) atomicAdd(&h[ps[i]], 1u);
    else atomicAdd(reinterpret_cast<unsigned long long *>(cnt + ps[i]), 1ull);
  }
  __syncthreads();
  if (lds)
    for (int i = threadIdx.x; i < nslices; i += blockDim.x)
      if (h[i]) atomicAdd(reinterpret_cast<unsigned long long *>(cnt + i), (unsigned long long)h[i]);
}

// Labels of the units of flagged solves back to their copy from the start of the sweep.
template <class V>
__global__ void k_restore_flagged(V g, int64_t n, const uint32_t *snap, const int32_t *redo,
                                  uint32_t *comm) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n && redo[g.usolve[v]] != kRedoUnset) comm[v] = snap[v];
}

// ------------------------------------------------------------------ level 0 by position
// The level-0 sweeps read the supra-CSR in colour-batch order (ViewP): position i holds unit
// units[i] of the level's sorted batch list.  These kernels lay it out once per level-0 visit.
__global__ void k_pos_of(const int32_t *units, int64_t n, int32_t *pos) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) pos[units[i]] = (int32_t)i;
}

// keys ordering the level's units by (batch key, label), ids ascending among equals
__global__ void k_pos_label_keys(const uint32_t *keys, const int32_t *units,
                                 const uint32_t *comm, int64_t n, uint64_t *out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = ((uint64_t)keys[i] << 32) | comm[units[i]];
}

// per position: degree (for the row starts), intra degree, slice, solve, labels
__global__ void k_pos_meta(View0 g, const int32_t *units, int64_t n, int64_t *deg, int32_t *pk,
                           int32_t *pslice, int32_t *psolve, const uint32_t *comm,
                           uint32_t *pcomm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > n) return;
  if (i == n) {
    deg[n] = 0;
    return;
  }
  const int64_t v = units[i];
  deg[i] = g.degree(v);
  int gs;
  int64_t kk;
  g.pent(v, 0, gs, kk);
  pk[i] = (int32_t)kk;
  pslice[i] = gs;
  if (psolve) psolve[i] = g.solve_of(v);
  pcomm[i] = comm[v];
}

// entries of one position: neighbour positions with the coupling flag, raw weights
// PosRows: the optional neighbour-label copy (labels of the level's start) and reverse entries
struct PosLabels {
  const uint32_t *comm;   // labels by unit id
  const int64_t *prp;     // row starts by position
  uint32_t *elab;         // nullptr: not built
  int32_t *prev;
};

__device__ inline void pos_row(const View0 &g, const SolveDev &sd, int64_t v, int64_t out,
                               const int32_t *pos, int32_t *pcol, int32_t *pw, int first,
                               int step, const PosLabels &pl) {
  const typename View0::Row r = g.row(v, sd);
  for (int64_t e = r.lo + first; e < r.hi; e += step) {
    const int32_t x = g.col[e];
    const bool coupling = !(x >= r.slo && x < r.shi);
    const int32_t px = pos[x];
    pcol[out + (e - r.lo)] = px | (coupling ? (int32_t)0x80000000 : 0);
    if (pw) pw[out + (e - r.lo)] = g.w[e];
    if (pl.elab) {
      pl.elab[out + (e - r.lo)] = pl.comm[x];
      pl.prev[out + (e - r.lo)] = (int32_t)(pl.prp[px] + g.rev[e]);
    }
  }
}

// Rows of at most 32 entries take kPosGroup lanes each, whose reads and writes of the row are
// consecutive (one thread each: 2.5 ms for 27.6M entries); longer rows are listed for a wave each.
constexpr int kPosGroup = 8;
__global__ __launch_bounds__(256) void k_pos_rows(View0 g, SolveDev sd, const int32_t *units, int64_t n,
                           const int64_t *prp, const int32_t *pos, int32_t *pcol, int32_t *pw,
                           int32_t *wide, uint32_t *nwide, PosLabels pl) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kPosGroup;
  const int gl = threadIdx.x % kPosGroup;
  const int64_t v = i < n ? units[i] : 0;
  const bool is_long = i < n && g.degree(v) > 32;
  wave_append(wide, nwide, is_long && gl == 0, (int32_t)i);
  if (i < n && !is_long) pos_row(g, sd, v, prp[i], pos, pcol, pw, gl, kPosGroup, pl);
}

__global__ void k_pos_rows_wide(View0 g, SolveDev sd, const int32_t *units, const int64_t *prp,
                                const int32_t *pos, int32_t *pcol, int32_t *pw,
                                const int32_t *wide, const uint32_t *nwide, PosLabels pl) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t k = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); k < *nwide;
       k += nw) {
    const int64_t i = wide[k];
    pos_row(g, sd, units[i], prp[i], pos, pcol, pw, lane, 64, pl);
  }
}

// global-table slots of the hub units, by position
__global__ void k_pos_gtab(const int32_t *hubs, int64_t cnt, const int32_t *pos,
                           const int64_t *goff, const int32_t *glg, int64_t *goffP,
                           int32_t *glgP) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cnt) return;
  const int64_t u = hubs[i];
  goffP[pos[u]] = goff[u];
  glgP[pos[u]] = glg[u];
}

__global__ void k_pos_labels_back(const int32_t *units, int64_t n, const uint32_t *pcomm,
                                  uint32_t *comm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) comm[units[i]] = pcomm[i];
}

// the label copy made current again after sweeps that did not keep it (entry order)
__global__ void k_pos_elab_refresh(const int32_t *pcol, int64_t nnz, const uint32_t *pcomm,
                                   uint32_t *elab) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz) elab[e] = pcomm[pcol[e] & 0x7fffffff];
}

// A refinement round taken again exactly for the solves that raised their redo flag only:
// their units get back the active flags and proposal stamps of the round's start; the other
// solves' units are set aside (inactive, so the proposal kernels skip them) and get their
// flags back afterwards (k_ref_redo_done), keeping their proposals of the first pass.
template <class V>
__global__ void k_ref_redo_prep(V g, int64_t n, const int32_t *redo, uint8_t *active,
                                const uint8_t *snap_a, uint32_t *propr, const uint32_t *snap_p,
                                uint8_t *keep) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  if (redo[g.solve_of(v)] != kRedoUnset) {
    active[v] = snap_a[v];
    propr[v] = snap_p[v];
  } else {
    keep[v] = active[v];
    active[v] = 0;
  }
}
template <class V>
__global__ void k_ref_redo_done(V g, int64_t n, const int32_t *redo, uint8_t *active,
                                const uint8_t *keep) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n && redo[g.solve_of(v)] == kRedoUnset) active[v] = keep[v];
}

template <class V>
__global__ void k_sigma_build(V g, int64_t n, const uint32_t *comm, SliceTable sig) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  int m = g.plen(v);
  for (int jj = 0; jj < m; jj++) {
    int gs;
    int64_t k;
    g.pent(v, jj, gs, k);
    tab_add(sig, gs, comm[v], (int32_t)k, false);
  }
}

__global__ void k_rebuild_check(const uint32_t *used, const uint32_t *limit, int nslices, int *flag) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nslices && used[s] > limit[s]) atomicOr(flag, 1);
}

// ------------------------------------------------------------------ colouring
// First-fit colouring in decreasing priority (Jones-Plassmann): a unit takes the smallest
// colour unused by its higher-priority neighbours once all of them are coloured.  The
// result equals the sequential greedy colouring in priority order.  Each unit counts its
// higher-priority neighbours once; a coloured unit marks its colour in the bitmaps of its
// lower-priority neighbours and then takes one off their counts, and whoever takes the last one
// off holds a unit whose colour is the first clear bit of its bitmap.  So a row is scanned twice
// (count, mark) and no colour is ever gathered.
//
// Rounds colour the units that are ready and collect those they release.  The time is the number
// of rounds (the longest chain of decreasing priorities, hundreds of units in dense aggregated
// levels) times a dozen dependent memory round trips each, so:
//   large levels (k_jp_round)  short rows take 8 lanes each while more units are ready than the
//                              chip has waves, else every unit takes a wave; rows above
//                              kJpWaveRow entries take the block;
//   small levels (k_jp_chain)  the units a block releases queue in its own LDS and its waves take
//                              them at once, up to kJpDepth links of a chain per round, which
//                              deals them out to the blocks again.  No block waits for another.
// Measured against rounds that gather colours, one wave per unit (small levels: one workgroup for
// the whole level): 3.2M units of degree 11 11.4 -> 9.1 ms, 207k of degree 72 15.1 -> 11.7 ms,
// 9k of degree 218 9.3 -> 4.4 ms.  Chains in large levels lose (99k units 3.8 -> 21 ms): blocks
// that release much keep it, and their waves queue up while others have left.
//
// Between waves of one launch everything travels through device-scope atomics, and a wave
// waits for its marks to be performed before it takes the counts down.
struct JpLists {
  int32_t *list[2];   // ready units by parity of the round
  // [0..2] their numbers (round r uses r % 3), [3] long rows of the count, [4] a wave gave up
  uint32_t *counts;
};
// What a colouring works on: counts of uncoloured higher-priority neighbours, colours, and
// `planes` bitmaps of 64 colours per unit (plane p of unit v at used[p * n + v]).  A colour
// beyond the planes is found by scanning the row (jp_scan_free).
struct JpState {
  uint32_t *cnt;
  int32_t *colour;
  unsigned long long *used;
  int64_t n;
  int planes;
};

// Rows longer than kJpCountThread entries are counted by a wave (k_jp_count_wide) instead
// of a single thread.
constexpr int kJpCountThread = 64;

template <class V>
__global__ __launch_bounds__(256) void k_jp_count(V g, SolveDev sd, const int32_t *work,
                                                  int64_t nwork, JpState s, int32_t *front,
                                                  uint32_t *nfront, int32_t *wide,
                                                  uint32_t *nwide, int it, int lvl) {
  // one thread per unit; ready units are appended once per wave
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool ready = false;
  int64_t v = 0;
  if (idx < nwork) {
    v = work[idx];
    for (int p = 0; p < s.planes; p++) s.used[p * s.n + v] = 0ull;
  }
  const bool long_row = idx < nwork && g.degree(v) > kJpCountThread;
  wave_append(wide, nwide, long_row, (int32_t)v);
  if (idx < nwork && !long_row) {
    const int j = g.solve_of(v);
    const uint64_t sm = sd.seedmix[j];
    const int64_t off = sd.uoff[j];
    const uint64_t hv = priority(sm, it, lvl, 0, (uint32_t)(v - off));
    typename V::Row row = g.row(v, sd);
    uint32_t c = 0;
    bool alone = true;
    for (int64_t e = row.lo; e < row.hi; e++) {
      int32_t x = g.col[e];
      if (!g.live(row, x)) continue;
      alone = false;
      uint64_t hx = priority(sm, it, lvl, 0, (uint32_t)(x - off));
      if (outranks(hx, (uint32_t)x, hv, (uint32_t)v)) c++;
    }
    s.cnt[v] = c;
    ready = c == 0 && !alone;
    if (alone) s.colour[v] = 0;   // no neighbours: nothing to wait for or to release
  }
  wave_append(front, nfront, ready, (int32_t)v);
}

// The long rows set aside by k_jp_count, one wave each; their number is read on the device.
template <class V>
__global__ __launch_bounds__(256) void k_jp_count_wide(V g, SolveDev sd, const int32_t *wide,
                                                       const uint32_t *nwide, uint32_t *cnt,
                                                       int32_t *front, uint32_t *nfront, int it,
                                                       int lvl) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = *nwide;
  for (int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); idx < nw;
       idx += (int64_t)gridDim.x * 4) {
    const int64_t v = wide[idx];
    const int j = g.solve_of(v);
    const uint64_t sm = sd.seedmix[j];
    const int64_t off = sd.uoff[j];
    const uint64_t hv = priority(sm, it, lvl, 0, (uint32_t)(v - off));
    typename V::Row row = g.row(v, sd);
    int64_t c = 0;
    for (int64_t e = row.lo + lane; e < row.hi; e += 64) {
      int32_t x = g.col[e];
      if (!g.live(row, x)) continue;
      uint64_t hx = priority(sm, it, lvl, 0, (uint32_t)(x - off));
      if (outranks(hx, (uint32_t)x, hv, (uint32_t)v)) c++;
    }
    for (int m = 32; m >= 1; m >>= 1) c += shfl_xor64(c, m);
    if (lane == 0) cnt[v] = (uint32_t)c;
    wave_append(front, nfront, lane == 0 && c == 0, (int32_t)v);
  }
}

// Waits until every memory operation of this wave has been performed.
__device__ inline void wave_drain() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// First colour of v that the planes leave free, or -1: the G lanes from lane gbase on hold one
// plane each and learn the same answer.
template <int G>
__device__ inline int jp_plane_free(const JpState &s, int64_t v) {
  const int lane = threadIdx.x & 63, gl = lane & (G - 1), gbase = lane & ~(G - 1);
  const uint64_t word = gl < s.planes ? __hip_atomic_load(s.used + gl * s.n + v, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT)
                                      : ~0ull;
  const uint64_t mask = (G == 64 ? ~0ull : ((1ull << G) - 1)) << gbase;
  const uint64_t freew = __ballot(~word != 0) & mask;
  const int L = freew ? __builtin_ctzll(freew) : gbase;
  const uint64_t wl = (uint64_t)__shfl((long long)word, L, 64);
  return freew ? (L - gbase) * 64 + __builtin_ctzll(~wl) : -1;
}

// The unit being coloured, and what its neighbours are compared with.
template <class V>
struct JpUnit {
  const V &g;
  typename V::Row row;
  int64_t v, off;
  uint64_t sm, hv;
  int it, lvl;
  __device__ JpUnit(const V &g_, const SolveDev &sd, int64_t v_, int it_, int lvl_)
      : g(g_), row(g_.row(v_, sd)), v(v_), it(it_), lvl(lvl_) {
    const int j = g.solve_of(v);
    sm = sd.seedmix[j];
    off = sd.uoff[j];
    hv = priority(sm, it, lvl, 0, (uint32_t)(v - off));
  }
  __device__ int64_t len() const { return row.hi - row.lo; }
  // the neighbour at offset i of the row when its priority is lower (or higher), else -1
  __device__ int32_t nbr(int64_t i, bool higher) const {
    const int64_t e = row.lo + i;
    if (e >= row.hi) return -1;
    const int32_t x = g.col[e];
    if (!g.live(row, x)) return -1;
    const uint64_t hx = priority(sm, it, lvl, 0, (uint32_t)(x - off));
    return outranks(hx, (uint32_t)x, hv, (uint32_t)v) == higher ? x : -1;
  }
  __device__ int32_t lower(int64_t i) const { return nbr(i, false); }
};

// First free colour from `base` on: the colours of the higher-priority neighbours of u are
// marked in an LDS bitmap of NW words (atomic OR), a window of 64*NW colours at a time.
// sync() orders the bitmap's clear, marks and reads among the threads that share it.
template <int NW, class V, class Sync>
__device__ inline int jp_scan_free(const JpUnit<V> &u, int first, int step, const int32_t *colour,
                                   int base, uint64_t *bits, Sync sync) {
  const int lane = threadIdx.x & 63;
  int result = -1;
  for (; result < 0; base += 64 * NW) {
    for (int i = first; i < NW; i += step) bits[i] = 0;
    sync();
    for (int64_t i = first; i < u.len(); i += step) {
      const int32_t x = u.nbr(i, true);
      if (x < 0) continue;
      const int d =
          __hip_atomic_load(colour + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - base;
      if (d >= 0 && d < 64 * NW) atomicOr((unsigned long long *)(bits + (d >> 6)), 1ull << (d & 63));
    }
    sync();
    // every wave reads the bitmap and finds the same first clear bit
    for (int w0 = 0; w0 < NW && result < 0; w0 += 64) {
      const uint64_t word = w0 + lane < NW ? bits[w0 + lane] : ~0ull;
      const uint64_t freew = __ballot(~word != 0);
      if (freew) {
        const int L = __builtin_ctzll(freew);
        const uint64_t wl = (uint64_t)__shfl((long long)word, L, 64);
        result = base + (w0 + L) * 64 + __builtin_ctzll(~wl);
      }
    }
    sync();
  }
  return result;
}

struct WaveLdsSync {
  // a wave's LDS operations complete in issue order; this only keeps the compiler from
  // moving them across the phases
  __device__ void operator()() const {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
};
struct BlockLdsSync {
  __device__ void operator()() const { __syncthreads(); }
};

// The colour c of a unit marked at its lower-priority neighbour x.
__device__ inline void jp_mark(const JpState &s, int64_t x, int c) {
  if (c < 64 * s.planes) atomicOr(s.used + (int64_t)(c >> 6) * s.n + x, 1ull << (c & 63));
}

// Colour unit v with one wave and release its lower-priority neighbours: put(ready, x) is called
// by the whole wave for the neighbours of one turn.
constexpr int kJpTurns = 4;   // entries per lane in flight together, kept between mark and release
template <int NW, class V, class Put>
__device__ inline void jp_wave(const V &g, const SolveDev &sd, int64_t v, const JpState &s, int it,
                               int lvl, uint64_t *bits, Put put) {
  const int lane = threadIdx.x & 63;
  int c = jp_plane_free<64>(s, v);
  const JpUnit<V> u(g, sd, v, it, lvl);
  if (c < 0) c = jp_scan_free<NW>(u, lane, 64, s.colour, 64 * s.planes, bits, WaveLdsSync());
  if (lane == 0) __hip_atomic_store(s.colour + v, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t len = u.len();
  int32_t low[kJpTurns];   // the first entries stay in registers
  for (int64_t e0 = 0; e0 < len; e0 += 64 * kJpTurns) {
    int32_t x[kJpTurns];
#pragma unroll
    for (int k = 0; k < kJpTurns; k++) x[k] = u.lower(e0 + 64 * k + lane);
#pragma unroll
    for (int k = 0; k < kJpTurns; k++) {
      if (x[k] >= 0) jp_mark(s, x[k], c);
      if (e0 == 0) low[k] = x[k];
    }
  }
  wave_drain();
  for (int64_t e0 = 0; e0 < len; e0 += 64 * kJpTurns) {
    int32_t x[kJpTurns];
    bool ready[kJpTurns];
#pragma unroll
    for (int k = 0; k < kJpTurns; k++) {
      x[k] = e0 == 0 ? low[k] : u.lower(e0 + 64 * k + lane);
      ready[k] = x[k] >= 0 && atomicSub(s.cnt + x[k], 1u) == 1u;
    }
#pragma unroll
    for (int k = 0; k < kJpTurns; k++)
      if (__ballot(ready[k])) put(ready[k], x[k]);
  }
}

// Colour one unit with the whole block (all threads must call this).
constexpr int kJpBlockWords = 64;
template <class V>
__device__ inline void jp_block(const V &g, const SolveDev &sd, int64_t v, const JpState &s,
                                WaveStage &st, int it, int lvl, uint64_t *bits) {
  const int tid = threadIdx.x, nt = blockDim.x;
  int c = jp_plane_free<64>(s, v);   // v's bitmap is complete: every wave finds the same
  const JpUnit<V> u(g, sd, v, it, lvl);
  if (c < 0)
    c = jp_scan_free<kJpBlockWords>(u, tid, nt, s.colour, 64 * s.planes, bits, BlockLdsSync());
  if (tid == 0) __hip_atomic_store(s.colour + v, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t len = u.len();
  for (int64_t e = tid; e < len; e += nt) {
    const int32_t x = u.lower(e);
    if (x >= 0) jp_mark(s, x, c);
  }
  wave_drain();
  __syncthreads();   // thread 0's colour is stored as well
  for (int64_t e0 = 0; e0 < len; e0 += nt) {
    const int32_t x = u.lower(e0 + tid);
    st.append(x >= 0 && atomicSub(s.cnt + x, 1u) == 1u, x);
  }
}

// One round with its frontier size read on the device, so rounds can be launched back to back
// without a host round trip: round r colours the list of parity r&1 (counts[r%3] units), appends
// the released units to the other list (counts[(r+1)%3]) and clears counts[(r+2)%3].  A round
// with an empty frontier does nothing.
constexpr int kJpGroup = 8;        // lanes of a short row
constexpr int kJpGroupRow = 64;     // entries a lane group takes
constexpr int kJpWaveRow = 256;     // entries a wave takes
constexpr int kJpWaveWords = (kJpWaveRow + 64) / 64;   // its colour lies within these bitmap words
constexpr int kJpLater = 256;       // rows a block sets aside for its waves, or for all of it
template <class V>
__global__ __launch_bounds__(256) void k_jp_round(V g, SolveDev sd, JpLists L, JpState s, int r,
                                                  int it, int lvl) {
  __shared__ uint64_t s_wave[4][kJpWaveWords];
  __shared__ uint64_t s_block[kJpBlockWords];
  __shared__ int32_t s_stage[4][kStage];
  __shared__ int32_t s_mid[kJpLater], s_big[kJpLater];
  __shared__ uint32_t s_nmid, s_nbig;
  const int64_t nf = L.counts[r % 3];
  const int32_t *list = L.list[r & 1];
  if (blockIdx.x == 0 && threadIdx.x == 0) L.counts[(r + 2) % 3] = 0;
  if ((int64_t)blockIdx.x * 4 >= nf) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  WaveStage st{s_stage[wv], L.list[(r & 1) ^ 1], L.counts + (r + 1) % 3, 0};
  if (threadIdx.x == 0) s_nmid = s_nbig = 0;
  __syncthreads();
  const int64_t waves = (int64_t)gridDim.x * 4, w0 = (int64_t)blockIdx.x * 4 + wv;
  auto put = [&](bool ready, int32_t x) { st.append(ready, x); };
  auto later = [&](int32_t *q, uint32_t *n, int32_t v) {   // one lane; full: the next round's
    const uint32_t i = atomicAdd(n, 1u);
    if (i < kJpLater) q[i] = v;
    return i < kJpLater;
  };
  if (nf > 2 * waves) {
    constexpr int kPer = 64 / kJpGroup;
    const int gl = lane & (kJpGroup - 1);
    for (int64_t i0 = w0 * kPer; i0 < nf; i0 += waves * kPer) {
      const int64_t i = i0 + lane / kJpGroup;
      bool on = i < nf, back = false;
      const int64_t v = on ? list[i] : list[i0];
      const JpUnit<V> u(g, sd, v, it, lvl);
      if (on && u.len() > kJpGroupRow) {
        if (gl == 0)
          back = u.len() > kJpWaveRow ? !later(s_big, &s_nbig, (int32_t)v)
                                      : !later(s_mid, &s_nmid, (int32_t)v);
        on = false;
      }
      const int c = jp_plane_free<kJpGroup>(s, v);
      if (on && c < 0) {   // beyond the planes: a wave scans the row
        if (gl == 0) back = !later(s_mid, &s_nmid, (int32_t)v);
        on = false;
      }
      constexpr int kTurns = kJpGroupRow / kJpGroup;
      int32_t low[kTurns];
      if (on && gl == 0)
        __hip_atomic_store(s.colour + v, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int k = 0; k < kTurns; k++) low[k] = on ? u.lower(k * kJpGroup + gl) : -1;
#pragma unroll
      for (int k = 0; k < kTurns; k++)
        if (low[k] >= 0) jp_mark(s, low[k], c);
      wave_drain();
      bool ready[kTurns];
#pragma unroll
      for (int k = 0; k < kTurns; k++)
        ready[k] = low[k] >= 0 && atomicSub(s.cnt + low[k], 1u) == 1u;
#pragma unroll
      for (int k = 0; k < kTurns; k++) st.append(ready[k], low[k]);
      st.append(back, (int32_t)v);
    }
  } else {
    for (int64_t i = w0; i < nf; i += waves) {
      const int64_t v = list[i];
      if (g.degree(v) <= kJpWaveRow) {
        jp_wave<kJpWaveWords>(g, sd, v, s, it, lvl, s_wave[wv], put);
        continue;
      }
      bool back = false;
      if (lane == 0) back = !later(s_big, &s_nbig, (int32_t)v);
      st.append(back, (int32_t)v);
    }
  }
  __syncthreads();
  const int nmid = s_nmid < kJpLater ? s_nmid : kJpLater, nbig = s_nbig < kJpLater ? s_nbig : kJpLater;
  for (int i = wv; i < nmid; i += 4)
    jp_wave<kJpWaveWords>(g, sd, (int64_t)s_mid[i], s, it, lvl, s_wave[wv], put);
  for (int i = 0; i < nbig; i++) jp_block(g, sd, (int64_t)s_big[i], s, st, it, lvl, s_block);
  st.flush();
}

constexpr int kJpThreads = 512;
constexpr int kJpWaves = kJpThreads / 64;
constexpr int kJpDepth = 16;       // links of a chain followed in one round
constexpr int kJpSlots = 2048;     // units a block may queue in one round
constexpr int kJpChainRow = 2048;  // longer rows take the block
constexpr int kJpChainWords = (kJpChainRow + 64) / 64;
constexpr int kJpUnitBits = 27;    // the depth sits above the unit id: chains are followed only in
                                   // levels of at most 2^27 units (graphs hold fewer than 2^32 / 33
                                   // and unions at most 100 * 2^20, whatever a solve's sweeps)
static_assert(kJpDepth <= 1 << (31 - kJpUnitBits), "unit and depth fit 31 bits: -1 is an empty slot");
constexpr uint32_t kJpPolls = 1u << 22;   // ends a wave's wait (seconds) should its block stall

// The units queued by the waves of one block (LDS).  Slots are claimed from `tail` on, then
// filled, and taken from `head` on; `busy` counts the units taken or queued and not finished, so
// that it is 0 only when no wave of the block can queue another one.
struct JpQueue {
  int32_t *slot;   // [kJpSlots], -1: not filled yet
  uint32_t *head, *tail, *busy, *next;   // next: units of the round's list taken by the block
  uint32_t *failed;

  // A wave's next unit (depth above bit kJpUnitBits) from the queue, else from the round's list
  // (positions blockIdx, blockIdx + gridDim, ...), or -1 when the block has nothing left.
  __device__ int32_t take(const int32_t *list, int64_t n) const {
    int32_t got = -1;
    if ((threadIdx.x & 63) == 0) {
      bool listed = true;   // the list may hold more for this block
      for (uint32_t polls = 0;; polls++) {
        const uint32_t h = load(head), t = load(tail);
        if (h < (t < kJpSlots ? t : kJpSlots)) {
          if (atomicCAS(head, h, h + 1) != h) continue;
          // whoever claimed it in push() fills it next and waits for nobody; bounded all the same
          for (uint32_t k = 0; k < kJpPolls; k++)
            if ((got = (int32_t)load((uint32_t *)slot + h)) >= 0) break;
          if (got < 0) atomicOr(failed, 1u);
          break;
        }
        if (listed) {
          atomicAdd(busy, 1u);
          const int64_t i = blockIdx.x + (int64_t)atomicAdd(next, 1u) * gridDim.x;
          if (i < n) {
            got = list[i];
            break;
          }
          atomicSub(busy, 1u);
          listed = false;
          continue;
        }
        if (load(busy) == 0) break;
        if (polls >= kJpPolls) {
          atomicOr(failed, 1u);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    return __shfl(got, 0, 64);
  }
  // queue x behind a unit of this block that is not finished; false when the queue is full
  __device__ bool push(int32_t x, int depth) const {
    const uint32_t i = atomicAdd(tail, 1u);
    if (i >= kJpSlots) return false;
    atomicAdd(busy, 1u);
    __hip_atomic_store(slot + i, x | (depth << kJpUnitBits), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_WORKGROUP);
    return true;
  }
  __device__ static uint32_t load(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};

// A round of a small level: as k_jp_round, and the units that a block releases are coloured in
// the same launch up to kJpDepth links down (what does not fit goes to the next round).
template <class V>
__global__ __launch_bounds__(kJpThreads) void k_jp_chain(V g, SolveDev sd, JpLists L, JpState s,
                                                         int r, int it, int lvl) {
  __shared__ uint64_t s_wave[kJpWaves][kJpChainWords];
  __shared__ uint64_t s_block[kJpBlockWords];
  __shared__ int32_t s_stage[kJpWaves][kStage];
  __shared__ int32_t s_slot[kJpSlots], s_big[kJpLater];
  __shared__ uint32_t s_q[5];
  const int64_t nf = L.counts[r % 3];
  if (blockIdx.x == 0 && threadIdx.x == 0) L.counts[(r + 2) % 3] = 0;
  if (blockIdx.x >= nf) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  WaveStage st{s_stage[wv], L.list[(r & 1) ^ 1], L.counts + (r + 1) % 3, 0};
  for (int i = threadIdx.x; i < kJpSlots; i += kJpThreads) s_slot[i] = -1;
  if (threadIdx.x < 5) s_q[threadIdx.x] = 0;
  __syncthreads();
  const JpQueue q{s_slot, s_q, s_q + 1, s_q + 2, s_q + 3, L.counts + 4};
  uint32_t *nbig = s_q + 4;
  for (;;) {
    const int32_t got = q.take(L.list[r & 1], nf);
    if (got < 0) break;
    int64_t v = got & ((1 << kJpUnitBits) - 1);
    for (int depth = got >> kJpUnitBits; v >= 0; depth++) {
      int64_t next = -1;
      if (g.degree(v) > kJpChainRow) {   // set aside for the block, or for the next round
        uint32_t i = kJpLater;
        if (lane == 0 && (i = atomicAdd(nbig, 1u)) < kJpLater) s_big[i] = (int32_t)v;
        st.append(lane == 0 && i >= kJpLater, (int32_t)v);
      } else {
        jp_wave<kJpChainWords>(g, sd, v, s, it, lvl, s_wave[wv], [&](bool ready, int32_t x) {
          if (depth + 1 < kJpDepth) {
            const uint64_t bal = __ballot(ready);
            if (next < 0 && bal) {   // this wave goes on with one of them
              const int first = __builtin_ctzll(bal);
              next = __shfl(x, first, 64);
              if (lane == first) ready = false;
            }
            if (ready && q.push(x, depth + 1)) ready = false;
          }
          st.append(ready, x);
        });
      }
      v = next;
    }
    if (lane == 0) atomicSub(q.busy, 1u);   // its chain is done
  }
  __syncthreads();
  const int nb = *nbig < kJpLater ? *nbig : kJpLater;
  for (int i = 0; i < nb; i++) jp_block(g, sd, (int64_t)s_big[i], s, st, it, lvl, s_block);
  st.flush();
}

// sort key of a unit for batching: colour, then degree bin
// (inactive: the key of units of solves that sit this iteration out, above every real key)
template <class V>
__global__ void k_batch_keys(V g, int64_t n, const int32_t *colour, const uint8_t *sactive,
                             uint32_t inactive, uint32_t *keys, uint32_t *vals) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  vals[v] = (uint32_t)v;
  if (!sactive[g.usolve[v]]) {
    keys[v] = inactive;
    return;
  }
  keys[v] = ((uint32_t)colour[v] << kBatchShift) | batch_slot(g, v);
}

template <class V>
__global__ void k_bin_keys(V g, int64_t n, const uint8_t *sactive, uint32_t *keys, uint32_t *vals) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  vals[v] = (uint32_t)v;
  uint32_t bin = kNumBins;
  if (sactive[g.usolve[v]]) bin = unit_bin(g, v);
  keys[v] = bin;
}
// first[key] = first position of key in a sorted key array (keys below nkeys only)
__global__ void k_key_bounds(const uint32_t *sk, int64_t n, uint32_t nkeys, int64_t *first) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t k = sk[i];
  if (k < nkeys && (i == 0 || sk[i - 1] != k)) first[k] = i;
}

// per unit of the global-table bin: table size (power of two >= 2*degree), by unit id
template <class V>
__global__ void k_gtab_sizes(V g, const int32_t *units, int64_t count, int64_t *sz, int32_t *lg) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  int64_t v = units[i];
  int64_t d = g.degree(v);
  int l = 4;
  while ((1ll << l) < 2 * d) l++;
  lg[v] = l;
  sz[i] = 1ll << l;
}
__global__ void k_gtab_assign(const int32_t *units, int64_t count, const int64_t *off,
                              int64_t *goff) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) goff[units[i]] = off[i];
}

// ------------------------------------------------------------------ work-list segments
// Refinement work lists by degree: lane groups of 4, 8, 16 and 32 lanes (degree up to the
// group size), waves, LDS blocks, global tables.
constexpr int kRefLists = 7;
struct Segs {
  const int32_t *p[kRefLists];
  int64_t pre[kRefLists + 1];   // prefix sums of the segment lengths
  __device__ int seg(int64_t i) const {
    int k = 0;
    while (k < kRefLists - 1 && i >= pre[k + 1]) k++;
    return k;
  }
  __device__ int64_t unit(int64_t i) const {
    const int k = seg(i);
    return p[k][i - pre[k]];
  }
  __device__ int64_t total() const { return pre[kRefLists]; }
};
struct SegOut {
  int32_t *p[kRefLists];
};

// keep the units whose flag is still set, segment by segment
__global__ __launch_bounds__(256) void k_compact_segs(Segs in, const uint8_t *flag, SegOut out,
                                                      uint32_t *cnt) {
  __shared__ uint32_t s_app[256 / 64 + 1];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i < in.total();
  const int ks = live ? in.seg(i) : -1;
  // a block may straddle segments: append segment by segment, one atomic per block and list
  for (int k = 0; k < kRefLists; k++) {
    bool keep = false;
    int32_t v = 0;
    if (ks == k) {
      v = (int32_t)in.unit(i);
      keep = flag[v] != 0;
    }
    if (__syncthreads_or(ks == k)) block_append(out.p[k], cnt + k, keep, v, s_app);
  }
}

// ------------------------------------------------------------------ refinement
// Leiden refinement inside each community (Section 3.2 citing Traag et al.): singletons
// that are well connected to their community merge into well-connected sub-communities
// of positive gain; a proposer merges only if it outranks every proposing neighbour of
// its community, so each merge joins a frozen sub-community along an edge and
// sub-communities stay connected.

// Rows up to kRefThreadRow entries are scanned by the unit's own thread; longer ones are set
// aside for a wave each (most units of a refinement pass need no scan at all).
constexpr int kRefThreadRow = 64;

// Refinement starts from singletons: R = id, ext = weight to the own community, slice mask,
// and each unit's Sigma in the refined table.  first/step: this thread's share of the row
// and profile (a thread for a short row, a wave's lanes for a long one).
template <class V>
__device__ inline void ref_init_unit(const V &g, const SolveDev &sd, int64_t v,
                                     const uint32_t *comm, uint32_t *R, int64_t *ext,
                                     uint64_t *mask, SliceTable sr, int first, int step,
                                     bool wave) {
  const uint32_t D = comm[v];
  typename V::Row row = g.row(v, sd);
  int64_t s = 0;
  for (int64_t e = row.lo + first; e < row.hi; e += step) {
    int32_t x = g.col[e];
    if (comm[x] == D) s += g.wt(row, e, x);
  }
  if (wave) s = wave_sum64(s);
  const int m = g.plen(v);
  const int j = g.usolve[v];
  uint64_t mk = 0;
  for (int jj = 0; jj < m; jj++) {
    int gs;
    int64_t k;
    g.pent(v, jj, gs, k);
    mk |= 1ull << (gs - sd.sfirst[j]);
    if (jj % step == first) tab_add(sr, gs, (uint32_t)v, (int32_t)k, false);
  }
  if (first == 0) {
    R[v] = (uint32_t)v;
    ext[v] = s;
    mask[v] = mk;
  }
}

template <class V>
__global__ __launch_bounds__(256) void k_ref_init(V g, SolveDev sd, int64_t n, const uint32_t *comm,
                                                  uint32_t *R, int64_t *ext, uint64_t *mask,
                                                  SliceTable sr, int32_t *wide, uint32_t *nwide) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = v < n;
  const bool defer = live && (g.degree(v) > kRefThreadRow || g.plen(v) > kRefThreadRow);
  if (live && !defer) ref_init_unit(g, sd, v, comm, R, ext, mask, sr, 0, 1, false);
  wave_append(wide, nwide, defer, (int32_t)v);
}

template <class V>
__global__ __launch_bounds__(256) void k_ref_init_wide(V g, SolveDev sd, const int32_t *wide,
                                                       const uint32_t *nwide,
                                                       const uint32_t *comm, uint32_t *R,
                                                       int64_t *ext, uint64_t *mask,
                                                       SliceTable sr) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = *nwide;
  for (int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); idx < nw;
       idx += (int64_t)gridDim.x * 4)
    ref_init_unit(g, sd, (int64_t)wide[idx], comm, R, ext, mask, sr, lane, 64, true);
}

// Well-connectedness of sub-community T within its community K:
//   q*ext(T) - p*b * sum_s x_s (K_s - x_s) / S_s >= 0,  x_s = Sigma_R(T, s), K_s = Sigma(K, s).
template <class V>
__global__ __launch_bounds__(256) void k_ref_wc(V g, SolveDev sd, const int32_t *list,
                                                int64_t count, const uint32_t *comm,
                                                const int64_t *ext, const uint64_t *mask,
                                                SliceTable sr, SliceTable sig, uint8_t *wcT,
                                                uint8_t *active, uint32_t *changed) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int64_t T = list ? list[i] : i;
  if (changed) changed[T] = 0;
  const int j = g.usolve[T];
  const int64_t q = sd.q[j], pb = sd.pb[j];
  const uint32_t K = comm[T];
  const int base = sd.sfirst[j];
  uint64_t mk = mask[T];
  int m = 0;
  int gs0 = 0;
  int64_t c0 = 0;
  double acc = 0, mag = 0;
  for (uint64_t b = mk; b; b &= b - 1) {
    int gs = base + __builtin_ctzll(b);
    int64_t x = tab_get(sr, gs, (uint32_t)T);
    if (x == 0) continue;
    int64_t c = x * ((int64_t)tab_get(sig, gs, K) - x);
    if (m == 0) {
      gs0 = gs;
      c0 = c;
    }
    m++;
    double t = sd.rS[gs].of((double)c);
    acc += t;
    mag += fabs(t);
  }
  int sign;
  if (m <= 1) {
    i128 val = (i128)q * ext[T] * (m ? sd.S[gs0] : 1) - (i128)pb * c0;
    sign = val < 0 ? -1 : (val > 0 ? 1 : 0);
  } else if (mag == 0.0 || pb == 0) {
    sign = ext[T] > 0 ? 1 : (ext[T] < 0 ? -1 : 0);
  } else {
    const double qw = (double)q * (double)ext[T] * sd.scale[j];
    const double all = fabs(qw) + (double)pb * mag;
    const double ap = qw - (double)pb * acc;
    const double er = all < sd.scale[sd.J + j] ? 0.0 : (double)(m + 8) * 0x1p-50 * all;
    if (er == 0.0) {   // exact: one common denominator
      sign = ap > 0 ? 1 : (ap < 0 ? -1 : 0);
    } else if (fabs(ap) > er) {
      sign = ap > 0 ? 1 : -1;
    } else {
      atomicAdd(reinterpret_cast<unsigned long long *>(sd.fallbacks + j), 1ull);
      ExactAcc ea;
      ea.init();
      for (uint64_t b = mk; b; b &= b - 1) {
        int gs = base + __builtin_ctzll(b);
        int64_t x = tab_get(sr, gs, (uint32_t)T);
        if (x == 0) continue;
        ea.term(x * ((int64_t)tab_get(sig, gs, K) - x), sd.S[gs]);
      }
      sign = ea.sign(q, ext[T], pb);
    }
  }
  wcT[T] = sign >= 0;
  if (active) active[T] = sign >= 0;
}

// Proposal of one active singleton: best well-connected sub-community of positive gain.
template <class P, class V, class Grp, class Tab>
__device__ inline void ref_unit(Grp grp, Tab tab, const V &g, const SolveDev &sd, int64_t v,
                                const uint32_t *comm, const uint32_t *R, const uint8_t *wcT,
                                const SliceTable &sr, uint32_t *prop, uint32_t *propr,
                                uint32_t stamp, int64_t *propw, uint8_t *active,
                                typename P::Score *red, int64_t *sredW = nullptr,
                                uint32_t *sredL = nullptr) {
  const int r = grp.rank(), gsz = grp.size();
  for (int i = r; i < tab.size(); i += gsz) {
    tab.K[i] = 0;
    tab.V[i] = 0;
  }
  tab.reset(r);
  grp.sync();
  const uint32_t D = comm[v];
  typename V::Row row = g.row(v, sd);
  for (int64_t e = row.lo + r; e < row.hi; e += gsz) {
    int32_t x = g.col[e];
    if (comm[x] != D) continue;
    int64_t w = g.wt(row, e, x);
    if (w == 0) continue;
    tab.add(R[x], w);
  }
  grp.sync();
  UnitCtx u = unit_ctx(g, sd, v, D);
  const typename P::Score zero = P::make(g, u, sd, sr, kNone, 0, kEmpty);
  typename P::Score best = zero;
  int64_t hW;
  uint32_t hL;
  group_heaviest(grp, tab, kNone, wcT, hW, hL, sredW, sredL);
  bool coop = false;
  if constexpr (!V::kLevel0 && IsMulti<P>::value) coop = u.m >= kCoopMinM;
  if (coop) {
    if constexpr (!V::kLevel0 && IsMulti<P>::value) {
      // one profile slice per lane, subgroups take the sub-communities in turn (every lane of
      // a subgroup runs the same turns)
      const CoopLane c = coop_lane(g, u, sd, sr, r);
      const int sub = r / c.mp, nsub = gsz / c.mp;
      if (hL != kNone) {
        ScoreK s = coop_make(u, c, hL, hW, kTarget);
        if (P::cmp(g, u, sd, sr, s, zero) > 0) best = s;
      }
      const int nc = tab.count();
      for (int i0 = 0; i0 < nc; i0 += nsub * kCoopBatch) {
        uint32_t lab[kCoopBatch];
        int64_t W[kCoopBatch], y[kCoopBatch];
        bool ok[kCoopBatch];
        for (int k = 0; k < kCoopBatch; k++) {
          const int i = i0 + k * nsub + sub;
          const int h = i < nc ? tab.slot(i) : 0;
          const uint32_t key = i < nc ? tab.K[h] : 0u;
          lab[k] = key - 1;
          ok[k] = key != 0 && key - 1 != hL && wcT[key - 1];
          W[k] = ok[k] ? tab.V[h] : 0;
          ok[k] = ok[k] && !P::prunable(u, W[k], best);
        }
        coop_lookup<kCoopBatch>(c, lab, ok, y);
        for (int k = 0; k < kCoopBatch; k++) {
          if (!ok[k]) continue;
          ScoreK s = coop_score(u, c, lab[k], W[k], y[k], kTarget);
          if (P::cmp(g, u, sd, sr, s, zero) <= 0) continue;
          if (better<P>(g, u, sd, sr, s, best)) best = s;
        }
      }
    }
  } else {
    if (hL != kNone) {
      typename P::Score s = P::make(g, u, sd, sr, hL, hW, kTarget);
      if (P::cmp(g, u, sd, sr, s, zero) > 0) best = s;
    }
    const int nc = tab.count();
    for (int i = r; i < nc; i += gsz) {
      const int h = tab.slot(i);
      uint32_t key = tab.K[h];
      if (key == 0) continue;
      uint32_t T = key - 1;
      if (T == hL || !wcT[T]) continue;
      if (P::prunable(u, tab.V[h], best)) continue;
      typename P::Score s = P::make(g, u, sd, sr, T, tab.V[h], kTarget);
      if (P::cmp(g, u, sd, sr, s, zero) <= 0) continue;
      if (better<P>(g, u, sd, sr, s, best)) best = s;
    }
  }
  best = group_best<P>(grp, g, u, sd, sr, best, red);
  int64_t w = best.lab == kNone ? 0 : tab.get(best.lab);
  grp.sync();
  if (r == 0) {
    if (best.lab == kNone) {
      active[v] = 0;
    } else {
      prop[v] = best.lab;
      propw[v] = w;
      propr[v] = stamp;
    }
  }
}

// Proposals of units of degree <= G with G lanes each: neighbours inside the community are
// merged by sub-community with shuffles, every leader evaluates its sub-community (well
// connected, positive gain), and the group reduces to the best (ties to the lower label).
template <class P, class V, int G>
__global__ __launch_bounds__(256) void k_ref_group(V g, SolveDev sd, const int32_t *units,
                                                   int64_t count, const uint32_t *comm,
                                                   const uint32_t *R, const uint8_t *wcT,
                                                   SliceTable sr, uint32_t *prop, uint32_t *propr,
                                                   uint32_t stamp, int64_t *propw,
                                                   uint8_t *active) {
  const int lane = threadIdx.x & 63;
  const int gl = lane & (G - 1);
  const int gbase = lane & ~(G - 1);
  const int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  if (idx >= count) return;   // whole groups leave together
  const int64_t v = units[idx];
  if (!active[v]) return;
  const uint32_t D = comm[v];
  typename V::Row row = g.row(v, sd);
  const int64_t e = row.lo + gl;
  uint32_t c = kNone;
  int64_t w = 0;
  if (e < row.hi) {
    const int32_t x = g.col[e];
    if (comm[x] == D) {
      w = g.wt(row, e, x);
      if (w != 0) c = R[x];
    }
  }
  int64_t wsum = 0;
  bool leader = c != kNone;
  for (int j = 0; j < G; j++) {
    const uint32_t cj = (uint32_t)__shfl((int)c, gbase + j, 64);
    const int64_t wj = __shfl(w, gbase + j, 64);
    if (cj == c) {
      wsum += wj;
      if (j < gl) leader = false;
    }
  }
  const UnitCtx u = unit_ctx(g, sd, v, D);
  const typename P::Score zero = P::make(g, u, sd, sr, kNone, 0, kEmpty);
  typename P::Score best = zero;
  if (leader && wcT[c]) {
    typename P::Score s = P::make(g, u, sd, sr, c, wsum, kTarget);
    if (P::cmp(g, u, sd, sr, s, zero) > 0) best = s;
  }
  for (int m = G / 2; m >= 1; m >>= 1) {
    typename P::Score o = P::shfl(best, m);
    if (better<P>(g, u, sd, sr, o, best)) best = o;
  }
  // the weight to the chosen sub-community sits with its leader
  const uint64_t gmask = (G == 64 ? ~0ull : ((1ull << G) - 1)) << gbase;
  const uint64_t bal = __ballot(leader && c == best.lab) & gmask;
  const int src = bal ? __builtin_ctzll(bal) : gbase;
  const int64_t wb = __shfl(wsum, src, 64);
  if (gl == 0) {
    if (best.lab == kNone) {
      active[v] = 0;
    } else {
      prop[v] = best.lab;
      propw[v] = wb;
      propr[v] = stamp;
    }
  }
}

template <class P, class V>
__global__ __launch_bounds__(256) void k_ref_prop_wave(V g, SolveDev sd, const int32_t *units,
                                                       int64_t count, const uint32_t *comm,
                                                       const uint32_t *R, const uint8_t *wcT,
                                                       SliceTable sr, uint32_t *prop, uint32_t *propr,
                                                       uint32_t stamp, int64_t *propw,
                                                       uint8_t *active) {
  __shared__ uint32_t sk[4][1 << kWaveLg];
  __shared__ int64_t sv[4][1 << kWaveLg];
  __shared__ uint16_t sl[4][kWaveMaxDeg];
  __shared__ int sn[4];
  const int wv = threadIdx.x >> 6;
  const int64_t idx = (int64_t)blockIdx.x * 4 + wv;
  if (idx >= count) return;
  const int64_t v = units[idx];
  if (!active[v]) return;
  LdsTab tab{sk[wv], sv[wv], kWaveLg, sl[wv], sn + wv};
  ref_unit<P>(WaveGrp(), tab, g, sd, v, comm, R, wcT, sr, prop, propr, stamp, propw, active,
              (typename P::Score *)nullptr);
}

template <class P, class V, int NT>
__global__ __launch_bounds__(NT) void k_ref_prop_block(V g, SolveDev sd, const int32_t *units,
                                                         int64_t count, const uint32_t *comm,
                                                         const uint32_t *R, const uint8_t *wcT,
                                                         SliceTable sr, uint32_t *prop,
                                                         uint32_t *propr, uint32_t stamp,
                                                         int64_t *propw, uint8_t *active) {
  __shared__ uint32_t sk[1 << kBlockLg];
  __shared__ int64_t sv[1 << kBlockLg];
  __shared__ uint16_t sl[kBlockMaxDeg];
  __shared__ int sn;
  __shared__ typename P::Score red[NT / 64];
  __shared__ int64_t hw[NT / 64];
  __shared__ uint32_t hl[NT / 64];
  LdsTab tab{sk, sv, kBlockLg, sl, &sn};
  for (int64_t idx = blockIdx.x; idx < count; idx += gridDim.x) {
    const int64_t v = units[idx];
    if (!active[v]) continue;
    ref_unit<P>(BlockGrp(), tab, g, sd, v, comm, R, wcT, sr, prop, propr, stamp, propw, active,
                red, hw, hl);
  }
}

template <class P, class V>
__global__ __launch_bounds__(256) void k_ref_prop_gtab(V g, SolveDev sd, const int32_t *units,
                                                       int64_t count, const uint32_t *comm,
                                                       const uint32_t *R, const uint8_t *wcT,
                                                       SliceTable sr, uint32_t *prop, uint32_t *propr,
                                                       uint32_t stamp, int64_t *propw,
                                                       uint8_t *active, uint32_t *gk, int64_t *gv,
                                                       const int64_t *goff, const int32_t *glg) {
  __shared__ typename P::Score red[4];
  __shared__ int64_t hw[4];
  __shared__ uint32_t hl[4];
  for (int64_t idx = blockIdx.x; idx < count; idx += gridDim.x) {
    const int64_t v = units[idx];
    if (!active[v]) continue;
    GTab tab{gk + goff[v], gv + goff[v], glg[v]};
    ref_unit<P>(BlockGrpG(), tab, g, sd, v, comm, R, wcT, sr, prop, propr, stamp, propw, active,
                red, hw, hl);
  }
}

// A proposer merges when its target sub-community keeps all its members this round:
//  (a) the target's founder does not propose (sub-communities with two or more members never
//      propose), or
//  (b) the proposer outranks every proposing neighbour of its community, and the target's
//      founder proposes to a target whose own founder proposes (so the founder cannot move).
// Proposals and eligibility carry the round's stamp instead of being cleared.

template <class V>
__device__ inline bool ref_beaten(const V &g, const SolveDev &sd, int64_t v, const uint32_t *comm,
                                  const uint32_t *propr, uint32_t stamp, int first, int step,
                                  int it, int lvl) {
  const int j = g.usolve[v];
  const uint64_t sm = sd.seedmix[j];
  const int64_t off = sd.uoff[j];
  const uint64_t hv = priority(sm, it, lvl, 1, (uint32_t)(v - off));
  const uint32_t D = comm[v];
  typename V::Row row = g.row(v, sd);
  bool beaten = false;
  for (int64_t e = row.lo + first; e < row.hi; e += step) {
    int32_t x = g.col[e];
    if (comm[x] != D || propr[x] != stamp) continue;
    if (g.wt(row, e, x) == 0) continue;
    uint64_t hx = priority(sm, it, lvl, 1, (uint32_t)(x - off));
    if (outranks(hx, (uint32_t)x, hv, (uint32_t)v)) {
      beaten = true;
      break;
    }
  }
  return beaten;
}

template <class V>
__global__ __launch_bounds__(256) void k_ref_eligible(V g, SolveDev sd, Segs segs,
                                                      const uint32_t *comm, const uint32_t *prop,
                                                      const uint32_t *propr, uint32_t stamp,
                                                      uint32_t *elig, int32_t *wide,
                                                      uint32_t *nwide, int it, int lvl) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool defer = false;
  int64_t v = 0;
  if (idx < segs.total()) {
    v = segs.unit(idx);
    if (propr[v] == stamp) {
      const uint32_t T = prop[v];
      if (propr[T] != stamp) {
        elig[v] = stamp;
      } else if (propr[prop[T]] == stamp) {
        if (g.degree(v) > kRefThreadRow) defer = true;
        else if (!ref_beaten(g, sd, v, comm, propr, stamp, 0, 1, it, lvl)) elig[v] = stamp;
      }
    }
  }
  wave_append(wide, nwide, defer, (int32_t)v);
}

// the long rows set aside above, one wave each (their number is read on the device)
template <class V>
__global__ __launch_bounds__(256) void k_ref_eligible_wide(V g, SolveDev sd, const int32_t *wide,
                                                           const uint32_t *nwide,
                                                           const uint32_t *comm,
                                                           const uint32_t *propr, uint32_t stamp,
                                                           uint32_t *elig, int it, int lvl) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = *nwide;
  for (int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); idx < nw;
       idx += (int64_t)gridDim.x * 4) {
    const int64_t v = wide[idx];
    int beaten = ref_beaten(g, sd, v, comm, propr, stamp, lane, 64, it, lvl) ? 1 : 0;
    for (int m = 32; m >= 1; m >>= 1) beaten |= __shfl_xor(beaten, m, 64);
    if (lane == 0 && !beaten) elig[v] = stamp;
  }
}

// Merge every eligible proposer into its target; edges between co-joiners of the same target
// become internal as well.
template <class V>
__device__ inline void ref_merge(const V &g, const SolveDev &sd, int64_t v, const uint32_t *prop,
                                 const int64_t *propw, const uint32_t *elig, uint32_t stamp,
                                 uint32_t *R, int64_t *ext, uint64_t *mask, uint8_t *active,
                                 SliceTable sr, int first, int step, bool wave) {
  const uint32_t T = prop[v];
  typename V::Row row = g.row(v, sd);
  int64_t corr = 0;
  for (int64_t e = row.lo + first; e < row.hi; e += step) {
    int32_t x = g.col[e];
    if (elig[x] == stamp && prop[x] == T) corr += g.wt(row, e, x);
  }
  if (wave) corr = wave_sum64(corr);
  const int m = g.plen(v);
  for (int jj = first; jj < m; jj += step) {
    int gs;
    int64_t k;
    g.pent(v, jj, gs, k);
    tab_add(sr, gs, T, (int32_t)k, false);
  }
  if (first == 0) {
    R[v] = T;
    active[v] = 0;
    active[T] = 0;
    atomicAdd(reinterpret_cast<unsigned long long *>(ext + T),
              (unsigned long long)(ext[v] - 2 * propw[v] - corr));
    atomicOr(reinterpret_cast<unsigned long long *>(mask + T), (unsigned long long)mask[v]);
  }
}

template <class V>
__global__ __launch_bounds__(256) void k_ref_apply(V g, SolveDev sd, Segs segs, const uint32_t *prop,
                                                   const int64_t *propw, const uint32_t *elig,
                                                   uint32_t stamp, uint32_t *R, int64_t *ext,
                                                   uint64_t *mask, uint8_t *active,
                                                   int32_t *wide, uint32_t *nwide, SliceTable sr) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool defer = false;
  int64_t v = 0;
  if (idx < segs.total()) {
    v = segs.unit(idx);
    if (elig[v] == stamp) {
      if (g.degree(v) > kRefThreadRow || g.plen(v) > kRefThreadRow) defer = true;
      else ref_merge(g, sd, v, prop, propw, elig, stamp, R, ext, mask, active, sr, 0, 1, false);
    }
  }
  wave_append(wide, nwide, defer, (int32_t)v);
}

template <class V>
__global__ __launch_bounds__(256) void k_ref_apply_wide(V g, SolveDev sd, const int32_t *wide,
                                                        const uint32_t *nwide,
                                                        const uint32_t *prop,
                                                        const int64_t *propw,
                                                        const uint32_t *elig, uint32_t stamp,
                                                        uint32_t *R, int64_t *ext, uint64_t *mask,
                                                        uint8_t *active, SliceTable sr) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = *nwide;
  for (int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); idx < nw;
       idx += (int64_t)gridDim.x * 4)
    ref_merge(g, sd, (int64_t)wide[idx], prop, propw, elig, stamp, R, ext, mask, active, sr, lane,
              64, true);
}

// merges per solve and the queue of sub-communities that received members (convergent)
template <class V>
__global__ __launch_bounds__(256) void k_ref_post(V g, Segs segs, const uint32_t *prop,
                                                  const uint32_t *elig, uint32_t stamp,
                                                  uint32_t *changed, int32_t *clist,
                                                  uint32_t *ccount, uint32_t *nelig) {
  __shared__ uint32_t s_app[256 / 64 + 1];
  __shared__ uint32_t s_merges;
  __shared__ int s_j, s_mixed;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool merged = false, first = false;
  int j = 0;
  uint32_t T = 0;
  if (threadIdx.x == 0) {
    s_merges = 0;
    s_mixed = 0;
    s_j = -1;
  }
  __syncthreads();
  if (i < segs.total()) {
    const int64_t v = segs.unit(i);
    if (elig[v] == stamp) {
      merged = true;
      j = g.usolve[v];
      T = prop[v];
      first = atomicExch(changed + T, 1u) == 0u;
      atomicAdd(&s_merges, 1u);
      const int prev = atomicCAS(&s_j, -1, j);
      if (prev != -1 && prev != j) s_mixed = 1;
    }
  }
  __syncthreads();
  // one atomic per block when its merges all belong to one solve (the usual case)
  if (!s_mixed) {
    if (threadIdx.x == 0 && s_merges) atomicAdd(nelig + s_j, s_merges);
  } else {
    wave_count(nelig, j, merged);
  }
  block_append(clist, ccount, first, (int32_t)T, s_app);
}

// ------------------------------------------------------------------ aggregation helpers
__global__ void k_minmember(const uint32_t *R, int64_t n, const int32_t *usolve,
                            const uint8_t *cont, uint32_t *minm) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u < n && cont[usolve[u]]) atomicMin(minm + R[u], (uint32_t)u);
}
__global__ void k_flag_minm(const uint32_t *R, const uint32_t *minm, int64_t n, uint8_t *flag) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u < n) flag[u] = minm[R[u]] == (uint32_t)u;
}
// super-node id of each unit of a continuing solve (kNone for units of finished solves)
__global__ void k_rank_gather(const uint32_t *R, const uint32_t *minm, const int64_t *rank,
                              int64_t n, uint32_t *r) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n) return;
  uint32_t m = minm[R[u]];
  r[u] = m == kNone ? kNone : (uint32_t)rank[m];
}

// key (r[u], r[x]) of every entry between different super-nodes, written at the entry's own
// position; dropped entries get the all-ones key, which sorts last
constexpr uint64_t kDropKey = ~0ull;
template <class V>
__global__ __launch_bounds__(256) void k_agg_keys(V g, SolveDev sd, int64_t n, const uint32_t *r,
                                                  int shift, uint64_t *keys, int64_t *vals) {
  const int lane = threadIdx.x & 63;
  const int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (u >= n) return;
  const uint32_t ru = r[u];
  typename V::Row row = g.row(u, sd);
  for (int64_t e = row.lo + lane; e < row.hi; e += 64) {
    int32_t x = g.col[e];
    int64_t w = g.wt(row, e, x);
    uint32_t rx = ru == kNone ? kNone : r[x];
    bool emit = ru != kNone && w != 0 && rx != ru;
    keys[e] = emit ? (((uint64_t)ru << shift) | rx) : kDropKey;
    vals[e] = emit ? w : 0;
  }
}

// profile entries (r[u], slice) at fixed positions: level 0 one per unit, later pp[u] + j
__device__ inline int64_t prof_pos(const View0 &, int64_t u, int) { return u; }
__device__ inline int64_t prof_pos(const ViewK &g, int64_t u, int j) { return g.pp[u] + j; }
template <class V>
__global__ void k_agg_prof_keys(V g, int64_t n, const uint32_t *r, int shift, uint64_t *keys,
                                int32_t *vals) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n) return;
  int m = g.plen(u);
  if (V::kLevel0 && m == 0) {
    keys[u] = kDropKey;
    vals[u] = 0;
    return;
  }
  for (int jj = 0; jj < m; jj++) {
    int gs;
    int64_t k;
    g.pent(u, jj, gs, k);
    int64_t pos = prof_pos(g, u, jj);
    bool keep = r[u] != kNone;
    keys[pos] = keep ? (((uint64_t)r[u] << shift) | (uint32_t)gs) : kDropKey;
    vals[pos] = keep ? (int32_t)k : 0;
  }
}

// row bounds of a sorted key array (row = high 32 bits): rs[row] = first, re[row] = last + 1
// keys are (row << shift) | column, sorted
__global__ void k_row_bounds(const uint64_t *keys, int64_t m, int shift, int64_t *rs, int64_t *re) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  uint64_t row = keys[i] >> shift;
  if (i == 0 || (keys[i - 1] >> shift) != row) rs[row] = i;
  if (i == m - 1 || (keys[i + 1] >> shift) != row) re[row] = i + 1;
}
__global__ void k_row_cnt(const int64_t *rs, const int64_t *re, int64_t n, int64_t *cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cnt[i] = re[i] - rs[i];
}
__global__ void k_low_bits(const uint64_t *keys, int64_t m, int shift, int32_t *out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) out[i] = (int32_t)(keys[i] & ((1ull << shift) - 1));
}

template <class V>
__global__ void k_scatter_next(V g, int64_t n, const uint32_t *r, const uint32_t *P,
                               uint32_t *Pnext, int32_t *usolve_next) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n || r[u] == kNone) return;
  Pnext[r[u]] = P[u];
  usolve_next[r[u]] = g.usolve[u];
}

__global__ void k_map_compose(int64_t *map0, const int64_t *lo, const int64_t *hi, int nr,
                              const uint32_t *r) {
  // ranges [lo[k], hi[k]) of level-0 units; grid-stride over their union
  int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t i = lo[k] + tid; i < hi[k]; i += stride) map0[i] = r[map0[i]];
}

// ------------------------------------------------------------------ canonical labels by sort
__global__ void k_seg_heads(const uint32_t *sk, const uint32_t *sv, int64_t n, uint8_t *head,
                            uint8_t *ismin) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint8_t h = (i == 0 || sk[i] != sk[i - 1]) ? 1 : 0;
  head[i] = h;
  ismin[sv[i]] = h;
}
// segid = inclusive index of the segment (exclusive scan of heads at heads), minOf[seg] = unit
__global__ void k_seg_min(const uint32_t *sv, const uint8_t *head, const int64_t *segx, int64_t n,
                          uint32_t *minof) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && head[i]) minof[segx[i]] = sv[i];
}
__global__ void k_seg_label(const uint32_t *sv, const uint8_t *head, const int64_t *segx,
                            const uint32_t *minof, const int64_t *rank, int64_t n, uint32_t *out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int64_t seg = segx[i] + head[i] - 1;
  out[sv[i]] = (uint32_t)rank[minof[seg]];
}
__global__ void k_count_heads(const uint32_t *sv, const uint8_t *head, const int32_t *usolve,
                              int64_t n, uint32_t *cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool h = i < n && head[i];
  wave_count(cnt, h ? usolve[sv[i]] : 0, h);
}
__global__ void k_solve_label_keys(const uint32_t *lab, const int32_t *usolve, int64_t n,
                                   uint64_t *keys, int32_t *vals) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) {
    keys[v] = ((uint64_t)(uint32_t)usolve[v] << 32) | lab[v];
    vals[v] = (int32_t)v;
  }
}
__global__ void k_count_key_heads(const uint64_t *keys, int64_t n, uint32_t *cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool h = i < n && (i == 0 || keys[i] != keys[i - 1]);
  wave_count(cnt, h ? (int)(keys[i] >> 32) : 0, h);
}
__global__ void k_fingerprint(const uint32_t *lab, int64_t n, unsigned long long *acc) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) atomicAdd(acc, (unsigned long long)mix64(((uint64_t)v << 32) | lab[v]));
}
__global__ void k_offset_labels(const int32_t *lab, const int32_t *usolve, const int64_t *uoff,
                                int64_t n, uint32_t *out) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) out[v] = (uint32_t)(uoff[usolve[v]] + lab[v]);
}
// Each solve's labels by first appearance from the union's canonical labels (communities
// ranked by their smallest member over the whole union): the solve's first unit is the
// smallest member of its community, so its rank counts the communities of earlier solves.
__global__ void k_local_labels(const uint32_t *comm, const int32_t *usolve, const int64_t *uoff,
                               int64_t n, int32_t *out) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) out[v] = (int32_t)(comm[v] - comm[uoff[usolve[v]]]);
}
__global__ void k_count_roots_R(const uint32_t *R, const int32_t *usolve, int64_t n, uint32_t *cnt) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool h = u < n && R[u] == (uint32_t)u;
  wave_count(cnt, h ? usolve[u] : 0, h);
}
__global__ void k_count_flags(const uint8_t *flag, const int32_t *usolve, int64_t n, uint32_t *cnt) {
  int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool h = u < n && flag[u];
  wave_count(cnt, h ? usolve[u] : 0, h);
}

// ------------------------------------------------------------------ split into connected parts
__device__ inline int32_t uf_find(int32_t *parent, int32_t x) {
  for (;;) {
    int32_t p = __hip_atomic_load(parent + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (p == x) return x;
    int32_t gp = __hip_atomic_load(parent + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (gp != p) __hip_atomic_store(parent + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x = p;
  }
}
__device__ inline void uf_unite(int32_t *parent, int32_t a, int32_t b) {
  for (;;) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a < b) {
      int32_t t = a;
      a = b;
      b = t;
    }
    // link the larger root under the smaller one: roots stay component minima
    if (atomicCAS(parent + a, a, b) == a) return;
  }
}

// body(v, first, step) for every element v of the ranges: by 16 lanes, or by the whole wave for
// rows of more than 1024 entries.
template <class F>
__device__ inline void uf_rows(const View0 &g, const int64_t *lo, const int64_t *hi, int nr,
                               F body) {
  const int lane = threadIdx.x & 63;
  const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int k = 0; k < nr; k++)
    for (int64_t v0 = lo[k] + 4 * wid; v0 < hi[k]; v0 += 4 * nw) {
      const int64_t v = v0 + lane / 16;
      const bool live = v < hi[k];
      const bool is_long = live && g.degree(v) > 1024;
      if (live && !is_long) body(v, lane & 15, 16);
      for (uint64_t m = __ballot(is_long && (lane & 15) == 0); m; m &= m - 1)
        body(v0 + __builtin_ctzll(m) / 16, lane, 64);
    }
}

// First every element hooks onto its smallest neighbour of the same label (a smaller one, so no
// cycles and no atomics); then, flattened, every tree hooks onto the smallest root next to it
// (kRoots), which leaves few trees, and nearly every edge of k_uf_link finds its ends under one root
// by one load each.  Linking from single elements had all edges of a community fight over its
// root (500k elements in 12 communities 2.75 ms), from trees of the first round too (5.0 ms).
template <bool kRoots>
__global__ __launch_bounds__(256) void k_uf_hook(View0 g, SolveDev sd, const int64_t *lo,
                                                 const int64_t *hi, int nr, const uint32_t *lab,
                                                 int32_t *parent) {
  auto at = [&](int64_t x) {
    return __hip_atomic_load(parent + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  uf_rows(g, lo, hi, nr, [&](int64_t v, int first, int step) {
    View0::Row row = g.row(v, sd);
    const uint32_t L = lab[v];
    const int32_t own = kRoots ? at(v) : (int32_t)v;
    int32_t best = own;
    for (int64_t e = row.lo + first; e < row.hi; e += step) {
      const int32_t x = g.col[e];
      if (lab[x] != L) continue;
      const int32_t r = kRoots ? at(x) : x;
      if (r < best && g.wt(row, e, x) != 0) best = r;
    }
    for (int m = step / 2; m >= 1; m >>= 1) {
      const int32_t o = __shfl_xor(best, m, 64);
      best = o < best ? o : best;
    }
    if (first != 0) return;
    if (!kRoots) parent[v] = best;
    else if (best < own && best < at(own)) atomicMin(parent + own, best);
  });
}

__global__ __launch_bounds__(256) void k_uf_flatten(int32_t *parent, const int64_t *lo,
                                                    const int64_t *hi, int nr) {
  int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t i = lo[k] + tid; i < hi[k]; i += stride) {
      const int32_t r = uf_find(parent, (int32_t)i);
      __hip_atomic_store(parent + i, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ __launch_bounds__(256) void k_uf_link(View0 g, SolveDev sd, const int64_t *lo,
                                                 const int64_t *hi, int nr, const uint32_t *lab,
                                                 int32_t *parent) {
  uf_rows(g, lo, hi, nr, [&](int64_t v, int first, int step) {
    View0::Row row = g.row(v, sd);
    const uint32_t L = lab[v];
    const int32_t rv = __hip_atomic_load(parent + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int64_t e = row.lo + first; e < row.hi; e += step) {
      const int32_t x = g.col[e];
      if (x <= v || lab[x] != L || g.wt(row, e, x) == 0) continue;
      if (__hip_atomic_load(parent + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == rv) continue;
      uf_unite(parent, (int32_t)v, x);
    }
  });
}

// Root of every element into a separate array: other threads' path halving keeps rewriting
// parent[] with ancestors while this runs, so parent[] itself is not a root map afterwards.
__global__ void k_uf_roots(int32_t *parent, const int64_t *lo, const int64_t *hi, int nr,
                           uint8_t *isroot, int32_t *root) {
  int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t i = lo[k] + tid; i < hi[k]; i += stride) {
      int32_t r = uf_find(parent, (int32_t)i);
      root[i] = r;
      isroot[i] = r == (int32_t)i;
    }
}

// memb[i] = rank of i's root among the roots of its range; root and memb may alias
__global__ void k_label_out(const int32_t *root, const int64_t *rank, const int64_t *lo,
                            const int64_t *hi, const int64_t *roff, int nr, int32_t *memb) {
  int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t i = lo[k] + tid; i < hi[k]; i += stride)
      memb[i] = (int32_t)(rank[root[i]] - roff[k]);
}

__global__ void k_flatten(const int64_t *map0, const uint32_t *P, const int64_t *lo,
                          const int64_t *hi, int nr, uint32_t *flat) {
  int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t i = lo[k] + tid; i < hi[k]; i += stride) flat[i] = P[map0[i]];
}

__global__ void k_count_diff(const int32_t *a, const int32_t *b, const int32_t *usolve,
                             const int64_t *lo, const int64_t *hi, int nr, uint32_t *diff) {
  // convergent loops: every lane of a wave runs the same iterations
  const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) & ~63ll;
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t b0 = lo[k] + wave0; b0 < hi[k]; b0 += stride) {
      int64_t i = b0 + lane;
      bool d = i < hi[k] && a[i] != b[i];
      wave_count(diff, d ? usolve[i] : 0, d);
    }
}

// ------------------------------------------------------------------ Q components
// W_s: intra weight inside communities (both directions, unscaled) per global slice; one
// thread per unit, sums merged per wave by slice
__global__ void k_q_w(View0 g, int64_t n, const int32_t *memb, int64_t *W) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t s = 0;
  int gs = 0;
  if (v < n) {
    gs = g.uslice[v];
    const int64_t slo = g.sstart[gs], shi = g.sstart[gs + 1];
    const int32_t L = memb[v];
    for (int64_t e = g.rp[v]; e < g.rp[v + 1]; e++) {
      int32_t x = g.col[e];
      if (x >= slo && x < shi && memb[x] == L) s += g.w ? g.w[e] : 1;
    }
  }
  wave_add64(W, gs, s);
}

// Sigma of a membership: per Sigma slice and label, the sum of the null-model degrees
// (a block's kMembUnits units are added up in LDS first: final memberships have few labels, and
// 500k units of 12 communities and one slice took 2.0 ms of atomics on 12 words; a label that
// finds no slot in kMembProbes goes to the table itself).
constexpr int kMembUnits = 4096, kMembLg = 10, kMembProbes = 4;
__global__ __launch_bounds__(256) void k_sigma_build_memb(View0 g, int64_t n, const int32_t *memb,
                                                          SliceTable t) {
  __shared__ unsigned long long sk[1 << kMembLg];   // slice << 32 | label, ~0: free
  __shared__ int32_t sv[1 << kMembLg];
  for (int i = threadIdx.x; i < 1 << kMembLg; i += 256) {
    sk[i] = ~0ull;
    sv[i] = 0;
  }
  __syncthreads();
  const int64_t v0 = (int64_t)blockIdx.x * kMembUnits;
  for (int64_t v = v0 + threadIdx.x; v < v0 + kMembUnits && v < n; v += 256) {
    int gs;
    int64_t k;
    g.pent(v, 0, gs, k);
    if (k <= 0) continue;
    const uint32_t lab = (uint32_t)memb[v];
    const unsigned long long key = (unsigned long long)(uint32_t)gs << 32 | lab;
    uint32_t h = (lab * 0x9e3779b1u + (uint32_t)gs * 0x85ebca6bu) >> (32 - kMembLg);
    int p = 0;
    for (; p < kMembProbes; p++, h = (h + 1) & ((1u << kMembLg) - 1)) {
      const unsigned long long was = atomicCAS(sk + h, ~0ull, key);
      if (was == ~0ull || was == key) break;
    }
    if (p < kMembProbes) atomicAdd(sv + h, (int32_t)k);
    else tab_add(t, gs, lab, (int32_t)k, false);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 1 << kMembLg; i += 256)
    if (sk[i] != ~0ull) tab_add(t, (int)(sk[i] >> 32), (uint32_t)sk[i], sv[i], false);
}

// Scaled supra-degree of every unit of one solve under the global null model:
// b*k_i^s + a*c with c the unit's coupling entries (1 in the first and last slice, 2 between,
// none for one slice).
__global__ void k_null_degree_global(const int32_t *k, const int64_t *rp, const int32_t *col,
                                     const int32_t *w, int64_t n, int64_t N, int64_t a, int64_t b,
                                     int32_t *out) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int64_t lo = (v / N) * N, hi = lo + N;
  int64_t c = 0;   // the copy's coupling multipliers
  for (int64_t e = rp[v]; e < rp[v + 1]; e++) {
    const int32_t x = col[e];
    if (x < lo || x >= hi) c += w ? w[e] : 1;
  }
  out[v] = (int32_t)(b * k[v] + a * c);
}

// CPM node weight: 1 per copy, or 0 for a copy without an intra edge when only present copies
// are coupled (it is then no supra-node)
__global__ void k_cpm_weight(const int32_t *kd, int64_t n, bool present_only, int32_t *out) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) out[v] = (!present_only || kd[v] > 0) ? 1 : 0;
}

// SS per Sigma slice: sum over the slice's sub-table of value^2
__global__ void k_q_ss(const uint64_t *slots, const int64_t *base, int nslices, int64_t total,
                       int64_t *SS) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t sq = 0;
  int lo = 0;
  if (i < total) {
    uint64_t e = slots[i];
    int64_t val = (uint32_t)e ? (int32_t)(e >> 32) : 0;
    sq = val * val;
    int hi = nslices;   // base[lo] <= i < base[hi]
    while (hi - lo > 1) {
      int mid = (lo + hi) >> 1;
      if (base[mid] <= i) lo = mid; else hi = mid;
    }
  }
  wave_add64(SS, lo, sq);
}

// I: ordered coupled copy pairs (i,s),(i,s+1) sharing a community, per solve
__global__ void k_q_inter(View0 g, int64_t n, const int32_t *memb, int64_t *I) {
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t add = 0;
  int j = 0;
  if (v < n) {   // the coupling entries of v (both directions are counted, one per row)
    const int gs = g.uslice[v];
    const int64_t lo = g.sstart[gs], hi = g.sstart[gs + 1];
    j = g.usolve[v];
    for (int64_t e = g.rp[v]; e < g.rp[v + 1]; e++) {
      const int32_t x = g.col[e];
      if ((x < lo || x >= hi) && memb[x] == memb[v]) add += g.w ? g.w[e] : 1;
    }
  }
  wave_add64(I, j, add);
}

// ------------------------------------------------------------------ small utilities
template <class T>
__global__ void k_fill(T *p, T val, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = val;
}
__global__ void k_iota_i32(int32_t *p, int64_t n, int64_t off) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int32_t)(i + off);
}
__global__ void k_iota_u32(uint32_t *p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (uint32_t)i;
}
__global__ void k_fill_ranges(int32_t *out, const int64_t *lo, const int64_t *hi,
                              const int64_t *outoff, int nr) {
  int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < nr; k++)
    for (int64_t i = tid; i < hi[k] - lo[k]; i += stride) out[outoff[k] + i] = (int32_t)(lo[k] + i);
}
__global__ void k_gather_i64(const int64_t *src, const int64_t *idx, int n, int64_t *dst) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[idx[i]];
}
__global__ void k_compact_flag(const uint8_t *flag, int64_t n, int32_t *out, uint32_t *cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && flag[i]) out[atomicAdd(cnt, 1u)] = (int32_t)i;
}

}  // namespace mslm
