// zeus_bfgs_common.h -- pieces shared by the two BFGS kernels (one group of
// lanes per start, and one block per start for wide problems).
#pragma once

#include "zeus_device.h"
#include "zeus_group.h"
#include "zeus_internal.h"

namespace zeus {

// The scalars of a start's request that every iteration reads, kept in LDS
// (registers hold only the request index; output pointers are read from the
// request table when a start retires).
struct ReqHot {
  int d, m;                  // dimension, number of terms
  int iter_bfgs, iter_ls, trace_len, ri;
  int stop_status;           // status at the iteration budget
  int m_hist;                // L-BFGS pairs kept
  double armijo_c, tol, shrink;
  int32_t *es;               // early-stop state while a start may stop at its bound
  int64_t es_c;              // converged starts that stop the request
};
constexpr int kHotDoubles = (sizeof(ReqHot) + 7) / 8;

// Term sums an objective's outer function combines (Ackley has two).
constexpr int kMaxSums = 2;

// Per-start counts of two decisions of Alg. 4, kept in LDS and touched only
// by the start's first lane (no registers): steps whose rank-2 update was
// skipped because y's <= 0, and search directions reset to -g because g'p
// was not negative.
struct StartCounts {
  int32_t skips, resets;
};

// Step lengths alpha_t = shrink^t of the first kTabTrials trials, each the
// product of the previous one and shrink, as Alg. 6 forms them.
constexpr int kTabTrials = 32;

__device__ __forceinline__ double step_length(const double *al, double shrink, int t) {
  // the load does not wait for the test, which hardly ever holds
  double alpha = al[t < kTabTrials ? t : kTabTrials - 1];
  if (t >= kTabTrials)
    for (int e = kTabTrials - 1; e < t; ++e) alpha = alpha * shrink;
  return alpha;
}

// Lanes lane0, lane0 + stride, ... below kTabTrials fill the table.
__device__ __forceinline__ void fill_step_lengths(double *al, double shrink, int lane0, int stride) {
  for (int t = lane0; t < kTabTrials; t += stride) {
    double a = 1.0;
    for (int e = 0; e < t; ++e) a = a * shrink;
    al[t] = a;
  }
}

// In the second early-stop pass almost every claimed start keeps its
// first-pass result, so a claim is mostly a skip and the agent-scope work
// counter would serialise the pass (one same-address atomic per start).
// There a worker (group or block) `self` of `workers` takes the starts
// self, self + workers, self + 2 workers, ... instead: the reruns are short
// and alike, so a static split balances them.  Returns the worker's n-th
// start (n >= 1) in that split.
__device__ __forceinline__ unsigned long long strided_claim(unsigned long long self,
                                                            unsigned long long workers, int n) {
  return self + (unsigned long long)n * workers;
}

// The request of a launch group that holds global start `got` (the start
// offsets of the table ascend from 0).
__device__ __forceinline__ int request_of(const ReqDev *reqs, int nreq, int64_t got) {
  int lo = 0, hi = nreq - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (reqs[mid].start_offset <= got) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// sqrt(gg) < bound, the norm test of a start (gg = g'g).  kWave: the starts of
// the wave nearly always fail it together (one start per wave, above all); then
// a branch skips the root when gg >= 4 bound^2: there it is at least twice the
// bound up to a few roundings.  (Below a bound of about 1e-154 the square loses
// its digits and then vanishes, so a subnormal or zero gg always goes to the
// root.)  With many starts in a wave the branch costs more than the root
// (Rosenbrock d = 4, 256 starts 0.193 -> 0.188 ms).
template <bool kWave = true>
__device__ __forceinline__ bool norm_below(double gg, double bound) {
  if constexpr (kWave)
    if (__ballot(gg < __builtin_fmax((4.0 * bound) * bound, 0x1p-1022)) == 0ull) return false;
  return sqrt(gg) < bound;
}

// Relaxed agent-scope access to the early-stop state: its values are only
// ever bounds (a stale bound is a larger one), so no ordering is needed.
__device__ __forceinline__ int es_load(const int32_t *p) {
  // as device memory, not a generic address: a generic load would also count as
  // an LDS access, and every later LDS read would wait for it
  typedef const __attribute__((address_space(1))) int32_t *Global;
  return __hip_atomic_load((Global)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Smallest iteration k at which the counts of the Fenwick tree (nodes
// 1 .. n, node i for iteration i - 1) reach c convergences at iterations
// <= k, or -1 when they do not.  With counts read while they still grow the
// answer can only be too large, never too small.
__device__ __forceinline__ int es_search(const int32_t *es, int n, int64_t c) {
  const int32_t *tree = es + kEsTree;
  int step = 1;
  while (2 * step <= n) step *= 2;
  int pos = 0;
  int64_t rem = c;
  for (; step > 0; step >>= 1)
    if (pos + step <= n) {
      const int64_t t = (uint32_t)es_load(tree + pos + step);
      if (t < rem) {
        pos += step;
        rem -= t;
      }
    }
  return pos < n ? pos : -1;
}

// A start of a request with early stop has converged at iteration k (one
// lane per start): count it, and lower the stopping bound to the c-th
// smallest convergence iteration counted so far.
__device__ __forceinline__ void es_converged(int32_t *es, int k, int iter_bfgs, int64_t c) {
  const int n = iter_bfgs + 1;
  for (int i = k + 1; i <= n; i += i & -i)
    __hip_atomic_fetch_add(es + kEsTree + i, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t cnt =
      (int64_t)(uint32_t)__hip_atomic_fetch_add(es + kEsCount, 1, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT) + 1;
  if (cnt < c || k >= es_load(es + kEsBound)) return;
  const int kc = es_search(es, n, c);
  if (kc >= 0) __hip_atomic_fetch_min(es + kEsBound, kc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Early-stop pass of a launch group (BatchDev::es_pass), read once per kernel.
__device__ __forceinline__ int es_pass_of(const BatchDev *hdr) {
  return (int)__hip_atomic_load(&hdr->es_pass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// In the second pass a claimed start reruns only if its request stops early
// and the start went past K* in the first pass; every other start keeps the
// results of the first pass.
__device__ __forceinline__ bool es_rerun(const ReqDev &rq, int64_t idx) {
  if (!rq.ws.es) return false;
  const int ks = es_load(rq.ws.es + kEsKstar);
  return ks >= 0 && rq.out_iters[idx] > ks;
}

// The request's scalars for the start a group claimed; in the second
// early-stop pass the start reruns with K* as its budget and ends STOPPED.
template <int OBJ>
__device__ __forceinline__ void load_hot(ReqHot &w, const ReqDev &rq, int ri, int es_pass) {
  w.d = rq.d;
  w.m = Elem<OBJ>::terms(rq.d);
  w.iter_bfgs = rq.iter_bfgs;
  w.stop_status = rq.stop_status;
  w.m_hist = rq.lbfgs_m;
  w.iter_ls = rq.iter_ls;
  w.trace_len = rq.trace ? rq.trace_len : 0;
  w.ri = ri;
  w.armijo_c = rq.armijo_c;
  w.tol = rq.tol;
  w.shrink = rq.shrink;
  w.es = es_pass == 1 ? rq.ws.es : nullptr;
  w.es_c = rq.required_c;
  if (es_pass == 2) {
    w.iter_bfgs = es_load(rq.ws.es + kEsKstar);
    w.stop_status = ZEUS_ST_STOPPED;
  }
}

// Status of a start at iteration k that is neither non-finite nor converged:
// the budget, else (first early-stop pass) the stopping bound read at the top
// of the iteration, else still running (-1).
__device__ __forceinline__ int budget_status(const ReqHot &q, int iter_bfgs, int k, int bound) {
  if (k == iter_bfgs) return q.stop_status;  // MAXITER, or STOPPED in the rerun
  if (k >= bound) return ZEUS_ST_STOPPED;
  return -1;
}

// Stopping bound of the start's request for this iteration (no bound without
// early stop).
__device__ __forceinline__ int es_bound(const ReqHot &q) {
  return q.es ? es_load(q.es + kEsBound) : 0x7fffffff;
}

// The request's scalars that every iteration of a start needs, in registers: in
// the LDS copy (ReqHot) each is a wait of its own on the iteration's path.
// Where a group is a whole wave they are taken from one lane, so that they
// sit in scalar registers.
template <int G>
struct HotRegs {
  int d, iter_bfgs, iter_ls, trace_len;
  double tol, armijo_c;
  bool es;  // the start may stop at its request's bound
  __device__ __forceinline__ static int uni(int v) {
    return G == 64 ? __builtin_amdgcn_readfirstlane(v) : v;
  }
  __device__ __forceinline__ static double uni(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(
        double, ((uint64_t)(uint32_t)uni((int)(b >> 32)) << 32) | (uint32_t)uni((int)(uint32_t)b));
  }
  // after the group's wave_sync that publishes q
  __device__ __forceinline__ void take(const ReqHot &q) {
    d = uni(q.d);
    iter_bfgs = uni(q.iter_bfgs);
    iter_ls = uni(q.iter_ls);
    trace_len = uni(q.trace_len);
    tol = uni(q.tol);
    armijo_c = uni(q.armijo_c);
    es = uni(q.es != nullptr ? 1 : 0) != 0;
  }
};

// Objectives with starts that stall: near a minimum their value is a small
// difference of larger numbers, so at some point no trial passes any more and a
// start whose gradient is still above the tolerance fails every search to its
// budget.  Where the minimum is zero the value keeps its relative precision.
template <int OBJ>
constexpr bool kStalls = !(OBJ == kRosenbrock || OBJ == kSphere || OBJ == kQuartic);

// Whether the groups of a BFGS wave share their lanes in the line searches
// (wave_search).  That helps the starts that stall, and costs the others the
// loop that keeps a wave's groups together: where nothing stalls each group
// searches, claims and ends by itself (Rosenbrock, shared and by itself: d = 4,
// 1,024 starts 0.227 and 0.207 ms; d = 14 in mixed precision, 65,536 starts 1.83
// and 1.72 ms).  Two groups of 32 lanes gain little: nothing in whole form, where 32
// lanes already try 32 lengths (a user's chain of 20 terms, 32,768 starts: 0.92 of
// the speed), and less than they pay for Styblinski-Tang (d = 24, 65,536 starts
// 1.37 and 1.31 ms), but a third for Ackley (d = 18, 4,096 starts 4.8 and 6.3 ms).
template <int OBJ, int G>
constexpr bool kShareLanes = G < 64 && kStalls<OBJ> &&
                             !(G == 32 && (whole_form<Elem<OBJ>>::value || OBJ == kStyblinskiTang));

// Lanes per line-search trial.  A lane then holds SLOTS / TP consecutive term
// slots, and a round gives a group of G lanes R = G / TP trials.  64-lane
// groups take R = 2 (one trial a round was slower, four evaluate trials past
// the accepted one: d = 50 BFGS 3-7% slower), smaller groups R = 4 (R = 2:
// Ackley d = 2, 4,096 starts 12.9 ms against 7.6; Rosenbrock and Rastrigin
// d = 10 within 2%); objectives in whole form take a trial per lane.  The
// L-BFGS kernels choose their own (zeus_lbfgs_kernels.h).
template <int OBJ, int G>
constexpr int kTrialLanes = whole_form<Elem<OBJ>>::value ? 1 : G == 64 ? 32 : G < 4 ? 1 : G / 4;

// What a search reads from its group's LDS slice: offsets in doubles.
struct SearchLayout {
  int stride;     // between the slices of a wave's groups
  int xs, ps;     // the point and the direction, zero past the dimension
  int al, q;      // step lengths, request
  int fd;         // room for f and g'p at the point
  int pick;       // one double of scratch
  int acc;        // the accepted trial's term sums (-1: not kept)
};

// One trial's value, formed by TP lanes (this lane is number c of them) over
// SLOTS term slots, at xs + alpha ps: a lane adds its B = SLOTS / TP consecutive
// slots pairwise (zero past the last term) and the trial's lanes finish the
// pairwise sum with a butterfly, so the value does not depend on which lanes
// form it.  sums receives the term sums.
template <int OBJ, int SLOTS, int TP, class U>
__device__ __forceinline__ double trial_value(const double *xs, const double *ps, double alpha, int d,
                                              int m, int c, U (&sums)[Elem<OBJ>::K]) {
  using E = Elem<OBJ>;
  constexpr int B = SLOTS / TP;
  // Every slot is evaluated (indices clamped into the vectors) and the
  // slots past the last term are replaced by zero afterwards: no branch
  // per slot, so the loads of a chunk of CB slots are in flight together.
  // A lane's B slots are taken CB at a time (a memory clobber between
  // chunks keeps the next chunk's loads from being hoisted, which bounds
  // the live registers); the pairwise tree over B is the tree over the
  // chunk sums.
  constexpr int CB = B < 4 ? B : 4;
  U csum[E::K][B / CB];
#pragma unroll
  for (int cb = 0; cb < B / CB; ++cb) {
    if (cb > 0) asm volatile("" ::: "memory");
    U tv[E::K][CB];
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int i = c * B + cb * CB + b;
      U w[E::W], out[E::K];
#pragma unroll
      for (int e = 0; e < E::W; ++e) {
        const int ie = i + e < SLOTS ? i + e : SLOTS - 1;
        w[e] = (U)(xs[ie] + alpha * ps[ie]);
      }
      // With a trial per lane, slot b is term b on every lane, and no lane of
      // the wave may need it (d = 2 and 3 in groups of four lanes).  Asking costs
      // more than a polynomial term (Rosenbrock d = 4, 256 starts 0.193 and 0.202
      // ms), not more than the others (Rastrigin d = 3, 1,024 starts 2.91 and 2.72).
      constexpr bool kAsk = TP == 1 && (OBJ == kRastrigin || OBJ == kAckley || OBJ == kGoldsteinPrice);
      bool any = true;
      if constexpr (kAsk)
        if (b > 0) any = __ballot(i < m) != 0ull;
#pragma unroll
      for (int kk = 0; kk < E::K; ++kk) tv[kk][b] = U(0);
      if (any) {
        E::template term<U>(w, out);
#pragma unroll
        for (int kk = 0; kk < E::K; ++kk) tv[kk][b] = i < m ? out[kk] : U(0);
      }
    }
#pragma unroll
    for (int kk = 0; kk < E::K; ++kk) csum[kk][cb] = reg_tree_sum<CB, U>(tv[kk]);
  }
#pragma unroll
  for (int kk = 0; kk < E::K; ++kk)
    sums[kk] = lane_tree_sum<TP, U>(reg_tree_sum<B / CB, U>(csum[kk]));
  return (double)E::template outer<U>(d, sums);
}

// v of one lane of the wave (the same number on every lane).
__device__ __forceinline__ double read_lane(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), lane) << 32) |
                                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane));
}

// The Armijo searches (Alg. 6) of a wave's groups, the objective evaluated in
// number type U.  With SHARE every lane of the wave must call it and need (the
// same on all lanes of a group) says which groups search, the others lending
// their lanes; without, the lanes of each searching group call it by themselves.
// hot, f and ddir are the scalars, the value and g'p of the lane's own group.
// Returns, on the lanes of a searching group, the index of the first trial
// that passes, or -1 when none of the iter_ls trials does: the step the
// sequential loop of Alg. 6 returns.
//
// A round evaluates 64 / TP trials, TP lanes each.  While more than half of
// the wave's groups search (always, without SHARE), each tries R = G / TP trials a round on its own
// lanes.  After that the lanes are shared out among the groups that have not
// found their step (as many equal shares as the next power of two), so the
// fewer they are the more trials each tries at once.  A start that stalls,
// every trial of every search failing, sets the end of a launch by itself;
// with its own lanes alone it took 5 rounds an iteration beside idle ones.
// Bound by latency there.  BFGS phase with fixed lanes and with shared ones:
// Ackley d = 10, 16,384 starts 15.9 -> 7.4 ms, Rastrigin d = 6, 16,384 starts
// 5.5 -> 3.4 ms, d = 2, 65,536 starts 9.2 -> 8.1 ms.  (Where no start stalls it
// costs up to a tenth, see kShareLanes.)
// Sharing from the first failed round on, whatever the number of groups left,
// was slower (Ackley d = 2, 4,096 starts 9.4 ms against 7.6), and so was
// sharing after two rounds (Rastrigin d = 6 4.3 ms).
//
// The group sees what is written to acc after its next wave_sync.  kept, where a
// wave has one group, receives the accepted trial's term sums on every lane.
template <int OBJ, int G, int SLOTS, int TP, bool SHARE, class U>
__device__ __forceinline__ int wave_search(const GroupLanes<G> &L, const HotRegs<G> &hot, bool need,
                                           double f, double ddir, double *wave_lds,
                                           const SearchLayout &lay, double *kept = nullptr) {
  using E = Elem<OBJ>;
  constexpr int R = G / TP, S = SHARE ? 64 / G : 1;  // S: groups that share lanes
  static_assert(TP >= 1 && TP <= G && G % TP == 0 && SLOTS % TP == 0, "whole trials per group");
  static_assert(E::K <= kMaxSums, "more term sums than the slots kept for them");
  const int lane = threadIdx.x & 63, c = lane % TP;
  const double *own = wave_lds + L.grp * lay.stride;
  const ReqHot &oq = *reinterpret_cast<const ReqHot *>(own + lay.q);
  constexpr uint64_t leaders = [] {  // bit r * TP for every trial r of a group
    uint64_t b = 0;
    for (int r = 0; r < R; ++r) b |= 1ull << (r * TP);
    return b;
  }();
  const int r = L.j / TP, iter_ls = hot.iter_ls;
  int taken = -1;
  bool open = need;  // the lane's own group still searches
  int base = 0;
  uint64_t todo;     // the groups that search, bit G * group
  {
    do {
      const int t = base + r;
      // lanes past the last trial take a length that costs nothing, and in whole
      // form no value either (a round of one start's lanes reaches far past it;
      // one trial a round is within the loop's test)
      const bool tries = (S == 1 && R == 1) || t < iter_ls;
      const double alpha = step_length(own + lay.al, oq.shrink, tries ? t : 0);
      // the trial's bound, formed before the terms rather than behind them
      const double bound = f + (hot.armijo_c * alpha) * ddir;
      double ft = 0.0;
      U sums[E::K];
      if constexpr (whole_form<E>::value) {
        // a group that has not searched yet has no request in its slice
        if (open & tries) ft = E::template trial<U>(own + lay.xs, own + lay.ps, alpha, oq.d);
      } else {
        ft = trial_value<OBJ, SLOTS, TP, U>(own + lay.xs, own + lay.ps, alpha, oq.d, oq.m, c, sums);
      }
      const bool ok = open & (t < iter_ls) & (ft <= bound);
      const uint64_t mine = L.ballot(ok) & leaders;
      if (mine != 0ull) {
        const int first = (__ffsll((unsigned long long)mine) - 1) / TP;  // the passing trial's place
        taken = base + first;
        open = false;
        if constexpr (!whole_form<E>::value)
          if (lay.acc >= 0 && L.j == first * TP)
#pragma unroll
            for (int kk = 0; kk < E::K; ++kk)
              wave_lds[L.grp * lay.stride + lay.acc + kk] = (double)sums[kk];
        if constexpr (G == 64 && !whole_form<E>::value) {
          if (kept)
#pragma unroll
            for (int kk = 0; kk < E::K; ++kk) kept[kk] = read_lane((double)sums[kk], first * TP);
        }
        if constexpr (S == 1) return taken;
      }
      base += R;
      open = open && base < iter_ls;
      todo = S == 1 ? 0ull : __ballot(open && L.j == 0);
    } while (S == 1 ? base < iter_ls : __popcll(todo) > S / 2);
  }
  if constexpr (S > 1) {
    constexpr uint64_t all_leaders = [] {  // bit s * TP for every trial s of a round
      uint64_t b = 0;
      for (int s = 0; s < 64 / TP; ++s) b |= 1ull << (s * TP);
      return b;
    }();
    while (todo != 0ull) {
      // share the lanes out: 64 >> (6 - share) of them per group, in group order
      const int n = __popcll(todo);
      int share = 6;  // log2 of a share's lanes
      while ((64 >> share) < n) --share;
      const int per = (1 << share) / TP;  // trials per share
      const int rank = __popcll(todo & ((1ull << (L.grp * G)) - 1ull));
      wave_sync();  // every lane has read the previous shares
      if (open && L.j == 0) {
        *reinterpret_cast<int *>(wave_lds + rank * lay.stride + lay.pick) = L.grp;
        wave_lds[L.grp * lay.stride + lay.fd] = f;
        wave_lds[L.grp * lay.stride + lay.fd + 1] = ddir;
      }
      wave_sync();
      const int s = lane >> share;
      const bool valid = s < n;
      const int target = *reinterpret_cast<const int *>(wave_lds + (valid ? s : 0) * lay.stride + lay.pick);
      double *sl = wave_lds + target * lay.stride;  // the slice of the group the lane works for
      const ReqHot &q = *reinterpret_cast<const ReqHot *>(sl + lay.q);
      const int t = base + ((lane / TP) & (per - 1));
      const int target_ls = q.iter_ls;
      const bool tries = t < target_ls;
      const double alpha = step_length(sl + lay.al, q.shrink, tries ? t : 0);
      const double bound = sl[lay.fd] + (q.armijo_c * alpha) * sl[lay.fd + 1];
      double ft = 0.0;
      U sums[E::K];
      if constexpr (whole_form<E>::value) {
        if (valid & tries) ft = E::template trial<U>(sl + lay.xs, sl + lay.ps, alpha, q.d);
      } else {
        ft = trial_value<OBJ, SLOTS, TP, U>(sl + lay.xs, sl + lay.ps, alpha, q.d, q.m, c, sums);
      }
      const bool ok = valid & tries & (ft <= bound);
      const uint64_t hits = __ballot(ok) & all_leaders;
      const uint64_t field = share == 6 ? ~0ull : (1ull << (1 << share)) - 1ull;  // a share's lanes
      if constexpr (!whole_form<E>::value) {
        // the first lane of a share's first passing trial keeps its sums
        const uint64_t before = hits & ((1ull << lane) - 1ull);
        if (lay.acc >= 0 && ((hits >> lane) & 1ull) && (before >> (s << share)) == 0ull)
#pragma unroll
          for (int kk = 0; kk < E::K; ++kk) sl[lay.acc + kk] = (double)sums[kk];
      }
      if (open) {
        const uint64_t mine = (hits >> ((rank << share) & 63)) & field;
        if (mine != 0ull) {
          taken = base + (__ffsll((unsigned long long)mine) - 1) / TP;
          open = false;
        } else {
          open = base + per < iter_ls;
        }
      }
      base += per;
      todo = __ballot(open && L.j == 0);
    }
  }
  return taken;
}

}  // namespace zeus

