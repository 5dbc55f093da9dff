// zeus_lbfgs_kernels.h -- limited-memory BFGS kernel template for gfx950: the BFGS run of Alg. 4 /
// Alg. 10 with the dual-number gradient of Alg. 5 and the Armijo search of
// Alg. 6, but the search direction comes from the m most recent (s, y) pairs
// by the two-loop recursion (Nocedal and Wright, "Numerical Optimization",
// 2nd ed., Alg. 7.4; H0 = gamma I with gamma = s'y / y'y of the newest pair,
// their eq. 7.20), the remedy the paper names for the O(d^2) update.
//
// Mapping: one group of G lanes per start (G a power of two <= 64, so a group
// never spans two wavefronts); lane j owns the CPL consecutive coordinates
// CPL j .. CPL j + CPL - 1, so a single wavefront covers up to 256
// coordinates.  Each lane keeps its coordinates of the stored pairs in
// registers (2 m CPL doubles); there is no d x d matrix anywhere.  Sums over
// coordinates are the pairwise trees used everywhere: a lane's own coordinates
// first, then one lane butterfly.  The claim loop, termination, mixed
// precision and retirement follow the BFGS kernel.
//
// Bound by VALU issue: the two-loop recursion is a chain of 2 m sums over
// coordinates.  With the coordinates j, j + G, ... in lane j every block of G
// coordinates took a butterfly of its own (four per sum at 256 slots), which
// was most of the kernel.  Rosenbrock, m = 8: d = 200, 8,192 starts 40.1 ->
// 21.3 ms (with one trial a round, below), d = 50, 65,536 starts 26.9 -> 11.9 ms,
// d = 100, 8,192 starts 13.3 -> 6.3 ms.  Launches with few starts, and those that
// end with a stalled one, wait for single iterations instead; they run with a
// coordinate per lane (lbfgs_spread).
#pragma once

#include "zeus_bfgs_common.h"

namespace zeus {
namespace {

constexpr int kHist = kLbfgsMaxHistory;  // pairs kept in registers (m <= kHist)

// Per-group LDS slice: the point under evaluation and the search direction
// (the line search reads both in full), the step lengths, the accepted
// trial's term sums, the start's counts, the request, f and g'p of the point
// whose search runs, and the searches' scratch.
__device__ __host__ __forceinline__ constexpr int lbfgs_stride(int slots) {
  return 2 * slots + kTabTrials + kMaxSums + 1 + kHotDoubles + 3 + kHist;
}
__device__ __host__ __forceinline__ constexpr SearchLayout lbfgs_search_layout(int slots) {
  const int al = 2 * slots, acc = al + kTabTrials, q = acc + kMaxSums + 1, fd = q + kHotDoubles;
  return SearchLayout{lbfgs_stride(slots), 0, slots, al, q, fd, fd + 2, acc};
}

template <int OBJ, int G, int CPL, class T>
__device__ __forceinline__ double value_slots(const GroupLanes<G> &L, int d, const double *xs) {
  return group_value_slots<OBJ, G, CPL, T>(L, d, xs);
}

// Two waves per SIMD for the 4-coordinate kernels of the polynomial
// objectives, which then take 245 to 256 registers: with 64 lanes up to 4 spilled,
// with fewer 16 to 20 for Rosenbrock (18 to 30 in mixed precision) and 4 to 10 for
// the others.  (The transcendental ones would spill over a hundred and stay at
// one wave, and user code is of unknown size.)
template <int OBJ, int CPL>
constexpr int kLbfgsWaves =
    CPL == 4 && OBJ != kRastrigin && OBJ != kAckley && OBJ != kUser ? 2 : 1;

template <int OBJ, int G, int CPL, class T>
__global__ __launch_bounds__(kBfgsBlock) __attribute__((amdgpu_waves_per_eu(kLbfgsWaves<OBJ, CPL>)))
void lbfgs_kernel(const ReqDev *reqs, int nreq, BatchDev *hdr, int64_t total) {
  constexpr bool kMixed = sizeof(T) != sizeof(double);
  constexpr int S = 64 / G;  // groups per wave
  constexpr int SLOTS = G * CPL;
  extern __shared__ double smem[];
  const GroupLanes<G> L;
  const int j = L.j;
  double *xs, *ps, *al, *acc, *av;
  StartCounts *cnt;  // the start's pair skips and direction resets (lane 0)
  ReqHot *qh;
  constexpr SearchLayout lay = lbfgs_search_layout(SLOTS);
  // Lanes per trial.  With several coordinates per lane a trial takes all the
  // group's lanes, a lane its own coordinates' terms: at one to two trials per
  // iteration more of them a round are mostly wasted (two a round: d = 200 26.5 ms
  // against 22.3, d = 100 7.2 against 6.4), and wave_search gives a search that
  // goes on the other groups' lanes.  Groups of four lanes take two or four, for
  // the starts that stall at small d (Ackley d = 4, 8,192 starts: 13.4 ms with one,
  // 7.7 with four).  With a coordinate per lane a round has four trials as in
  // the BFGS kernels, on 64 lanes two (Styblinski-Tang d = 120, 1,024 starts that
  // stall, 300 iterations: 2.2 ms with one, 1.4 with two).
  constexpr bool kCostly = OBJ == kRastrigin || OBJ == kAckley;
  constexpr int TP = whole_form<Elem<OBJ>>::value || SLOTS == 4      ? 1
                     : G == 64 && CPL <= 2 && !(CPL == 2 && kCostly) ? 32
                     : CPL == 1                                      ? G / 4
                     : G == 4                                        ? 2
                                                                     : G;
  double *wave_lds = smem + (size_t)((threadIdx.x >> 6) * S) * lay.stride;
  {
    double *base = wave_lds + L.grp * lay.stride;
    xs = base + lay.xs;
    ps = base + lay.ps;
    al = base + lay.al;
    acc = base + lay.acc;
    cnt = reinterpret_cast<StartCounts *>(acc + kMaxSums);
    qh = reinterpret_cast<ReqHot *>(base + lay.q);
    av = base + lay.pick + 1;
  }

  const int j0 = CPL * j;  // the lane's first coordinate
  bool own[CPL];
  double gj[CPL], sj[CPL];  // x and p stay in LDS (xs, ps)
  // The stored pairs, newest last: pair i holds from kHist - count on.  The
  // newest has a fixed place, so a new pair moves the others down one place
  // (a register copy each) and nothing is selected by a run-time index.
  double hs[kHist][CPL], hy[kHist][CPL], hrho[kHist];
  double gamma = 0.0;                                    // s'y / y'y of the newest pair
  int count = 0;                                         // pairs stored
  double f = 0.0;
  int64_t idx = -1;
  int k = 0, ls_trials = 0;
  bool fresh = false, first = true, alive = true;
  bool hi = !kMixed;
#pragma unroll
  for (int c = 0; c < CPL; ++c) own[c] = false, gj[c] = sj[c] = 0.0;
#pragma unroll
  for (int i = 0; i < kHist; ++i) {
    hrho[i] = 0.0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) hs[i][c] = hy[i][c] = 0.0;
  }
  const int es_pass = es_pass_of(hdr);
  int claims = 0;  // starts claimed after the first (second early-stop pass)
  int cur_ri = -1;  // the request whose scalars and step lengths the group's LDS holds
  HotRegs<G> hot{};
  bool have_acc = false;  // acc holds the term sums at xs (value_grad_slots)

  for (;;) {
    // -- claim a start when idle (as the BFGS kernel) -----------------------
    while (alive && idx < 0) {
      const unsigned long long groups = (unsigned long long)gridDim.x * (kBfgsBlock / G);
      const unsigned long long self =
          (unsigned long long)blockIdx.x * (kBfgsBlock / G) + (threadIdx.x >> 6) * S + L.grp;
      unsigned long long got = 0;
      if (first) {
        got = self;
        first = false;
      } else if (es_pass == 2) {
        got = strided_claim(self, groups, ++claims);
      } else {
        if (j == 0) got = groups + atomicAdd((unsigned long long *)&hdr->queue, 1ull);
        got = __shfl(got, L.grp * G, 64);
      }
      if (got >= (unsigned long long)total) {
        alive = false;
        break;
      }
      const int ri = request_of(reqs, nreq, (int64_t)got);
      const ReqDev &rq = reqs[ri];
      idx = (int64_t)got - rq.start_offset + rq.slice_first;
      if (es_pass == 2 && !es_rerun(rq, idx)) {  // keeps its first-pass result
        idx = -1;
        continue;
      }
      const int d0 = rq.d;
      if (ri != cur_ri) {  // the LDS slice still holds the previous start's request
        if (j == 0) load_hot<OBJ>(*qh, rq, ri, es_pass);
        fill_step_lengths(al, rq.shrink, j, G);
        cur_ri = ri;
        wave_sync();
        hot.take(*qh);
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        own[c] = j0 + c < d0;
        xs[j0 + c] = own[c] ? rq.ws.x[idx * d0 + j0 + c] : 0.0;  // x <- swarm[i]
      }
      if (j == 0) *cnt = StartCounts{0, 0};
      count = 0;
      k = 0;
      ls_trials = 0;
      fresh = true;
      hi = !kMixed;
    }
    if (S == 1 ? !alive : __ballot(alive) == 0ull) break;
    wave_sync();
    const ReqHot &q = *qh;
    const int d = hot.d;
    bool search = false;  // the group's start goes on to a line search
    double ddir = 0.0;
    if (S == 1 || alive) do {
      // the group's stopping bound, read early (its use is at the termination
      // test) and taken from one lane: the bound falls while the kernel runs
      int bound = 0x7fffffff;
      if (hot.es) bound = __shfl(es_load(q.es + kEsBound), L.grp * G, 64);

      // -- value and gradient at xs -------------------------------------------
      double gn[CPL];
      double fn;
      if (hi)
        fn = value_grad_slots<OBJ, G, CPL, double>(L, d, xs, gn, have_acc ? acc : nullptr);
      else
        fn = value_grad_slots<OBJ, G, CPL, T>(L, d, xs, gn, have_acc ? acc : nullptr);
      have_acc = false;

      // y's, y'y and g'g are formed together (independent sums overlap);
      // right after a claim or an escalation the first two are not used
      double yj[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) yj[c] = gn[c] - gj[c];
      const double sy = slot_dot<G, CPL>(yj, sj);
      const double yy = slot_dot<G, CPL>(yj, yj);
      const double gg = slot_dot<G, CPL>(gn, gn);

      // -- after a step: keep (s, y) when y's > 0, dropping the oldest pair ----
      if (!fresh) {
        if (sy > 0.0) {
#pragma unroll
          for (int i = 0; i + 1 < kHist; ++i) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
              hs[i][c] = hs[i + 1][c];
              hy[i][c] = hy[i + 1][c];
            }
            hrho[i] = hrho[i + 1];
          }
#pragma unroll
          for (int c = 0; c < CPL; ++c) {
            hs[kHist - 1][c] = sj[c];
            hy[kHist - 1][c] = yj[c];
          }
          hrho[kHist - 1] = 1.0 / sy;
          gamma = sy / yy;
          if (count < q.m_hist) ++count;
        } else if (j == 0) {
          ++cnt->skips;
        }
        ++k;
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) gj[c] = gn[c];
      f = fn;
      fresh = false;
      if (k < hot.trace_len)
#pragma unroll
        for (int c = 0; c < CPL; ++c)
          if (own[c]) reqs[q.ri].trace[(idx * hot.trace_len + k) * d + j0 + c] = xs[j0 + c];

      // -- termination -----------------------------------------------------------
      bool bad = !__builtin_isfinite(f);
#pragma unroll
      for (int c = 0; c < CPL; ++c) bad = bad || (own[c] && !__builtin_isfinite(gj[c]));
      const bool any_bad = L.ballot(bad) != 0ull;
      if (kMixed && !hi && (any_bad || norm_below(gg, 10.0 * hot.tol))) {
        hi = true;  // escalate: re-evaluate this point in FP64
        fresh = true;
        break;
      }
      int status = -1;
      if (any_bad)
        status = ZEUS_ST_NONFINITE;
      else if (norm_below(gg, hot.tol))
        status = ZEUS_ST_CONVERGED;
      else
        status = budget_status(q, hot.iter_bfgs, k, bound);
      if (status >= 0) {
        const ReqDev &rq = reqs[q.ri];
        const int tl = hot.trace_len;
        if (status == ZEUS_ST_CONVERGED && hot.es && j == 0) es_converged(q.es, k, q.iter_bfgs, q.es_c);
#pragma unroll
        for (int c = 0; c < CPL; ++c)
          if (own[c]) rq.out_x[idx * d + j0 + c] = xs[j0 + c];
        if (kMixed && !hi) f = value_slots<OBJ, G, CPL, double>(L, d, xs);
        if (j == 0) {
          rq.out_f[idx] = f;
          rq.out_iters[idx] = k;
          rq.out_status[idx] = status;
          if (rq.out_ls) rq.out_ls[idx] = ls_trials;
          if (rq.out_skips) rq.out_skips[idx] = cnt->skips;
          if (rq.out_resets) rq.out_resets[idx] = cnt->resets;
        }
        if (tl)
#pragma unroll
          for (int c = 0; c < CPL; ++c)
            if (own[c])
              for (int kk = k + 1; kk < tl; ++kk)
                rq.trace[(idx * tl + kk) * d + j0 + c] = __builtin_nan("");
        idx = -1;
        break;
      }

      // -- search direction: two-loop recursion over the stored pairs -----------
      double qv[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) qv[c] = gj[c];
#pragma unroll
      for (int i = kHist - 1; i >= 0; --i) {
        if (i >= kHist - count) {  // newest pair first: alpha_i = rho_i s_i'q, q <- q - alpha_i y_i
          const double alpha = hrho[i] * slot_dot<G, CPL>(hs[i], qv);
          av[i] = alpha;
#pragma unroll
          for (int c = 0; c < CPL; ++c) qv[c] = __builtin_fma(-alpha, hy[i][c], qv[c]);
        }
      }
      if (count > 0)  // r = gamma q
#pragma unroll
        for (int c = 0; c < CPL; ++c) qv[c] = gamma * qv[c];
#pragma unroll
      for (int i = 0; i < kHist; ++i)
        if (i >= kHist - count) {  // oldest pair first: beta = rho_i y_i'r, r <- r + (alpha_i - beta) s_i
          const double beta = hrho[i] * slot_dot<G, CPL>(hy[i], qv);
#pragma unroll
          for (int c = 0; c < CPL; ++c) qv[c] = __builtin_fma(av[i] - beta, hs[i][c], qv[c]);
        }
      double pj[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) pj[c] = own[c] ? -qv[c] : 0.0;
      ddir = slot_dot<G, CPL>(gj, pj);
      if (!(ddir < 0.0)) {  // not a descent direction: forget the pairs, p = -g
        if (j == 0) ++cnt->resets;
        count = 0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) pj[c] = own[c] ? -gj[c] : 0.0;
        ddir = slot_dot<G, CPL>(gj, pj);
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) ps[j0 + c] = pj[c];
      search = true;
    } while (false);

    // -- Armijo backtracking, by every lane of the wave -------------------------
    if (S == 1 ? !search : __ballot(search) == 0ull) continue;
    wave_sync();
    int taken = -1;
    if constexpr (kMixed) {
      if (__ballot(search && !hi) != 0ull) {
        const int tk = wave_search<OBJ, G, SLOTS, TP, true, T>(L, hot, search && !hi, f, ddir, wave_lds, lay);
        if (search && !hi) {
          taken = tk;
          if (tk < 0) {
            ls_trials += hot.iter_ls;
            hi = true;
            fresh = true;
            search = false;
          }
        }
      }
      if (__ballot(search && taken < 0) != 0ull) {
        const bool need = search && taken < 0;
        const int tk = wave_search<OBJ, G, SLOTS, TP, true, double>(L, hot, need, f, ddir, wave_lds, lay);
        if (need) taken = tk;
      }
    } else {
      taken = wave_search<OBJ, G, SLOTS, TP, true, double>(L, hot, search, f, ddir, wave_lds, lay);
    }
    wave_sync();  // every lane has read xs and ps in the line search

    // -- step ---------------------------------------------------------------------
    if (search) {
      // the accepted trial's term sums are those of the next evaluation
      have_acc = taken >= 0 && !whole_form<Elem<OBJ>>::value;
      const int nshrink = taken >= 0 ? taken : hot.iter_ls;
      ls_trials += taken >= 0 ? taken + 1 : hot.iter_ls;
      const double a = step_length(al, q.shrink, nshrink);
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const double x = xs[j0 + c], xnew = x + a * ps[j0 + c];
        sj[c] = own[c] ? xnew - x : 0.0;
        xs[j0 + c] = own[c] ? xnew : 0.0;
      }
    }
  }
}

}  // namespace
}  // namespace zeus
