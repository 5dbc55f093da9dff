// zeus_bfgs_wide.hip -- the BFGS phase for 208 < d <= 256 on gfx950 (Alg. 4 /
// Alg. 10 with the dual-number gradient of Alg. 5 and the Armijo search of
// Alg. 6): one block of eight wavefronts per start, the inverse Hessian spread
// over registers, LDS and a device-memory slot of the block.
//
//  * H is 256 x 256 (zero-padded past the dimension, ones on the padded
//    diagonal), a 4 x 4 grid of 64 x 64 tiles.  512 KB are the whole register
//    file of a CU, so it cannot stay there beside the rest of an iteration;
//    wavefront w holds two tiles of rows 64 (w & 3) .. + 63: the one of
//    columns 64 (w >> 2) .. + 63 in its registers, in the 4 x 16 lane tiles of
//    the narrow kernel's 64-lane groups (zeus_group.h Tile), and the one 128
//    columns to the right, a row per lane, as four strips of 16 columns:
//    strips 0 and 1 in LDS (128 KB for the block), strips 2 and 3 in the slot
//    (at most 128 KB a block: 32 MB for the chip, which its caches hold).
//    Strips wholly in the padding are skipped.
//  * Every wavefront keeps all coordinates (lane l the coordinates 4 l .. 4 l + 3)
//    and evaluates value, gradient and sums for itself, so an iteration has
//    three barriers: one after each product's partial sums (u = H y and
//    H_new g) and one per line-search round (eight trials, one per wavefront).
//    The vectors of an iteration are shared in LDS: all wavefronts write the
//    same values, and a vector is written again only after a barrier that
//    follows its last reader.
//  * A row's product with a vector is a fused multiply-add chain over each
//    block of 16 consecutive columns, the block sums added pairwise over the
//    16 blocks (the order of every other kernel): each tile's four blocks meet
//    in its wavefront, the four tiles of a row through LDS.
//  * The strips are updated and multiplied by g in one pass.
//  * Starts are claimed as by the other kernels: first the block's own index,
//    then an agent-scope work counter.
// The control flow is uniform across the block (one start per block), so
// every barrier is reached by all its threads.  One block fills a CU's LDS.
//
// Bound by the strips' traffic and by latency between the barriers: per
// iteration and block 128 KB of LDS and up to 128 KB of the slot are read twice
// and written once.  With all of H in the slot, streamed from device memory,
// Rosenbrock with 509 starts took 169 ms at d = 256 against 33.5 ms, 101 ms at
// d = 209 against 23.6 ms, and with 2,048 starts 645 ms at d = 256 against 106 ms.
// With a coordinate per lane and every sum finished across the block (seven
// barriers, less arithmetic) d = 256 took 42.3 and 148 ms.
#include "zeus_block.h"

namespace zeus {
namespace {

constexpr int kWW = 8;                    // wavefronts per start
constexpr int kWLanes = 64 * kWW;         // lanes per start
constexpr int kWVec = tile_vec_len(256);  // doubles of a padded operand vector (vpos<256>)
constexpr int kStripLds = 2;              // strips of a wavefront in LDS (the other two in the slot)
// doubles of a wavefront's strips in the slot
constexpr int kSlotWave = (4 - kStripLds) * 16 * 64;
static_assert(kWW * kSlotWave == kWideSlotDoubles, "the slot holds the strips that are not in LDS");
static_assert(128 + 16 * kStripLds == 160, "up to dimension 160 no strip is in the slot");

struct alignas(16) Pair {
  double a, b;  // two consecutive columns
};

struct WideShm {
  // two buffers where the old vector is still read while the new one is
  // written (x in the step, g for y)
  alignas(16) double xs[2][256];    // iterate under evaluation (x, then x_new), zero past d
  alignas(16) double ps[256];       // search direction
  alignas(16) double gs[2][kWVec];  // g, operand of p = -H g, padded layout
  alignas(16) double vs[kWVec];     // y, operand of u = H y, then u, padded layout
  alignas(16) double ss[kWVec];     // s = x_new - x, padded layout
  alignas(16) double part[2][4][256];  // [product][tile column][row] partial sums
  double red[1][1][kWW];         // (its extent is the number of wavefronts)
  double tsum[2 * kWW][kMaxSums];     // [phase * waves + wave][sum] line-search trials' term sums
  double al[kTabTrials];
  int pass[2][kWW];              // [phase][wave] line-search outcome
  StartCounts cnt;               // update skips and direction resets (thread 0)
  unsigned long long got;
  int bound;                     // early-stop bound
  ReqHot q;
  // [wave][strip][column pair][row]; last, so that the fields above stay within
  // reach of the 16-bit offsets of LDS instructions from one base
  Pair hl[kWW][kStripLds][8][64];
};
static_assert(sizeof(WideShm) <= 160 * 1024, "the block's state fits the LDS of a CU");

// The strips of a wavefront's second tile: strip s, column pair k of this
// lane's row.
struct Strips {
  Pair *lds;   // this lane's entry of strip 0, pair 0 in LDS
  Pair *slot;  // ... of strip kStripLds in the slot
  int live;    // strips that hold a column below the dimension (0: none, or no such row)
  __device__ __forceinline__ Pair *at(int s, int k) const {
    return s < kStripLds ? lds + (s * 8 + k) * 64 : slot + ((s - kStripLds) * 8 + k) * 64;
  }
};

__device__ __forceinline__ void strips_identity(const Strips &t, int row, int c0) {
  row = Tile<64>::opaque(row);  // once per start: keeps the pattern out of registers
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if (s < t.live)
#pragma unroll 1
      for (int k = 0; k < 8; ++k) {
        const int c = c0 + 16 * s + 2 * k;
        *t.at(s, k) = Pair{row == c ? 1.0 : 0.0, row == c + 1 ? 1.0 : 0.0};
      }
}

// This lane's row of the second tile times a vector: vec is the padded vector
// from the tile's first column; the four strips' chains added pairwise.  The
// pairs are loaded four at a time (a memory clobber keeps the next four from
// being hoisted, which bounds the live registers).
__device__ __forceinline__ double strips_matvec(const Strips &t, const double *vec, int lane) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  static_for<0, 4>([&](auto ss) {
    constexpr int s = 3 - decltype(ss)::value;  // the slot's strips first
    if (s < t.live) {
      const double v = vec[18 * s + (lane & 15)];  // padded: strip s starts at 18 s
      static_for<0, 2>([&](auto hh) {
        constexpr int k0 = 4 * decltype(hh)::value;
        asm volatile("" ::: "memory");
        Pair h[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = *t.at(s, k0 + k);
        static_for<0, 4>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          fmac_bcast<2 * (k0 + k)>(acc[s], v, h[k].a);
          fmac_bcast<2 * (k0 + k) + 1>(acc[s], v, h[k].b);
        });
      });
    }
  });
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The rank-2 update of the second tile and its product with g in one pass:
// element (r, c) by fma(e_r, s_c, fma(a_r, u_c, H_rc)); us, ss, gs are the padded
// vectors from the tile's first column.  fin false: a or e is not finite and
// the padding's columns get the identity back.
__device__ __forceinline__ double strips_update_matvec(const Strips &t, const double *us,
                                                       const double *ss, const double *gs, double a,
                                                       double e, bool fin, int row, int c0, int d,
                                                       int lane) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  static_for<0, 4>([&](auto st) {
    constexpr int s = 3 - decltype(st)::value;
    if (s < t.live) {
      const int o = 18 * s + (lane & 15);
      const double u = us[o], sv = ss[o], g = gs[o];
      static_for<0, 2>([&](auto hh) {
        constexpr int k0 = 4 * decltype(hh)::value;
        asm volatile("" ::: "memory");
        Pair h[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = *t.at(s, k0 + k);
        static_for<0, 4>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          upd_bcast<2 * (k0 + k)>(h[k].a, u, sv, a, e);
          upd_bcast<2 * (k0 + k) + 1>(h[k].b, u, sv, a, e);
        });
        if (!fin) {
          const int r = Tile<64>::opaque(row);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int c = c0 + 16 * s + 2 * (k0 + k);
            if (c >= d) h[k].a = r == c ? 1.0 : 0.0;
            if (c + 1 >= d) h[k].b = r == c + 1 ? 1.0 : 0.0;
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) *t.at(s, k0 + k) = h[k];
        static_for<0, 4>([&](auto kk) {
          constexpr int k = decltype(kk)::value;
          fmac_bcast<2 * (k0 + k)>(acc[s], g, h[k].a);
          fmac_bcast<2 * (k0 + k) + 1>(acc[s], g, h[k].b);
        });
      });
    }
  });
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The sums of rows 4 lane .. + 3 over the four tile columns (all wavefronts).
__device__ __forceinline__ void wide_rows(const WideShm &sh, int buf, int j0, double (&r)[4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int i = j0 + c;
    r[c] = (sh.part[buf][0][i] + sh.part[buf][1][i]) + (sh.part[buf][2][i] + sh.part[buf][3][i]);
  }
}

// See the narrow kernel for the mixed-precision rules (T = float).
template <int OBJ, class T>
__global__ __launch_bounds__(kWLanes) __attribute__((amdgpu_waves_per_eu(2)))
void bfgs_wide_kernel(const ReqDev *reqs, int nreq, BatchDev *hdr, int64_t total, double *slots,
                      int64_t slot_doubles) {
  constexpr bool kMixed = sizeof(T) != sizeof(double);
  __shared__ WideShm sh;
  const GroupLanes<64> L;
  const int j = threadIdx.x;
  const int lane = j & 63, w = __builtin_amdgcn_readfirstlane(j >> 6);
  const int r0 = 64 * (w & 3), tq = w >> 2;  // the wavefront's rows, its register tile's column
  const int c0 = 64 * tq, c1 = c0 + 128;     // first columns of its two tiles
  const int row = r0 + lane;                 // this lane's row of the second tile
  const int j0 = 4 * lane;                   // the lane's coordinates j0 .. j0 + 3
  const int v0 = vpos<256>(j0);              // their place in a padded vector
  Tile<64> H;
  Strips st;
  st.lds = &sh.hl[w][0][0][lane];
  st.slot = reinterpret_cast<Pair *>(slots + (int64_t)blockIdx.x * slot_doubles + w * kSlotWave) + lane;
  st.live = 0;
  int lsphase = 0;
  int acc = -1;  // slot of sh.tsum with the accepted trial's term sums (block_armijo), or -1
  bool first = true, fresh = false, hi = !kMixed;
  double f = 0.0;
  int xb = 0, gb = 0;  // the buffers of xs and gs that hold the current x and g
  int64_t idx = -1;
  int k = 0, ls_trials = 0, bound = 0;
  const int es_pass = es_pass_of(hdr);
  int claims = 0;  // starts claimed after the first (second early-stop pass; thread 0)

  for (;;) {
    if (idx < 0) {
      if (j == 0) {
        sh.got = first           ? (unsigned long long)blockIdx.x
                 : es_pass == 2 ? strided_claim(blockIdx.x, gridDim.x, ++claims)
                                : gridDim.x + atomicAdd((unsigned long long *)&hdr->queue, 1ull);
      }
      first = false;
      __syncthreads();
      const unsigned long long got = sh.got;
      if (got >= (unsigned long long)total) break;
      const int ri = request_of(reqs, nreq, (int64_t)got);
      const ReqDev &rq = reqs[ri];
      idx = (int64_t)got - rq.start_offset + rq.slice_first;
      if (es_pass == 2 && !es_rerun(rq, idx)) {  // keeps its first-pass result
        idx = -1;
        __syncthreads();  // every thread has read sh.got before the next claim writes it
        continue;
      }
      const int d0 = __builtin_amdgcn_readfirstlane(rq.d);
      if (j == 0) {
        load_hot<OBJ>(sh.q, rq, ri, es_pass);
        sh.cnt = StartCounts{0, 0};
        sh.bound = es_bound(sh.q);
      }
      fill_step_lengths(sh.al, rq.shrink, j, kWLanes);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sh.xs[xb][j0 + c] = j0 + c < d0 ? rq.ws.x[idx * d0 + j0 + c] : 0.0;  // x <- swarm[i]
        sh.gs[gb][v0 + c] = sh.ss[v0 + c] = 0.0;
      }
      st.live = r0 < d0 && c1 < d0 ? (d0 - c1 + 15) / 16 : 0;
      if (st.live > 4) st.live = 4;
      strips_identity(st, row, c1);  // H <- I (the register tile before the first product)
      k = 0;
      ls_trials = 0;
      fresh = true;
      hi = !kMixed;
      __syncthreads();  // the request and the bound are visible
      bound = sh.bound;
    }
    wave_sync();
    const ReqHot &q = sh.q;
    const int d = __builtin_amdgcn_readfirstlane(q.d);

    // -- value and gradient at xs, on every wavefront ---------------------------
    const double *xs = sh.xs[xb];
    double gn[4], fn;
    {
      const double *known = acc >= 0 ? sh.tsum[acc] : nullptr;
      if (hi)
        fn = value_grad_slots<OBJ, 64, 4, double>(L, d, xs, gn, known);
      else
        fn = value_grad_slots<OBJ, 64, 4, T>(L, d, xs, gn, known);
    }
    acc = -1;

    // y's, g'g and the non-finite test; right after a claim or an escalation
    // y's is not used
    double yj[4], sj[4];
    bool bad = !__builtin_isfinite(fn);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      yj[c] = gn[c] - sh.gs[gb][v0 + c];  // zero beyond the dimension
      sj[c] = sh.ss[v0 + c];
      bad = bad || (j0 + c < d && !__builtin_isfinite(gn[c]));
      sh.vs[v0 + c] = yj[c];
      sh.gs[gb ^ 1][v0 + c] = gn[c];
    }
    gb ^= 1;
    const double *gs = sh.gs[gb];
    const double sy = slot_dot<64, 4>(yj, sj);
    const double gg = slot_dot<64, 4>(gn, gn);
    const bool any_bad = __ballot(bad) != 0ull;

    // -- after a step: u = H y and the rank-2 update, the strips' part of the
    //    product H_new g with it --------------------------------------------
    bool updated = false;
    if (!fresh) {
      if (sy > 0.0) {  // curvature condition; skip the update otherwise
        const double rho = 1.0 / sy;
        wave_sync();
        sh.part[0][tq + 2][row] = strips_matvec(st, sh.vs + vpos<256>(c1), lane);
        sh.part[0][tq][row] = H.matvec_bcast(sh.vs[vpos<256>(c0 + lane)]);
        __syncthreads();
        double uj[4];
        wide_rows(sh, 0, j0, uj);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          uj[c] = j0 + c < d ? uj[c] : 0.0;
          sh.vs[v0 + c] = uj[c];  // every wavefront has formed its products of y
        }
        const double yu = slot_dot<64, 4>(yj, uj);
        const double beta = (rho * rho) * yu + rho;
        wave_sync();
        // H+ = H - rho (s u' + u s') + beta s s'   (u = H y); inf * 0 would
        // have reached the padding when a coefficient is not finite
        const double sr = sh.ss[vpos<256>(row)], ur = sh.vs[vpos<256>(row)];
        const double a = -rho * sr, e = beta * sr - rho * ur;
        sh.part[1][tq + 2][row] = strips_update_matvec(
            st, sh.vs + vpos<256>(c1), sh.ss + vpos<256>(c1), gs + vpos<256>(c1), a, e,
            __builtin_isfinite(a) && __builtin_isfinite(e), row, c1, d, lane);
        if (!H.rank2_bcast(rho, beta, sh.vs + vpos<256>(r0), sh.ss + vpos<256>(r0),
                           sh.vs[vpos<256>(c0 + lane)], sh.ss[vpos<256>(c0 + lane)], lane, 0.0, 0.0))
          H.restore_padding_at(lane, d, r0, c0);
        updated = true;
      } else if (j == 0) {
        ++sh.cnt.skips;
      }
      ++k;
    }
    f = fn;
    fresh = false;
    if (q.trace_len && w == 0 && k < q.trace_len)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (j0 + c < d) reqs[q.ri].trace[(idx * q.trace_len + k) * d + j0 + c] = xs[j0 + c];

    // -- termination: non-finite, ||g|| < Theta, budget ---------------------
    if (kMixed && !hi && (any_bad || norm_below(gg, 10.0 * q.tol))) {
      hi = true;  // escalate: re-evaluate this point in FP64
      fresh = true;
      __syncthreads();  // every wavefront has read the vectors that are written again
      continue;
    }
    int status = -1;
    if (any_bad)
      status = ZEUS_ST_NONFINITE;
    else if (norm_below(gg, q.tol))
      status = ZEUS_ST_CONVERGED;
    else
      status = budget_status(q, q.iter_bfgs, k, bound);
    if (status >= 0) {
      const ReqDev &rq = reqs[q.ri];
      const int tl = q.trace_len;
      if (status == ZEUS_ST_CONVERGED && q.es && j == 0) es_converged(q.es, k, q.iter_bfgs, q.es_c);
      if (kMixed && !hi) f = group_value_slots<OBJ, 64, 4, double>(L, d, xs);
      if (w == 0)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (j0 + c < d) {
            rq.out_x[idx * d + j0 + c] = xs[j0 + c];
            for (int kk = k + 1; kk < tl; ++kk)
              rq.trace[(idx * tl + kk) * d + j0 + c] = __builtin_nan("");
          }
      if (j == 0) {
        rq.out_f[idx] = f;
        rq.out_iters[idx] = k;
        rq.out_status[idx] = status;
        if (rq.out_ls) rq.out_ls[idx] = ls_trials;
        if (rq.out_skips) rq.out_skips[idx] = sh.cnt.skips;
        if (rq.out_resets) rq.out_resets[idx] = sh.cnt.resets;
      }
      idx = -1;
      __syncthreads();  // every wavefront is done with the request before the next claim
      continue;
    }

    // -- search direction p = -H g (reset to -g if not a descent direction) -
    // The register tile is the identity until the first update (k = 0);
    // setting it here rather than at the claim keeps the old tile's registers
    // from being live beside the new one's.
    if (k == 0) H.identity_at(lane, r0, c0);
    wave_sync();
    if (!updated) sh.part[1][tq + 2][row] = strips_matvec(st, gs + vpos<256>(c1), lane);
    sh.part[1][tq][row] = H.matvec_bcast(gs[vpos<256>(c0 + lane)]);
    __syncthreads();
    double pj[4], gj[4];
    wide_rows(sh, 1, j0, pj);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      gj[c] = gs[v0 + c];
      pj[c] = j0 + c < d ? -pj[c] : 0.0;
    }
    double ddir = slot_dot<64, 4>(gj, pj);
    if (!(ddir < 0.0)) {
      if (j == 0) ++sh.cnt.resets;
      H.identity_at(lane, r0, c0);
      strips_identity(st, row, c1);
#pragma unroll
      for (int c = 0; c < 4; ++c) pj[c] = j0 + c < d ? -gj[c] : 0.0;
      ddir = slot_dot<64, 4>(gj, pj);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) sh.ps[j0 + c] = pj[c];
    wave_sync();
    // the stopping bound for the next test, read by one thread for the block
    // and published by the search's first barrier: the bound falls while the
    // kernel runs
    if (j == 0) sh.bound = es_bound(q);

    // -- Armijo backtracking (Alg. 6) ---------------------------------------
    int taken;
    if (hi) {
      taken = block_armijo<OBJ, double, 256>(sh, xs, sh.ps, f, ddir, lsphase, &acc);
    } else {
      taken = block_armijo<OBJ, T, 256>(sh, xs, sh.ps, f, ddir, lsphase, &acc);
      if (taken < 0) {
        ls_trials += q.iter_ls;
        hi = true;  // escalate: FP32 cannot resolve this decrease
        fresh = true;
        continue;
      }
    }
    bound = sh.bound;
    const int nshrink = taken >= 0 ? taken : q.iter_ls;
    ls_trials += taken >= 0 ? taken + 1 : q.iter_ls;
    const double alpha = step_length(sh.al, q.shrink, nshrink);

    // -- step: x_new = x + alpha p, s = x_new - x -----------------------------
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double x = xs[j0 + c], xnew = x + alpha * sh.ps[j0 + c];
      sh.ss[v0 + c] = j0 + c < d ? xnew - x : 0.0;
      sh.xs[xb ^ 1][j0 + c] = j0 + c < d ? xnew : 0.0;
    }
    xb ^= 1;
  }
}

template <int OBJ, class T>
hipError_t launch_wide_t(const Group &g, int64_t want, int cus) {
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void *>(&bfgs_wide_kernel<OBJ, T>), kWLanes, 0);
  if (e != hipSuccess) return e;
  if (per_cu < 1) return hipErrorInvalidConfiguration;  // the block does not fit a CU
  int64_t cap = (int64_t)cus * per_cu;
  if (g.resident) {
    *g.resident = cap;
    return hipSuccess;
  }
  if (cap > g.wide_slots) cap = g.wide_slots;
  const int blocks = (int)(want < cap ? want : cap);
  hipLaunchKernelGGL((bfgs_wide_kernel<OBJ, T>), dim3(blocks), dim3(kWLanes), 0, g.stream, g.reqs,
                     g.nreq, g.hdr, g.total_starts, g.hslots, g.wide_slot_doubles);
  return hipGetLastError();
}

template <class T>
hipError_t launch_wide_prec(const Group &g, int64_t want, int cus) {
  switch (g.objective) {
    case kRosenbrock: return launch_wide_t<kRosenbrock, T>(g, want, cus);
    case kRastrigin: return launch_wide_t<kRastrigin, T>(g, want, cus);
    case kAckley: return launch_wide_t<kAckley, T>(g, want, cus);
    case kStyblinskiTang: return launch_wide_t<kStyblinskiTang, T>(g, want, cus);
    case kSphere: return launch_wide_t<kSphere, T>(g, want, cus);
    case kQuartic: return launch_wide_t<kQuartic, T>(g, want, cus);
    default: return hipErrorInvalidValue;  // Goldstein-Price has d == 2
  }
}

}  // namespace

hipError_t launch_bfgs_wide(const Group &g, int cus) {
  if (!g.hslots || g.wide_slots < 1) return hipErrorInvalidValue;
  const int64_t want = g.total_starts;
  if (g.precision == ZEUS_MIXED) return launch_wide_prec<float>(g, want, cus);
  return launch_wide_prec<double>(g, want, cus);
}

}  // namespace zeus
