// zeus_bfgs_tile_kernels.h -- the BFGS phase for 64 < d <= 128 with the
// inverse Hessian on chip (Alg. 4 / Alg. 10 with the dual-number gradient of
// Alg. 5 and the Armijo search of Alg. 6): one block of four wavefronts per
// start.  Built into the library (zeus_bfgs_tile.hip) and into the run-time
// program of a user objective.
//
//  * H is 128 x 128 (zero-padded past the dimension, ones on the padded
//    diagonal) and split into four 64 x 64 quarters, one per wavefront:
//    wavefront w holds rows 64 (w & 1) .. + 63 and columns 64 (w >> 1) .. + 63
//    in its registers, in the 4 x 16 tiles of the narrow kernel's 64-lane
//    groups (zeus_group.h Tile), so H never leaves the chip;
//  * a row's product with a vector is a fused multiply-add chain over each
//    block of 16 consecutive columns, the block sums added pairwise: inside a
//    wavefront the four blocks of its quarter meet in two lane-swap levels,
//    then the two quarters of a row are added through LDS, which is the
//    pairwise tree over the eight blocks (the order of every other kernel);
//    lane i of wavefronts w and w + 2 both end with row 64 (w & 1) + i;
//  * every wavefront keeps all coordinates (lane l the coordinates 2 l and
//    2 l + 1) and forms value, gradient and sums for itself, so an iteration
//    has three barriers: one after each product's quarters (u = H y and
//    H_new g) and one per line-search round (four trials, one per wavefront).
//    The vectors the lanes exchange are shared in LDS: all wavefronts write
//    the same values, and a vector is written again only after a barrier that
//    follows its last reader (a copy per wavefront cost a user objective, which
//    reads the whole point for every coordinate, 13%).  With a coordinate per
//    lane and every sum finished across the block an iteration had seven
//    barriers; the second coordinate's gradient and the repeated sums cost
//    less than they did: Rosenbrock d = 128, 16,384 starts 89.7 -> 83.8 ms,
//    Styblinski-Tang 6.84 -> 6.37 ms, Ackley d = 128, 8,192 starts 2.10 -> 1.92 ms
//    (with the sine and cosine's branches gone).  Bound by VALU issue and by
//    latency between the barriers;
//  * a user objective's gradient is still formed once in the block, a
//    coordinate per lane, with a barrier of its own;
//  * starts are claimed as by the other kernels: first the block's own index,
//    then an agent-scope work counter.
// The control flow is uniform across the block (one start per block), so
// every barrier is reached by all its threads.
#pragma once

#include "zeus_block.h"

namespace zeus {
namespace {

constexpr int kTDim = kTileBlockDim;            // rows and columns of the padded H
constexpr int kQuarter = 64;                    // rows and columns of a wavefront's part
constexpr int kTVec = tile_vec_len(kTDim);      // doubles of a padded operand vector
static_assert(kTDim == 2 * kQuarter, "four wavefronts hold two by two quarters");

struct TileShm {
  double xs[kTDim];  // iterate under evaluation (x, then x_new), zero past d
  double ps[kTDim];  // search direction
  double vs[kTVec];  // y, then g: operand of u = H y and p = -H g, padded layout
  double ss[kTVec];  // s = x_new - x, padded layout
  double us[kTVec];  // u = H y, padded layout
  double part[2][kBlockWaves][kQuarter];  // each wavefront's products over its quarter (u, H g)
  double gx[kTDim];                       // the gradient, lane by lane (whole-form objectives)
  double red[1][1][kBlockWaves];          // (its extent is the number of wavefronts)
  double tsum[2 * kBlockWaves][kMaxSums];   // [phase * waves + wave][sum] line-search trials' term sums
  double al[kTabTrials];
  int pass[2][kBlockWaves];            // [phase][wave] line-search outcome
  StartCounts cnt;                     // update skips and direction resets (thread 0)
  unsigned long long got;
  int bound;                           // early-stop bound
  ReqHot q;
};

// Row products of H with the vector whose entries this wavefront left in v
// (padded layout): rows 2 lane and 2 lane + 1 in r.  Every wavefront forms its
// quarter's products; after the barrier each adds the two quarters of every
// row for itself.  The two products of an iteration use a buffer each, so a
// buffer is written again only after the barrier of the other.
__device__ __forceinline__ void tile_block_matvec(const Tile<64> &H, const double *v, TileShm &sh,
                                                  int buf, int lane, int w, int c0, double (&r)[2]) {
  sh.part[buf][w][lane] = H.matvec_bcast(v[vpos<kTDim>(c0 + lane)]);
  __syncthreads();
  const int hf = lane >> 5, i = (2 * lane) & 63;  // rows 2 lane, 2 lane + 1: half hf, place i, i + 1
#pragma unroll
  for (int c = 0; c < 2; ++c) r[c] = sh.part[buf][hf][i + c] + sh.part[buf][hf + 2][i + c];
}

// See the narrow kernel for the mixed-precision rules (T = float).
template <int OBJ, class T>
__global__ __launch_bounds__(kBlockLanes) __attribute__((amdgpu_waves_per_eu(2)))
void bfgs_tile_kernel(const ReqDev *reqs, int nreq, BatchDev *hdr, int64_t total) {
  constexpr bool kMixed = sizeof(T) != sizeof(double);
  constexpr bool kWhole = whole_form<Elem<OBJ>>::value;
  __shared__ TileShm sh;
  const GroupLanes<64> L;
  const int j = threadIdx.x;
  const int lane = j & 63, w = __builtin_amdgcn_readfirstlane(j >> 6);
  const int r0 = kQuarter * (w & 1), c0 = kQuarter * (w >> 1);  // this wavefront's quarter
  const int j0 = 2 * lane;                                      // the lane's coordinates j0, j0 + 1
  Tile<64> H;
  int lsphase = 0;
  int acc = -1;  // slot of sh.tsum with the accepted trial's term sums (block_armijo), or -1
  bool first = true, fresh = false, hi = !kMixed;
  double xj[2] = {0.0, 0.0}, gj[2] = {0.0, 0.0}, sj[2] = {0.0, 0.0}, f = 0.0;
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
      const int d0 = rq.d;
      if (j == 0) {
        load_hot<OBJ>(sh.q, rq, ri, es_pass);
        sh.cnt = StartCounts{0, 0};
        sh.bound = es_bound(sh.q);
      }
      fill_step_lengths(sh.al, rq.shrink, j, kBlockLanes);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        xj[c] = j0 + c < d0 ? rq.ws.x[idx * d0 + j0 + c] : 0.0;  // x <- swarm[i]
        sh.xs[j0 + c] = xj[c];
      }
      k = 0;  // H <- I before the first product (below)
      ls_trials = 0;
      fresh = true;
      hi = !kMixed;
      __syncthreads();  // the request and the bound are visible
      bound = sh.bound;
    }
    wave_sync();
    const ReqHot &q = sh.q;
    const int d = q.d;

    // -- value and gradient at xs, on every wavefront ---------------------------
    double gn[2], fn;
    if constexpr (kWhole) {
      // user code of unknown cost: a pass per coordinate, once in the block
      double g1[1];
      if (hi)
        fn = Elem<OBJ>::template value_grad<double>(sh.xs, d, j < d ? j : -1, &g1[0]);
      else
        fn = Elem<OBJ>::template value_grad<T>(sh.xs, d, j < d ? j : -1, &g1[0]);
      if (j < kTDim) sh.gx[j] = j < d ? g1[0] : 0.0;
      __syncthreads();
      gn[0] = sh.gx[j0];
      gn[1] = sh.gx[j0 + 1];
    } else {
      const double *known = acc >= 0 ? sh.tsum[acc] : nullptr;
      if (hi)
        fn = value_grad_slots<OBJ, 64, 2, double>(L, d, sh.xs, gn, known);
      else
        fn = value_grad_slots<OBJ, 64, 2, T>(L, d, sh.xs, gn, known);
    }
    acc = -1;

    // y's, g'g and the non-finite test; right after a claim or an escalation
    // y's is not used
    const double yj[2] = {gn[0] - gj[0], gn[1] - gj[1]};  // zero beyond the dimension
    const double sy = slot_dot<64, 2>(yj, sj);
    const double gg = slot_dot<64, 2>(gn, gn);
    const bool bad = (j0 < d && !__builtin_isfinite(gn[0])) ||
                     (j0 + 1 < d && !__builtin_isfinite(gn[1])) || !__builtin_isfinite(fn);
    const bool any_bad = __ballot(bad) != 0ull;

    // -- after a step: u = H y and the rank-2 update --------------------------
    if (!fresh) {
      if (sy > 0.0) {  // curvature condition; skip the update otherwise
        const double rho = 1.0 / sy;
#pragma unroll
        for (int c = 0; c < 2; ++c) sh.vs[vpos<kTDim>(j0) + c] = yj[c];
        wave_sync();
        double uj[2];
        tile_block_matvec(H, sh.vs, sh, 0, lane, w, c0, uj);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          uj[c] = j0 + c < d ? uj[c] : 0.0;
          sh.us[vpos<kTDim>(j0) + c] = uj[c];
          sh.ss[vpos<kTDim>(j0) + c] = sj[c];
        }
        const double yu = slot_dot<64, 2>(yj, uj);
        const double beta = (rho * rho) * yu + rho;
        wave_sync();
        // H+ = H - rho (s u' + u s') + beta s s'   (u = H y); inf * 0 would
        // have reached the padding when a coefficient is not finite
        if (!H.rank2_bcast(rho, beta, sh.us + vpos<kTDim>(r0), sh.ss + vpos<kTDim>(r0),
                           sh.us[vpos<kTDim>(c0 + lane)], sh.ss[vpos<kTDim>(c0 + lane)], lane, 0.0,
                           0.0))
          H.restore_padding_at(lane, d, r0, c0);
      } else if (j == 0) {
        ++sh.cnt.skips;
      }
      ++k;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) gj[c] = gn[c];
    f = fn;
    fresh = false;
    if (q.trace_len && w == 0 && k < q.trace_len)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (j0 + c < d) reqs[q.ri].trace[(idx * q.trace_len + k) * d + j0 + c] = xj[c];

    // -- termination: non-finite, ||g|| < Theta, budget ---------------------
    if (kMixed && !hi && (any_bad || norm_below(gg, 10.0 * q.tol))) {
      hi = true;  // escalate: re-evaluate this point in FP64
      fresh = true;
      if constexpr (kWhole) __syncthreads();  // gx has been read
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
      if (kMixed && !hi) f = group_value_slots<OBJ, 64, 2, double>(L, d, sh.xs);
      if (w == 0)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (j0 + c < d) {
            rq.out_x[idx * d + j0 + c] = xj[c];
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
    // H is the identity until the first update (k = 0).  Setting it here
    // rather than at the claim keeps the old tile's registers from being
    // live beside the new one's (the claim path rejoins the loop with H).
    if (k == 0) H.identity_at(lane, r0, c0);
    wave_sync();  // the product of y has read vs
#pragma unroll
    for (int c = 0; c < 2; ++c) sh.vs[vpos<kTDim>(j0) + c] = gj[c];
    wave_sync();
    double pj[2];
    tile_block_matvec(H, sh.vs, sh, 1, lane, w, c0, pj);
#pragma unroll
    for (int c = 0; c < 2; ++c) pj[c] = j0 + c < d ? -pj[c] : 0.0;
    double ddir = slot_dot<64, 2>(gj, pj);
    if (!(ddir < 0.0)) {
      if (j == 0) ++sh.cnt.resets;
      H.identity_at(lane, r0, c0);
#pragma unroll
      for (int c = 0; c < 2; ++c) pj[c] = j0 + c < d ? -gj[c] : 0.0;
      ddir = slot_dot<64, 2>(gj, pj);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) sh.ps[j0 + c] = pj[c];
    wave_sync();
    // the stopping bound for the next test, read by one thread for the block
    // and published by the search's first barrier: the bound falls while the
    // kernel runs
    if (j == 0) sh.bound = es_bound(q);

    // -- Armijo backtracking (Alg. 6) ---------------------------------------
    int taken;
    if (hi) {
      taken = block_armijo<OBJ, double, kTDim>(sh, sh.xs, sh.ps, f, ddir, lsphase, &acc);
    } else {
      taken = block_armijo<OBJ, T, kTDim>(sh, sh.xs, sh.ps, f, ddir, lsphase, &acc);
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
    wave_sync();  // the wavefront has read xs in its trials
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const double xnew = xj[c] + alpha * sh.ps[j0 + c];
      sj[c] = j0 + c < d ? xnew - xj[c] : 0.0;
      xj[c] = j0 + c < d ? xnew : 0.0;
      sh.xs[j0 + c] = xj[c];
    }
  }
}

}  // namespace
}  // namespace zeus
