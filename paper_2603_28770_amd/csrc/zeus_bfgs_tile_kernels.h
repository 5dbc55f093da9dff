// zeus_bfgs_tile_kernels.h -- the BFGS phase for 64 < d <= 128 with the
// inverse Hessian on chip (Alg. 4 / Alg. 10 with the dual-number gradient of
// Alg. 5 and the Armijo search of Alg. 6): one block of three (d <= 96) or
// four wavefronts per start.  Built into the library (zeus_bfgs_tile.hip) and,
// with four wavefronts, into the run-time program of a user objective.
//
//  * H is padded to 96 x 96 or 128 x 128 (zeros past the dimension, ones on
//    the padded diagonal), all of it in the wavefronts' registers.  Three
//    wavefronts hold two blocks of 16 columns each (ColumnTile); four hold a
//    64 x 64 quarter each, in the 4 x 16 tiles of the narrow kernel's 64-lane
//    groups (QuarterTile);
//  * a row's product with a vector is a fused multiply-add chain over each
//    block of 16 consecutive columns, the block sums added pairwise: a
//    wavefront's blocks of a row meet in lane swaps, its pieces of a row are
//    added through LDS, which is the pairwise tree over the blocks (the order
//    of every other kernel);
//  * in the 128 columns of four wavefronts, d = 65 .. 96 did 1.8 times the work
//    on H, with 224 registers and two blocks on a CU.  Three wavefronts of 96
//    columns fit 168 registers and four blocks.  Rosenbrock, 8,192 starts:
//    d = 96 35.0 -> 21.2 ms, d = 65 25.7 -> 15.4 ms (at two blocks still 32.5 and
//    23.8); Styblinski-Tang d = 90 3.1 -> 1.9 ms; Ackley d = 70 1.77 -> 1.55 ms,
//    with 67 registers spilled (not in small launches, see tile_three).  Columns
//    split this way among four wavefronts need four pieces per row instead of
//    two: d = 128 86.0 ms against 83.1;
//  * every wavefront keeps all coordinates (lane l the coordinates 2 l and
//    2 l + 1) and forms value, gradient and sums for itself, so an iteration
//    has three barriers: one after each product's pieces (u = H y and
//    H_new g) and one per line-search round (a trial per wavefront).
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

constexpr int kTDim = kTileBlockDim;            // coordinate slots (two per lane)
constexpr int kTVec = tile_vec_len(kTDim);      // doubles of a padded operand vector
template <int NB>
constexpr int kTWaves = NB / 2;                 // wavefronts per start

template <int NB>
struct TileShm {
  static constexpr int NW = kTWaves<NB>;
  double xs[kTDim];  // iterate under evaluation (x, then x_new), zero past d
  double ps[kTDim];  // search direction
  double vs[kTVec];  // y, then g: operand of u = H y and p = -H g, padded layout
  double ss[kTVec];  // s = x_new - x, padded layout
  double us[kTVec];  // u = H y, padded layout
  double part[2][3][kTDim];   // [product: u, H g][piece][row]
  double gx[kTDim];           // the gradient, lane by lane (whole-form objectives)
  double red[1][1][NW];       // (its extent is the number of wavefronts)
  double tsum[2 * NW][kMaxSums];   // [phase * waves + wave][sum] line-search trials' term sums
  double al[kTabTrials];
  int pass[2][NW];                 // [phase][wave] line-search outcome
  StartCounts cnt;                 // update skips and direction resets (thread 0)
  unsigned long long got;
  int bound;                       // early-stop bound
  ReqHot q;
};

// The columns of one of three wavefronts: its 16-lane rows hold its two column
// blocks for the upper and the lower 48 rows.  Lane l holds, for t < 3, row
// 48 (l / 32) + 16 t + l mod 16 at the 16 columns of block 2 w + (l / 16) mod 2.
struct ColumnTile {
  static constexpr int R = 3;
  double h[16 * R];
  __device__ __forceinline__ static int row(int lane, int t) {
    return 16 * R * (lane >> 5) + 16 * t + (lane & 15);
  }
  __device__ __forceinline__ static int col(int lane, int w) { return 16 * (2 * w + ((lane >> 4) & 1)); }

  __device__ __forceinline__ void identity(int lane, int w) {
    lane = Tile<64>::opaque(lane);
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int k = 0; k < 16; ++k) h[16 * t + k] = row(lane, t) == col(lane, w) + k ? 1.0 : 0.0;
  }
  __device__ __forceinline__ void restore_padding(int lane, int w, int d) {
    lane = Tile<64>::opaque(lane);
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int r = row(lane, t), c = col(lane, w) + k;
        if (r >= d || c >= d) h[16 * t + k] = r == c ? 1.0 : 0.0;
      }
  }
  // The rows' sums over the wavefront's two blocks, piece w of the product with
  // the padded vector v.
  __device__ __forceinline__ void matvec(const double *v, int lane, int w, double (*part)[kTDim]) const {
    const double vc = v[vpos<kTDim>(col(lane, w)) + (lane & 15)];
    double *out = part[w];
    double p[R];
#pragma unroll
    for (int t = 0; t < R; ++t) p[t] = 0.0;
    static_for<0, 16>([&](auto kk) {
      constexpr int k = decltype(kk)::value;
      fmac_bcast<k>(p[0], p[1], p[2], vc, h[k], h[16 + k], h[32 + k]);
    });
    // one swap leaves row t's sum in the first block's lanes, row t + 1's in
    // the second's
    const int r = row(lane, 0), up = lane & 16;
    out[r + up] = half_pair_sum<16>(p[0], p[1]);
    out[r + 32] = half_pair_sum<16>(p[2], p[2]);  // the same value in both
  }
  // H <- H - rho (s u' + u s') + beta s s', as Tile::rank2_bcast; false when a
  // coefficient is not finite.
  __device__ __forceinline__ bool rank2(double rho, double beta, const double *us, const double *ss,
                                        int lane, int w) {
    double a[R], e[R];
    bool fin = true;
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const int r = vpos<kTDim>(row(lane, t));
      const double sr = ss[r], ur = us[r];
      a[t] = -rho * sr;
      e[t] = beta * sr - rho * ur;
      fin = fin && __builtin_isfinite(a[t]) && __builtin_isfinite(e[t]);
    }
    const int c = vpos<kTDim>(col(lane, w)) + (lane & 15);
    const double uc = us[c], sc = ss[c];
    static_for<0, 16>([&](auto kk) {
      constexpr int k = decltype(kk)::value;
      upd_bcast<k>(h[k], h[16 + k], h[32 + k], uc, sc, a, e);
    });
    return fin;
  }
};

// The 64 x 64 quarters of four wavefronts: rows 64 (w & 1) .., columns
// 64 (w >> 1) ...
struct QuarterTile {
  Tile<64> t;
  __device__ __forceinline__ void identity(int lane, int w) {
    t.identity_at(lane, 64 * (w & 1), 64 * (w >> 1));
  }
  __device__ __forceinline__ void restore_padding(int lane, int w, int d) {
    t.restore_padding_at(lane, d, 64 * (w & 1), 64 * (w >> 1));
  }
  __device__ __forceinline__ void matvec(const double *v, int lane, int w, double (*part)[kTDim]) const {
    part[w >> 1][64 * (w & 1) + lane] = t.matvec_bcast(v[vpos<kTDim>(64 * (w >> 1) + lane)]);
  }
  __device__ __forceinline__ bool rank2(double rho, double beta, const double *us, const double *ss,
                                        int lane, int w) {
    const int r0 = vpos<kTDim>(64 * (w & 1)), c = vpos<kTDim>(64 * (w >> 1) + lane);
    return t.rank2_bcast(rho, beta, us + r0, ss + r0, us[c], ss[c], lane, 0.0, 0.0);
  }
};
template <int NB>
struct TileOf {
  using type = QuarterTile;
};
template <>
struct TileOf<6> {
  using type = ColumnTile;
};

// Row products of H with the padded vector v: rows 2 lane and 2 lane + 1 in r.
// Every wavefront forms its columns' part; after the barrier each adds the
// pieces of every row for itself.  The two products of an iteration use a
// buffer each, so a buffer is written again only after the barrier of the
// other.
template <int NB>
__device__ __forceinline__ void tile_block_matvec(const typename TileOf<NB>::type &H, const double *v,
                                                  TileShm<NB> &sh, int buf, int lane, int w,
                                                  double (&r)[2]) {
  H.matvec(v, lane, w, sh.part[buf]);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int i = 2 * lane + c;
    r[c] = sh.part[buf][0][i] + sh.part[buf][1][i];
    if constexpr (NB == 6) r[c] = r[c] + sh.part[buf][2][i];
  }
}

// Waves per SIMD the register allocation must allow.
template <int NB>
constexpr int kTileWavesPerSimd = NB == 6 ? 3 : 2;

// See the narrow kernel for the mixed-precision rules (T = float).
template <int OBJ, class T, int NB>
__global__ __launch_bounds__(64 * kTWaves<NB>) __attribute__((amdgpu_waves_per_eu(kTileWavesPerSimd<NB>)))
void bfgs_tile_kernel(const ReqDev *reqs, int nreq, BatchDev *hdr, int64_t total) {
  constexpr bool kMixed = sizeof(T) != sizeof(double);
  constexpr bool kWhole = whole_form<Elem<OBJ>>::value;
  __shared__ TileShm<NB> sh;
  const GroupLanes<64> L;
  const int j = threadIdx.x;
  const int lane = j & 63, w = __builtin_amdgcn_readfirstlane(j >> 6);
  const int j0 = 2 * lane;                                      // the lane's coordinates j0, j0 + 1
  typename TileOf<NB>::type H;
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
      fill_step_lengths(sh.al, rq.shrink, j, 64 * kTWaves<NB>);
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
      static_assert(!kWhole || 64 * kTWaves<NB> >= kTDim, "a lane per coordinate");
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
        tile_block_matvec<NB>(H, sh.vs, sh, 0, lane, w, uj);
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
        if (!H.rank2(rho, beta, sh.us, sh.ss, lane, w)) H.restore_padding(lane, w, d);
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
    if (k == 0) H.identity(lane, w);
    wave_sync();  // the product of y has read vs
#pragma unroll
    for (int c = 0; c < 2; ++c) sh.vs[vpos<kTDim>(j0) + c] = gj[c];
    wave_sync();
    double pj[2];
    tile_block_matvec<NB>(H, sh.vs, sh, 1, lane, w, pj);
#pragma unroll
    for (int c = 0; c < 2; ++c) pj[c] = j0 + c < d ? -pj[c] : 0.0;
    double ddir = slot_dot<64, 2>(gj, pj);
    if (!(ddir < 0.0)) {
      if (j == 0) ++sh.cnt.resets;
      H.identity(lane, w);
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
