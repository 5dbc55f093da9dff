// zeus_bfgs_hybrid_kernels.h -- the BFGS phase for 128 < d <= 208 with the
// inverse Hessian on chip, in registers and LDS (Alg. 4 / Alg. 10 with the
// dual-number gradient of Alg. 5 and the Armijo search of Alg. 6): one block
// of eight wavefronts per start.  Built into the library
// (zeus_bfgs_hybrid.hip) and into the run-time program of a user objective.
//
//  * H is 208 x 208 (zero-padded past the dimension, ones on the padded
//    diagonal).  Rows and columns 0 .. 191 form a 3 x 3 grid of 64 x 64
//    tiles; eight of them sit in the registers of the eight wavefronts, in
//    the 4 x 16 lane tiles of the narrow kernel's 64-lane groups (zeus_group.h
//    Tile).  The rest is held in LDS in units of 64 chains of 16 consecutive
//    columns, a chain per lane: the ninth tile (rows and columns 128 .. 191)
//    as four units of 16 rows, the row strip (rows 192 .. 207, columns
//    0 .. 191) as three units of 64 columns, and the column strip (columns
//    192 .. 207, all rows) as four units of 64 rows.  A wavefront holds one
//    unit, the first three a second one;
//  * a row's product with a vector is a fused multiply-add chain over each
//    block of 16 consecutive columns, the block sums added pairwise over the
//    13 blocks (the order of every other kernel): four blocks meet inside a
//    wavefront in two lane-swap levels, whether of a register tile or of a
//    unit, and lane i < 208 adds row i's four pieces;
//  * a chain takes the vectors' entries of its columns by row broadcasts from
//    the lanes' own entries, as the register tiles do, and its elements two at
//    a time; the update and the product with the new gradient are one pass.
//    (Every operand read from LDS, and the update and the product two passes,
//    a chain took 128 LDS instructions per iteration instead of 28, and the LDS
//    was what the iteration waited for: Rosenbrock, 2,048 starts, d = 200
//    64.0 -> 47.1 ms, d = 160 45.1 -> 36.1 ms; Ackley d = 200, 4,096 starts 5.0 -> 4.3 ms.)
//  * units that lie wholly in the padding are skipped;
//  * lanes 0 .. 207 own the coordinates (x, g, p, s, y); the vectors the
//    tiles and chains read go through LDS in the padded layout, written
//    before a reduction whose barrier publishes them;
//  * gradient, sums, line search (eight trials per round, one per wavefront),
//    termination and retirement are those of the other block kernels
//    (zeus_block.h), over 256 term slots;
//  * starts are claimed as by the other kernels: first the block's own index,
//    then an agent-scope work counter.
// The control flow is uniform across the block (one start per block), so
// every barrier is reached by all its threads.  One block fills a CU's LDS.
#pragma once

#include "zeus_block.h"

namespace zeus {
namespace {

constexpr int kHD = kHybridDim;            // rows and columns of the padded H
constexpr int kHW = 8;                     // wavefronts per start
constexpr int kHLanes = 64 * kHW;          // lanes per start
constexpr int kHB = kHD / 16;              // column blocks
constexpr int kHReg = 192;                 // rows and columns of the 3 x 3 tile grid
constexpr int kUnits = 11;                 // units in LDS
constexpr int kUnitRows = 4, kUnitCols = 7;  // first unit of the row strip, of the column strip
constexpr int kHVec = tile_vec_len(256);   // doubles of a padded operand vector (vpos<256>)
constexpr int kHSlots = 256;               // term slots of a line-search trial
static_assert(kHD == kHReg + 16 && kHB == 13, "one 16-wide strip past the tile grid");

struct alignas(16) ChainPair {
  double a, b;  // two consecutive columns of a chain
};

struct HybridShm {
  double xs[kHSlots];            // iterate under evaluation (x, then x_new), zero past d
  double ps[kHSlots];            // search direction
  double vs[kHVec];              // y, operand of u = H y, padded layout
  double gs[kHVec];              // g, operand of p = -H g, padded layout
  double ss[kHVec];              // s = x_new - x, padded layout
  double us[kHVec];              // u = H y, padded layout
  double part[4][kHSlots];       // [64-column piece][row] products (piece 3: the column strip)
  double red[2][3][kHW];         // [phase][sum][wave] partial sums
  double tsum[2 * kHW][kMaxSums];     // [phase * waves + wave][sum] line-search trials' term sums
  double al[kTabTrials];
  int pass[2][kHW];              // [phase][wave] line-search outcome
  StartCounts cnt;               // update skips and direction resets (thread 0)
  unsigned long long got;
  int bound;                     // early-stop bound of this iteration
  ReqHot q;
  // last: the fields above stay within reach of the 16-bit offsets of LDS
  // instructions from one base, which keeps their addresses out of registers
  ChainPair hl[kUnits][8][64];   // the LDS part of H: [unit][column pair][lane]
};

// The chains of one unit: this lane's row and the columns of its chain.
struct Unit {
  ChainPair *h;  // column pair k at h[64 k]
  int row, c0;   // the chain's row and first column
  int piece;     // the 64-column piece of the row it belongs to
  bool across;   // the four 16-lane rows hold four blocks of the same rows
  bool live;     // some chain of the unit lies below the dimension
};

__device__ __forceinline__ Unit unit_of(HybridShm &sh, int u, int lane, int d) {
  const int i = lane & 15, b = lane >> 4;
  Unit t;
  t.h = &sh.hl[u < kUnits ? u : 0][0][lane];
  t.across = u < kUnitCols;
  if (u < kUnitRows) {
    t.row = 128 + 16 * u + i;
    t.c0 = 128 + 16 * b;
    t.piece = 2;
    t.live = 128 + 16 * u < d;
  } else if (u < kUnitCols) {
    t.row = kHReg + i;
    t.c0 = 64 * (u - kUnitRows) + 16 * b;
    t.piece = u - kUnitRows;
    t.live = kHReg < d;
  } else {  // the last one holds 16 rows (the same in its four 16-lane rows)
    t.row = u + 1 < kUnits ? 64 * (u - kUnitCols) + lane : kHReg + i;
    t.c0 = kHReg;
    t.piece = 3;
    t.live = kHReg < d && u < kUnits;
  }
  return t;
}

// Place in a padded vector of the entry a lane holds for its chain's row
// broadcasts: the chain's column at the lane's position in its row of 16.
__device__ __forceinline__ int unit_entry(const Unit &t, int lane) {
  return vpos<256>(t.c0) + (lane & 15);
}

// The wavefront's units: unit w, and unit w + 8 of the first three.  The
// wavefronts with two are the block's first ones: issue favours a SIMD's
// older wavefronts, so there the longer path between two barriers is served
// first.
template <class F>
__device__ __forceinline__ void for_wave_units(HybridShm &sh, int w, int lane, int d, F &&f) {
#pragma unroll 1
  for (int u = w; u < kUnits; u += kHW) {
    const Unit t = unit_of(sh, u, lane, d);
    if (t.live) f(t);
  }
}

__device__ __forceinline__ void units_identity(HybridShm &sh, int w, int lane, int d) {
  for_wave_units(sh, w, lane, d, [&](const Unit &t) {
    const int diag = Tile<64>::opaque(t.row - t.c0);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      t.h[64 * k] = ChainPair{diag == 2 * k ? 1.0 : 0.0, diag == 2 * k + 1 ? 1.0 : 0.0};
  });
}

// The unit's piece of its rows' products, from the lanes' chains.
__device__ __forceinline__ void unit_piece(HybridShm &sh, const Unit &t, double acc) {
  if (t.across) {
    acc = half_pair_sum<16>(acc, acc);
    acc = half_pair_sum<32>(acc, acc);
  }
  sh.part[t.piece][t.row] = acc;
}

// H v over the units, v the padded vector vec.
__device__ __forceinline__ void units_matvec(HybridShm &sh, const double *vec, int w, int lane, int d) {
  for_wave_units(sh, w, lane, d, [&](const Unit &t) {
    const double v = vec[unit_entry(t, lane)];
    double acc = 0.0;
    static_for<0, 2>([&](auto hh) {
      constexpr int k0 = 4 * decltype(hh)::value;
      // four pairs at a time: a memory clobber keeps the next loads from
      // being hoisted, which bounds the live registers
      asm volatile("" ::: "memory");
      ChainPair h[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) h[k] = t.h[64 * (k0 + k)];
      static_for<0, 4>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        fmac_bcast<2 * (k0 + k)>(acc, v, h[k].a);
        fmac_bcast<2 * (k0 + k) + 1>(acc, v, h[k].b);
      });
    });
    unit_piece(sh, t, acc);
  });
}

// The rank-2 update of the units (the register tiles update themselves) and
// their product with g in one pass: element (r, c) by
// fma(e_r, s_c, fma(a_r, u_c, H_rc)), a_r = -rho s_r, e_r = beta s_r - rho u_r; a
// chain whose coefficients are not finite gets its padding back.
__device__ __forceinline__ void units_update_matvec(HybridShm &sh, int w, int lane, int d, double rho,
                                                    double beta) {
  for_wave_units(sh, w, lane, d, [&](const Unit &t) {
    const double sr = sh.ss[vpos<256>(t.row)], ur = sh.us[vpos<256>(t.row)];
    const double a = -rho * sr;
    const double e = beta * sr - rho * ur;
    const bool fin = __builtin_isfinite(a) && __builtin_isfinite(e);
    const int o = unit_entry(t, lane);
    const double u = sh.us[o], s = sh.ss[o], g = sh.gs[o];
    double acc = 0.0;
    static_for<0, 2>([&](auto hh) {
      constexpr int k0 = 4 * decltype(hh)::value;
      asm volatile("" ::: "memory");
      ChainPair h[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) h[k] = t.h[64 * (k0 + k)];
      static_for<0, 4>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        upd_bcast<2 * (k0 + k)>(h[k].a, u, s, a, e);
        upd_bcast<2 * (k0 + k) + 1>(h[k].b, u, s, a, e);
      });
      if (!fin) {
        const int c = Tile<64>::opaque(t.c0) + 2 * k0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (c + 2 * k >= d) h[k].a = t.row == c + 2 * k ? 1.0 : 0.0;
          if (c + 2 * k + 1 >= d) h[k].b = t.row == c + 2 * k + 1 ? 1.0 : 0.0;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) t.h[64 * (k0 + k)] = h[k];
      static_for<0, 4>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        fmac_bcast<2 * (k0 + k)>(acc, g, h[k].a);
        fmac_bcast<2 * (k0 + k) + 1>(acc, g, h[k].b);
      });
    });
    unit_piece(sh, t, acc);
  });
}

// Row t of the product whose pieces the wavefronts have written (lane t < kHD,
// after the barrier): the pairwise tree over the 13 blocks,
// ((b0..b3 + b4..b7) + (b8..b11 + b12)).  Pieces that hold no live column are
// not written: rows take the first 64-column pieces that do.
__device__ __forceinline__ double hybrid_row(const HybridShm &sh, int t, int d) {
  if (t >= kHD) return 0.0;
  const double lo = sh.part[0][t] + sh.part[1][t];
  const double hi = kHReg < d ? sh.part[2][t] + sh.part[3][t] : sh.part[2][t];
  return lo + hi;
}

// See the narrow kernel for the mixed-precision rules (T = float).
template <int OBJ, class T>
__global__ __launch_bounds__(kHLanes) __attribute__((amdgpu_waves_per_eu(2)))
void bfgs_hybrid_kernel(const ReqDev *reqs, int nreq, BatchDev *hdr, int64_t total) {
  constexpr bool kMixed = sizeof(T) != sizeof(double);
  __shared__ HybridShm sh;
  const int j = threadIdx.x;  // coordinate of lanes below kHD
  const int lane = j & 63, w = __builtin_amdgcn_readfirstlane(j >> 6);
  const int r0 = 64 * (w / 3), c0 = 64 * (w % 3);  // this wavefront's register tile
  const bool coord = j < kHD;
  Tile<64> H;
  int phase = 0, lsphase = 0;
  int acc = -1;  // slot of sh.tsum with the accepted trial's term sums (block_armijo), or -1
  bool own = false, first = true, fresh = false, hi = !kMixed;
  double xj = 0.0, gj = 0.0, pj = 0.0, sj = 0.0, f = 0.0;
  int64_t idx = -1;
  int k = 0, ls_trials = 0;
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
      }
      fill_step_lengths(sh.al, rq.shrink, j, kHLanes);
      own = j < d0;
      xj = own ? rq.ws.x[idx * d0 + j] : 0.0;  // x <- swarm[i]
      if (coord) sh.xs[j] = xj;
      units_identity(sh, w, lane, d0);  // H <- I (the register tiles before the first product)
      k = 0;
      ls_trials = 0;
      fresh = true;
      hi = !kMixed;
    }
    // the stopping bound, read early (its use is at the termination test) by
    // one thread for the block: the bound falls while the kernel runs
    if (j == 0) sh.bound = es_bound(sh.q);
    __syncthreads();  // xs, the request and the bound are visible; earlier reads are done
    const ReqHot &q = sh.q;
    const int d = q.d;
    const int bound = sh.bound;

    // -- value and gradient at xs -------------------------------------------
    double gn, fn;
    if (hi)
      fn = block_eval<OBJ, double, true>(d, sh.xs, &gn, sh, phase, acc);
    else
      fn = block_eval<OBJ, T, true>(d, sh.xs, &gn, sh, phase, acc);
    acc = -1;

    // y's, g'g and the non-finite test in one reduction, whose barrier also
    // publishes y and g for the products below; right after a claim or an
    // escalation y's is not used
    const double yj = gn - gj;  // zero beyond the dimension and on lanes >= kHD
    if (coord) {
      sh.vs[vpos<256>(j)] = yj;
      sh.gs[vpos<256>(j)] = gn;
    }
    const bool bad = (own && !__builtin_isfinite(gn)) || !__builtin_isfinite(fn);
    double sums[3] = {yj * sj, gn * gn, bad ? 1.0 : 0.0};
    block_tree_sums<3, double>(sums, sh, phase);
    const double sy = sums[0], gg = sums[1];
    const bool any_bad = sums[2] != 0.0;

    // -- after a step: u = H y and the rank-2 update --------------------------
    bool updated = false;
    if (!fresh) {
      if (sy > 0.0) {  // curvature condition; skip the update otherwise
        const double rho = 1.0 / sy;
        units_matvec(sh, sh.vs, w, lane, d);
        sh.part[w % 3][r0 + lane] = H.matvec_bcast(sh.vs[vpos<256>(c0 + lane)]);
        __syncthreads();
        double uj = hybrid_row(sh, j, d);
        uj = own ? uj : 0.0;
        if (coord) {  // published by the barrier of the next reduction
          sh.us[vpos<256>(j)] = uj;
          sh.ss[vpos<256>(j)] = sj;
        }
        const double yu = block_tree_sum(yj * uj, sh, phase);
        const double beta = (rho * rho) * yu + rho;
        // H+ = H - rho (s u' + u s') + beta s s'   (u = H y); inf * 0 would
        // have reached the padding when a coefficient is not finite
        if (!H.rank2_bcast(rho, beta, sh.us + vpos<256>(r0), sh.ss + vpos<256>(r0),
                           sh.us[vpos<256>(c0 + lane)], sh.ss[vpos<256>(c0 + lane)], lane, 0.0, 0.0))
          H.restore_padding_at(lane, d, r0, c0);
        units_update_matvec(sh, w, lane, d, rho, beta);  // and their pieces of H_new g
        updated = true;
      } else if (j == 0) {
        ++sh.cnt.skips;
      }
      ++k;
    }
    gj = gn;
    f = fn;
    fresh = false;
    if (q.trace_len && own && k < q.trace_len) reqs[q.ri].trace[(idx * q.trace_len + k) * d + j] = xj;

    // -- termination: non-finite, ||g|| < Theta, budget ---------------------
    if (kMixed && !hi && (any_bad || norm_below(gg, 10.0 * q.tol))) {
      hi = true;  // escalate: re-evaluate this point in FP64
      fresh = true;
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
      if (own) rq.out_x[idx * d + j] = xj;
      if (kMixed && !hi) f = block_eval<OBJ, double, false>(d, sh.xs, nullptr, sh, phase);
      if (j == 0) {
        rq.out_f[idx] = f;
        rq.out_iters[idx] = k;
        rq.out_status[idx] = status;
        if (rq.out_ls) rq.out_ls[idx] = ls_trials;
        if (rq.out_skips) rq.out_skips[idx] = sh.cnt.skips;
        if (rq.out_resets) rq.out_resets[idx] = sh.cnt.resets;
      }
      if (tl && own)
        for (int kk = k + 1; kk < tl; ++kk) rq.trace[(idx * tl + kk) * d + j] = __builtin_nan("");
      idx = -1;
      continue;
    }

    // -- search direction p = -H g (reset to -g if not a descent direction) -
    // The register tiles are the identity until the first update (k = 0);
    // setting them here rather than at the claim keeps the old tile's
    // registers from being live beside the new one's.
    if (k == 0) H.identity_at(lane, r0, c0);
    if (!updated) units_matvec(sh, sh.gs, w, lane, d);
    sh.part[w % 3][r0 + lane] = H.matvec_bcast(sh.gs[vpos<256>(c0 + lane)]);
    __syncthreads();
    const double hg = hybrid_row(sh, j, d);
    pj = own ? -hg : 0.0;
    if (coord) sh.ps[j] = pj;  // published by the barrier of the next reduction
    double ddir = block_tree_sum(gj * pj, sh, phase);
    if (!(ddir < 0.0)) {
      if (j == 0) ++sh.cnt.resets;
      H.identity_at(lane, r0, c0);
      units_identity(sh, w, lane, d);
      pj = own ? -gj : 0.0;
      if (coord) sh.ps[j] = pj;
      ddir = block_tree_sum(gj * pj, sh, phase);
    }

    // -- Armijo backtracking (Alg. 6) ---------------------------------------
    int taken;
    if (hi) {
      taken = block_armijo<OBJ, double, kHSlots>(sh, sh.xs, sh.ps, f, ddir, lsphase, &acc);
    } else {
      taken = block_armijo<OBJ, T, kHSlots>(sh, sh.xs, sh.ps, f, ddir, lsphase, &acc);
      if (taken < 0) {
        ls_trials += q.iter_ls;
        hi = true;  // escalate: FP32 cannot resolve this decrease
        fresh = true;
        continue;
      }
    }
    const int nshrink = taken >= 0 ? taken : q.iter_ls;
    ls_trials += taken >= 0 ? taken + 1 : q.iter_ls;
    const double alpha = step_length(sh.al, q.shrink, nshrink);

    // -- step: x_new = x + alpha p, s = x_new - x -----------------------------
    // every lane has read xs and ps before the last barrier of the line search
    const double xnew = xj + alpha * pj;
    sj = own ? xnew - xj : 0.0;
    xj = own ? xnew : 0.0;
    if (coord) sh.xs[j] = xj;
  }
}

}  // namespace
}  // namespace zeus
