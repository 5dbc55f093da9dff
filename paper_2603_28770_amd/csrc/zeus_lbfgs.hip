// zeus_lbfgs.hip -- limited-memory BFGS on gfx950: the launches (the
// kernel template is in zeus_lbfgs_kernels.h).
#include "zeus_lbfgs_kernels.h"

namespace zeus {
namespace {

template <int OBJ, int G, int CPL, class T>
hipError_t launch_l(const Group &g, int cus) {
  const size_t lds = sizeof(double) * (size_t)lbfgs_stride(G * CPL) * (kBfgsBlock / G);
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void *>(&lbfgs_kernel<OBJ, G, CPL, T>), kBfgsBlock, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) per_cu = 1;
  const int64_t per_block = kBfgsBlock / G;
  const int64_t want = (g.total_starts + per_block - 1) / per_block;
  const int64_t cap = (int64_t)cus * per_cu;
  if (g.resident) {
    *g.resident = cap * per_block;
    return hipSuccess;
  }
  const int blocks = (int)(want < cap ? want : cap);
  hipLaunchKernelGGL((lbfgs_kernel<OBJ, G, CPL, T>), dim3(blocks), dim3(kBfgsBlock), lds, g.stream,
                     g.reqs, g.nreq, g.hdr, g.total_starts);
  return hipGetLastError();
}

// A launch with SLOTS coordinate slots per start, which two kernels can run:
//  * dense: four coordinates per lane, so that a wave holds 256 / SLOTS starts and
//    a sum needs one butterfly over SLOTS / 4 lanes; two at 8 slots and for the
//    transcendental objectives, whose four-coordinate kernels pass 256
//    registers and run one wave per SIMD (Ackley d = 50, 16,384 starts: 0.84 ms
//    with four, 0.65 with two);
//  * spread: a coordinate per lane (two at 128 slots), which is done sooner with
//    one start's iteration.
// lbfgs_spread says which.  At 128 slots the transcendental objectives' kernels
// are the same one.
template <int OBJ, int SLOTS, class T>
hipError_t launch_l_slots(const Group &g, int cus) {
  constexpr int kDense = SLOTS == 8 || OBJ == kRastrigin || OBJ == kAckley ? 2 : 4;
  constexpr int kSpreadLanes = SLOTS < 64 ? SLOTS : 64, kSpread = SLOTS / kSpreadLanes;
  if constexpr (kDense != kSpread) {
    int64_t room = 0;  // starts that the spread kernel keeps resident
    Group ask = g;
    ask.resident = &room;
    const hipError_t e = launch_l<OBJ, kSpreadLanes, kSpread, T>(ask, cus);
    if (e != hipSuccess) return e;
    // (a caller that asks for the room gets that of the largest launches' kernel)
    if (lbfgs_spread(OBJ, g.precision, SLOTS, g.resident ? INT64_MAX / 256 : g.total_starts, room, cus))
      return launch_l<OBJ, kSpreadLanes, kSpread, T>(g, cus);
  }
  return launch_l<OBJ, SLOTS / kDense, kDense, T>(g, cus);
}

template <int OBJ, class T>
hipError_t launch_l_obj(const Group &g, int cus) {
  switch (g.g_bfgs) {  // coordinate slots per start
    case 4: return launch_l<OBJ, 4, 1, T>(g, cus);
    case 8: return launch_l_slots<OBJ, 8, T>(g, cus);
    case 16: return launch_l_slots<OBJ, 16, T>(g, cus);
    case 32: return launch_l_slots<OBJ, 32, T>(g, cus);
    case 64: return launch_l_slots<OBJ, 64, T>(g, cus);
    case 128: return launch_l_slots<OBJ, 128, T>(g, cus);
    case 256: return launch_l<OBJ, 64, 4, T>(g, cus);
    default: return hipErrorInvalidValue;
  }
}

template <class T>
hipError_t launch_l_prec(const Group &g, int cus) {
  switch (g.objective) {
    case kRosenbrock: return launch_l_obj<kRosenbrock, T>(g, cus);
    case kRastrigin: return launch_l_obj<kRastrigin, T>(g, cus);
    case kAckley: return launch_l_obj<kAckley, T>(g, cus);
    case kStyblinskiTang: return launch_l_obj<kStyblinskiTang, T>(g, cus);
    case kGoldsteinPrice: return launch_l<kGoldsteinPrice, 4, 1, T>(g, cus);
    case kSphere: return launch_l_obj<kSphere, T>(g, cus);
    case kQuartic: return launch_l_obj<kQuartic, T>(g, cus);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

size_t lbfgs_lds_bytes(int slots) {
  const int lanes = slots < 64 ? slots : 64;
  return sizeof(double) * (size_t)lbfgs_stride(slots) * (kBfgsBlock / lanes);
}

int lbfgs_slots(int dim) {
  int s = 4;
  while (s < dim) s <<= 1;
  return s;
}

// Whether a launch takes the spread kernel:
//  * while every start has lanes of it at once, at most three wavefronts on a SIMD
//    (at 8 slots, where the dense kernel's wave has only twice the starts, for
//    Rosenbrock; for the others up to half a wavefront).  Spread against dense,
//    m = 5: Rosenbrock d = 14, 1,024 starts 0.39 / 0.53 ms, d = 50, 256 starts 0.84 /
//    1.22, 2,048 starts 1.08 / 1.25 and from there on 4,096 starts 1.60 / 1.30, 16,384
//    starts 5.09 / 2.95, d = 7, 16,384 starts 0.48 / 0.53; Styblinski-Tang d = 30,
//    4,096 starts 0.192 / 0.210, 8,192 starts 0.250 / 0.247; Rastrigin d = 6, 4,096
//    starts 0.175 / 0.179, 8,192 starts 0.202 / 0.195;
//  * in mixed precision, where many starts stall after the change to FP64 and one
//    of them sets the end of the launch by itself, always for the objectives
//    that have such starts: Styblinski-Tang d = 30, 16,384 starts 4.9 / 8.6 ms,
//    Rastrigin d = 45, 30,000 starts 5.6 / 7.9, Ackley d = 10, 30,000 starts 7.8 /
//    11.8.  (Ackley from d = 17 on loses more without stalls than it gains with
//    them: d = 30, 30,000 starts 0.71 / 0.60; and so does Styblinski-Tang d = 6 0.42 /
//    0.34.)
bool lbfgs_spread(int objective, int precision, int slots, int64_t starts, int64_t room, int cus) {
  const int64_t lanes = (int64_t)starts * (slots < 64 ? slots : 64);
  const int64_t per_wave = 4 * 64 * (int64_t)cus;  // lanes of one wavefront per SIMD
  if (slots == 8 && objective != kRosenbrock) return 2 * lanes <= per_wave;
  if (starts <= room && lanes <= 3 * per_wave) return true;
  if (precision != ZEUS_MIXED) return false;
  return objective == kRastrigin || objective == kStyblinskiTang ||
         (objective == kAckley && slots == 16);
}

hipError_t launch_lbfgs(const Group &g, int cus) {
  if (g.objective == kUser) return launch_user_lbfgs(g, cus);
  if (g.precision == ZEUS_MIXED) return launch_l_prec<float>(g, cus);
  return launch_l_prec<double>(g, cus);
}

}  // namespace zeus
