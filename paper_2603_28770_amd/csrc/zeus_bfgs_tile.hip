// zeus_bfgs_tile.hip -- launches of the on-chip block kernels for 64 < d <= 128:
// three wavefronts per start up to 96, four above
// (the kernel template is in zeus_bfgs_tile_kernels.h).
#include "zeus_bfgs_tile_kernels.h"

namespace zeus {
namespace {

// The kernel is persistent: as many blocks as can be resident at once.
template <int OBJ, class T, int NB>
hipError_t launch_tile_nb(const Group &g, int cus) {
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &per_cu, reinterpret_cast<const void *>(&bfgs_tile_kernel<OBJ, T, NB>), 64 * kTWaves<NB>, 0);
  if (e != hipSuccess) return e;
  if (per_cu < 1) per_cu = 1;
  const int64_t cap = (int64_t)cus * per_cu;
  if (g.resident) {
    *g.resident = cap;
    return hipSuccess;
  }
  const int blocks = (int)(g.total_starts < cap ? g.total_starts : cap);
  hipLaunchKernelGGL((bfgs_tile_kernel<OBJ, T, NB>), dim3(blocks), dim3(64 * kTWaves<NB>), 0, g.stream,
                     g.reqs, g.nreq, g.hdr, g.total_starts);
  return hipGetLastError();
}

template <int OBJ, class T>
hipError_t launch_tile_t(const Group &g, int cus) {
  if (g.g_bfgs == kTile3Dim && (g.resident || tile_three(OBJ, g.precision, g.total_starts, cus)))
    return launch_tile_nb<OBJ, T, 6>(g, cus);
  return launch_tile_nb<OBJ, T, 8>(g, cus);
}

template <class T>
hipError_t launch_tile_prec(const Group &g, int cus) {
  switch (g.objective) {
    case kRosenbrock: return launch_tile_t<kRosenbrock, T>(g, cus);
    case kRastrigin: return launch_tile_t<kRastrigin, T>(g, cus);
    case kAckley: return launch_tile_t<kAckley, T>(g, cus);
    case kStyblinskiTang: return launch_tile_t<kStyblinskiTang, T>(g, cus);
    case kSphere: return launch_tile_t<kSphere, T>(g, cus);
    case kQuartic: return launch_tile_t<kQuartic, T>(g, cus);
    default: return hipErrorInvalidValue;  // Goldstein-Price has d == 2
  }
}

}  // namespace

// Whether a launch of problems that fit the three-wavefront block takes it.  With
// the polynomial terms always (Rosenbrock d = 81: 256 starts 2.08 ms against 2.15
// with four wavefronts, 8,192 starts 18.5 / 30.5).  With the transcendental terms
// it spills 57 to 74 registers, and a search has three trials a round instead
// of four: an iteration takes a fifth longer and a search that fails seven rounds
// instead of five.  Its four blocks on a CU against two make up for it from about
// eight starts per CU on, in mixed precision sixteen; the lines lie where no start
// stalls (a launch that ends with one stalled start is slower up to many more:
// Rastrigin d = 72, 4,094 starts 7.7 / 6.0).  Three against four wavefronts, d = 66 ..
// 96, ms: Ackley, 256 starts 0.26 / 0.20, 1,024 starts 0.37 / 0.36, 2,048 starts 0.55 /
// 0.56, 4,096 starts 0.89 / 0.96; Rastrigin 4,096 starts 1.84 / 1.99; in mixed
// precision Rastrigin 512 starts 0.71 / 0.51, 4,096 starts 2.07 / 1.94, 8,192 starts
// 2.82 / 2.90, Ackley 4,096 starts 1.02 / 0.98, 8,192 starts 1.69 / 1.73.
bool tile_three(int objective, int precision, int64_t starts, int cus) {
  if (objective != kRastrigin && objective != kAckley) return true;
  return starts > (precision == ZEUS_MIXED ? 16 : 8) * (int64_t)cus;
}

hipError_t launch_bfgs_tile(const Group &g, int cus) {
  if (g.precision == ZEUS_MIXED) return launch_tile_prec<float>(g, cus);
  return launch_tile_prec<double>(g, cus);
}

}  // namespace zeus
