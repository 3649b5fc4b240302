// Four level steps in one launch (gfx950), for the captured step loop of small
// homogeneous levels whose patches have extrapolation boundaries.
//
// On a small level a step is bound by its launch (4 us for 128 x 128, where the
// arithmetic of all its cells takes a few hundred nanoseconds) and by the
// march of one wavefront.  Here a workgroup keeps a region of 32 x 32 cells,
// one per thread, in registers and takes four steps on it, of which the middle
// 16 x 16 cells are valid at the end (a step reaches two cells to each side):
// four times the arithmetic, but a quarter of the launches, and no march.
// x-neighbours come through lane shifts (a wavefront holds two rows), what a
// cell needs of the rows around it through LDS: the state, to form the cell's
// bottom edge, and then the edges and x-fluctuations, with a barrier for each.
// 128 x 128 FP64 in a loop of 100 steps: 2.0 us per step, 3.5 with two steps
// per launch (which is the faster one again past one region per CU).
//
// Every quantity has the expression the one-step sweeps give it
// (march_up, cell_update), so a cell's result is bitwise that of four steps.

#include <hip/hip_runtime.h>

#include "ws_device.h"
#include "ws_internal.h"
#include "../../include/wavestep.h"

namespace ws {
namespace {

constexpr int kSide = kBlockCells + 4 * kBlockSteps;  // cells per side of a region
static_assert(kSide == 32, "a wavefront holds two rows of a region");
constexpr int kPitch = kSide + 1;
constexpr int kBlockThreads = kSide * kSide;

template <typename T>
struct Shared {
  T p[kSide][kPitch], u[kSide][kPitch], v[kSide][kPitch];
  T b1[kSide][kPitch], b2[kSide][kPitch], xs[kSide][kPitch];
  Coef<T> k[kBlockSteps];
};

__device__ inline double block_next_dt(double dt, double c, const InstMin &m, double cfl_desired,
                                       double &cfl) {
  cfl = fmax(c * (dt / m.dx), c * (dt / m.dy));
  return cfl_desired > 0.0 && cfl > 0.0 ? dt * cfl_desired / cfl : dt;
}

template <typename T, int LIM>
__global__ __launch_bounds__(kBlockThreads) void step_kernel_block(StepArgs a) {
  if ((int)blockIdx.x == a.n_tiles) {
    // file the four steps' Courant numbers; the level maximum is left to the
    // one-step launch that ends every loop
    const CflSlots &c = a.slots;
    for (int n = (int)threadIdx.x; n < c.n_inst; n += kBlockThreads) {
      const InstMin m = c.inst_min[n];
      double dt = a.dt[n], cfl = 0.0, top = c.cfl_max[n];
      for (int s = 0; s < kBlockSteps; ++s) {
        dt = block_next_dt(dt, a.inst[n].c, m, a.cfl_desired, cfl);
        top = fmax(top, cfl);
      }
      c.dt[n] = dt;
      c.cfl_last[n] = cfl;
      c.cfl_max[n] = top;
    }
    return;
  }
  __shared__ Shared<T> S;
  const int tid = (int)threadIdx.x, x = tid % kSide, y = tid / kSide;
  // (a level of one patch needs no list)
  const TileEntry listed = a.tiles ? uniform_row(a.tiles[blockIdx.x]) : TileEntry{0, 0, 0};
  const PatchRow pr = uniform_row(a.patches[listed.patch]);
  const int ntx = (pr.mx + kBlockCells - 1) / kBlockCells;
  const int tile = (int)blockIdx.x;
  const TileEntry te = a.tiles ? listed
                               : TileEntry{0, (uint16_t)(tile % ntx), (uint16_t)(tile / ntx)};
  const int mx = pr.mx, my = pr.my;
  const int i0 = te.tx * kBlockCells - 2 * kBlockSteps, j0 = te.ty * kBlockCells - 2 * kBlockSteps;
  const int i = i0 + x, j = j0 + y;
  // the interior cell this one is (itself, or the one its ghost copies), in
  // the region's numbering, and the one below it; the first step reads the
  // ghosts as the state holds them
  const int ci = min(max(i, 0), mx - 1), cj = min(max(j, 0), my - 1);
  const int cx = ci - i0, cy = min(max(cj - j0, 0), kSide - 1);
  const int by = min(max(min(max(j - 1, 0), my - 1) - j0, 0), kSide - 1);
  const int cxr = min(max(cx, 0), kSide - 1);
  const bool ghost = i != ci || j != cj;
  const bool ghosts = i0 < 0 || j0 < 0 || i0 + kSide > mx || j0 + kSide > my;  // of the workgroup
  const int64_t org = pr.q_off + 2 * (int64_t)pr.ld + pr.col0;
  const T *q = reinterpret_cast<const T *>(a.qin) + org +
               (int64_t)min(max(j, -2), my + 1) * pr.ld + min(max(i, -2), mx + 1);
  T p = q[0], u = q[pr.plane], v = q[2 * pr.plane];
  if (tid < kBlockSteps) {
    // lane s: the coefficients of step s
    const InstRow in = a.inst[pr.inst];
    const InstMin m = a.slots.inst_min[pr.inst];
    double dt = a.dt[pr.inst], cfl;
    for (int s = 0; s < tid; ++s) dt = block_next_dt(dt, in.c, m, a.cfl_desired, cfl);
    S.k[tid] = lane_coef<T, LIM>(in.c, in.Z, dt, pr.dx, pr.dy);
  }
  const int y1 = min(y + 1, kSide - 1), y2 = min(y + 2, kSide - 1), ym = max(y - 1, 0);
  for (int s = 0; s < kBlockSteps; ++s) {
    S.p[y][x] = p, S.u[y][x] = u, S.v[y][x] = v;
    __syncthreads();
    const Coef<T> k = uniform_row(S.k[s]);
    const T Z = k.Z;
    if (ghosts && ghost && s > 0) p = S.p[cy][cxr], u = S.u[cy][cxr], v = S.v[cy][cxr];
    const int yb = s > 0 ? by : ym, xb = s > 0 ? cxr : x;
    const T pb = S.p[yb][xb], vb = S.v[yb][xb];
    // left x-edge and bottom y-edge of the cell
    const T dp = p - shr(p), du = u - shr(u);
    const T a1L = s1(Z, dp, du), a2L = s2(Z, dp, du);
    const T a1R = shl(a1L);
    const T xs0 = a2L + a1R;
    const T b1B = s1(Z, p - pb, v - vb), b2B = s2(Z, p - pb, v - vb);
    S.b1[y][x] = b1B, S.b2[y][x] = b2B, S.xs[y][x] = xs0;
    __syncthreads();
    const T b1T = S.b1[y1][x], b2T = S.b2[y1][x], b1TT = S.b1[y2][x], b2BB = S.b2[ym][x];
    const T xsm = S.xs[ym][x], xsp = S.xs[y1][x];
    const T ys0 = b2B + b1T;
    T FL1, FL2, GB1, GB2, GT1, GT2;
    ftilde<T, LIM>(k, a1L, a2L, a1R, shr(a2L), shr(ys0), ys0, FL1, FL2);
    const T FR1 = shl(FL1), FR2 = shl(FL2);
    gtilde<T, LIM>(k, b1B, b2B, b1T, b2BB, xsm, xs0, GB1, GB2);
    gtilde<T, LIM>(k, b1T, b2T, b1TT, b2B, xs0, xsp, GT1, GT2);
    update<T>(k, p, u, v, a2L, a1R, b2B, b1T, FL1, FL2, FR1, FR2, GB1, GB2, GT1, GT2, p, u, v);
  }
  if (ghosts) {  // (the same for the whole workgroup)
    S.p[y][x] = p, S.u[y][x] = u, S.v[y][x] = v;
    __syncthreads();
    if (ghost) p = S.p[cy][cxr], u = S.u[cy][cxr], v = S.v[cy][cxr];
  }
  // the tile's cells, and the ghosts that copy one of them
  const bool mine = ci >= te.tx * kBlockCells && ci < (te.tx + 1) * kBlockCells &&
                    cj >= te.ty * kBlockCells && cj < (te.ty + 1) * kBlockCells;
  if (mine && i >= -2 && i <= mx + 1 && j >= -2 && j <= my + 1) {
    T *o = reinterpret_cast<T *>(a.qout) + org + (int64_t)j * pr.ld + i;
    o[0] = p, o[pr.plane] = u, o[2 * pr.plane] = v;
  }
}

template <typename T>
hipError_t block_t(int limiter, const StepArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)a.n_tiles + 1), block(kBlockThreads);
  switch (limiter) {
    case WS_LIM_NONE:
      hipLaunchKernelGGL((step_kernel_block<T, WS_LIM_NONE>), grid, block, 0, s, a);
      break;
    case WS_LIM_VANLEER:
      hipLaunchKernelGGL((step_kernel_block<T, WS_LIM_VANLEER>), grid, block, 0, s, a);
      break;
    default:
      hipLaunchKernelGGL((step_kernel_block<T, WS_LIM_MC>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_step_block(int dtype, int limiter, const StepArgs &a, hipStream_t s) {
  if (a.n_tiles <= 0) return hipErrorInvalidValue;
  return dtype == WS_F32 ? block_t<float>(limiter, a, s) : block_t<double>(limiter, a, s);
}

}  // namespace ws
