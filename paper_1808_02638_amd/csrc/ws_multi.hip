// Two level steps in one launch (gfx950), for the captured step loop of
// homogeneous levels whose patches have extrapolation boundaries.
//
// The step's rate is set by HBM (or the Infinity Cache): every launch reads
// and writes the whole state, while its arithmetic takes well under half of
// that time.  Here a state read once is advanced twice before it is written.
// A wavefront marches up a segment of rows exactly as a MARCH segment does,
// and the rows its first step produces feed a second step that follows two
// rows behind, all in registers: the second step's three-row window takes the
// first step's new rows, and its x-neighbours come through the same lane
// shifts.  A step reaches two columns and two rows to each side, so of the 64
// lanes the middle 56 are updated (60 with one step), and a segment's first
// step covers two rows more at each end than its second.
//
// Every quantity has the expression the one-step sweeps give it
// (march_up, cell_update), so a cell's result is bitwise that of two steps.

#include <hip/hip_runtime.h>

#include "ws_device.h"
#include "ws_internal.h"
#include "../../include/wavestep.h"

namespace ws {
namespace {

// What a step carries up its column between rows.
template <typename T>
struct Carry {
  T yb2, b1h, b2h;       // b2 of the cell's bottom edge; b1, b2 of its top edge
  T GBp, GBv;            // G~ of the bottom edge
  T xs0, a1L, a2L, a1R;  // x-fluctuation sum and x-edge strengths of the row
};

// Carry for row r from rows r-2 (p, v), r-1, r and r+1 (p, v).
template <typename T, int LIM>
__device__ __attribute__((always_inline)) inline Carry<T> carry_in(const Coef<T> &k,
                                                                   const Row3<T> &M2,
                                                                   const Row3<T> &M1,
                                                                   const Row3<T> &A,
                                                                   const Row3<T> &B) {
  const T Z = k.Z;
  Carry<T> S;
  const T b2mm = s2(Z, M1.p - M2.p, M1.v - M2.v);
  const T b1m = s1(Z, A.p - M1.p, A.v - M1.v), b2m = s2(Z, A.p - M1.p, A.v - M1.v);
  S.b1h = s1(Z, B.p - A.p, B.v - A.v);
  S.b2h = s2(Z, B.p - A.p, B.v - A.v);
  S.yb2 = b2m;
  const T plm = shr(M1.p), ulm = shr(M1.u);
  const T xsm = s2(Z, M1.p - plm, M1.u - ulm) + shl(s1(Z, M1.p - plm, M1.u - ulm));
  const T pl = shr(A.p), ul = shr(A.u);
  S.a1L = s1(Z, A.p - pl, A.u - ul);
  S.a2L = s2(Z, A.p - pl, A.u - ul);
  S.a1R = shl(S.a1L);
  S.xs0 = S.a2L + S.a1R;
  gtilde<T, LIM>(k, b1m, b2m, S.b1h, b2mm, xsm, S.xs0, S.GBp, S.GBv);
  return S;
}

// The update of row r from rows r (A), r+1 (B) and r+2 (C; p, v); slides the
// carry up one row.
template <typename T, int LIM>
__device__ __attribute__((always_inline)) inline Row3<T> row_step(const Coef<T> &k, Carry<T> &S,
                                                                  const Row3<T> &A,
                                                                  const Row3<T> &B,
                                                                  const Row3<T> &C) {
  const T Z = k.Z;
  const T b1hh = s1(Z, C.p - B.p, C.v - B.v), b2hh = s2(Z, C.p - B.p, C.v - B.v);
  const T ys0 = S.yb2 + S.b1h, yd0 = S.yb2 - S.b1h;
  const T pl = shr(B.p), ul = shr(B.u);
  const T a1Ln = s1(Z, B.p - pl, B.u - ul), a2Ln = s2(Z, B.p - pl, B.u - ul);
  const T a1Rn = shl(a1Ln);
  const T xsp = a2Ln + a1Rn;
  const T xd0 = S.a2L - S.a1R;
  T FLp, FLu, GTp, GTv;
  ftilde<T, LIM>(k, S.a1L, S.a2L, S.a1R, shr(S.a2L), shr(ys0), ys0, FLp, FLu);
  const T FRp = shl(FLp), FRu = shl(FLu);
  gtilde<T, LIM>(k, S.b1h, S.b2h, b1hh, S.yb2, S.xs0, xsp, GTp, GTv);
  Row3<T> N;
  update<T>(k, A.p, A.u, A.v, S.xs0, xd0, ys0, yd0, FLp, FLu, FRp, FRu, S.GBp, S.GBv, GTp, GTv,
            N.p, N.u, N.v);
  S.yb2 = S.b2h, S.b1h = b1hh, S.b2h = b2hh;
  S.GBp = GTp, S.GBv = GTv;
  S.xs0 = xsp, S.a1L = a1Ln, S.a2L = a2Ln, S.a1R = a1Rn;
  return N;
}

// Row sets of a segment: a set holds a row from its load until its last use
// as row r, then is refilled with the row kMultiSets further up.
constexpr int kMultiSets = 6;

// Lanes of one segment: lane l holds column i of the patch, lanes kHalo ..
// 63 - kHalo are updated.  Reads take the nearest interior cell (the
// extrapolation ghosts); 32-bit byte offsets as in a MARCH segment.
template <typename T>
struct MultiLanes {
  const char *base;
  __amdgpu_buffer_rsrc_t ob;
  unsigned ld, plb, colb, ocolb;
  int my, rmax;
  bool xbc;   // the wavefront holds ghost columns
  int gx;     // ghost column: 1, 2 -> i = -1, -2; 3, 4 -> i = mx, mx+1; else 0
  bool st;    // the lane stores

  __device__ MultiLanes(const T *qi, T *qo, const PatchRow &pr, int i0, int l, int r1) {
    constexpr int halo = kMultiHalo;
    ld = (unsigned)pr.ld;
    plb = (unsigned)pr.plane * (unsigned)sizeof(T);
    my = pr.my;
    rmax = min(r1 + 3, pr.my - 1);
    base = reinterpret_cast<const char *>(qi - 2 * (int64_t)ld - 2);
    ob = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char *>(qo - 2 * (int64_t)ld - 2), 0,
                                           (int)(3 * plb), kRawBufferWord3);
    const int i = i0 + l, mx = pr.mx;
    colb = (unsigned)(min(max(i, 0), mx - 1) + 2) * (unsigned)sizeof(T);
    ocolb = (unsigned)(i + 2) * (unsigned)sizeof(T);
    xbc = i0 < 0 || i0 + kMarchWidth > mx;
    gx = i == -1 ? 1 : i == -2 ? 2 : i == mx ? 3 : i == mx + 1 ? 4 : 0;
    const bool out = l >= halo && l < kMarchWidth - halo && i < mx;
    // ghost columns are stored next to the updated column they copy
    const int s = gx == 1 ? l + 1 : gx == 2 ? l + 2 : gx == 3 ? l - 1 : l - 2;
    st = out || (gx != 0 && s >= halo && s < kMarchWidth - halo);
  }
  __device__ void fetch(Row3<T> &S, int r) const {
    const unsigned o = (unsigned)(min(max(r, 0), rmax) + 2) * ld * (unsigned)sizeof(T) + colb;
    S.p = *reinterpret_cast<const T *>(base + o);
    S.u = *reinterpret_cast<const T *>(base + o + plb);
    S.v = *reinterpret_cast<const T *>(base + o + 2 * plb);
  }
  // The lanes on ghost columns take the new value of the nearest column.
  __device__ void ghost_columns(Row3<T> &N) const {
    if (!xbc) return;
    const T p1 = shl(N.p), u1 = shl(N.u), v1 = shl(N.v);
    const T p2 = shl(p1), u2 = shl(u1), v2 = shl(v1);
    const T p3 = shr(N.p), u3 = shr(N.u), v3 = shr(N.v);
    const T p4 = shr(p3), u4 = shr(u3), v4 = shr(v3);
    if (gx == 1) N.p = p1, N.u = u1, N.v = v1;
    if (gx == 2) N.p = p2, N.u = u2, N.v = v2;
    if (gx == 3) N.p = p3, N.u = u3, N.v = v3;
    if (gx == 4) N.p = p4, N.u = u4, N.v = v4;
  }
  __device__ void put(const Row3<T> &N, int r) const {
    const unsigned o = st ? (unsigned)(r + 2) * ld * (unsigned)sizeof(T) + ocolb : kDropOffset;
    bstore(ob, N.p, o);
    bstore(ob, N.u, o + plb);
    bstore(ob, N.v, o + 2 * plb);
  }
  __device__ void emit(Row3<T> N, int r) const {
    ghost_columns(N);
    put(N, r);
    if (r == 0) put(N, -1), put(N, -2);
    if (r == my - 1) put(N, my), put(N, my + 1);
  }
};

// Rows [r0, r1) advanced by two steps.  Set j holds row r0-2+j of the input
// at first; iteration I works the first step's row r0-2+I and, from I = 4,
// the second step's row r0-4+I.  The first step's rows below the patch are
// copies of its row 0 and those above it of its last row.
template <typename T, int LIM>
__device__ __attribute__((always_inline)) inline void march_two(const MultiLanes<T> &M,
                                                                const Coef<T> &ka,
                                                                const Coef<T> &kb, int r0,
                                                                int r1) {
  const bool bottom = r0 == 0;
  Row3<T> R[kMultiSets], W[3], M2, M1, e0, e1;
  const int q0 = bottom ? 0 : r0 - 2;  // first row of the first step
  M.fetch(M2, q0 - 2);
  M.fetch(M1, q0 - 1);
  // at the bottom sets 0 and 1 start with the rows they would hold next
  M.fetch(R[0], bottom ? r0 + 4 : r0 - 2);
  M.fetch(R[1], bottom ? r0 + 5 : r0 - 1);
  M.fetch(R[2], r0);
  M.fetch(R[3], r0 + 1);
  M.fetch(R[4], r0 + 2);
  M.fetch(R[5], r0 + 3);
  Carry<T> S, S2;
  if (!bottom) {
    S = carry_in<T, LIM>(ka, M2, M1, R[0], R[1]);
    e0 = row_step<T, LIM>(ka, S, R[0], R[1], R[2]);
    M.fetch(R[0], r0 + 4);
    e1 = row_step<T, LIM>(ka, S, R[1], R[2], R[3]);
    M.fetch(R[1], r0 + 5);
    M.ghost_columns(e0);
    M.ghost_columns(e1);
  } else {
    S = carry_in<T, LIM>(ka, M2, M1, R[2], R[3]);
  }
  W[2] = row_step<T, LIM>(ka, S, R[2], R[3], R[4]);
  M.ghost_columns(W[2]);
  M.fetch(R[2], r0 + 6);
  if (bottom) e0 = W[2], e1 = W[2];
  W[0] = row_step<T, LIM>(ka, S, R[3], R[4], R[5]);
  M.ghost_columns(W[0]);
  M.fetch(R[3], r0 + 7);
  if (r0 + 1 >= M.my) W[0] = W[2];
  S2 = carry_in<T, LIM>(kb, e0, e1, W[2], W[0]);

  // one row: first step's row r+2 from sets A, B, C into Wc, then the second
  // step's row r from Wa, Wb, Wc; set A is refilled
  auto row = [&](Row3<T> &A, const Row3<T> &B, const Row3<T> &C, const Row3<T> &Wa,
                 const Row3<T> &Wb, Row3<T> &Wc, int r) {
    __builtin_amdgcn_sched_barrier(0);
    Wc = row_step<T, LIM>(ka, S, A, B, C);
    M.ghost_columns(Wc);
    if (r + 2 >= M.my) Wc = Wb;
    const Row3<T> N = row_step<T, LIM>(kb, S2, Wa, Wb, Wc);
    M.emit(N, r);
    __builtin_amdgcn_sched_barrier(0);
    M.fetch(A, r + 2 + kMultiSets);
  };
  for (int r = r0;;) {
    row(R[4], R[5], R[0], W[2], W[0], W[1], r);
    if (++r == r1) break;
    row(R[5], R[0], R[1], W[0], W[1], W[2], r);
    if (++r == r1) break;
    row(R[0], R[1], R[2], W[1], W[2], W[0], r);
    if (++r == r1) break;
    row(R[1], R[2], R[3], W[2], W[0], W[1], r);
    if (++r == r1) break;
    row(R[2], R[3], R[4], W[0], W[1], W[2], r);
    if (++r == r1) break;
    row(R[3], R[4], R[5], W[1], W[2], W[0], r);
    if (++r == r1) break;
  }
}

// The time step after one of Courant number cfl (Sec. 2.5 eq. (2.11)), as
// the one-step launch computes it.
__device__ inline double next_dt(double dt, double c, const InstMin &m, double cfl_desired,
                                 double &cfl) {
  cfl = fmax(c * (dt / m.dx), c * (dt / m.dy));
  return cfl > 0.0 ? dt * cfl_desired / cfl : dt;
}

// Workgroup t works tile t: four segments of seg_rows rows, one per
// wavefront, stacked up the patch.  Workgroups are dispatched round-robin
// over the XCDs; each XCD takes a contiguous run of tiles, whose halos
// overlap.  The last workgroup files the two steps' Courant numbers.
template <typename T, int LIM>
__global__ __launch_bounds__(kThreads, 2) void step_kernel_two(StepArgs a) {
  if (blockIdx.x == gridDim.x - 1) {
    const CflSlots &c = a.slots;
    for (int k = (int)threadIdx.x; k < c.n_inst; k += kThreads) {
      const InstMin m = c.inst_min[k];
      double cfl0, cfl1;
      const double dt1 = next_dt(a.dt[k], a.inst[k].c, m, a.cfl_desired, cfl0);
      c.dt[k] = next_dt(dt1, a.inst[k].c, m, a.cfl_desired, cfl1);
      c.cfl_last[k] = cfl1;
      c.cfl_max[k] = fmax(fmax(c.cfl_max[k], cfl0), cfl1);
    }
    // the level maximum is left to the one-step launch that ends every loop
    return;
  }
  const int x = (int)blockIdx.x % kGroups, y = (int)blockIdx.x / kGroups;
  const int t = (int)((int64_t)a.n_tiles * x / kGroups) + y;
  if (t >= (int)((int64_t)a.n_tiles * (x + 1) / kGroups)) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const TileEntry te = uniform_row(a.tiles[t]);
  const PatchRow pr = uniform_row(a.patches[te.patch]);
  const int r0 = (te.ty * 4 + wave) * a.seg_rows, r1 = min(r0 + a.seg_rows, pr.my);
  if (r0 >= r1) return;
  const InstRow in = uniform_row(a.inst[pr.inst]);
  const InstMin m = uniform_row(a.slots.inst_min[pr.inst]);
  const double dt0 = a.dt[pr.inst];
  double cfl;
  const double dt1 = next_dt(dt0, in.c, m, a.cfl_desired, cfl);
  const Coef<T> ka = make_coef<T>(in.c, in.Z, dt0, pr.dx, pr.dy);
  const Coef<T> kb = make_coef<T>(in.c, in.Z, dt1, pr.dx, pr.dy);
  const int64_t org = pr.q_off + 2 * (int64_t)pr.ld + pr.col0;
  const MultiLanes<T> M(reinterpret_cast<const T *>(a.qin) + org,
                        reinterpret_cast<T *>(a.qout) + org, pr,
                        te.tx * kMultiCols - kMultiHalo, (int)threadIdx.x & 63, r1);
  march_two<T, LIM>(M, ka, kb, r0, r1);
}

template <typename T>
hipError_t two_t(int limiter, const StepArgs &a, hipStream_t s) {
  // the XCDs' runs differ by at most one tile: the grid covers the longest on
  // each, and the filing workgroup comes after them
  const dim3 grid((unsigned)((a.n_tiles + kGroups - 1) / kGroups * kGroups + 1)), block(kThreads);
  switch (limiter) {
    case WS_LIM_NONE:
      hipLaunchKernelGGL((step_kernel_two<T, WS_LIM_NONE>), grid, block, 0, s, a);
      break;
    case WS_LIM_VANLEER:
      hipLaunchKernelGGL((step_kernel_two<T, WS_LIM_VANLEER>), grid, block, 0, s, a);
      break;
    default:
      hipLaunchKernelGGL((step_kernel_two<T, WS_LIM_MC>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_step_two(int dtype, int limiter, const StepArgs &a, hipStream_t s) {
  if (a.n_tiles <= 0 || a.seg_rows <= 0) return hipErrorInvalidValue;
  return dtype == WS_F32 ? two_t<float>(limiter, a, s) : two_t<double>(limiter, a, s);
}

}  // namespace ws
