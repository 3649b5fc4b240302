// Two level steps in one launch (gfx950), for the captured step loop of
// homogeneous levels whose patches have extrapolation boundaries, and of tiled
// levels.
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
// A tiled level whose patches cut the domain along full columns and rows is
// worked as that one domain.
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
  unsigned ybits;        // branches of the row's bottom edge (recording only)
  T yb2, b1h, b2h;       // b2 of the cell's bottom edge; b1, b2 of its top edge
  T GB1, GB2;            // G~ of the bottom edge (characteristic)
  T a1L, a2L;            // strengths of the row's left x-edge
};

// Carry for row r from rows r-2 (p, v), r-1, r and r+1 (p, v).
template <typename T, int LIM, bool MASKS>
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
  gtilde<T, LIM>(k, b1m, b2m, S.b1h, b2mm, xsm, S.a2L + shl(S.a1L), S.GB1, S.GB2);
  if constexpr (MASKS) S.ybits = (mc_branch(b1m, S.b1h) << 4) | (mc_branch(b2m, b2mm) << 6);
  return S;
}

// The update of row r from rows r (A), r+1 (B) and r+2 (C; p, v); slides the
// carry up one row.  branches: those of its left and bottom edges, as a
// branch byte (recording only).
template <typename T, int LIM, bool MASKS>
__device__ __attribute__((always_inline)) inline Row3<T> row_step(const Coef<T> &k, Carry<T> &S,
                                                                  const Row3<T> &A,
                                                                  const Row3<T> &B,
                                                                  const Row3<T> &C,
                                                                  unsigned &branches) {
  const T Z = k.Z;
  const T b1hh = s1(Z, C.p - B.p, C.v - B.v), b2hh = s2(Z, C.p - B.p, C.v - B.v);
  const T ys0 = S.yb2 + S.b1h;
  const T pl = shr(B.p), ul = shr(B.u);
  const T a1Ln = s1(Z, B.p - pl, B.u - ul), a2Ln = s2(Z, B.p - pl, B.u - ul);
  const T xsp = a2Ln + shl(a1Ln);
  const T a1R = shl(S.a1L);
  T FL1, FL2, GT1, GT2;
  ftilde<T, LIM>(k, S.a1L, S.a2L, a1R, shr(S.a2L), shr(ys0), ys0, FL1, FL2);
  const T FR1 = shl(FL1), FR2 = shl(FL2);
  gtilde<T, LIM>(k, S.b1h, S.b2h, b1hh, S.yb2, S.a2L + a1R, xsp, GT1, GT2);
  Row3<T> N;
  update<T>(k, A.p, A.u, A.v, S.a2L, a1R, S.yb2, S.b1h, FL1, FL2, FR1, FR2, S.GB1, S.GB2, GT1, GT2,
            N.p, N.u, N.v);
  if constexpr (MASKS) {
    branches = mc_branch(S.a1L, a1R) | (mc_branch(S.a2L, shr(S.a2L)) << 2) | S.ybits;
    S.ybits = (mc_branch(S.b1h, b1hh) << 4) | (mc_branch(S.b2h, S.yb2) << 6);
  }
  S.yb2 = S.b2h, S.b1h = b1hh, S.b2h = b2hh;
  S.GB1 = GT1, S.GB2 = GT2;
  S.a1L = a1Ln, S.a2L = a2Ln;
  return N;
}

// Row sets of a segment: a set holds a row from its load until its last use
// as row r, then is refilled with the row kMultiSets further up.
constexpr int kMultiSets = 6;

// Lane `from` of the wavefront (a scalar) as a wave-uniform value.
__device__ inline double lane_value(double v, int from) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), from),
                          __builtin_amdgcn_readlane(__double2loint(v), from));
}
__device__ inline float lane_value(float v, int from) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), from));
}

// The lanes on ghost columns (glo, ghi: of the low, the high side) take the
// new value of the nearest column, on lane lo or hi, through scalar registers:
// two lane reads per value and side.  lo <= 0 or hi >= 63: no such lanes.
template <typename T>
__device__ inline void nearest_columns(Row3<T> &N, int lo, int hi, bool glo, bool ghi) {
  if (lo > 0) {
    const T p = lane_value(N.p, lo), u = lane_value(N.u, lo), v = lane_value(N.v, lo);
    if (glo) N.p = p, N.u = u, N.v = v;
  }
  if (hi < kMarchWidth - 1) {
    const int from = max(hi, 0);
    const T p = lane_value(N.p, from), u = lane_value(N.u, from), v = lane_value(N.v, from);
    if (ghi) N.p = p, N.u = u, N.v = v;
  }
}

// Lanes of one segment: lane l holds column i of the patch, lanes kMultiHalo
// .. 63 - kMultiHalo are updated.  The first step reads the ghosts as the state
// holds them (they need not be extrapolated: a state may be uploaded with
// others); the lanes and rows past them read the last ones.  Rows are addressed
// by a scalar offset that is stepped along, columns by the lane's: no vector
// instruction goes into addresses.
template <typename T>
struct MultiLanes {
  __amdgpu_buffer_rsrc_t ib, ob;  // the patch in the two pools, from padded cell (-2, -2)
  unsigned ldb, plb;     // row and plane strides (bytes)
  unsigned colb, ocolb;  // the lane's offsets in a row: the column read, the column stored
  int my, rmax;          // rmax: last row the segment needs
  int lo, hi;            // lanes of columns 0 and mx-1 (negative, over 63: not in the segment)
  bool glo, ghi;         // the lane holds a ghost column of the low, the high side
  int i, mx, r0, r1;     // the lane's column; the segment's rows
  bool own, edge;        // the lane updates its column; holds the one past the last updated

  __device__ MultiLanes(const T *qi, T *qo, const PatchRow &pr, int i0, int l, int r0_,
                        int r1_) {
    constexpr int halo = kMultiHalo;
    ldb = (unsigned)pr.ld * (unsigned)sizeof(T);
    plb = (unsigned)pr.plane * (unsigned)sizeof(T);
    my = pr.my;
    r0 = r0_;
    r1 = r1_;
    rmax = min(r1 + 3, pr.my + 1);
    const int64_t first = 2 * (int64_t)pr.ld + 2;
    ib = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(qi - first), 0, (int)(3 * plb),
                                           kRawBufferWord3);
    ob = __builtin_amdgcn_make_buffer_rsrc(qo - first, 0, (int)(3 * plb), kRawBufferWord3);
    i = i0 + l;
    mx = pr.mx;
    colb = (unsigned)(min(max(i, -2), mx + 1) + 2) * (unsigned)sizeof(T);
    lo = -i0;
    hi = mx - 1 - i0;
    glo = i < 0;
    ghi = i >= mx;
    // ghost columns are stored by the segment that updates the column they copy
    const int s = i < 0 ? lo : i >= mx ? hi : l;
    const bool st = i >= -2 && i <= mx + 1 && s >= halo && s < kMarchWidth - halo;
    ocolb = st ? (unsigned)(i + 2) * (unsigned)sizeof(T) : kDropOffset;
    own = l >= halo && l < kMarchWidth - halo && i < mx;
    edge = i == mx && l > halo && l <= kMarchWidth - halo;
  }
  // The branch byte of row r, and above the last row that of its top edges.
  __device__ void record(uint8_t *masks, int r, unsigned branches, unsigned top) const {
    if (r < r0 || r >= r1) return;
    uint8_t *row = masks + (int64_t)r * (mx + 1) + i;
    if (own || edge) row[0] = (uint8_t)(own ? branches : branches & 15u);
    if (r == my - 1 && (own || edge)) row[mx + 1] = (uint8_t)(own ? top : 0u);  // no edge owns the corner
  }
  // The new rows outside the patch copy its first and last row.
  __device__ bool clamp_y() const { return true; }
  // Whether the segment holds ghost columns.
  __device__ bool ghosts() const { return lo > 0 || hi < kMarchWidth - 1; }
  // A place in the rows read or stored, stepped up row by row.
  struct Cursor {
    unsigned o;
  };
  __device__ unsigned row_offset(int r) const {
    return (unsigned)(min(max(r, -2), rmax) + 2) * ldb;
  }
  __device__ void fetch_at(Row3<T> &S, unsigned o) const {
    S.p = bload<T>(ib, colb, o);
    S.u = bload<T>(ib, colb, o + plb);
    S.v = bload<T>(ib, colb, o + 2 * plb);
  }
  __device__ void fetch(Row3<T> &S, int r) const { fetch_at(S, row_offset(r)); }
  __device__ Cursor read_from(int r) const { return Cursor{row_offset(r)}; }
  __device__ void fetch_next(Row3<T> &S, Cursor &c) const {
    fetch_at(S, c.o);
    c.o = min(c.o + ldb, row_offset(rmax));
  }
  __device__ Cursor store_from(int r) const { return Cursor{(unsigned)(r + 2) * ldb}; }
  // Row r, with its ghost rows (EDGE).
  template <bool EDGE>
  __device__ void store_next(const Row3<T> &N, Cursor &c, int r) const {
    if constexpr (EDGE) {
      if (r == 0) put_at(N, 0), put_at(N, ldb);
      if (r == my - 1) put_at(N, c.o + ldb), put_at(N, c.o + 2 * ldb);
    }
    put_at(N, c.o);
    c.o += ldb;
  }
  __device__ void ghost_columns(Row3<T> &N) const {
    nearest_columns(N, lo, hi, glo, ghi);
  }
  __device__ void put_at(const Row3<T> &N, unsigned o) const {
    bstore(ob, N.p, ocolb, o);
    bstore(ob, N.u, ocolb, o + plb);
    bstore(ob, N.v, ocolb, o + 2 * plb);
  }
};

// Lanes of one segment of a tiled level, whose patches cut one domain along
// full columns and rows: lane l holds column i of the domain, wherever the
// patches' edges fall, and the march crosses from a patch to the one above it.
// So the segment reads what the ghosts stand for, and no ghosts are needed
// between the launches.  A lane keeps its patch's addressing (the patches of a
// wavefront may have different strides) and takes the next patch's from the
// table when the march leaves a row of patches.  Outside the domain, columns
// and rows wrap around or copy the nearest one.  Pools under 2^31 bytes.
template <typename T>
struct DomainLanes {
  __amdgpu_buffer_rsrc_t ib, ob;  // the two pools
  const DomainPatch *tab;         // row of patches by row of patches
  int ycut;                       // lane b: where row b of patches starts (b = nb: the end)
  int na, nb, my, rmax, r0, r1;   // patches per row, rows of patches; the domain's rows
  bool wrap;                      // rows wrap around
  int a;                          // the lane's column of patches
  unsigned colb;                  // its offset in a row of its patch
  int lo, hi;                     // lanes of columns 0 and mx-1 (clamped columns only)
  bool glo, ghi, own;

  struct Cursor {
    unsigned o, ldb, plb;  // the lane's place, row and plane strides (bytes)
    int row, end, b;       // row of the domain, end of the row of patches, its index
  };

  __device__ DomainLanes(const StepArgs &A, int i0, int l, int r0_, int r1_) {
    constexpr int halo = kMultiHalo;
    ib = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(A.qin), 0, A.pool_bytes,
                                           kRawBufferWord3);
    ob = __builtin_amdgcn_make_buffer_rsrc(A.qout, 0, A.pool_bytes, kRawBufferWord3);
    const Domain &D = A.domain;
    tab = D.patches;
    na = D.na;
    nb = D.nb;
    ycut = D.ycut[min(l, nb)];
    const int xcut = D.xcut[min(l, na)];
    my = D.my;
    wrap = (D.periodic & 2) != 0;
    r0 = r0_;
    r1 = r1_;
    rmax = r1 + 3;
    const int i = i0 + l, mx = D.mx;
    own = l >= halo && l < kMarchWidth - halo && i < mx;
    const bool wrap_x = (D.periodic & 1) != 0;
    lo = wrap_x ? 0 : -i0;
    hi = wrap_x ? kMarchWidth : mx - 1 - i0;
    glo = !wrap_x && i < 0;
    ghi = !wrap_x && i >= mx;
    const int c = wrap_x ? (i % mx + mx) % mx : min(max(i, 0), mx - 1);
    a = 0;
    int x0 = 0;
    for (int n = 1; n < na; ++n) {
      const int x = __builtin_amdgcn_readlane(xcut, n);
      if (c >= x) a = n, x0 = x;
    }
    colb = (unsigned)(c - x0 + 2) * (unsigned)sizeof(T);
  }
  __device__ bool clamp_y() const { return !wrap; }
  __device__ bool ghosts() const { return lo > 0 || hi < kMarchWidth - 1; }
  __device__ Cursor cursor(int r, bool store) const {
    Cursor c;
    c.row = wrap ? (r % my + my) % my : min(max(r, 0), my - 1);
    c.b = 0;
    while (c.b + 1 < nb && c.row >= __builtin_amdgcn_readlane(ycut, c.b + 1)) ++c.b;
    place(c, store);
    return c;
  }
  // The lane's addressing in the cursor's row of patches.
  __device__ void place(Cursor &c, bool store) const {
    const DomainPatch p = tab[c.b * na + a];
    const int y0 = __builtin_amdgcn_readlane(ycut, c.b);
    c.end = __builtin_amdgcn_readlane(ycut, c.b + 1);
    c.ldb = p.ldb;
    c.plb = p.plb;
    c.o = p.off + (unsigned)(c.row - y0 + 2) * p.ldb + colb;
    if (store && !own) c.o = kDropOffset, c.ldb = 0, c.plb = 0;
  }
  __device__ void step(Cursor &c, bool store) const {
    if (c.row + 1 < c.end) {
      c.row += 1;
      c.o += c.ldb;
      return;
    }
    if (c.b + 1 == nb && !wrap) return;  // the last row stands for those above it
    c.b = c.b + 1 == nb ? 0 : c.b + 1;
    c.row = __builtin_amdgcn_readlane(ycut, c.b);
    place(c, store);
  }
  __device__ void load(Row3<T> &S, const Cursor &c) const {
    S.p = bload<T>(ib, c.o, 0);
    S.u = bload<T>(ib, c.o + c.plb, 0);
    S.v = bload<T>(ib, c.o + 2 * c.plb, 0);
  }
  __device__ void fetch(Row3<T> &S, int r) const { load(S, cursor(r, false)); }
  __device__ Cursor read_from(int r) const { return cursor(min(r, rmax), false); }
  __device__ void fetch_next(Row3<T> &S, Cursor &c) const {
    load(S, c);
    step(c, false);
  }
  __device__ Cursor store_from(int r) const { return cursor(r, true); }
  template <bool EDGE>
  __device__ void store_next(const Row3<T> &N, Cursor &c, int) const {
    bstore(ob, N.p, c.o);
    bstore(ob, N.u, c.o + c.plb);
    bstore(ob, N.v, c.o + 2 * c.plb);
    step(c, true);
  }
  __device__ void ghost_columns(Row3<T> &N) const {
    nearest_columns(N, lo, hi, glo, ghi);
  }
  __device__ void record(uint8_t *, int, unsigned, unsigned) const {}
};

// Rows [r0, r1) advanced by two steps.  Set j holds row r0-2+j of the input
// at first; the first step's rows r0-2 .. r0+1 come before the loop, and its
// iteration for row r works the first step's row r+2 and the second step's
// row r.  EDGE: the segment holds ghost columns, or rows next to the patch's
// first or last one; the first step's rows below the patch are then copies of
// its row 0 and those above it of its last row.  The other segments' loop has
// no branches: a wavefront alone on its SIMD issues one instruction of any
// kind per four cycles, so what goes into branches and addresses counts.
template <typename T, int LIM, bool EDGE, bool MASKS, class L>
__device__ __attribute__((always_inline)) inline void march_two(const L &M,
                                                                const Coef<T> &ka,
                                                                const Coef<T> &kb,
                                                                uint8_t *masks,
                                                                uint8_t *masks2) {
  const int r0 = M.r0, r1 = M.r1;
  const bool clamp = EDGE && M.clamp_y();  // (without: the rows wrap around)
  const bool bottom = clamp && r0 == 0;
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
  // the first step's row r from sets A, B, C; A is refilled
  auto first = [&](Row3<T> &A, const Row3<T> &B, const Row3<T> &C, int r) {
    unsigned br = 0;
    Row3<T> N = row_step<T, LIM, MASKS>(ka, S, A, B, C, br);
    if constexpr (MASKS) M.record(masks, r, br, S.ybits);
    if constexpr (EDGE) M.ghost_columns(N);
    M.fetch(A, r + kMultiSets);
    return N;
  };
  if (!bottom) {
    S = carry_in<T, LIM, MASKS>(ka, M2, M1, R[0], R[1]);
    e0 = first(R[0], R[1], R[2], r0 - 2);
    e1 = first(R[1], R[2], R[3], r0 - 1);
  } else {
    S = carry_in<T, LIM, MASKS>(ka, M2, M1, R[2], R[3]);
  }
  W[0] = first(R[2], R[3], R[4], r0);
  if (bottom) e0 = W[0], e1 = W[0];
  W[1] = first(R[3], R[4], R[5], r0 + 1);
  if (clamp && r0 + 1 >= M.my) W[1] = W[0];
  S2 = carry_in<T, LIM, MASKS>(kb, e0, e1, W[0], W[1]);

  // the row fetched next and the row stored
  typename L::Cursor in = M.read_from(r0 + 8), out = M.store_from(r0);
  auto row = [&](Row3<T> &A, const Row3<T> &B, const Row3<T> &C, const Row3<T> &Wa,
                 const Row3<T> &Wb, Row3<T> &Wc, int r) {
    __builtin_amdgcn_sched_barrier(0);
    unsigned br = 0;
    Wc = row_step<T, LIM, MASKS>(ka, S, A, B, C, br);
    if constexpr (MASKS) M.record(masks, r + 2, br, S.ybits);
    if constexpr (EDGE) {
      M.ghost_columns(Wc);
      if (clamp && r + 2 >= M.my) {
        asm volatile("");  // a branch taken on two rows, not selects on each
        Wc = Wb;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    Row3<T> N = row_step<T, LIM, MASKS>(kb, S2, Wa, Wb, Wc, br);
    if constexpr (MASKS) M.record(masks2, r, br, S2.ybits);
    if constexpr (EDGE) M.ghost_columns(N);
    M.template store_next<EDGE>(N, out, r);
    __builtin_amdgcn_sched_barrier(0);
    M.fetch_next(A, in);
  };
  for (int r = r0;;) {
    row(R[4], R[5], R[0], W[0], W[1], W[2], r);
    if (++r == r1) break;
    row(R[5], R[0], R[1], W[1], W[2], W[0], r);
    if (++r == r1) break;
    row(R[0], R[1], R[2], W[2], W[0], W[1], r);
    if (++r == r1) break;
    row(R[1], R[2], R[3], W[0], W[1], W[2], r);
    if (++r == r1) break;
    row(R[2], R[3], R[4], W[1], W[2], W[0], r);
    if (++r == r1) break;
    row(R[3], R[4], R[5], W[2], W[0], W[1], r);
    if (++r == r1) break;
  }
}

// The time step after one of Courant number cfl (Sec. 2.5 eq. (2.11)), as
// the one-step launch computes it.
__device__ inline double next_dt(double dt, double c, const InstMin &m, double cfl_desired,
                                 double &cfl) {
  cfl = fmax(c * (dt / m.dx), c * (dt / m.dy));
  return cfl_desired > 0.0 && cfl > 0.0 ? dt * cfl_desired / cfl : dt;
}

// Receivers: p before the launch's first step, read, and after it, from the
// cell's 13-point footprint (cell_update, whose bits are the sweep's).  The
// state after the second step is the next launch's first.
template <typename T, int LIM>
__device__ inline void gather_receivers(const StepArgs &a, int first) {
  const int n = first + (int)threadIdx.x;
  if (n >= a.rec_n) return;
  const PatchRow pr = a.patches[a.rec_patch];
  const int i = a.rec_ij[2 * n], j = a.rec_ij[2 * n + 1];
  double now = __builtin_nan(""), mid = now;
  if (i >= 0 && i < pr.mx && j >= 0 && j < pr.my) {
    const T *q = reinterpret_cast<const T *>(a.qin) + pr.q_off + 2 * (int64_t)pr.ld + pr.col0;
    const InstRow in = a.inst[pr.inst];
    const double dt = a.dt_override > 0.0 ? a.dt_override : a.dt[pr.inst];
    const Coef<T> k = make_coef<T, LIM>(in.c, in.Z, dt, pr.dx, pr.dy);
    const Planes<T> Q{q, q + pr.plane, q + 2 * pr.plane, pr.ld};
    T pn, un, vn;
    cell_update<T, LIM, false>(Q, i, j, k, pn, un, vn, nullptr);
    now = (double)Q.P(i, j), mid = (double)pn;
  }
  if (a.rec_now) a.rec_now[n] = now;
  a.rec_mid[n] = mid;
}

// Measured, MC, us per launch of two steps and of one step: 2048 x 2048 FP64
// (200 MB of state, within the Infinity Cache) 43.8 and 34.2, 4096 x 4096 FP64
// 194 and 197, 2048 x 2048 FP32 29.1 and 21.1.  What bounds it is instruction
// issue and memory together: 183 instructions per row and wavefront for the two
// steps (164 of them vector), 24 us of the 44 us a 2048 x 2048 launch takes, and
// 235 MB of traffic at 5.4 TB/s; 4096 x 4096 runs at 4.8 TB/s, 93% of a large
// copy's.
//
// Workgroup t works tile t: four segments of seg_rows rows, one per
// wavefront, stacked up the patch.  Workgroups are dispatched round-robin
// over the XCDs; each XCD takes a contiguous run of tiles, whose halos
// overlap.  The last workgroup files the two steps' Courant numbers.
// Wavefronts per SIMD the registers are kept for: three (153 registers in
// FP64; four spilled and ran 4x slower), two where branches are recorded
// (197) and on a tiled level, whose lanes carry their own addressing (three
// spilled 66).
template <typename T, int LIM, bool MASKS, bool DOMAIN>
constexpr int two_waves() {
  return sizeof(T) == 8 && (MASKS || DOMAIN) ? 2 : 3;
}

// DOMAIN: a tiled level, worked as the one domain its patches cut.
template <typename T, int LIM, bool MASKS, bool DOMAIN>
__global__ __launch_bounds__(kThreads, (two_waves<T, LIM, MASKS, DOMAIN>())) void step_kernel_two(StepArgs a) {
  const int work = (a.n_tiles + kGroups - 1) / kGroups * kGroups;  // workgroups of the tiles
  if ((int)blockIdx.x >= work) {
    if ((int)blockIdx.x > work) {
      if constexpr (sizeof(T) == 8)
        gather_receivers<T, LIM>(a, ((int)blockIdx.x - work - 1) * kThreads);
      return;
    }
    const CflSlots &c = a.slots;
    for (int k = (int)threadIdx.x; k < c.n_inst; k += kThreads) {
      const InstMin m = c.inst_min[k];
      const double dt0 = a.dt_override > 0.0 ? a.dt_override : a.dt[k];
      double cfl0, cfl1;
      const double dt1 = next_dt(dt0, a.inst[k].c, m, a.cfl_desired, cfl0);
      c.dt[k] = next_dt(dt1, a.inst[k].c, m, a.cfl_desired, cfl1);
      c.cfl_last[k] = cfl1;
      c.cfl_max[k] = fmax(fmax(c.cfl_max[k], cfl0), cfl1);
    }
    // the level maximum is left to the one-step launch that ends every loop
    return;
  }
  const int x = (int)blockIdx.x % kGroups, y = (int)blockIdx.x / kGroups;
  const int beg = (int)((int64_t)a.n_tiles * x / kGroups);
  const int end = (int)((int64_t)a.n_tiles * (x + 1) / kGroups);
  if (beg + y >= end) return;
  const int t = a.reverse ? end - 1 - y : beg + y;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const TileEntry te = uniform_row(a.tiles[t]);
  const PatchRow pr = uniform_row(a.patches[te.patch]);
  const int rows = DOMAIN ? a.domain.my : pr.my;
  const int r0 = (te.ty * 4 + wave) * a.seg_rows, r1 = min(r0 + a.seg_rows, rows);
  if (r0 >= r1) return;
  const InstRow in = uniform_row(a.inst[pr.inst]);
  const InstMin m = uniform_row(a.slots.inst_min[pr.inst]);
  const double dt0 = a.dt_override > 0.0 ? a.dt_override : a.dt[pr.inst];
  double cfl;
  const double dt1 = next_dt(dt0, in.c, m, a.cfl_desired, cfl);
  const Coef<T> ka = make_coef<T, LIM>(in.c, in.Z, dt0, pr.dx, pr.dy);
  const Coef<T> kb = make_coef<T, LIM>(in.c, in.Z, dt1, pr.dx, pr.dy);
  if constexpr (DOMAIN) {
    const DomainLanes<T> M(a, te.tx * kMultiCols - kMultiHalo, (int)threadIdx.x & 63, r0, r1);
    if (M.ghosts() || (M.clamp_y() && (r0 == 0 || r1 + 2 > rows)))
      march_two<T, LIM, true, false>(M, ka, kb, nullptr, nullptr);
    else
      march_two<T, LIM, false, false>(M, ka, kb, nullptr, nullptr);
    return;
  }
  const int64_t org = pr.q_off + 2 * (int64_t)pr.ld + pr.col0;
  const MultiLanes<T> M(reinterpret_cast<const T *>(a.qin) + org,
                        reinterpret_cast<T *>(a.qout) + org, pr,
                        te.tx * kMultiCols - kMultiHalo, (int)threadIdx.x & 63, r0, r1);
  uint8_t *m1 = MASKS ? a.masks + pr.mask_off : nullptr;
  uint8_t *m2 = MASKS ? a.masks2 + pr.mask_off : nullptr;
  if (M.ghosts() || r0 == 0 || r1 + 2 > pr.my)
    march_two<T, LIM, true, MASKS>(M, ka, kb, m1, m2);
  else
    march_two<T, LIM, false, MASKS>(M, ka, kb, m1, m2);
}

template <typename T, int LIM>
hipError_t two_l(const StepArgs &a, hipStream_t s) {
  // the XCDs' runs differ by at most one tile: the grid covers the longest on
  // each; the filing workgroup and the receivers' come after them
  const dim3 grid((unsigned)((a.n_tiles + kGroups - 1) / kGroups * kGroups + 1 +
                             (a.rec_n + kThreads - 1) / kThreads));
  if constexpr (sizeof(T) == 8 && LIM == WS_LIM_MC) {
    if (a.masks) {
      if (a.domain.na > 0) return hipErrorInvalidValue;
      hipLaunchKernelGGL((step_kernel_two<T, LIM, true, false>), grid, dim3(kThreads), 0, s, a);
      return hipGetLastError();
    }
  }
  if (a.masks) return hipErrorInvalidValue;
  if (a.domain.na > 0)
    hipLaunchKernelGGL((step_kernel_two<T, LIM, false, true>), grid, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((step_kernel_two<T, LIM, false, false>), grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t two_t(int limiter, const StepArgs &a, hipStream_t s) {
  switch (limiter) {
    case WS_LIM_NONE: return two_l<T, WS_LIM_NONE>(a, s);
    case WS_LIM_VANLEER: return two_l<T, WS_LIM_VANLEER>(a, s);
    default: return two_l<T, WS_LIM_MC>(a, s);
  }
}

}  // namespace

hipError_t launch_step_two(int dtype, int limiter, const StepArgs &a, hipStream_t s) {
  if (a.n_tiles <= 0 || a.seg_rows <= 0) return hipErrorInvalidValue;
  if (a.rec_n > 0 && dtype != WS_F64) return hipErrorInvalidValue;
  return dtype == WS_F32 ? two_t<float>(limiter, a, s) : two_t<double>(limiter, a, s);
}

template <typename T, int LIM>
static int two_occupancy_of(bool domain) {
  int n = 0;
  const hipError_t e =
      domain ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                   &n, step_kernel_two<T, LIM, false, true>, kThreads, 0)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                   &n, step_kernel_two<T, LIM, false, false>, kThreads, 0);
  return e == hipSuccess ? n : 0;
}

template <typename T>
static int two_occupancy_t(int limiter, bool domain) {
  return limiter == WS_LIM_NONE      ? two_occupancy_of<T, WS_LIM_NONE>(domain)
         : limiter == WS_LIM_VANLEER ? two_occupancy_of<T, WS_LIM_VANLEER>(domain)
                                     : two_occupancy_of<T, WS_LIM_MC>(domain);
}

int step_two_occupancy(int dtype, int limiter, bool domain) {
  return dtype == WS_F32 ? two_occupancy_t<float>(limiter, domain)
                         : two_occupancy_t<double>(limiter, domain);
}

}  // namespace ws
