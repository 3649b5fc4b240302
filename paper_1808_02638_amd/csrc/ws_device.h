// Device helpers shared by the forward and adjoint kernels of the
// wave-propagation library.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/wavestep.h"

namespace ws {

// --------------------------------------------------------------------------
// Per-patch coefficients of the closed forms (computed in FP64, rounded once
// to T)
// --------------------------------------------------------------------------
template <typename T>
struct Coef {
  T Z;
  T h, hz;                // c/2, c/(2Z): fluctuation factors
  T fx, fxz, fy, fyz;     // c(1-nu)/4 and /Z: correction factors
  T gx, gxz, gy, gyz;     // dtdx c^2/8 and /Z: transverse factors
  T dtdx, dtdy;
  T iz, dtdxz, dtdyz;     // 1/Z, dtdx/Z, dtdy/Z
  T lx, ly;               // fx, fy on the limiter's scale
  T tx, ty;               // 1 - nu on it: the correction moved into the split vectors
};

// limited() returns its strength divided by this power of two (it goes into
// the factors, exactly).
template <typename T>
constexpr double limiter_scale(int lim) {
  return lim == WS_LIM_NONE ? 1.0 : lim == WS_LIM_VANLEER && sizeof(T) == 8 ? 2.0 : 0.5;
}

// Wave-uniform values are moved to scalar registers.
__device__ inline double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ inline float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// lane_coef: each lane's own; make_coef: those of a wave-uniform dt.
template <typename T, int LIM = WS_LIM_NONE>
__device__ inline Coef<T> lane_coef(double c, double Z, double dt, double dx, double dy) {
  const double dtdx = dt / dx, dtdy = dt / dy, iz = 1.0 / Z;
  const double fx = 0.25 * c * (1.0 - c * dtdx), fy = 0.25 * c * (1.0 - c * dtdy);
  const double gx = 0.125 * dtdx * c * c, gy = 0.125 * dtdy * c * c;
  Coef<T> k;
  k.Z = (T)Z;
  k.h = (T)(0.5 * c);
  k.hz = (T)(0.5 * c * iz);
  k.fx = (T)fx;
  k.fxz = (T)(fx * iz);
  k.fy = (T)fy;
  k.fyz = (T)(fy * iz);
  k.gx = (T)gx;
  k.gxz = (T)(gx * iz);
  k.gy = (T)gy;
  k.gyz = (T)(gy * iz);
  k.dtdx = (T)dtdx;
  k.dtdy = (T)dtdy;
  k.iz = (T)iz;
  k.dtdxz = (T)(dtdx * iz);
  k.dtdyz = (T)(dtdy * iz);
  k.lx = (T)(limiter_scale<T>(LIM) * fx);
  k.ly = (T)(limiter_scale<T>(LIM) * fy);
  k.tx = (T)(limiter_scale<T>(LIM) * (1.0 - c * dtdx));
  k.ty = (T)(limiter_scale<T>(LIM) * (1.0 - c * dtdy));
  return k;
}

template <typename T, int LIM = WS_LIM_NONE>
__device__ inline Coef<T> make_coef(double c, double Z, double dt, double dx, double dy) {
  Coef<T> k = lane_coef<T, LIM>(c, Z, dt, dx, dy);
  T *f = &k.Z;
  for (int n = 0; n < (int)(sizeof(Coef<T>) / sizeof(T)); ++n) f[n] = uniform(f[n]);
  return k;
}

// A table row read by a whole workgroup, moved to scalar registers word by
// word (the kernel stores to memory, so the compiler cannot use scalar loads
// for it and would otherwise treat its fields as per-lane values).
template <typename S>
__device__ inline S uniform_row(const S &v) {
  static_assert(sizeof(S) % 4 == 0, "row must be whole words");
  uint32_t w[sizeof(S) / 4];
  __builtin_memcpy(w, &v, sizeof(S));
#pragma unroll
  for (int n = 0; n < (int)(sizeof(S) / 4); ++n) w[n] = __builtin_amdgcn_readfirstlane(w[n]);
  S out;
  __builtin_memcpy(&out, w, sizeof(S));
  return out;
}

// Whole-wavefront lane shifts (DPP): shr gives lane l the value of lane l-1,
// shl the value of lane l+1.  Lanes without a source read 0 (never used).
__device__ inline int dpp_shr_i(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ inline int dpp_shl_i(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
__device__ inline double shr(double v) {
  return __hiloint2double(dpp_shr_i(__double2hiint(v)), dpp_shr_i(__double2loint(v)));
}
__device__ inline double shl(double v) {
  return __hiloint2double(dpp_shl_i(__double2hiint(v)), dpp_shl_i(__double2loint(v)));
}
__device__ inline float shr(float v) { return __int_as_float(dpp_shr_i(__float_as_int(v))); }
__device__ inline float shl(float v) { return __int_as_float(dpp_shl_i(__float_as_int(v))); }

// --------------------------------------------------------------------------
// Limiter on unscaled strengths: psi(a, a_up) = phi(a_up/a) a (the limiters
// are positively homogeneous), divided by limiter_scale.  MC:
// minmod(2a, 2a_up, (a + a_up)/2).  FP64: min(4 min(a, a_up), a + a_up), half
// of it, on |a| and on a_up with a's sign taken out of it (a negative minimum:
// the signs differ, and the result is 0); five FP64 and three integer
// instructions, where max(min(2a, 2a_up, m), 0) + min(max(2a, 2a_up, m), 0)
// takes eleven.  The minima are written as instructions because the compiler
// first quiets every operand whose bits were edited (two more each).  FP32:
// the median of (0, x, y) is minmod(x, y), so four instructions instead of
// nine.
// --------------------------------------------------------------------------
__device__ inline double flip(double v, int sign) {
  return __hiloint2double(__double2hiint(v) ^ sign, __double2loint(v));
}
__device__ inline double min_abs(double a, double b) {  // min(|a|, b)
  double r;
  asm("v_min_f64 %0, |%1|, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ inline double min_raw(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ inline double max_zero(double a) {
  double r;
  asm("v_max_f64 %0, %1, 0" : "=v"(r) : "v"(a));
  return r;
}
// 2 ab / (a + b) over its scale, from x = ab > 0 and s = a + b: the hardware
// reciprocal, refined once in FP64 by Newton's iteration, then the quotient
// corrected by its residual.  On 4 million random pairs of strengths in
// 2^+-500 (FP32: 2^+-20) every result is that of the division of ab + ab by
// a + b; past those, where products or quotients are subnormal, some differ in
// their last places.  A general division scales its operands on top of that.
// s is never small here (s >= 2 sqrt(x), and x is at least the smallest
// subnormal), but it may be large: FP32's reciprocal of s > 2^126 would be
// subnormal, which the hardware rounds to 0, so s is divided by 4 first (FP64's
// reciprocals may be subnormal).  Where ab overflowed the division fixup puts
// the infinite quotient in the place of the residual's NaN.  7 instructions in
// FP64 and 6 in FP32 instead of 11 and 10: 48 problems of 128 to 512 cells a
// side in FP64, loops of 40 steps, 31.1 us per step, 33.9 with the division.
__device__ inline double quotient(double x, double s) {
  double r = __builtin_amdgcn_rcp(s);
  r = fma(r, fma(-s, r, 1.0), r);
  const double q = x * r;
  return __builtin_amdgcn_div_fixup(fma(fma(-q, s, x), r, q), s, x);
}
__device__ inline float quotient(float x, float s) {  // 4 x / s
  const float d = 0.25f * s, r = __builtin_amdgcn_rcpf(d), q = x * r;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, d, x), r, q), d, x);
}
template <typename T, int LIM>
__device__ inline T limited(T a, T b) {
  if constexpr (LIM == WS_LIM_NONE) {
    return a;
  } else if constexpr (LIM == WS_LIM_VANLEER) {
    // van Leer, phi(theta) = (theta + |theta|)/(1 + |theta|) with theta = b/a:
    // 0 unless a and b share a sign, then 2ab/(a + b)
    // (the quotient is formed either way: a select costs less than a branch)
    const T ab = a * b, r = quotient(ab, a + b);
    return ab > T(0) ? r : T(0);
  } else if constexpr (sizeof(T) == 4) {
    const float t = __builtin_amdgcn_fmed3f(0.0f, a, b);
    return __builtin_amdgcn_fmed3f(0.0f, a + b, 4.0f * t);
  } else {
    const int sign = __double2hiint(a) & (int)0x80000000;
    const double y = flip(b, sign);
    return flip(max_zero(min_raw(4.0 * min_abs(a, y), fabs(a) + y)), sign);
  }
}

// Strengths at an edge from the jumps of (p, normal velocity).
template <typename T>
__device__ inline T s1(T Z, T dp, T dn) { return fma(Z, dn, -dp); }
template <typename T>
__device__ inline T s2(T Z, T dp, T dn) { return fma(Z, dn, dp); }

// F~ at an x-edge is carried in characteristic form: with the limited
// strengths l1, l2 of the waves -c, +c and the y-fluctuation sums of the cells
// left and right,
//   F~_p = c2 - c1, Z F~_u = c2 + c1, c2 = fx l2 - gy ys_left,
//   c1 = fx l1 - gy ys_right,
// since the transverse waves A-+ of a y-term reach one characteristic each.
// Two multiplies and two FMAs per edge instead of ten operations.
template <typename T>
__device__ inline void ftilde_l(const Coef<T> &k, T l1, T l2, T ys_left, T ys_right, T &c1,
                                T &c2) {
  c1 = fma(-k.gy, ys_right, k.lx * l1);
  c2 = fma(-k.gy, ys_left, k.lx * l2);
}

// G~ at a y-edge, the mirror image: the x-terms of the cells below (lo) and
// above (hi).
template <typename T>
__device__ inline void gtilde_l(const Coef<T> &k, T l1, T l2, T xs_lo, T xs_hi, T &c1, T &c2) {
  c1 = fma(-k.gx, xs_hi, k.ly * l1);
  c2 = fma(-k.gx, xs_lo, k.ly * l2);
}

// F~ from the raw strengths (wave -c takes its upwind neighbour on the right,
// wave +c on the left) and the y-fluctuations of the cells left and right.
template <typename T, int LIM>
__device__ inline void ftilde(const Coef<T> &k, T a1, T a2, T a1_right, T a2_left, T ys_left,
                              T ys_right, T &c1, T &c2) {
  ftilde_l<T>(k, limited<T, LIM>(a1, a1_right), limited<T, LIM>(a2, a2_left), ys_left, ys_right,
              c1, c2);
}

// G~ from the raw strengths and the x-fluctuations of the cells below and above.
template <typename T, int LIM>
__device__ inline void gtilde(const Coef<T> &k, T b1, T b2, T b1_up, T b2_down, T xs_lo, T xs_hi,
                              T &c1, T &c2) {
  gtilde_l<T>(k, limited<T, LIM>(b1, b1_up), limited<T, LIM>(b2, b2_down), xs_lo, xs_hi, c1, c2);
}

// Flux-differencing update of one cell, eq. (2.3), from the strengths that
// enter it (a2 of its left and a1 of its right edge, b2 of its bottom and b1
// of its top edge) and the characteristic F~, G~ of its four edges: the
// fluctuation h (a2 +- a1) and the flux difference meet per characteristic.
template <typename T>
__device__ inline void update(const Coef<T> &k, T p0, T u0, T v0, T a2L, T a1R, T b2B, T b1T,
                              T FL1, T FL2, T FR1, T FR2, T GB1, T GB2, T GT1, T GT2, T &pn, T &un,
                              T &vn) {
  const T x2 = fma(k.h, a2L, FR2 - FL2), x1 = fma(k.h, a1R, FL1 - FR1);
  const T y2 = fma(k.h, b2B, GT2 - GB2), y1 = fma(k.h, b1T, GB1 - GT1);
  pn = p0 - fma(k.dtdy, y2 + y1, k.dtdx * (x2 + x1));  // one rounding at p's size
  un = fma(-k.dtdxz, x2 - x1, u0);
  vn = fma(-k.dtdyz, y2 - y1, v0);
}

// Raw buffer stores (gfx9 buffer resource, no format conversion).  An offset
// at or past the resource's size is dropped by the hardware.  The stores are
// device-scope (cache policy SC1: written through the XCD's L2), so the L2s
// hold no dirty output to write back when the launch ends; the next step's
// workgroups read it on whichever XCD they run.
constexpr int kRawBufferWord3 = 0x00020000;
constexpr unsigned kDropOffset = 0x80000000u;
constexpr int kStoreDeviceScope = 16;  // SC1
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// off: per lane; soff: the same for the wavefront (a scalar register).  Only
// off decides whether a lane's store is dropped.
__device__ inline void bstore(__amdgpu_buffer_rsrc_t r, double v, unsigned off,
                              unsigned soff = 0) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, soff,
                                        kStoreDeviceScope);
}
__device__ inline void bstore(__amdgpu_buffer_rsrc_t r, float v, unsigned off,
                              unsigned soff = 0) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, soff,
                                        kStoreDeviceScope);
}
template <typename T>
__device__ inline T bload(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}

// One row of (p, u, v) of a MARCH segment's column.
template <typename T>
struct Row3 {
  T p, u, v;
};

// MC branch taken: 0 -> 0, 1 -> (a+b)/2, 2 -> 2a, 3 -> 2b; ties -> lowest.
template <typename T>
__device__ inline unsigned mc_branch(T a, T b) {
  const bool same = (a > T(0) && b > T(0)) || (a < T(0) && b < T(0));
  if (!same) return 0u;
  const T m1 = fabs(a + b) * T(0.5), m2 = fabs(a) * T(2), m3 = fabs(b) * T(2);
  if (m1 <= m2 && m1 <= m3) return 1u;
  return (m2 <= m3) ? 2u : 3u;
}

// Padded planes of one patch, indexed by interior coordinates (i, j).
template <typename T>
struct Planes {
  const T *p, *u, *v;
  int64_t ld;
  __device__ T P(int i, int j) const { return p[(int64_t)j * ld + i]; }
  __device__ T U(int i, int j) const { return u[(int64_t)j * ld + i]; }
  __device__ T V(int i, int j) const { return v[(int64_t)j * ld + i]; }
};

struct CellMasks {
  unsigned own;    // bits of the cell's left x-edge (0-3) and bottom y-edge (4-7)
  unsigned right;  // bits 0-3 of the right x-edge (stored at cell i+1)
  unsigned top;    // bits 4-7 of the top y-edge (stored at cell j+1)
};

// DIRECT path: the whole update of one interior cell from its 13-point
// footprint.
template <typename T, int LIM, bool MASKS>
__device__ __attribute__((always_inline)) inline void cell_update(const Planes<T> &q, int i, int j, const Coef<T> &k, T &pn,
                                   T &un, T &vn, CellMasks *mk) {
  const T Z = k.Z;
  // ---- x-edges of row j: LL = i-3/2, L = i-1/2, R = i+1/2, RR = i+3/2
  const T pm2 = q.P(i - 2, j), pm1 = q.P(i - 1, j), p0 = q.P(i, j), pp1 = q.P(i + 1, j),
          pp2 = q.P(i + 2, j);
  const T um2 = q.U(i - 2, j), um1 = q.U(i - 1, j), u0 = q.U(i, j), up1 = q.U(i + 1, j),
          up2 = q.U(i + 2, j);
  const T a2LL = s2(Z, pm1 - pm2, um1 - um2);
  const T a1L = s1(Z, p0 - pm1, u0 - um1), a2L = s2(Z, p0 - pm1, u0 - um1);
  const T a1R = s1(Z, pp1 - p0, up1 - u0), a2R = s2(Z, pp1 - p0, up1 - u0);
  const T a1RR = s1(Z, pp2 - pp1, up2 - up1);
  // ---- y-edges of column i: BB = j-3/2, B = j-1/2, T = j+1/2, TT = j+3/2
  const T qm2 = q.P(i, j - 2), qm1 = q.P(i, j - 1), qp1 = q.P(i, j + 1), qp2 = q.P(i, j + 2);
  const T vm2 = q.V(i, j - 2), vm1 = q.V(i, j - 1), v0 = q.V(i, j), vp1 = q.V(i, j + 1),
          vp2 = q.V(i, j + 2);
  const T b2BB = s2(Z, qm1 - qm2, vm1 - vm2);
  const T b1B = s1(Z, p0 - qm1, v0 - vm1), b2B = s2(Z, p0 - qm1, v0 - vm1);
  const T b1T = s1(Z, qp1 - p0, vp1 - v0), b2T = s2(Z, qp1 - p0, vp1 - v0);
  const T b1TT = s1(Z, qp2 - qp1, vp2 - vp1);

  // ---- first-order fluctuations entering the cell (and its neighbours)
  const T xs0 = a2L + a1R, ys0 = b2B + b1T;
  const T pdm = q.P(i - 1, j - 1), pdp = q.P(i + 1, j - 1);
  const T udm = q.U(i - 1, j - 1), udp = q.U(i + 1, j - 1);
  const T xsm = s2(Z, qm1 - pdm, q.U(i, j - 1) - udm) + s1(Z, pdp - qm1, udp - q.U(i, j - 1));
  const T pum = q.P(i - 1, j + 1), pup = q.P(i + 1, j + 1);
  const T uum = q.U(i - 1, j + 1), uup = q.U(i + 1, j + 1);
  const T xsp = s2(Z, qp1 - pum, q.U(i, j + 1) - uum) + s1(Z, pup - qp1, uup - q.U(i, j + 1));
  const T vlm = q.V(i - 1, j - 1), vl0 = q.V(i - 1, j), vlp = q.V(i - 1, j + 1);
  const T ysl = s2(Z, pm1 - pdm, vl0 - vlm) + s1(Z, pum - pm1, vlp - vl0);
  const T vrm = q.V(i + 1, j - 1), vr0 = q.V(i + 1, j), vrp = q.V(i + 1, j + 1);
  const T ysr = s2(Z, pp1 - pdp, vr0 - vrm) + s1(Z, pup - pp1, vrp - vr0);

  // ---- F~ and G~ on the four edges, then the update
  T FL1, FL2, FR1, FR2, GB1, GB2, GT1, GT2;
  ftilde<T, LIM>(k, a1L, a2L, a1R, a2LL, ysl, ys0, FL1, FL2);
  ftilde<T, LIM>(k, a1R, a2R, a1RR, a2L, ys0, ysr, FR1, FR2);
  gtilde<T, LIM>(k, b1B, b2B, b1T, b2BB, xsm, xs0, GB1, GB2);
  gtilde<T, LIM>(k, b1T, b2T, b1TT, b2B, xs0, xsp, GT1, GT2);
  update<T>(k, p0, u0, v0, a2L, a1R, b2B, b1T, FL1, FL2, FR1, FR2, GB1, GB2, GT1, GT2, pn, un, vn);

  if constexpr (MASKS) {
    mk->own = mc_branch(a1L, a1R) | (mc_branch(a2L, a2LL) << 2) | (mc_branch(b1B, b1T) << 4) |
              (mc_branch(b2B, b2BB) << 6);
    mk->right = mc_branch(a1R, a1RR) | (mc_branch(a2R, a2L) << 2);
    mk->top = (mc_branch(b1T, b1TT) << 4) | (mc_branch(b2T, b2B) << 6);
  }
}

}  // namespace ws
