// gfx950 kernels of lbnlm: the fused pull / velocity-gradient / inlM stress /
// forcing / BGK sweep, its observation variant, the per-channel FP64
// reduction and the step-counter advance.
//
// Layout: ten fields per node (nine populations in the order
// (0,0),(1,0),(0,1),(-1,0),(0,-1),(1,1),(-1,1),(-1,-1),(1,-1), then the
// previous stress trace), stored as tiles of 64 consecutive nodes (row by
// row, x fastest, every channel starting on a tile): a tile holds field 0 of
// its 64 nodes, then field 1, ... (structure of arrays inside a 64-node
// tile, 2.5 KB in FP32). A slot holds the post-collision population of the
// previous step at its source node; the sweep pulls it along the lattice
// velocity (Sec. II.A, Eq. (lbupdate)), or from the same node with the
// opposite velocity where the link crosses a wall (half-way bounce-back,
// Sec. II.B).
//
// One wavefront marches up a strip of rows. It keeps the provisional
// velocity u~ = j/sum_i n_i of three consecutive row blocks in registers, so
// the central differences of Sec. II.C need no LDS: x neighbours come from
// lane moves, y neighbours from the previous/next block.
//  * narrow channels (nx a power of two up to 64) put whole periods into
//    lane groups of nx lanes (sweep_kernel);
//  * channels with nx a multiple of 64 run strips of 64 aligned columns
//    (sweep_wide64_kernel): every load is one aligned 64-lane run of a tile,
//    addressed from a wave-uniform tile base, and the x-shifted pulls are
//    DPP lane shifts of the aligned loads, with the two edge columns loaded
//    separately; this keeps the address arithmetic scalar;
//  * other widths run generic 64-column strips with wrapped lanes
//    (sweep_kernel, WIDE).
// The physics of one node (stencil, stress, forcing, collision) is one
// device function shared by all of them.
#include "lb_internal.h"

namespace lbnlm {
namespace {

#ifndef LB_WG_WAVES
#define LB_WG_WAVES 4
#endif
// Rows of loads in flight per wavefront in the vector sweep. A state that
// stays in the last-level cache (cached stores) runs best with two: the
// third row's registers push the FP32 kernel into accumulator registers
// (76 of them against 11), whose moves cost more than the deeper prefetch
// gains. A state written with nontemporal stores, streamed from HBM, runs
// best with three.
#ifndef LB_VEC_DEPTH
#define LB_VEC_DEPTH 2
#endif
#ifndef LB_VEC_DEPTH_NT
#define LB_VEC_DEPTH_NT 3
#endif

template <typename T>
__device__ __forceinline__ T shfl(T v, int src) {
  return __shfl(v, src, 64);
}

template <typename T>
__device__ __forceinline__ constexpr T weight(int i) {
  return i == 0 ? T(4.0 / 9.0) : (i < 5 ? T(1.0 / 9.0) : T(1.0 / 36.0));
}

template <typename T>
__device__ __forceinline__ T recip(T v) {
  if constexpr (sizeof(T) == 4) return __builtin_amdgcn_rcpf(v);
  return T(1) / v;
}
// Square root: FP32 takes the hardware instruction (1 ulp, like the
// reciprocal above) instead of the correctly rounded sequence.
template <typename T>
__device__ __forceinline__ T root(T v) {
  if constexpr (sizeof(T) == 4) return __builtin_amdgcn_sqrtf(v);
  return sqrt(v);
}

// Lane moves across the whole wavefront: shift_up gives lane i the value of
// lane i-1 (lane 0 gets `edge`), shift_down gives lane i the value of lane
// i+1 (lane 63 gets `edge`).
__device__ __forceinline__ int dpp_shr(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ int dpp_shl(int edge, int v) {
  return __builtin_amdgcn_update_dpp(edge, v, 0x130, 0xf, 0xf, false);
}
template <typename T>
__device__ __forceinline__ T shift_up(T edge, T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, dpp_shr(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v)));
  } else {
    const long long e = __builtin_bit_cast(long long, edge), x = __builtin_bit_cast(long long, v);
    const int lo = dpp_shr((int)e, (int)x), hi = dpp_shr((int)(e >> 32), (int)(x >> 32));
    return __builtin_bit_cast(T, ((long long)hi << 32) | (unsigned int)lo);
  }
}
template <typename T>
__device__ __forceinline__ T shift_down(T edge, T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, dpp_shl(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v)));
  } else {
    const long long e = __builtin_bit_cast(long long, edge), x = __builtin_bit_cast(long long, v);
    const int lo = dpp_shl((int)e, (int)x), hi = dpp_shl((int)(e >> 32), (int)(x >> 32));
    return __builtin_bit_cast(T, ((long long)hi << 32) | (unsigned int)lo);
  }
}
// The same with zero in the end lane (no register to keep for it).
__device__ __forceinline__ int dpp_shr0(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_shl0(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
template <typename T>
__device__ __forceinline__ T shift_in_up(T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, dpp_shr0(__builtin_bit_cast(int, v)));
  } else {
    const long long x = __builtin_bit_cast(long long, v);
    return __builtin_bit_cast(T, ((long long)dpp_shr0((int)(x >> 32)) << 32) | (unsigned int)dpp_shr0((int)x));
  }
}
template <typename T>
__device__ __forceinline__ T shift_in_down(T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, dpp_shl0(__builtin_bit_cast(int, v)));
  } else {
    const long long x = __builtin_bit_cast(long long, v);
    return __builtin_bit_cast(T, ((long long)dpp_shl0((int)(x >> 32)) << 32) | (unsigned int)dpp_shl0((int)x));
  }
}
// A value that is the same in every lane, kept in scalar registers.
__device__ __forceinline__ float uniform(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double uniform(double v) { return v; }
template <typename T>
__device__ __forceinline__ T lane_value(T v, int l) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
  } else {
    const long long x = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)x, l), hi = __builtin_amdgcn_readlane((int)(x >> 32), l);
    return __builtin_bit_cast(T, ((long long)hi << 32) | (unsigned int)lo);
  }
}

// Pulls the nine post-streaming populations of node (x, y), 0 <= y < ny;
// row = index of node (0, y).
// uw6 = u_w/6 of the top wall during the previous step: the populations
// reflected there gained -/+ u_w/6 (a_i c_ix u_w / cs2 for the diagonals).
template <typename T>
__device__ __forceinline__ void pull(const T *__restrict__ A, long long row, int nx, int ny, int x,
                                     int y, T uw6, T f[9]) {
  const int xm = (x == 0) ? nx - 1 : x - 1;
  const int xp = (x == nx - 1) ? 0 : x + 1;
  const long long dn = row - nx, up = row + nx;
  const bool bot = (y == 0), top = (y == ny - 1);
  f[0] = A[slot(0, row + x)];
  f[1] = A[slot(1, row + xm)];
  f[3] = A[slot(3, row + xp)];
  f[2] = A[bot ? slot(4, row + x) : slot(2, dn + x)];
  f[5] = A[bot ? slot(7, row + x) : slot(5, dn + xm)];
  f[6] = A[bot ? slot(8, row + x) : slot(6, dn + xp)];
  f[4] = A[top ? slot(2, row + x) : slot(4, up + x)];
  f[7] = A[top ? slot(5, row + x) : slot(7, up + xp)] - (top ? uw6 : T(0));
  f[8] = A[top ? slot(6, row + x) : slot(8, up + xm)] + (top ? uw6 : T(0));
}

// Slot of population q of node m of a channel relative to the channel's first
// slot (channels start on a tile boundary, so slot(q, off + m) = kPlanes *
// off + lslot(q, m)); 32-bit, for channels of fewer than 2^32 / kPlanes
// nodes.
__device__ __forceinline__ unsigned lslot(int q, unsigned m) {
  return ((m >> 6) * kPlanes + q) * kTile + (m & (kTile - 1));
}

// pull() on a channel's own slots (C = the channel's first slot).
__device__ __forceinline__ void pull_local(const double *__restrict__ C, int nx, int ny, int x, int y, double uw6,
                                           double f[9]) {
  const unsigned row = (unsigned)y * nx;
  const unsigned xm = (x == 0) ? nx - 1 : x - 1, xp = (x == nx - 1) ? 0 : x + 1;
  const unsigned dn = row - nx, up = row + nx;
  const bool bot = (y == 0), top = (y == ny - 1);
  f[0] = C[lslot(0, row + x)];
  f[1] = C[lslot(1, row + xm)];
  f[3] = C[lslot(3, row + xp)];
  f[2] = C[bot ? lslot(4, row + x) : lslot(2, dn + x)];
  f[5] = C[bot ? lslot(7, row + x) : lslot(5, dn + xm)];
  f[6] = C[bot ? lslot(8, row + x) : lslot(6, dn + xp)];
  f[4] = C[top ? lslot(2, row + x) : lslot(4, up + x)];
  f[7] = C[top ? lslot(5, row + x) : lslot(7, up + xp)] - (top ? uw6 : 0.0);
  f[8] = C[top ? lslot(6, row + x) : lslot(8, up + xm)] + (top ? uw6 : 0.0);
}

// Zeroth and first moments of the stored values: sd = sum_i f_i, m = sum_i
// c_i f_i. With SHIFT the stored values are n_i - a_i, so sd is the density
// deviation rho - 1 (kept separate so FP32 does not round it against 1) and
// the momentum is unchanged.
template <typename T>
__device__ __forceinline__ void moments(const T f[9], T &sd, T &mx, T &my) {
  sd = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
  mx = (f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7]);
  my = (f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8]);
}

template <typename T>
struct U2 {
  T x, y;
};

template <typename T>
__device__ __forceinline__ U2<T> shfl2(U2<T> v, int src) {
  return U2<T>{shfl(v.x, src), shfl(v.y, src)};
}

// Provisional velocity u~ = (m + f/2) / sum_i n_i (reading R2 of the design
// notes: the stencil uses the velocity before the flow-induced density).
// With SHIFT the populations are stored relative to the equilibrium at the
// row's reference velocity (ur, 0), mx is the momentum beyond ur and the x
// component returned is u~_x - ur, kept small so that FP32 resolves it.
// No fused multiply-adds here or in the two helpers below: the nodes of a row
// and the halo columns beside a strip take these terms through differently
// shared code and must still round them identically (an x-uniform state
// stays exactly x-uniform).
template <typename T, bool SHIFT>
__device__ __forceinline__ U2<T> u_tilde(T sd, T mx, T my, T fx, T ur) {
#pragma clang fp contract(off)
  const T inv = recip<T>(SHIFT ? T(1) + sd : sd);
  if constexpr (SHIFT) return U2<T>{(mx + T(0.5) * fx - ur * sd) * inv, my * inv};
  return U2<T>{(mx + T(0.5) * fx) * inv, my * inv};
}

// FP32 storage: a population emitted by a node of row y is stored as
// n_i - a_i - E_i(ur_y), E_i(u) = a_i (3 c_ix u + (4.5 c_ix^2 - 1.5) u^2) the
// equilibrium excess at density 1 and velocity (u, 0). A value pulled from
// row y' != y therefore changes by E_i(ur_y') - E_i(ur_y); one reflected at a
// wall comes from the same node's opposite population and changes by
// E_opp(ur_y) - E_i(ur_y) = -6 a_i c_ix ur_y. Both are formed from
// differences, so the small stored values stay exact to FP32 rounding.
template <typename T>
__device__ __forceinline__ T ref_shift(T a, T cx, T us, T ud) {
#pragma clang fp contract(off)
  return a * (us - ud) * (T(3) * cx + (T(4.5) * cx * cx - T(1.5)) * (us + ud));
}
template <typename T>
__device__ __forceinline__ void to_row_reference(T f[9], T urd, T urc, T uru, bool bot, bool top) {
#pragma clang fp contract(off)
  constexpr T w1 = T(1.0 / 9.0), w5 = T(1.0 / 36.0);
  // from below (c_y = +1): 2 (c_x 0), 5 (+1), 6 (-1)
  f[2] += bot ? T(0) : ref_shift(w1, T(0), urd, urc);
  f[5] += bot ? -urc * T(1.0 / 6.0) : ref_shift(w5, T(1), urd, urc);
  f[6] += bot ? urc * T(1.0 / 6.0) : ref_shift(w5, T(-1), urd, urc);
  // from above (c_y = -1): 4 (0), 7 (-1), 8 (+1)
  f[4] += top ? T(0) : ref_shift(w1, T(0), uru, urc);
  f[7] += top ? urc * T(1.0 / 6.0) : ref_shift(w5, T(-1), uru, urc);
  f[8] += top ? -urc * T(1.0 / 6.0) : ref_shift(w5, T(1), uru, urc);
}

// Zou and He's velocity boundary on the top node row (Sec. II.B, the moving
// wall of planar Couette flow): the three populations a node of row ny - 1
// lacks after streaming (c_y = -1: 4, 7, 8) follow from the six it has. No
// flow through the wall gives the density s = f0 + f1 + f3 + 2 (f2 + f5 +
// f6); the normal non-equilibrium part bounces back, f4 = f2; the diagonals
// keep f7 + f8 = f5 + f6 and supply the x momentum for which the provisional
// velocity (m + f/2)/s is the wall's (uw, 0). With SHIFT the values are
// relative to the equilibrium at density 1 and the row reference (ur, 0):
// s is then the density deviation and the momentum the one beyond ur,
// (uw - ur) + s uw - f/2, and the relations between stored values are the
// same (the reference terms of 4 and 2, and of 7 + 8 and 5 + 6, are equal).
template <typename T, bool SHIFT>
__device__ __forceinline__ void zou_he_top(T f[9], T uw, T ur, T fx) {
#pragma clang fp contract(off)
  const T s = (f[0] + f[1] + f[3]) + T(2) * (f[2] + f[5] + f[6]);
  const T m = SHIFT ? (uw - ur) + s * uw - T(0.5) * fx : s * uw - T(0.5) * fx;
  const T d87 = m - ((f[1] - f[3]) + (f[5] - f[6]));
  const T s78 = f[5] + f[6];
  f[4] = f[2];
  f[8] = T(0.5) * (s78 + d87);
  f[7] = T(0.5) * (s78 - d87);
}
// x momentum a node of the top row gave a Zou-He wall in the previous step:
// what it emitted upwards (its own stored 5 and 6, a5 - a6) minus what the
// completion f supplies (f8 - f7). With SHIFT the reduction adds -ur/6 per
// node (the reference terms of both differences).
template <typename T>
__device__ __forceinline__ double zh_drag(T a5, T a6, const T f[9]) {
  return ((double)a5 - (double)a6) - ((double)f[8] - (double)f[7]);
}

// Wave-wide sum over a lane group of width GW (power of two).
template <int GW>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int m = 1; m < GW; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long x = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double read_lane(double v, int lane) {
  const long long x = __builtin_bit_cast(long long, v);
  return __builtin_bit_cast(double, ((long long)__builtin_amdgcn_readlane((int)(x >> 32), lane) << 32) |
                                        (unsigned int)__builtin_amdgcn_readlane((int)x, lane));
}
// The same pairs in the same order for a whole wavefront (all lanes active):
// once the lanes of a quad agree, mirrored lanes hold what xor 4 and xor 8
// would fetch, and four scalar reads replace the last two exchanges. No trip
// through the LDS crossbar per exchange.
template <>
__device__ __forceinline__ double group_sum<64>(double v) {
  v += dpp_move<0xB1>(v);   // quad_perm 1 0 3 2
  v += dpp_move<0x4E>(v);   // quad_perm 2 3 0 1
  v += dpp_move<0x141>(v);  // row_half_mirror
  v += dpp_move<0x140>(v);  // row_mirror
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// a * b, never contracted with what uses it.
template <typename T>
__device__ __forceinline__ T rounded_product(T a, T b) {
#pragma clang fp contract(off)
  return a * b;
}

// a * b + c rounded once.
template <typename T>
__device__ __forceinline__ T fused(T a, T b, T c) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
  return __builtin_fma(a, b, c);
}

// Channel constants in the arithmetic type.
template <typename T>
struct Coef {
  T om, kf, sp, G, inv_tau, inv_gc, lgt;
  bool stress_on;
  __device__ explicit Coef(const ChanDev &c)
      : om(uniform(T(c.omega))), kf(uniform(T(c.kf))), sp(uniform(T(c.sp))), G(uniform(T(c.G))),
        inv_tau(uniform(T(c.inv_tau))), inv_gc(uniform(T(c.inv_gc))), lgt(uniform(T(c.lgt))), stress_on(c.G > 0.0) {}
};

// Instantaneous stress (Eqs. (nlmaxwell), (sigtsum)) for the velocity
// gradient k_ab = d_b u_a: tau_M from the shear rate, then the steady sum
// through the relation it satisfies by Eq. (smalld),
// sigma - tau_M (kappa sigma + sigma kappa^T) = G tau_M D, solved in closed
// form (Cramer) for (sigma_xx, sigma_xy, sigma_yy). The relaxation rate
// vanishes only for tau = inf and D = 0; any finite tau_M then gives the
// right sigma = 0 (every right-hand side is zero), so tau_M = 1 is taken
// there instead of a branch.
template <typename T>
__device__ __forceinline__ void inlm_stress(T kxx, T kxy, T kyx, T kyy, const Coef<T> &q, T &sxx, T &sxy,
                                            T &syy) {
  const T Dxx = T(2) * kxx, Dxy = kxy + kyx, Dyy = T(2) * kyy;
  const T II = T(0.5) * (Dxx * Dxx + T(2) * Dxy * Dxy + Dyy * Dyy);
  const T r0 = q.inv_tau + root(II) * q.inv_gc;
  const T rate = r0 > T(0) ? r0 : T(1);
  {
    const T tM = recip<T>(rate);
    const T ka = tM * kxx, kb = tM * kxy, kc = tM * kyx, kd = tM * kyy;
    const T gt = q.G * tM;
    const T r1 = gt * Dxx, r2 = gt * Dxy, r3 = gt * Dyy;
    const T m11 = T(1) - T(2) * ka, m12 = T(-2) * kb, m21 = -kc;
    const T m22 = T(1) - ka - kd, m23 = -kb, m32 = T(-2) * kc, m33 = T(1) - T(2) * kd;
    const T c11 = m22 * m33 - m23 * m32;
    const T det = m11 * c11 - m12 * m21 * m33;
    const T idet = recip<T>(det);
    const T e2 = r2 * m33 - m23 * r3;
    sxx = (r1 * c11 - m12 * e2) * idet;
    sxy = (m11 * e2 - r1 * m21 * m33) * idet;
    syy = (m11 * (m22 * r3 - r2 * m32) - m12 * m21 * r3 + r1 * m21 * m32) * idet;
  }
}

// Everything that happens at one node once its populations and the stencil
// velocities are known: kappa (Sec. II.C), the inlM stress (Eqs.
// (nlmaxwell), (sigtsum)), the flow-induced density change (Eq. (rhoplus)),
// the density and velocity of Eq. (rhoj), and either the post-collision
// populations (equilibrium, forcing of Eq. (bodyforce), BGK) or the
// observables of the node.
// With SHIFT, f are stored relative to the row's reference (ur, 0), mx is
// the momentum beyond ur, the velocities lf, rt, dn, up carry u~_x minus
// their own row's reference, and kref = (ur_above - ur_below)/2 restores the
// reference's share of d_y u_x; the outputs are stored relative to ur.
// With VE the stress is the time-integrated one: sp holds (xx, xy, yy) of the
// previous step and sn receives those of this step.
template <typename T, bool SHIFT, bool OBS, bool VE>
__device__ __forceinline__ void node_update(const T f[9], T sd, T mx, T my, T Pc, T fx, U2<T> lf,
                                            U2<T> rt, U2<T> dn, U2<T> up, T ur, T kref, const Coef<T> &q,
                                            int nnp, const T sp[3], T sn[3], T out[9], T &trT_out,
                                            double obs[OF_COUNT]) {
  // velocity gradient kappa_ab = d_b u_a
  const T kxx = T(0.5) * (rt.x - lf.x);
  const T kxy = T(0.5) * (up.x - dn.x) + kref;
  const T kyx = T(0.5) * (rt.y - lf.y);
  const T kyy = T(0.5) * (up.y - dn.y);

  // tau_M of Eq. (nlmaxwell), then the steady series of Eq. (sigtsum) through
  // the relation it satisfies by Eq. (smalld),
  // sigma - tau_M (kappa sigma + sigma kappa^T) = G tau_M D, solved in closed
  // form (Cramer) for (sigma_xx, sigma_xy, sigma_yy).
  const T Dxx = T(2) * kxx, Dxy = kxy + kyx, Dyy = T(2) * kyy;
  T sxx = T(0), sxy = T(0), syy = T(0);
  if constexpr (VE) {
    // Time-integrated stress, Eq. (gkder) with d_t G = -G / tau_M(t): one
    // step with the upper-convected terms and the source explicit and the
    // relaxation implicit, sigma' = [sigma + kappa sigma + sigma kappa^T +
    // G D] / (1 + 1/tau_M), written as sigma plus its increment so that FP32
    // rounds only the increment.
    // (explicit fused operations: sums of two products, which the compiler
    // may contract either way, round alike in every kernel)
    const T II = T(0.5) * (Dxx * Dxx + T(2) * Dxy * Dxy + Dyy * Dyy);
    const T rate = q.inv_tau + root(II) * q.inv_gc;  // 1 / tau_M
    const T d = recip<T>(T(1) + rate);
    const T cxx = fused(kxx, sp[0], rounded_product(kxy, sp[1]));
    const T cyy = fused(kyx, sp[1], rounded_product(kyy, sp[2]));
    const T cxy = fused(kxx, sp[1], fused(kxy, sp[2], fused(kyx, sp[0], rounded_product(kyy, sp[1]))));
    sxx = fused(fused(-rate, sp[0], fused(q.G, Dxx, rounded_product(T(2), cxx))), d, sp[0]);
    sxy = fused(fused(-rate, sp[1], fused(q.G, Dxy, cxy)), d, sp[1]);
    syy = fused(fused(-rate, sp[2], fused(q.G, Dyy, rounded_product(T(2), cyy))), d, sp[2]);
    sn[0] = sxx;
    sn[1] = sxy;
    sn[2] = syy;
  } else if (q.stress_on) {
    inlm_stress<T>(kxx, kxy, kyx, kyy, q, sxx, sxy, syy);
  }
  // non-Newtonian stress carried by the forcing (viscosity split)
  const T Txx = sxx - q.lgt * Dxx, Txy = sxy - q.lgt * Dxy, Tyy = syy - q.lgt * Dyy;
  const T trT = Txx + Tyy;
  const T Sxx = T(0.5) * (Txx - Tyy);  // traceless part; Sbar_yy = -Sxx
  // Eq. (rhoplus): r = dt d(delta rho)/dt with delta rho = -tr Sigma^nN /(cs2 d)
  const T rr = nnp ? T(-1.5) * (trT - Pc) : T(0);

  const T jx = mx + T(0.5) * fx, jy = my;
  // Eq. (rhoj): the equilibrium density is sum (n* + n)/2 = s + r/2, carried
  // as its deviation from 1 in the shifted storage
  const T sdev = SHIFT ? sd : sd - T(1);
  const T rho_dev = sdev + T(0.5) * rr;
  const T rho_e = SHIFT ? T(1) + rho_dev : sd + T(0.5) * rr;
  const T irho = recip<T>(rho_e);
  // SHIFT: jx is j_x - ur, so u_x - ur = (jx - ur rho_dev) / rho_e
  const T dux = (SHIFT ? jx - ur * rho_dev : jx) * irho;
  const T ux = SHIFT ? ur + dux : dux, uy = jy * irho;
  trT_out = trT;

  if constexpr (OBS) {
    // SHIFT: u_x - ur and j_x - ur; the reduction adds ur once per row, so
    // that row sums of equal values stay exact in any summation order
    obs[OF_UX] = SHIFT ? (double)dux : (double)ux;
    obs[OF_UY] = (double)uy;
    obs[OF_SXX] = (double)sxx;
    obs[OF_SXY] = (double)sxy;
    obs[OF_SYY] = (double)syy;
    obs[OF_RHOE_DEV] = (double)rho_dev;
    obs[OF_MASS_DEV] = (double)sdev + (nnp ? 1.5 * (double)Pc : 0.0);
    obs[OF_MOMX] = (double)mx;
    obs[OF_KXY] = (double)kxy;
    obs[OF_TRT] = (double)trT;
    obs[OF_KXX] = (double)kxx;
  } else {
    // equilibrium, forcing of Eq. (bodyforce) and BGK collision:
    // n*_i = (1 - om) n_i + om n^eq_i + F_i. For a pair of opposite
    // velocities c_i = -c_j the parts even in c (constant, (c.u)^2, (c.u)(c.f),
    // the stress term) are shared and the odd parts ((c.u), (c.f)) change sign.
    const T usq = ux * ux + uy * uy;
    const T uf = ux * fx;
    const T K0 = q.kf * (rr + T(1.5) * rr * usq - T(3) * uf);
    const T om1 = T(1) - q.om;
    // Equilibrium excess n^eq_i - a_i (- E_i(ur) with SHIFT). SHIFT expands it
    // around the reference so that only small differences are rounded:
    // a_i [rho_dev (1 + 3 cu + 4.5 cu^2 - 1.5 u^2) + 3 c.du + 4.5 (c.du)(c.(u+ur))
    //      - 1.5 du.(u + ur)], du = u - (ur, 0); with ur = 0 it is the plain
    // shifted form.
    T C0, Acu2, Bcu;
    if constexpr (SHIFT) {
      const T mix = dux * (ux + ur) + uy * uy;  // du.(u + ur)
      C0 = q.om * (rho_dev * (T(1) - T(1.5) * usq) - T(1.5) * mix) + K0;
      Acu2 = T(4.5) * (q.om * rho_dev - q.kf * rr);
      Bcu = T(3) * q.om * rho_dev;
    } else {
      C0 = q.om * rho_e * (T(1) - T(1.5) * usq) + K0;  // constant part
      Acu2 = T(4.5) * (q.om * rho_e - q.kf * rr);      // coefficient of (c.u)^2
      Bcu = T(3) * q.om * rho_e;                       // coefficient of (c.u), odd
    }
    const T E4 = SHIFT ? T(4.5) * q.om : T(0);  // (c.du)(c.(u+ur)), even
    const T B3 = SHIFT ? T(3) * q.om : T(0);    // c.du, odd
    // rounded by itself, also where it is not constant over a kernel's loop (a
    // node's result does not depend on the kernel it falls to)
    const T Ccf = rounded_product(T(3) * q.kf, fx);  // 3 kf (c.f) for c_x = 1, odd
    const T Dcf = T(9) * q.kf * fx;             // 9 kf (c.u)(c.f) for c_x = 1, even
    const T spS = q.sp * Sxx, spT = T(2) * q.sp * Txy;
    const T usx = ux + ur;                      // (u + ur)_x (ur = 0 without SHIFT)
    constexpr T w0 = weight<T>(0), w1 = weight<T>(1), w5 = weight<T>(5);
    out[0] = om1 * f[0] + w0 * C0;
    {  // (1,0) and (-1,0): c.u = ux, c.f = fx, stress term Sxx
      const T cu = ux, cdu = dux, cs = usx;
      const T ev = w1 * (C0 + Acu2 * cu * cu + E4 * cdu * cs + spS + Dcf * cu);
      const T od = w1 * (Bcu * cu + B3 * cdu + Ccf);
      out[1] = om1 * f[1] + ev + od;
      out[3] = om1 * f[3] + ev - od;
    }
    {  // (0,1) and (0,-1): c.u = uy, c.f = 0, stress term -Sxx
      const T cu = uy;
      const T ev = w1 * (C0 + Acu2 * cu * cu + E4 * cu * cu - spS);
      const T od = w1 * (Bcu * cu + B3 * cu);
      out[2] = om1 * f[2] + ev + od;
      out[4] = om1 * f[4] + ev - od;
    }
    {  // (1,1) and (-1,-1): c.u = ux + uy, c.f = fx, stress term 2 Sxy
      const T cu = ux + uy, cdu = dux + uy, cs = usx + uy;
      const T ev = w5 * (C0 + Acu2 * cu * cu + E4 * cdu * cs + spT + Dcf * cu);
      const T od = w5 * (Bcu * cu + B3 * cdu + Ccf);
      out[5] = om1 * f[5] + ev + od;
      out[7] = om1 * f[7] + ev - od;
    }
    {  // (-1,1) and (1,-1): c.u = uy - ux, c.f = -fx, stress term -2 Sxy
      const T cu = uy - ux, cdu = uy - dux, cs = uy - usx;
      const T ev = w5 * (C0 + Acu2 * cu * cu + E4 * cdu * cs - spT - Dcf * cu);
      const T od = w5 * (Bcu * cu + B3 * cdu - Ccf);
      out[6] = om1 * f[6] + ev + od;
      out[8] = om1 * f[8] + ev - od;
    }
  }
}

// Momentum handed to the walls in the previous step: the reflected
// populations sit in the wall rows with the opposite velocity.
// With the FP32 reference ur the pulled values are n_i - a_i - E_i(ur), and
// n6 - n5 = f6 - f5 - ur/6, n7 - n8 = f7 - f8 - ur/6; the -ur/3 of each wall
// node is added per row in the reduction.
// At a Zou-He top wall the top row's share is ztop (zh_drag).
template <typename T>
__device__ __forceinline__ double wall_drag(const T f[9], int y, int ny, T uw6, bool zh, double ztop) {
  double d = 0.0;
  if (y == 0) d += 2.0 * ((double)f[6] - (double)f[5]);
  // a moving top wall also received the momentum its reflection added
  if (y == ny - 1) d += zh ? ztop : 2.0 * ((double)f[7] - (double)f[8]) + 2.0 * (double)uw6;
  return d;
}

// Workgroup w of n runs on XCD w % 8; the work item it takes, such that
// each XCD takes a contiguous range of the n items (neighbouring items then
// share their halo rows through that XCD's L2).
__device__ __forceinline__ int xcd_item(int w, int n) {
  const int q = n >> 3, rem = n & 7, j = w & 7;
  return j * q + (j < rem ? j : rem) + (w >> 3);
}
// The same ranges, with back set each taken from its end: a launch that goes
// over what the last one wrote in reverse, every XCD over its own part (what
// fits the L2s is then found there: 1920 x 73 FP64 with the stress as a force
// 9.2 us per step, with the whole list reversed 13.8).
__device__ __forceinline__ int xcd_item(int w, int n, bool back) {
  const int q = n >> 3, rem = n & 7, j = w & 7;
  const int first = j * q + (j < rem ? j : rem), len = q + (j < rem), at = w >> 3;
  return first + (back ? len - 1 - at : at);
}

__device__ __forceinline__ int strip_index(const SweepArgs &a) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  return xcd_item(blockIdx.x, a.n_wg) * LB_WG_WAVES + wave;
}

template <typename T, bool SHIFT, int TXW, bool WIDE, bool OBS, bool VE>
__global__ void __launch_bounds__(64 * LB_WG_WAVES) sweep_kernel(SweepArgs a) {
  constexpr int TYW = 64 / TXW;
  const int lane = threadIdx.x & 63;
  const int sidx = strip_index(a);
  if (sidx >= a.n_strips) return;
  const Strip st = a.strips[sidx];
  const ChanDev c = a.ch[st.ch];
  const T *__restrict__ A = static_cast<const T *>(a.A);
  T *__restrict__ B = static_cast<T *>(a.B);
  const int nx = c.nx, ny = c.ny;
  const long long t = c.t + a.k;
  const T fx = (t < c.t_startup) ? T(c.g) : T(0);
  // moving top wall: its velocity at step t (stencil ghost) and u_w/6 of step
  // t - 1, whose reflected links step t pulls
  const T uwg = (t < c.t_startup) ? T(c.uw) : T(0);
  const T uw6 = (!c.zh && t >= 1 && t - 1 < c.t_startup) ? T(c.uw / 6.0) : T(0);
  const Coef<T> q(c);

  int lx, ly, x, hx = 0;
  bool colok;
  if (WIDE) {
    // 64 columns from x0; lanes past the end of the channel wrap onto valid
    // columns and only supply neighbours
    lx = lane;
    ly = 0;
    const int xr = st.x0 + lane;
    x = xr % nx;
    colok = xr < nx;
    // x halo: even lanes pull the column left of the strip, odd lanes the
    // column right of it
    hx = (lane & 1) ? (st.x0 + 64) % nx : (st.x0 - 1 + nx) % nx;
  } else {
    lx = lane & (TXW - 1);
    ly = lane / TXW;
    x = lx;
    colok = true;
  }
  const int left_src = WIDE ? (lane == 0 ? 0 : lane - 1) : ly * TXW + ((lx + TXW - 1) & (TXW - 1));
  const int right_src = WIDE ? (lane == 63 ? 63 : lane + 1) : ly * TXW + ((lx + 1) & (TXW - 1));
  const long long base = c.off;

  auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
  // FP32 reference velocity of row y (0 in FP64)
  auto ref = [&](int y) -> T {
    if constexpr (SHIFT) return a.uref[c.row_off + clampy(y)];
    return T(0);
  };
  // a row's loads (the pulled populations and P), then the populations
  // relative to that row's reference ur: split so that the loads of several
  // rows can be in flight before any is used
  struct RowLoad {
    T f[9], P;
  };
  auto load_row = [&](int y, RowLoad &L) {
    const int yc = clampy(y);
    const long long row = base + (long long)yc * nx;
    pull<T>(A, row, nx, ny, x, yc, uw6, L.f);
    L.P = A[slot(9, row + x)];
  };
  auto finish_row = [&](int y, const RowLoad &L, T f[9], T &Pv, T &ur) {
    const int yc = clampy(y);
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = L.f[i];
    Pv = L.P;
    ur = ref(yc);
    if constexpr (SHIFT) to_row_reference(f, ref(yc - 1), ur, ref(yc + 1), yc == 0, yc == ny - 1);
    if (c.zh && yc == ny - 1) zou_he_top<T, SHIFT>(f, uwg, ur, fx);
  };
  auto halo_u = [&](int y) -> U2<T> {
    const int yc = clampy(y);
    T f[9], sd, mx, my;
    pull<T>(A, base + (long long)yc * nx, nx, ny, hx, yc, uw6, f);
    const T ur = ref(yc);
    if constexpr (SHIFT) to_row_reference(f, ref(yc - 1), ur, ref(yc + 1), yc == 0, yc == ny - 1);
    if (c.zh && yc == ny - 1) zou_he_top<T, SHIFT>(f, uwg, ur, fx);
    moments<T>(f, sd, mx, my);
    return u_tilde<T, SHIFT>(sd, mx, my, fx, ur);
  };
  // viscoelastic model: the stress of the previous step at (x, y)
  const T *__restrict__ SA = static_cast<const T *>(a.SA);
  T *__restrict__ SB = static_cast<T *>(a.SB);
  auto load_sigma = [&](int y, T sg[3]) {
    if constexpr (VE) {
      const long long o = base + (long long)clampy(y) * nx + x;
#pragma unroll
      for (int p = 0; p < 3; ++p) sg[p] = SA[sslot(p, o)];
    } else {
      sg[0] = sg[1] = sg[2] = T(0);
    }
  };

  T fc[9], fn[9], Pc, Pn, urc, urn, sgc[3], sgn[3];
  U2<T> uPrev, uCur, uNext, uhCur = {T(0), T(0)}, uhNext = {T(0), T(0)};
  // the loads of the row groups below the strip, at its start and after it
  // (the first one the loop takes) go out together
  RowLoad Lp, Lc, Ln;
  load_row(st.y0 - TYW + ly, Lp);
  load_row(st.y0 + ly, Lc);
  load_row(st.y0 + TYW + ly, Ln);
  {
    T ftmp[9], Ptmp, sd, mx, my, urp;
    finish_row(st.y0 - TYW + ly, Lp, ftmp, Ptmp, urp);
    moments<T>(ftmp, sd, mx, my);
    uPrev = u_tilde<T, SHIFT>(sd, mx, my, fx, urp);
  }
  T sdc, mxc, myc;
  finish_row(st.y0 + ly, Lc, fc, Pc, urc);
  load_sigma(st.y0 + ly, sgc);
  moments<T>(fc, sdc, mxc, myc);
  uCur = u_tilde<T, SHIFT>(sdc, mxc, myc, fx, urc);
  if (WIDE) uhCur = halo_u(st.y0);

#pragma unroll 1
  for (int yb = st.y0; yb < st.y1; yb += TYW) {
    T sdn, mxn, myn;
    if (yb != st.y0) load_row(yb + TYW + ly, Ln);
    finish_row(yb + TYW + ly, Ln, fn, Pn, urn);
    load_sigma(yb + TYW + ly, sgn);
    if (WIDE) uhNext = halo_u(yb + TYW);
    moments<T>(fn, sdn, mxn, myn);
    uNext = u_tilde<T, SHIFT>(sdn, mxn, myn, fx, urn);
    const int y = yb + ly;

    U2<T> dn, up;
    if (TYW == 1) {
      dn = uPrev;
      up = uNext;
    } else {
      const U2<T> dc = shfl2(uCur, lane - TXW < 0 ? 0 : lane - TXW);
      const U2<T> dp = shfl2(uPrev, lane + (TYW - 1) * TXW > 63 ? 63 : lane + (TYW - 1) * TXW);
      const U2<T> uc = shfl2(uCur, lane + TXW > 63 ? 63 : lane + TXW);
      const U2<T> un = shfl2(uNext, lane - (TYW - 1) * TXW < 0 ? 0 : lane - (TYW - 1) * TXW);
      dn = (ly > 0) ? dc : dp;
      up = (ly < TYW - 1) ? uc : un;
    }
    U2<T> lf = shfl2(uCur, left_src);
    U2<T> rt = shfl2(uCur, right_src);
    if (WIDE) {
      const U2<T> hl = shfl2(uhCur, 0), hr = shfl2(uhCur, 1);
      if (lane == 0) lf = hl;
      if (lane == 63) rt = hr;
    }
    // no-slip ghosts behind the half-way walls, u~(-1) = -u~(0) and
    // u~(ny) = 2 u_w - u~(ny-1), or behind a Zou-He node wall
    // u~(ny) = 2 u_w - u~(ny-2); with SHIFT the ghost rows take the mirrored
    // references -ur and 2 u_w - ur, so their deltas are just mirrored
    if (y == 0) dn = U2<T>{-uCur.x, -uCur.y};
    if (y == ny - 1) {
      const U2<T> m = c.zh ? dn : uCur;
      up = U2<T>{(SHIFT ? T(0) : T(2) * uwg) - m.x, -m.y};
    }
    T kref = T(0);
    if constexpr (SHIFT) {
      const T urd = (y == 0) ? -urc : ref(y - 1);
      const T uru = (y >= ny - 1) ? T(2) * uwg - (c.zh ? urd : urc) : ref(y + 1);
      kref = T(0.5) * (uru - urd);
    }

    // Every lane computes; only valid lanes store. Lanes past the strip or
    // outside the channel read clamped rows and their results are dropped.
    const bool ok = (y < st.y1) && colok;
    T out[9], trT, sg[3];
    double obs[OF_COUNT];
    node_update<T, SHIFT, OBS, VE>(fc, sdc, mxc, myc, Pc, fx, lf, rt, dn, up, urc, kref, q, c.nnp, sgc, sg, out,
                                   trT, obs);
    if constexpr (OBS) {
      double ztop = 0.0;
      if (c.zh && y == ny - 1) {
        const long long o = base + (long long)y * nx + x;
        ztop = zh_drag<T>(A[slot(5, o)], A[slot(6, o)], fc);
      }
      obs[OF_DRAG] = wall_drag<T>(fc, y, ny, uw6, c.zh, ztop);
      constexpr int GW = WIDE ? 64 : TXW;
#pragma unroll
      for (int f = 0; f < OF_COUNT; ++f) obs[f] = group_sum<GW>(ok ? obs[f] : 0.0);
      const bool writer = WIDE ? (lane == 0) : (lx == 0);
      if (writer && y < st.y1) {
        const long long pr = (long long)c.poff + (long long)y * c.nxs + (WIDE ? st.x0 / 64 : 0);
        double *dst = a.part + pr * OF_COUNT;
#pragma unroll
        for (int f = 0; f < OF_COUNT; ++f) dst[f] = obs[f];
      }
    } else {
      if (ok) {
        const long long o = base + (long long)y * nx + x;
#pragma unroll
        for (int i = 0; i < 9; ++i) B[slot(i, o)] = out[i];
        B[slot(9, o)] = trT;
        if constexpr (VE) {
#pragma unroll
          for (int p = 0; p < 3; ++p) SB[sslot(p, o)] = sg[p];
        }
      }
    }

    uPrev = uCur;
    uCur = uNext;
    uhCur = uhNext;
    urc = urn;
#pragma unroll
    for (int p = 0; p < 3; ++p) sgc[p] = sgn[p];
#pragma unroll
    for (int i = 0; i < 9; ++i) fc[i] = fn[i];
    Pc = Pn;
    sdc = sdn;
    mxc = mxn;
    myc = myn;
  }
}

// Two steps per launch for the narrow widths of 32 and 64 columns (a row fits
// TXW = nx lanes and a wavefront holds TYW = 64 / nx rows), for the
// instantaneous model. A workgroup of two wavefronts takes the strip of rows
// [y0, y1) of one channel through steps t and t+1 with the narrow sweep's
// row machine in both:
//  * wavefront 0 (stage A, step t) marches groups of TYW rows from
//    max(y0 - 2, 0) to min(y1 + 2, ny), reading the state, and writes each
//    group's post-collision populations and trace into a ring of groups in
//    LDS;
//  * wavefront 1 (stage B, step t+1) marches the groups of [y0, y1), pulling
//    from the ring (any row of the last few groups, by index), and stores.
// A row of the channel is whole in one group, so no column beyond it is
// needed. Stage B runs L iterations behind stage A (4 and 5 where a group
// holds 2 and 1 rows), or sooner at the end of the strip, so that
// every group it reads is in the ring; one barrier per iteration orders the
// ring's writes and reads. Per node the arithmetic is the narrow sweep's.
//
// For the lattices that do not step in boxes (sweep_block_kernel): FP32 beyond
// about a million nodes (64 x 65536 73 us per step against 92), FP64 beyond a
// quarter of that. Narrower channels always step in boxes (or, beyond the nodes
// boxes address, one step per launch).
constexpr int kN2Ring = 8;  // groups in the ring
template <typename T, bool SHIFT, int TXW>
__global__ void __launch_bounds__(128) sweep_narrow2_kernel(SweepArgs a) {
  constexpr int TYW = 64 / TXW;
  constexpr int L = 3 + 2 / TYW;  // stage B's lag in iterations
  static_assert(L <= kN2Ring, "the ring must hold the groups stage B reads");
  __shared__ T ring[kN2Ring][kPlanes][64];
  const int lane = threadIdx.x & 63;
  const bool isA = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0;
  const int sidx = xcd_item(blockIdx.x, a.n_wg);
  if (sidx >= a.n_strips) return;  // the whole workgroup, before any barrier
  const Strip st = a.strips[sidx];
  const ChanDev c = a.ch[st.ch];
  const T *__restrict__ A = static_cast<const T *>(a.A);
  T *__restrict__ B = static_cast<T *>(a.B);
  const int nx = c.nx, ny = c.ny;
  const long long t = c.t + a.k, ts = isA ? t : t + 1;  // this stage's step
  const T fx = (ts < c.t_startup) ? T(c.g) : T(0);
  const T uwg = (ts < c.t_startup) ? T(c.uw) : T(0);
  const T uw6 = (!c.zh && ts >= 1 && ts - 1 < c.t_startup) ? T(c.uw / 6.0) : T(0);
  const Coef<T> q(c);
  const int lx = lane & (TXW - 1), ly = lane / TXW, x = lx;
  const int left_src = ly * TXW + ((lx + TXW - 1) & (TXW - 1));
  const int right_src = ly * TXW + ((lx + 1) & (TXW - 1));
  const long long base = c.off;
  auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
  auto ref = [&](int y) -> T {
    if constexpr (SHIFT) return a.uref[c.row_off + clampy(y)];
    return T(0);
  };
  // the groups of the two stages
  const int yA0 = st.y0 - 2 < 0 ? 0 : st.y0 - 2, yA1 = st.y1 + 2 > ny ? ny : st.y1 + 2;
  const int nA = (yA1 - yA0 + TYW - 1) / TYW, nB = (st.y1 - st.y0 + TYW - 1) / TYW;
  const int ys = isA ? yA0 : st.y0;  // this stage's first group

  // stage A's source: the state (the narrow sweep's pull)
  auto pull_mem = [&](int y, T f[9], T &Pv) {
    const int yc = clampy(y);
    const long long row = base + (long long)yc * nx;
    pull<T>(A, row, nx, ny, x, yc, uw6, f);
    Pv = A[slot(9, row + x)];
  };
  // stage B's source: row r, column col of step t from the ring (rows
  // outside stage A's range read a row inside it; their values are unused)
  auto at = [&](int r, int p, int col) -> T {
    const int rr = (r < yA0 ? yA0 : (r >= yA1 ? yA1 - 1 : r)) - yA0;
    const int g = rr / TYW;
    return ring[g & (kN2Ring - 1)][p][(rr - g * TYW) * TXW + col];
  };
  auto pull_ring = [&](int y, T f[9], T &Pv) {
    const int yc = clampy(y);
    const bool bot = (yc == 0), top = (yc == ny - 1);
    const int xm = (x == 0) ? nx - 1 : x - 1, xp = (x == nx - 1) ? 0 : x + 1;
    f[0] = at(yc, 0, x);
    f[1] = at(yc, 1, xm);
    f[3] = at(yc, 3, xp);
    f[2] = bot ? at(yc, 4, x) : at(yc - 1, 2, x);
    f[5] = bot ? at(yc, 7, x) : at(yc - 1, 5, xm);
    f[6] = bot ? at(yc, 8, x) : at(yc - 1, 6, xp);
    f[4] = top ? at(yc, 2, x) : at(yc + 1, 4, x);
    f[7] = top ? at(yc, 5, x) - uw6 : at(yc + 1, 7, xp);
    f[8] = top ? at(yc, 6, x) + uw6 : at(yc + 1, 8, xm);
    Pv = at(yc, 9, x);
  };
  // a row's pulled populations and P (split from the rest so that stage A
  // can have the loads of several groups in flight), then the populations
  // relative to the row's reference, moments and u~
  struct RowLoad {
    T f[9], P;
  };
  auto fetch = [&](int y, RowLoad &L) {
    if (isA) pull_mem(y, L.f, L.P);
    else pull_ring(y, L.f, L.P);
  };
  auto finish = [&](int y, const RowLoad &L, T f[9], T &Pv, T &ur, T &sd, T &mx, T &my, U2<T> &u) {
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = L.f[i];
    Pv = L.P;
    const int yc = clampy(y);
    ur = ref(yc);
    if constexpr (SHIFT) to_row_reference(f, ref(yc - 1), ur, ref(yc + 1), yc == 0, yc == ny - 1);
    if (c.zh && yc == ny - 1) zou_he_top<T, SHIFT>(f, uwg, ur, fx);
    moments<T>(f, sd, mx, my);
    u = u_tilde<T, SHIFT>(sd, mx, my, fx, ur);
  };

  T fc[9], Pc, urc, sdc, mxc, myc;
  U2<T> uPrev, uCur;
  RowLoad Ln;
  // the group below this stage's first and the first; stage A also fetches
  // the second (stage B cannot yet: stage A has not written all its rows)
  auto start = [&]() {
    RowLoad Lp, Lc;
    fetch(ys - TYW + ly, Lp);
    fetch(ys + ly, Lc);
    if (isA) fetch(ys + TYW + ly, Ln);
    T ftmp[9], Ptmp, urp, sd, mx, my;
    finish(ys - TYW + ly, Lp, ftmp, Ptmp, urp, sd, mx, my, uPrev);
    finish(ys + ly, Lc, fc, Pc, urc, sdc, mxc, myc, uCur);
  };
  // group g of this stage: fetch and finish the next group, update this one
  auto group = [&](int g) {
    const int yb = ys + g * TYW;
    T fn[9], Pn, urn, sdn, mxn, myn;
    U2<T> uNext;
    if (g != 0 || !isA) fetch(yb + TYW + ly, Ln);
    finish(yb + TYW + ly, Ln, fn, Pn, urn, sdn, mxn, myn, uNext);
    const int y = yb + ly;
    U2<T> dn, up;
    if (TYW == 1) {
      dn = uPrev;
      up = uNext;
    } else {
      const U2<T> dc = shfl2(uCur, lane - TXW < 0 ? 0 : lane - TXW);
      const U2<T> dp = shfl2(uPrev, lane + (TYW - 1) * TXW > 63 ? 63 : lane + (TYW - 1) * TXW);
      const U2<T> uc = shfl2(uCur, lane + TXW > 63 ? 63 : lane + TXW);
      const U2<T> un = shfl2(uNext, lane - (TYW - 1) * TXW < 0 ? 0 : lane - (TYW - 1) * TXW);
      dn = (ly > 0) ? dc : dp;
      up = (ly < TYW - 1) ? uc : un;
    }
    const U2<T> lf = shfl2(uCur, left_src), rt = shfl2(uCur, right_src);
    if (y == 0) dn = U2<T>{-uCur.x, -uCur.y};
    if (y == ny - 1) {
      const U2<T> m = c.zh ? dn : uCur;
      up = U2<T>{(SHIFT ? T(0) : T(2) * uwg) - m.x, -m.y};
    }
    T kref = T(0);
    if constexpr (SHIFT) {
      const T urd = (y == 0) ? -urc : ref(y - 1);
      const T uru = (y >= ny - 1) ? T(2) * uwg - (c.zh ? urd : urc) : ref(y + 1);
      kref = T(0.5) * (uru - urd);
    }
    T out[9], trT, sg[3];
    const T sp[3] = {T(0), T(0), T(0)};
    double obs[OF_COUNT];
    node_update<T, SHIFT, false, false>(fc, sdc, mxc, myc, Pc, fx, lf, rt, dn, up, urc, kref, q, c.nnp, sp, sg, out,
                                        trT, obs);
    if (isA) {
      // the whole group goes into the ring (rows past stage A's range are
      // never read)
      T *slotp = &ring[g & (kN2Ring - 1)][0][0];
#pragma unroll
      for (int i = 0; i < 9; ++i) slotp[i * 64 + lane] = out[i];
      slotp[9 * 64 + lane] = trT;
    } else if (y < st.y1 && y < ny) {
      const long long o = base + (long long)y * nx + x;
#pragma unroll
      for (int i = 0; i < 9; ++i) B[slot(i, o)] = out[i];
      B[slot(9, o)] = trT;
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) fc[i] = fn[i];
    Pc = Pn;
    urc = urn;
    sdc = sdn;
    mxc = mxn;
    myc = myn;
    uPrev = uCur;
    uCur = uNext;
  };

  // Iteration j: stage A runs group j (after starting at j = 0). Stage B
  // runs group b once stage A has written every group it reads, the groups
  // up to b + L - 1 or stage A's last, nA - 1: at iteration
  // jB(b) = max(min(b + L, nA), jB(0) + b), having started (groups -1 and
  // 0) at min(L - 1, nA). One barrier per iteration.
  const int jS = (L - 1 < nA) ? L - 1 : nA, jB0 = (L < nA) ? L : nA;
  auto jB = [&](int b) {
    const int r = (b + L < nA) ? b + L : nA;
    return (r > jB0 + b) ? r : jB0 + b;
  };
  const int niter = (nA > jB(nB - 1) + 1) ? nA : jB(nB - 1) + 1;
  if (isA) start();
  int bnext = 0;
#pragma unroll 1
  for (int j = 0; j < niter; ++j) {
    if (isA) {
      if (j < nA) group(j);
    } else {
      if (j == jS) start();
      if (bnext < nB && j == jB(bnext)) group(bnext++);
    }
    __syncthreads();
  }
}

// Generalised periodic boundaries (Sec. II.B), applied to the state a step
// writes: a population that the next pull carries across the period (+x out
// of the outlet column x = nx-1 into the inlet, -x out of the inlet column
// into the outlet) becomes the equilibrium at the far end's density plus its
// own non-equilibrium part. With the moments (rho, j) of its source node, a
// density shift d = p+-/cs2 - mean column density adds
// a_i [d + (4.5 (c.j)^2 - 1.5 j^2) (1/(rho + d) - 1/rho)]. Diagonal links
// that meet a wall are reflected, not carried, and stay. f: a node's stored
// populations (FP32: relative to the equilibrium at density 1 and the row's
// reference velocity ur, which carries momentum); put(i, v) receives the three
// that change.
template <bool SHIFT, typename Put>
__device__ __forceinline__ void gpbc_change(const double f[9], double ur, double d, bool outlet, int y, int ny,
                                            Put put) {
  double s = 0;
#pragma unroll
  for (int i = 0; i < 9; ++i) s += f[i];
  const double rho = SHIFT ? 1.0 + s : s;
  const double jx = (f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7]) + (SHIFT ? ur : 0.0);
  const double jy = (f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8]);
  const double j2 = jx * jx + jy * jy, w = 1.0 / (rho + d) - 1.0 / rho;
  auto change = [&](int i, double cx, int cy) __attribute__((always_inline)) {
    if (y + cy < 0 || y + cy >= ny) return;  // met a wall: reflected
    const double cj = cx * jx + cy * jy;
    const double a = (i < 5) ? 1.0 / 9.0 : 1.0 / 36.0;
    put(i, f[i] + a * (d + (4.5 * cj * cj - 1.5 * j2) * w));
  };
  if (outlet) {
    change(1, 1.0, 0);
    change(5, 1.0, 1);
    change(8, 1.0, -1);
  } else {
    change(3, -1.0, 0);
    change(6, -1.0, 1);
    change(7, -1.0, -1);
  }
}

// Density of node (x, y) after streaming, in FP64, from the channel's slots C
// (FP64 storage, fixed walls).
__device__ __forceinline__ double column_density(const double *__restrict__ C, int nx, int ny, int x, int y) {
  const unsigned row = (unsigned)y * nx;
  const unsigned xm = (x == 0) ? nx - 1 : x - 1, xp = (x == nx - 1) ? 0 : x + 1;
  const bool bot = (y == 0), top = (y == ny - 1);
  const unsigned dn = row - nx, up = row + nx;
  const double f0 = C[lslot(0, row + x)], f1 = C[lslot(1, row + xm)], f3 = C[lslot(3, row + xp)];
  const double f2 = C[bot ? lslot(4, row + x) : lslot(2, dn + x)], f5 = C[bot ? lslot(7, row + x) : lslot(5, dn + xm)],
          f6 = C[bot ? lslot(8, row + x) : lslot(6, dn + xp)];
  const double f4 = C[top ? lslot(2, row + x) : lslot(4, up + x)], f7 = C[top ? lslot(5, row + x) : lslot(7, up + xp)],
          f8 = C[top ? lslot(6, row + x) : lslot(8, up + xm)];
  return (f0 + f1 + f3) + (f2 + f5 + f6) + (f4 + f7 + f8);
}

// Sum of a column of n densities (stride s apart; at most 512, as a box of 1024
// nodes holds at least two of them) over a wavefront, all lanes active: the
// sums of the rows of one residue mod 256, 64 of them after 64, or (TREE) in the
// order of gpbc_kernel.
template <bool TREE>
__device__ __forceinline__ double column_sum(const double *col, int s, int n) {
  const int lane = threadIdx.x & 63;
  if constexpr (!TREE) {
    double sum = 0;
    for (int k = 0; k < min(n, 256); k += 64) {
      double v = k + lane < n ? col[(k + lane) * s] : 0.0;
      if (n > 256) v += k + 256 + lane < n ? col[(k + 256 + lane) * s] : 0.0;
      sum += group_sum<64>(v);
    }
    return sum;
  } else {
    double part[4] = {0, 0, 0, 0};
    for (int k = 0; k < n; k += 256) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + 64 * j < n) part[j] += k + 64 * j + lane < n ? col[(k + 64 * j + lane) * s] : 0.0;
    }
    double v = (part[0] + part[2]) + (part[1] + part[3]);
    v += __shfl_xor(v, 32, 64);
    v += __shfl_xor(v, 16, 64);
    // rows of 16 lanes hold the same now: rotations fetch what xor would
    v += dpp_move<0x128>(v);  // row_ror 8
    v += dpp_move<0x124>(v);
    v += dpp_move<0x122>(v);
    v += dpp_move<0x121>(v);
    return v;
  }
}

// Collision of the stress-force step of node n, row y of ny (sd its density,
// inv 1 / sd): div Sigma^nN by central differences of the neighbours' Sigma^nN (three
// planes of TH values: l left, r right, n + od below, n + ou above; ghost rows
// extrapolated linearly), then the forcing of the total force; put(i, v) takes
// the populations one by one (an array of them costs the fused kernel 1-2%).
template <typename Put>
__device__ __forceinline__ void saf_collide(const double f[9], double sd, double inv, double mx, double my, double g,
                                            double om, double kf, const double *S, int TH, int n, int l, int r, int od, int ou,
                                            int y, int ny, Put put) {
  constexpr int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  constexpr int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  double dn[3], up[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double *T = S + p * TH;
    const double Tc = T[n];
    if (ny == 1) {
      dn[p] = up[p] = Tc;
    } else {
      dn[p] = y > 0 ? T[n + od] : 2.0 * Tc - T[n + ou];
      up[p] = y < ny - 1 ? T[n + ou] : 2.0 * Tc - T[n + od];
    }
  }
  const double fsx = 0.5 * (S[r] - S[l]) + 0.5 * (up[1] - dn[1]);
  const double fsy = 0.5 * (S[TH + r] - S[TH + l]) + 0.5 * (up[2] - dn[2]);
  const double fx = g + fsx, fy = fsy;
  const double ux = (mx + 0.5 * fx) * inv, uy = (my + 0.5 * fy) * inv;
  const double usq = ux * ux + uy * uy, uf = ux * fx + uy * fy;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const double cu = cx[i] * ux + cy[i] * uy, cfo = cx[i] * fx + cy[i] * fy;
    const double a = weight<double>(i);
    const double neq = a * sd * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq);
    const double F = a * kf * (3.0 * cfo + 9.0 * cu * cfo - 3.0 * uf);
    put(i, f[i] - om * (f[i] - neq) + F);
  }
}

// Many steps per launch for small lattices: one workgroup takes a box of
// nodes [x0, x1) x [y0, y1) of one channel through S steps with the state in
// LDS. It loads the box and a halo of 2 S nodes around it (clipped at the
// walls; a box of the channel's whole width needs no columns beyond it), one
// node per thread, and each step consumes two nodes of the halo: a step's
// u~ needs the populations one node further out, and its stencil u~ another.
// Per step a node's thread pulls its nine populations from LDS, forms u~ into
// LDS, and after a barrier takes its four stencil velocities, updates the node
// and writes its populations back in place (every pull of the step is done
// by then); a second barrier ends the step. The trace, the stress of the
// viscoelastic model, the pull addresses and the row references' shifts are
// node-local and stay in registers for the whole launch. The last step
// stores the box. Per node the arithmetic is that of the one-step sweeps.
//
// Small lattices are bound by latency: a launch of one or two steps costs
// 4 to 10 us whatever it computes. Here a step costs its chain of two LDS
// exchanges and the node update, about 0.9 us at one wavefront per SIMD and
// 1.05 at two (FP64 1.0 and 1.4): one 8 x 64 channel 1.1 us per step against
// 4.7 at two steps per launch. With every CU full (256 ragged channels, 80
// VGPRs, six wavefronts per SIMD in FP32) it issues VALU work about three
// quarters of the time: 5.3 us per step against 13.2.
//
// GP: channels with the pressure drive, the generalised periodic boundaries
// (gpbc_change) in the same launch. A step needs the density of the inlet and
// outlet columns, summed over all rows. FP64 takes it from what the step pulls
// (a collision keeps every node's density): with S = 1 a workgroup whose box
// stores inlet or outlet nodes sums it from the state it reads, while its
// region loads; with S > 1 the region holds all rows, and the wavefronts with
// inlet or outlet nodes sum it every step from LDS, in the same order. 64 x 32
// FP64 takes 3.3 us per step against 5.9 with S = 1. FP32 rounding does not
// keep the density exactly, and the boundary acts on that of the stored
// values: S > 1 sums it after the update, behind a third barrier, in the order
// of gpbc_kernel, which with S = 1 follows every step.
//
// SAF: the stress as a force density (FP64), the stages and the arithmetic of
// saf_fused_kernel. Its step reaches three nodes: u~, the stress Sigma^nN of
// the neighbours' u~ (three more planes), the divergence of the neighbours'
// stress; a third barrier, and a halo of 3 S nodes. 143 x 43 takes 3.2 us per
// step against 7.7 in a launch each.
template <typename T, bool VE, bool GP, bool SAF, int TH>
__global__ void __launch_bounds__(TH, sizeof(T) == 4 && !GP ? 6 : 4) sweep_block_kernel(SweepArgs a, int S) {
  constexpr bool SHIFT = sizeof(T) == 4;
  static_assert(!SAF || (!SHIFT && !VE && !GP), "the stress as a force: FP64, instantaneous, no pressure drive");
  constexpr int kReach = SAF ? 3 : 2;  // nodes a step reaches
  // planes of TH values: the populations at P(i), u~ at U and V, placed so
  // that the pull addresses of populations 2 and 4 also address u~ of the
  // rows below and above (a wall row's read another plane and are not used)
  __shared__ T l[(SAF ? 14 : 11) * TH];
  constexpr int U = 2 * TH, V = 3 * TH, Sg = 11 * TH;
  auto P = [](int i) __attribute__((always_inline)) { return (i < 2 ? i : (i == 2 ? 4 : (i == 4 ? 5 : (i == 3 ? 6 : i + 2)))) * TH; };
  const Strip st = a.strips[xcd_item(blockIdx.x, a.n_wg)];
  const ChanDev c = a.ch[st.ch];
  const int nx = c.nx, ny = c.ny, halo = kReach * S;
  const Coef<T> q(c);
  // the region: the box and its halo
  const bool whole = st.x1 - st.x0 >= nx;
  const int cx0 = whole ? 0 : st.x0 - halo, cw = whole ? nx : st.x1 - st.x0 + 2 * halo;
  const int ry0 = st.y0 - halo < 0 ? 0 : st.y0 - halo, ry1 = st.y1 + halo > ny ? ny : st.y1 + halo;
  const int rows = ry1 - ry0;
  const bool in = (int)threadIdx.x < rows * cw;  // (the host keeps rows * cw <= TH)
  const int n = in ? threadIdx.x : 0;
  // nodes row by row, or column by column where only columns are cut and the
  // boxes are few (st.flip, see kColumnOrderBoxes): the halo is then at both ends
  // of the node order, and whole wavefronts drop out of the later steps
  const bool by_col = st.flip && !whole && rows == ny;
  const int sx = by_col ? rows : 1, sy = by_col ? 1 : cw;
  const int major = n / (by_col ? rows : cw), minor = n - major * (by_col ? rows : cw);
  const int r = by_col ? minor : major, cc = by_col ? major : minor, y = ry0 + r;
  int x = cx0 + cc;
  if (!whole) {
    x %= nx;
    x += x < 0 ? nx : 0;
  }
  const bool bot = y == 0, top = y == ny - 1;
  // neighbours inside the region (at its cut edges the node itself: what
  // they lead to is outside the part of the region still valid)
  const int il = cc > 0 ? n - sx : (whole ? n + cw - 1 : n), ir = cc < cw - 1 ? n + sx : (whole ? n - (cw - 1) : n);
  const int od = r > 0 ? -sy : 0, ou = r < rows - 1 ? sy : 0;
  const int i2 = bot ? P(4) + n : P(2) + n + od, i4 = top ? P(2) + n : P(4) + n + ou;
  const int i5 = bot ? P(7) + n : P(5) + il + od, i6 = bot ? P(8) + n : P(6) + ir + od;
  const int i7 = top ? P(5) + n : P(7) + ir + ou, i8 = top ? P(6) + n : P(8) + il + ou;
  // the channel's own slots, 32-bit (the host keeps nx * ny small enough)
  const unsigned o = (unsigned)y * nx + x;
  const unsigned o0 = lslot(0, o), oS = ((o >> 6) * kStressPlanes) * kTile + (o & (kTile - 1));
  const T *__restrict__ A = static_cast<const T *>(a.A) + c.off * kPlanes + o0;
  T Pc = T(0), sg[3] = {T(0), T(0), T(0)};
  if (in) {
#pragma unroll
    for (int i = 0; i < 9; ++i) l[P(i) + n] = A[i * kTile];
    Pc = A[9 * kTile];
    if constexpr (VE) {
#pragma unroll
      for (int p = 0; p < 3; ++p) sg[p] = static_cast<const T *>(a.SA)[c.off * kStressPlanes + oS + p * kTile];
    }
  }
  // FP32: the row's reference and what to_row_reference adds to each pulled
  // population
  T urc = T(0), urd = T(0), uru = T(0), sh[9] = {T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0)};
  if constexpr (SHIFT) {
    const float *ur = a.uref + c.row_off;
    urc = ur[y];
    urd = ur[bot ? y : y - 1];
    uru = ur[top ? y : y + 1];
    to_row_reference(sh, urd, urc, uru, bot, top);
    if (bot) urd = -urc;
  }
  // position in the box, for the part of the region a step still updates
  const int ylo = st.y0 - y, yhi = y - (st.y1 - 1);              // > 0 outside the box
  const int xlo = whole ? 0 : halo - cc, xhi = whole ? 0 : cc - (cw - 1 - halo);
  const int out_by = max(max(ylo, yhi), max(xlo, xhi));          // distance outside the box (<= 0: inside)
  double dcol = 0;  // GP: density shift of the links leaving this thread's column
  __shared__ double dens[GP ? TH : 1];
  const bool edge_column = GP && (x == 0 || x == nx - 1);
  // first inlet and outlet columns of the region (it may be several periods wide)
  const int inlet = !GP || cx0 == 0 ? 0 : (cx0 < 0 ? -cx0 % nx : nx - cx0);
  const int outlet = inlet == 0 ? nx - 1 : inlet - 1;
  if (GP && !SHIFT && S == 1) {
    // 256 threads to a column whatever TH, in the order of column_sum (from
    // 512 on the outlet's are others than the inlet's)
    __shared__ double colsum[2][4];
    const bool stores[2] = {st.x0 == 0, st.x1 >= nx};
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      if (TH > 256 && (wave >> 2) != side) continue;
      double sum = 0;
      if (stores[side])
        for (int yy = threadIdx.x & 255; yy < ny; yy += 256)
          sum += column_density(static_cast<const double *>(a.A) + c.off * kPlanes, nx, ny, side ? nx - 1 : 0, yy);
      sum = group_sum<64>(sum);
      if ((threadIdx.x & 63) == 0) colsum[side][wave & 3] = sum;
    }
    __syncthreads();
    double in_sum = 0, out_sum = 0;
    for (int w = 0; w < 4; ++w) {
      in_sum += colsum[0][w];
      out_sum += colsum[1][w];
    }
    const double dp = (c.t + a.k < c.t_startup) ? c.pd : 0.0;
    dcol = (x == 0 ? 1.0 - 1.5 * dp : 1.0 + 1.5 * dp) - (x == 0 ? in_sum : out_sum) / ny;
  }
  __syncthreads();
#pragma unroll 1
  for (int s = 0; s < S; ++s) {
    const long long t = c.t + a.k + s;
    const T fx = (t < c.t_startup) ? T(c.g) : T(0);
    const T uwg = (t < c.t_startup) ? T(c.uw) : T(0);
    const T uw6 = (!c.zh && t >= 1 && t - 1 < c.t_startup) ? T(c.uw / 6.0) : T(0);
    const int reach = kReach * (S - 1 - s);  // this step updates the box and `reach` nodes around it
    T f[9], sd, mx, my;
    U2<T> uc;
    if (in && out_by <= reach + kReach - 1) {
      f[0] = l[P(0) + n];
      f[1] = l[P(1) + il];
      f[3] = l[P(3) + ir];
      f[2] = l[i2];
      f[5] = l[i5];
      f[6] = l[i6];
      f[4] = l[i4];
      f[7] = l[i7] - (top ? uw6 : T(0));
      f[8] = l[i8] + (top ? uw6 : T(0));
      if (GP && !SHIFT && S > 1 && edge_column) {  // as column_density
        const double d = ((double)f[0] + (double)f[1] + (double)f[3]) + ((double)f[2] + (double)f[5] + (double)f[6]) +
                         ((double)f[4] + (double)f[7] + (double)f[8]);
        dens[n] = d;
      }
      if constexpr (SHIFT) {
#pragma clang fp contract(off)
        f[2] += sh[2];
        f[5] += sh[5];
        f[6] += sh[6];
        f[4] += sh[4];
        f[7] += sh[7];
        f[8] += sh[8];
      }
      if (c.zh && top) zou_he_top<T, SHIFT>(f, uwg, urc, fx);
      moments<T>(f, sd, mx, my);
      uc = u_tilde<T, SHIFT>(sd, mx, my, fx, urc);
      l[U + n] = uc.x;
      l[V + n] = uc.y;
    }
    __syncthreads();
    if constexpr (SAF) {
      // Sigma^nN, as in saf_fused_kernel
      if (in && out_by <= reach + 1) {
        const double uxd = y > 0 ? l[U - P(2) + i2] : -uc.x, uyd = y > 0 ? l[V - P(2) + i2] : -uc.y;
        const double uxu = y < ny - 1 ? l[U - P(4) + i4] : 2.0 * uwg - uc.x;
        const double uyu = y < ny - 1 ? l[V - P(4) + i4] : -uc.y;
        const double kxx = 0.5 * (l[U + ir] - l[U + il]);
        const double kxy = 0.5 * (uxu - uxd);
        const double kyx = 0.5 * (l[V + ir] - l[V + il]);
        const double kyy = 0.5 * (uyu - uyd);
        double sxx = 0, sxy = 0, syy = 0;
        if (q.stress_on) inlm_stress<double>(kxx, kxy, kyx, kyy, q, sxx, sxy, syy);
        l[Sg + n] = sxx - q.lgt * 2.0 * kxx;
        l[Sg + TH + n] = sxy - q.lgt * (kxy + kyx);
        l[Sg + 2 * TH + n] = syy - q.lgt * 2.0 * kyy;
      }
      __syncthreads();
    }
    const bool update = in && out_by <= reach;
    // the shift dcol of the wavefronts with inlet or outlet nodes to update
    const bool edge = update && edge_column;
    auto column_shift = [&]() __attribute__((always_inline)) {
      if (!__builtin_amdgcn_ballot_w64(edge)) return;
      double mine = 0;
#pragma unroll 1
      for (int i = inlet, o = outlet; i < cw || o < cw; i += nx, o += nx) {
        const double si = i < cw ? column_sum<SHIFT>(dens + i * sx, sy, ny) : 0.0;
        const double so = o < cw ? column_sum<SHIFT>(dens + o * sx, sy, ny) : 0.0;
        if (cc == i) mine = si;
        if (cc == o) mine = so;
      }
      const double dp = (t < c.t_startup) ? c.pd : 0.0;
      dcol = (x == 0 ? 1.0 - 1.5 * dp : 1.0 + 1.5 * dp) - mine / ny;
    };
    if (GP && !SHIFT && S > 1) column_shift();
    T out[9], trT, sn[3];
    if constexpr (SAF) {
      if (update)
        saf_collide(f, sd, recip<double>(sd), mx, my, fx, c.omega, c.kf, l + Sg, TH, n, il, ir, od, ou, y, ny,
                    [&](int i, double v) __attribute__((always_inline)) { out[i] = v; });
      trT = Pc;
    } else if (update) {
      const U2<T> lf{l[U + il], l[V + il]}, rt{l[U + ir], l[V + ir]};
      U2<T> dn{l[U - P(2) + i2], l[V - P(2) + i2]}, up{l[U - P(4) + i4], l[V - P(4) + i4]};
      if (bot) dn = U2<T>{-uc.x, -uc.y};
      T kref = T(0);
      if (top) {
        const U2<T> m = c.zh ? dn : uc;
        up = U2<T>{(SHIFT ? T(0) : T(2) * uwg) - m.x, -m.y};
      }
      if constexpr (SHIFT) {
        const T urt = top ? T(2) * uwg - (c.zh ? urd : urc) : uru;
        kref = T(0.5) * (urt - urd);
      }
      double obs[OF_COUNT];
      node_update<T, SHIFT, false, VE>(f, sd, mx, my, Pc, fx, lf, rt, dn, up, urc, kref, q, c.nnp, sg, sn, out, trT,
                                       obs);
      Pc = trT;
      if constexpr (VE) {
#pragma unroll
        for (int p = 0; p < 3; ++p) sg[p] = sn[p];
      }
    }
    if constexpr (GP) {
      double g[9];
      if (edge) {
#pragma unroll
        for (int i = 0; i < 9; ++i) g[i] = (double)out[i];
      }
      if (SHIFT) {
        if (edge) {
          double d = 0;
#pragma unroll
          for (int i = 0; i < 9; ++i) d += g[i];
          dens[n] = 1.0 + d;
        }
        __syncthreads();
      }
      if (SHIFT) column_shift();
      if (edge) gpbc_change<SHIFT>(g, (double)urc, dcol, x != 0, y, ny, [&](int i, double v) { out[i] = (T)v; });
    }
    if (update) {
      if (s < S - 1) {
#pragma unroll
        for (int i = 0; i < 9; ++i) l[P(i) + n] = out[i];
      } else {
        T *__restrict__ B = static_cast<T *>(a.B) + c.off * kPlanes + o0;
#pragma unroll
        for (int i = 0; i < 9; ++i) B[i * kTile] = out[i];
        B[9 * kTile] = trT;
        if constexpr (VE) {
#pragma unroll
          for (int p = 0; p < 3; ++p) static_cast<T *>(a.SB)[c.off * kStressPlanes + oS + p * kTile] = sn[p];
        }
      }
    }
    if (s < S - 1) __syncthreads();
  }
}

// FP64 step of the instantaneous or time-integrated model over tiles of
// kMainTileX x kMainTileY nodes, one workgroup per tile and one thread per
// node. Each thread pulls its node and keeps the populations; u~ of the tile
// and of the ring of one node around it go to LDS, and after one barrier each
// thread has its four stencil velocities (no-slip ghosts behind the walls, as
// in the strip sweeps) and runs the node update. Each XCD takes a contiguous
// run of the tile list, which the host orders as blocks of neighbouring tiles
// (they share the halo populations they pull through that XCD's L2).
constexpr int kMainUX = kMainTileX + 2, kMainUY = kMainTileY + 2;
constexpr int kMainRing = 2 * kMainUX + 2 * kMainTileY;
static_assert(kMainTileX * kMainTileY == kMainThreads, "one node per thread");
static_assert(kMainRing <= kMainThreads, "at most one ring node per thread");

template <bool VE, bool NT>
__global__ void __launch_bounds__(kMainThreads) sweep_tile_kernel(SweepArgs a) {
  __shared__ double su[2][kMainUY][kMainUX];
  const int item = xcd_item(blockIdx.x, gridDim.x, a.down);
  const Strip tl = a.strips[item];
  const ChanDev c = a.ch[tl.ch];
  if (!c.active) return;  // frozen channel (uniform over the workgroup)
  const int nx = c.nx, ny = c.ny;
  const long long t = c.t + a.k;
  const double fx = (t < c.t_startup) ? c.g : 0.0;
  const double uwg = (t < c.t_startup) ? c.uw : 0.0;
  const double uw6 = (!c.zh && t >= 1 && t - 1 < c.t_startup) ? c.uw / 6.0 : 0.0;
  const Coef<double> q(c);
  const double *__restrict__ Ac = static_cast<const double *>(a.A) + c.off * kPlanes;
  double *__restrict__ Bc = static_cast<double *>(a.B) + c.off * kPlanes;
  const bool wide = nx >= kMainTileX + 2;  // then halo columns wrap at most once
  auto wrapx = [&](int x) {
    if (wide) return x < 0 ? x + nx : (x >= nx ? x - nx : x);
    const int r = x % nx;
    return r < 0 ? r + nx : r;
  };
  auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
  // this thread's node and (threads below kMainRing) one node of the ring:
  // the row below, the row above, one column on either side; both pulled
  // before either is used (rows outside the channel pull a row inside and
  // store nothing)
  const int jo = threadIdx.x / kMainTileX, io = threadIdx.x - jo * kMainTileX;
  const int yo = tl.y0 + jo, xo = tl.x0 + io;
  const int h = threadIdx.x;
  int hj, hi;
  if (h < kMainUX) {
    hj = 0;
    hi = h;
  } else if (h < 2 * kMainUX) {
    hj = kMainTileY + 1;
    hi = h - kMainUX;
  } else {
    const int r = h - 2 * kMainUX;
    hj = 1 + (r >> 1);
    hi = (r & 1) ? kMainUX - 1 : 0;
  }
  const int hy = tl.y0 - 1 + hj;
  const bool ring = h < kMainRing;
  const unsigned m = (unsigned)clampy(yo) * nx + wrapx(xo);
  double f[9], fh[9], sgc[3] = {0.0, 0.0, 0.0};
  pull_local(Ac, nx, ny, wrapx(xo), clampy(yo), uw6, f);
  if (c.zh && clampy(yo) == ny - 1) zou_he_top<double, false>(f, uwg, 0.0, fx);
  const double Pc = Ac[lslot(9, m)];
  if constexpr (VE) {
    const double *__restrict__ SAc = static_cast<const double *>(a.SA) + c.off * kStressPlanes;
#pragma unroll
    for (int p = 0; p < 3; ++p) sgc[p] = SAc[((m >> 6) * kStressPlanes + p) * kTile + (m & (kTile - 1))];
  }
  if (ring) pull_local(Ac, nx, ny, wrapx(tl.x0 - 1 + hi), clampy(hy), uw6, fh);
  if (ring && c.zh && clampy(hy) == ny - 1) zou_he_top<double, false>(fh, uwg, 0.0, fx);
  double sd, mx, my;
  moments<double>(f, sd, mx, my);
  const U2<double> uc = u_tilde<double, false>(sd, mx, my, fx, 0.0);
  if (yo < ny) {
    su[0][jo + 1][io + 1] = uc.x;
    su[1][jo + 1][io + 1] = uc.y;
  }
  if (ring && hy >= 0 && hy < ny) {
    double hs, hx, hv;
    moments<double>(fh, hs, hx, hv);
    const U2<double> u = u_tilde<double, false>(hs, hx, hv, fx, 0.0);
    su[0][hj][hi] = u.x;
    su[1][hj][hi] = u.y;
  }
  __syncthreads();
  if (yo >= tl.y1 || xo >= nx) return;
  const int js = jo + 1, is = io + 1;
  const U2<double> lf{su[0][js][is - 1], su[1][js][is - 1]};
  const U2<double> rt{su[0][js][is + 1], su[1][js][is + 1]};
  U2<double> dn{su[0][js - 1][is], su[1][js - 1][is]};
  U2<double> up{su[0][js + 1][is], su[1][js + 1][is]};
  if (yo == 0) dn = U2<double>{-uc.x, -uc.y};
  if (yo == ny - 1) up = c.zh ? U2<double>{2.0 * uwg - dn.x, -dn.y} : U2<double>{2.0 * uwg - uc.x, -uc.y};
  double out[9], trT, sg[3], obs[OF_COUNT];
  node_update<double, false, false, VE>(f, sd, mx, my, Pc, fx, lf, rt, dn, up, 0.0, 0.0, q, c.nnp, sgc, sg, out,
                                        trT, obs);
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    if constexpr (NT) __builtin_nontemporal_store(out[i], &Bc[lslot(i, m)]);
    else Bc[lslot(i, m)] = out[i];
  }
  if constexpr (NT) __builtin_nontemporal_store(trT, &Bc[lslot(9, m)]);
  else Bc[lslot(9, m)] = trT;
  if constexpr (VE) {
    double *__restrict__ SBc = static_cast<double *>(a.SB) + c.off * kStressPlanes;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      double *d = &SBc[((m >> 6) * kStressPlanes + p) * kTile + (m & (kTile - 1))];
      if constexpr (NT) __builtin_nontemporal_store(sg[p], d);
      else *d = sg[p];
    }
  }
}

// Aligned 64-column strips of a channel whose width is a multiple of 64
// (and at least 128). Row y of the strip is tile (off + y nx + x0)/64; lane
// l owns column x0 + l.
template <typename T, bool SHIFT, bool OBS, bool VE>
__global__ void __launch_bounds__(64 * LB_WG_WAVES) sweep_wide64_kernel(SweepArgs a) {
  const int lane = threadIdx.x & 63;
  const int sidx = strip_index(a);
  if (sidx >= a.n_strips) return;
  const Strip st = a.strips[sidx];
  const ChanDev c = a.ch[st.ch];
  const T *__restrict__ A = static_cast<const T *>(a.A);
  T *__restrict__ B = static_cast<T *>(a.B);
  const int nx = c.nx, ny = c.ny;
  const long long t = c.t + a.k;
  const T fx = (t < c.t_startup) ? T(c.g) : T(0);
  // moving top wall: its velocity at step t (stencil ghost) and u_w/6 of step
  // t - 1, whose reflected links step t pulls
  const T uwg = (t < c.t_startup) ? T(c.uw) : T(0);
  const T uw6 = (!c.zh && t >= 1 && t - 1 < c.t_startup) ? T(c.uw / 6.0) : T(0);
  const Coef<T> q(c);

  const int tiles_row = nx >> 6;                 // tiles per row
  const long long tile0 = (c.off + st.x0) >> 6;  // tile of row 0 of this strip
  const int xt = st.x0 >> 6;                     // tile column of the strip
  // tile offsets (in tiles) of the left and right neighbour columns' tiles
  const int dl = (xt == 0) ? tiles_row - 1 : -1;
  const int dr = (xt == tiles_row - 1) ? -(tiles_row - 1) : 1;
  constexpr int F = kTile;  // stride between fields inside a tile

  // Wave-uniform addressing: tile index of row y in this strip's column and
  // in the columns left/right of it; ld() reads one field of one column of a
  // tile (every lane the same address).
  auto tile = [&](int y) -> long long { return tile0 + (long long)y * tiles_row; };
  // wave-uniform loads go through the scalar unit: A is not written during
  // the sweep, so it can be read as constant memory
  typedef const __attribute__((address_space(4))) T *cptr;
  const cptr Ac = (cptr)(A);
  auto ld = [&](long long tl, int col, int p) -> T { return Ac[(tl * kPlanes + p) * F + col]; };
  auto run = [&](long long tl, int p) -> T { return A[(tl * kPlanes + p) * F + lane]; };
  // FP32 reference velocity of row y (0 in FP64), rows clamped to the channel
  auto ref = [&](int y) -> T {
    if constexpr (SHIFT) return a.uref[c.row_off + (y < 0 ? 0 : (y >= ny ? ny - 1 : y))];
    return T(0);
  };

  // Pull of row y (0 <= y < ny) for every lane from aligned runs of the
  // strip's own tiles; the x-shifted directions are lane shifts whose edge
  // lanes take the neighbouring column's value.
  auto pull_row = [&](int y, T f[9], T &Pv) {
    const bool bot = (y == 0), top = (y == ny - 1);
    const long long t0 = tile(y), td = bot ? t0 : tile(y - 1), tu = top ? t0 : tile(y + 1);
    f[0] = run(t0, 0);
    f[1] = shift_up(ld(t0 + dl, 63, 1), run(t0, 1));
    f[3] = shift_down(ld(t0 + dr, 0, 3), run(t0, 3));
    Pv = run(t0, 9);
    if (bot) {
      f[2] = run(t0, 4);
      f[5] = run(t0, 7);
      f[6] = run(t0, 8);
    } else {
      f[2] = run(td, 2);
      f[5] = shift_up(ld(td + dl, 63, 5), run(td, 5));
      f[6] = shift_down(ld(td + dr, 0, 6), run(td, 6));
    }
    if (top) {
      f[4] = run(t0, 2);
      f[7] = run(t0, 5) - uw6;
      f[8] = run(t0, 6) + uw6;
    } else {
      f[4] = run(tu, 4);
      f[7] = shift_down(ld(tu + dr, 0, 7), run(tu, 7));
      f[8] = shift_up(ld(tu + dl, 63, 8), run(tu, 8));
    }
    if constexpr (SHIFT) to_row_reference(f, ref(y - 1), ref(y), ref(y + 1), bot, top);
    if (c.zh && top) zou_he_top<T, SHIFT>(f, uwg, ref(y), fx);
  };
  // u~ of the column left of the strip (column 63 of the left tile) and of
  // the column right of it (column 0 of the right tile), from wave-uniform
  // pulls.
  auto halo_u = [&](int y, U2<T> &uL, U2<T> &uR) {
    const bool bot = (y == 0), top = (y == ny - 1);
    const long long t0 = tile(y), L0 = t0 + dl, R0 = t0 + dr;
    T a[9], b[9];
    a[0] = ld(L0, 63, 0);
    a[1] = ld(L0, 62, 1);
    a[3] = ld(t0, 0, 3);
    b[0] = ld(R0, 0, 0);
    b[1] = ld(t0, 63, 1);
    b[3] = ld(R0, 1, 3);
    if (bot) {
      a[2] = ld(L0, 63, 4);
      a[5] = ld(L0, 63, 7);
      a[6] = ld(L0, 63, 8);
      b[2] = ld(R0, 0, 4);
      b[5] = ld(R0, 0, 7);
      b[6] = ld(R0, 0, 8);
    } else {
      const long long td = tile(y - 1);
      a[2] = ld(td + dl, 63, 2);
      a[5] = ld(td + dl, 62, 5);
      a[6] = ld(td, 0, 6);
      b[2] = ld(td + dr, 0, 2);
      b[5] = ld(td, 63, 5);
      b[6] = ld(td + dr, 1, 6);
    }
    if (top) {
      a[4] = ld(L0, 63, 2);
      a[7] = ld(L0, 63, 5) - uw6;
      a[8] = ld(L0, 63, 6) + uw6;
      b[4] = ld(R0, 0, 2);
      b[7] = ld(R0, 0, 5) - uw6;
      b[8] = ld(R0, 0, 6) + uw6;
    } else {
      const long long tu = tile(y + 1);
      a[4] = ld(tu + dl, 63, 4);
      a[7] = ld(tu, 0, 7);
      a[8] = ld(tu + dl, 62, 8);
      b[4] = ld(tu + dr, 0, 4);
      b[7] = ld(tu + dr, 1, 7);
      b[8] = ld(tu, 63, 8);
    }
    const T urc = ref(y);
    if constexpr (SHIFT) {
      to_row_reference(a, ref(y - 1), urc, ref(y + 1), bot, top);
      to_row_reference(b, ref(y - 1), urc, ref(y + 1), bot, top);
    }
    if (c.zh && top) {
      zou_he_top<T, SHIFT>(a, uwg, urc, fx);
      zou_he_top<T, SHIFT>(b, uwg, urc, fx);
    }
    T sd, mx, my;
    moments<T>(a, sd, mx, my);
    uL = u_tilde<T, SHIFT>(sd, mx, my, fx, urc);
    moments<T>(b, sd, mx, my);
    uR = u_tilde<T, SHIFT>(sd, mx, my, fx, urc);
  };
  auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
  // viscoelastic model: the stress of the previous step, one tile row of the
  // stress buffers (three fields per 64-node tile) per row
  const T *__restrict__ SA = static_cast<const T *>(a.SA);
  T *__restrict__ SB = static_cast<T *>(a.SB);
  auto load_sigma = [&](int y, T sg[3]) {
    if constexpr (VE) {
#pragma unroll
      for (int p = 0; p < 3; ++p) sg[p] = SA[(tile(y) * kStressPlanes + p) * F + lane];
    } else {
      sg[0] = sg[1] = sg[2] = T(0);
    }
  };

  T fc[9], fn[9], Pc, Pn, sgc[3], sgn[3];
  U2<T> uPrev, uCur, uNext, uLc, uRc, uLn, uRn;
  {
    T ftmp[9], Ptmp, sd, mx, my;
    pull_row(clampy(st.y0 - 1), ftmp, Ptmp);
    moments<T>(ftmp, sd, mx, my);
    uPrev = u_tilde<T, SHIFT>(sd, mx, my, fx, ref(st.y0 - 1));
  }
  T sdc, mxc, myc;
  pull_row(st.y0, fc, Pc);
  load_sigma(st.y0, sgc);
  moments<T>(fc, sdc, mxc, myc);
  uCur = u_tilde<T, SHIFT>(sdc, mxc, myc, fx, ref(st.y0));
  halo_u(st.y0, uLc, uRc);

#pragma unroll 1
  for (int y = st.y0; y < st.y1; ++y) {
    const int yn = clampy(y + 1);
    T sdn, mxn, myn;
    pull_row(yn, fn, Pn);
    load_sigma(yn, sgn);
    halo_u(yn, uLn, uRn);
    moments<T>(fn, sdn, mxn, myn);
    uNext = u_tilde<T, SHIFT>(sdn, mxn, myn, fx, ref(yn));

    U2<T> dn = uPrev, up = uNext;
    const U2<T> lf{shift_up(uLc.x, uCur.x), shift_up(uLc.y, uCur.y)};
    const U2<T> rt{shift_down(uRc.x, uCur.x), shift_down(uRc.y, uCur.y)};
    // no-slip ghosts behind the half-way walls; with SHIFT the ghost rows take
    // the mirrored references -ur and 2 u_w - ur (see sweep_kernel)
    const T urc = ref(y);
    if (y == 0) dn = U2<T>{-uCur.x, -uCur.y};
    if (y == ny - 1) {
      const U2<T> m = c.zh ? dn : uCur;
      up = U2<T>{(SHIFT ? T(0) : T(2) * uwg) - m.x, -m.y};
    }
    T kref = T(0);
    if constexpr (SHIFT) {
      const T urd = (y == 0) ? -urc : ref(y - 1);
      const T uru = (y == ny - 1) ? T(2) * uwg - (c.zh ? urd : urc) : ref(y + 1);
      kref = T(0.5) * (uru - urd);
    }

    T out[9], trT, sg[3];
    double obs[OF_COUNT];
    node_update<T, SHIFT, OBS, VE>(fc, sdc, mxc, myc, Pc, fx, lf, rt, dn, up, urc, kref, q, c.nnp, sgc, sg, out,
                                   trT, obs);
    if constexpr (OBS) {
      const double ztop = (c.zh && y == ny - 1) ? zh_drag<T>(run(tile(y), 5), run(tile(y), 6), fc) : 0.0;
      obs[OF_DRAG] = wall_drag<T>(fc, y, ny, uw6, c.zh, ztop);
#pragma unroll
      for (int f = 0; f < OF_COUNT; ++f) obs[f] = group_sum<64>(obs[f]);
      if (lane == 0) {
        const long long pr = (long long)c.poff + (long long)y * c.nxs + xt;
        double *dst = a.part + pr * OF_COUNT;
#pragma unroll
        for (int f = 0; f < OF_COUNT; ++f) dst[f] = obs[f];
      }
    } else {
      T *w = B + tile(y) * (kPlanes * F);
#pragma unroll
      for (int i = 0; i < 9; ++i) w[i * F + lane] = out[i];
      w[9 * F + lane] = trT;
      if constexpr (VE) {
        T *ws = SB + tile(y) * (kStressPlanes * F);
#pragma unroll
        for (int p = 0; p < 3; ++p) ws[p * F + lane] = sg[p];
      }
    }

    uPrev = uCur;
    uCur = uNext;
    uLc = uLn;
    uRc = uRn;
#pragma unroll
    for (int p = 0; p < 3; ++p) sgc[p] = sgn[p];
#pragma unroll
    for (int i = 0; i < 9; ++i) fc[i] = fn[i];
    Pc = Pn;
    sdc = sdn;
    mxc = mxn;
    myc = myn;
  }
}

// Vector accesses of NPL consecutive elements.
template <typename T, int NPL>
struct Vec;
template <>
struct Vec<float, 4> {
  typedef float type __attribute__((ext_vector_type(4)));
};
template <>
struct Vec<double, 2> {
  typedef double type __attribute__((ext_vector_type(2)));
};
template <>
struct Vec<float, 2> {
  typedef float type __attribute__((ext_vector_type(2)));
};
template <>
struct Vec<double, 1> {
  typedef double type __attribute__((ext_vector_type(1)));
};

// Side values of a row of a vector strip (see sweep_vec_kernel), packed as
// (dy + 1) | tile << 2 | column << 4 | field << 11 with tile 0: column left
// of the strip's tiles, 1: right of them, 2: first tile, 3: last tile.
#define SIDE(dy, t, col, p) ((dy) + 1 | (t) << 2 | (col) << 4 | (p) << 11)
constexpr int kSideIn[25] = {
    SIDE(0, 0, 63, 1),  SIDE(0, 1, 0, 3),   SIDE(-1, 0, 63, 5), SIDE(-1, 1, 0, 6),  SIDE(1, 1, 0, 7),
    SIDE(1, 0, 63, 8),  SIDE(0, 0, 63, 0),  SIDE(0, 0, 62, 1),  SIDE(0, 2, 0, 3),   SIDE(-1, 0, 63, 2),
    SIDE(-1, 0, 62, 5), SIDE(-1, 2, 0, 6),  SIDE(1, 0, 63, 4),  SIDE(1, 2, 0, 7),   SIDE(1, 0, 62, 8),
    SIDE(0, 1, 0, 0),   SIDE(0, 3, 63, 1),  SIDE(0, 1, 1, 3),   SIDE(-1, 1, 0, 2),  SIDE(-1, 3, 63, 5),
    SIDE(-1, 1, 1, 6),  SIDE(1, 1, 0, 4),   SIDE(1, 1, 1, 7),   SIDE(1, 3, 63, 8),  SIDE(0, 2, 0, 0)};
// bottom wall row: entries reading row y-1 take the bounce-back source (-1: unchanged)
constexpr int kSideBot[25] = {
    -1, -1, SIDE(0, 2, 0, 0), SIDE(0, 2, 0, 0), -1, -1, -1, -1, -1, SIDE(0, 0, 63, 4), SIDE(0, 0, 63, 7),
    SIDE(0, 0, 63, 8), -1, -1, -1, -1, -1, -1, SIDE(0, 1, 0, 4), SIDE(0, 1, 0, 7), SIDE(0, 1, 0, 8), -1, -1, -1, -1};
// top wall row: entries reading row y+1 take the bounce-back source
constexpr int kSideTop[25] = {
    -1, -1, -1, -1, SIDE(0, 2, 0, 0), SIDE(0, 2, 0, 0), -1, -1, -1, -1, -1, -1, SIDE(0, 0, 63, 2),
    SIDE(0, 0, 63, 5), SIDE(0, 0, 63, 6), -1, -1, -1, -1, -1, -1, SIDE(0, 1, 0, 2), SIDE(0, 1, 0, 5),
    SIDE(0, 1, 0, 6), -1};
#undef SIDE

// Aligned strips of 64 NPL columns of a channel whose width is a multiple of
// that: lane l owns the NPL consecutive columns x0 + NPL l + k, k < NPL, which
// sit in one tile (tile x0/64 + l/(64/NPL), first column NPL (l % (64/NPL))),
// so every field of a row is one NPL-element access per lane (16 bytes for
// four FP32 nodes). A pull along +x
// takes element k-1 of the same lane, and for k = 0 element NPL-1 of lane l-1
// (a DPP lane shift; lane 0 takes the column left of the strip); a pull along
// -x mirrors it.
//
// The march is software-pipelined two rows deep: while row y is computed,
// the loads of row y+2 are in flight and row y+1 (loaded one iteration
// earlier) is assembled for the stencil. The 24 values a row needs from the
// columns beside the strip (the six edge populations of the shifted pulls and
// the nine pulled populations of each neighbour column, for its u~) come in
// one lane-indexed vector load, lane i holding value i, so that they complete
// in order with the row's other loads; they are read out with readlane.
template <typename T, bool SHIFT, bool OBS, int NPL, bool NT, bool VE, bool ZH>
__global__ void __launch_bounds__(64 * LB_WG_WAVES) sweep_vec_kernel(SweepArgs a) {
  typedef typename Vec<T, NPL>::type V;
  constexpr int LPT = 64 / NPL;  // lanes per tile
  const int lane = threadIdx.x & 63;
  const int sidx = strip_index(a);
  if (sidx >= a.n_strips) return;
  const Strip st = a.strips[sidx];
  const ChanDev c = a.ch[st.ch];
  const T *__restrict__ A = static_cast<const T *>(a.A);
  T *__restrict__ B = static_cast<T *>(a.B);
  const int nx = c.nx, ny = c.ny;
  const long long t = c.t + a.k;
  const T fx = (t < c.t_startup) ? T(c.g) : T(0);
  // moving top wall: its velocity at step t (stencil ghost) and u_w/6 of step
  // t - 1, whose reflected links step t pulls
  const T uwg = (t < c.t_startup) ? T(c.uw) : T(0);
  const T uw6 = (!c.zh && t >= 1 && t - 1 < c.t_startup) ? T(c.uw / 6.0) : T(0);
  const Coef<T> q(c);

  const int tiles_row = nx >> 6;        // tiles per row
  const long long tile00 = c.off >> 6;  // tile of node (0, 0)
  const int xt = st.x0 >> 6;            // first tile column of the strip
  const int xe = xt + NPL - 1;          // last tile column of the strip
  const int xl = (xt == 0) ? tiles_row - 1 : xt - 1;  // tile column left of the strip
  const int xr = (xe == tiles_row - 1) ? 0 : xe + 1;  // tile column right of the strip
  const int lt = lane / LPT;            // tile of this lane inside the strip
  const int lo = NPL * (lane % LPT);    // first column of this lane inside its tile
  constexpr int F = kTile;

  auto tile = [&](int y, int tx) __attribute__((always_inline)) -> long long { return tile00 + (long long)y * tiles_row + tx; };
  // one field of this lane's NPL columns of row y
  // The time-integrated model's cached step (state and stress about 218 MB
  // per buffer on 4096 x 1024 FP32, near the last-level cache's 256 MB)
  // reads its rows with nontemporal loads: the buffer it reads is dead once
  // read, and letting it go first keeps more of what the previous step wrote
  // (+3 points there; the same loads cost 1 point on the instantaneous
  // model's 168 MB buffers and 6 on the streamed 10.7 GB ones).
  auto vrun = [&](int y, int p) __attribute__((always_inline)) -> V {
    const V *src = reinterpret_cast<const V *>(A + (tile(y, xt + lt) * kPlanes + p) * F + lo);
    if constexpr (VE && !NT && !OBS) return __builtin_nontemporal_load(src);
    return *src;
  };

  // Side values of a row, by lane i < 24 (kSide* below): lanes 0..5 hold the
  // edge populations of the shifted pulls, lanes 6..14 the pulled
  // populations of the column left of the strip, lanes 15..23 those of the
  // column right of it; wall rows take the bounce-back sources. With FP32
  // storage lanes 24..26 hold the reference velocities of rows y-1, y, y+1
  // (clamped to the channel), so that they arrive with the row's loads and
  // not through a dependent load in the row step. Other lanes read node
  // (x0, y). Each lane decodes its entry into an element offset
  // relative to row 0: once per strip for interior rows, again on the wall
  // rows (bottom, top, or both when ny = 1).
  auto side_off = [&](int code) __attribute__((always_inline)) -> long long {
    const int dy = (code & 3) - 1, tsel = (code >> 2) & 3, col = (code >> 4) & 127, p = code >> 11;
    // a blend of values, not a choice between the captured variables (which
    // the compiler would turn into a load through a chosen address and so
    // keep those variables in scratch memory)
    const int tc = (tsel == 0) * xl + (tsel == 1) * xr + (tsel == 2) * xt + (tsel == 3) * xe;
    return ((tile00 + (long long)dy * tiles_row + tc) * kPlanes + p) * F + col;
  };
  const int li = lane < 24 ? lane : 24;
  const int c_in = kSideIn[li];
  const int c_bot = kSideBot[li] >= 0 ? kSideBot[li] : c_in;
  const int c_top = kSideTop[li] >= 0 ? kSideTop[li] : c_in;
  const int c_both = kSideBot[li] >= 0 ? kSideBot[li] : c_top;
  const long long o_in = side_off(c_in);
  const long long row_stride = (long long)tiles_row * kPlanes * F;  // elements per row

  // Raw loads of row y: the ten runs (fields 0, 1, 3, 9 of row y; 2, 5, 6 of
  // row y-1 or, at the bottom wall, 4, 7, 8 of row y; 4, 7, 8 of row y+1 or,
  // at the top wall, 2, 5, 6 of row y) and the side values.
  // viscoelastic model: the stress of the previous step comes with each
  // row's loads (three fields of this lane's NPL columns)
  const T *__restrict__ SA = static_cast<const T *>(a.SA);
  T *__restrict__ SB = static_cast<T *>(a.SB);
  struct Raw {
    V sg[VE ? 3 : 1];
    V r[10];
    T side;
  };
  auto load_raw = [&](int y, Raw &R) __attribute__((always_inline)) {
    const bool bot = (y == 0), top = (y == ny - 1);
    const int yd = bot ? y : y - 1, yu = top ? y : y + 1;
    R.r[0] = vrun(y, 0);
    R.r[1] = vrun(y, 1);
    R.r[3] = vrun(y, 3);
    R.r[9] = vrun(y, 9);
    R.r[2] = vrun(yd, bot ? 4 : 2);
    R.r[5] = vrun(yd, bot ? 7 : 5);
    R.r[6] = vrun(yd, bot ? 8 : 6);
    R.r[4] = vrun(yu, top ? 2 : 4);
    R.r[7] = vrun(yu, top ? 5 : 7);
    R.r[8] = vrun(yu, top ? 6 : 8);
    long long o = o_in;
    if (bot || top)  // wall rows only
      o = side_off(bot * top * c_both + bot * (1 - top) * c_bot + (1 - bot) * c_top);
    const T *ps = A + o + (long long)y * row_stride;
    if constexpr (SHIFT) {
      const int yr = y + lane - 25;
      const T *pu = a.uref + c.row_off + (yr < 0 ? 0 : (yr >= ny ? ny - 1 : yr));
      ps = (lane >= 24 && lane <= 26) ? pu : ps;
    }
    R.side = *ps;
    if constexpr (VE) {
#pragma unroll
      for (int p = 0; p < 3; ++p)
        R.sg[p] = *reinterpret_cast<const V *>(SA + (tile(y, xt + lt) * kStressPlanes + p) * F + lo);
    }
  };
  // Pulled populations, P, moments and u~ of the NPL columns of row y, and u~
  // of the two columns beside the strip.
  auto assemble = [&](int y, const Raw &R, T f[9][NPL], T P[NPL], T sd[NPL], T mx[NPL], T my[NPL],
                      U2<T> u[NPL], U2<T> &uL, U2<T> &uR, T ur3[3]) __attribute__((always_inline)) {
    const bool bot = (y == 0), top = (y == ny - 1);
    auto from_left = [&](const V &r, T edge, T out[NPL]) __attribute__((always_inline)) {
      out[0] = shift_up(edge, r[NPL - 1]);
#pragma unroll
      for (int k = 1; k < NPL; ++k) out[k] = r[k - 1];
    };
    auto from_right = [&](const V &r, T edge, T out[NPL]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NPL - 1; ++k) out[k] = r[k + 1];
      out[NPL - 1] = shift_down(edge, r[0]);
    };
    auto split = [&](const V &r, T out[NPL]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NPL; ++k) out[k] = r[k];
    };
    split(R.r[0], f[0]);
    from_left(R.r[1], lane_value(R.side, 0), f[1]);
    from_right(R.r[3], lane_value(R.side, 1), f[3]);
    split(R.r[9], P);
    split(R.r[2], f[2]);
    split(R.r[4], f[4]);
    if (bot) {
      split(R.r[5], f[5]);
      split(R.r[6], f[6]);
    } else {
      from_left(R.r[5], lane_value(R.side, 2), f[5]);
      from_right(R.r[6], lane_value(R.side, 3), f[6]);
    }
    if (top) {
      split(R.r[7], f[7]);
      split(R.r[8], f[8]);
#pragma unroll
      for (int k = 0; k < NPL; ++k) {
        f[7][k] -= uw6;
        f[8][k] += uw6;
      }
    } else {
      from_right(R.r[7], lane_value(R.side, 4), f[7]);
      from_left(R.r[8], lane_value(R.side, 5), f[8]);
    }
    // a Zou-He top wall completes the top row's populations from above (a
    // variant of its own: the completion's registers cost the plain sweep
    // about a fifth of a point of occupancy headroom)
    const bool zhtop = ZH && top && c.zh;
    // FP32: every pulled value relative to this row's reference
    const T urd = SHIFT ? lane_value(R.side, 24) : T(0);
    const T urc = SHIFT ? lane_value(R.side, 25) : T(0);
    const T uru = SHIFT ? lane_value(R.side, 26) : T(0);
    ur3[0] = urd;
    ur3[1] = urc;
    ur3[2] = uru;
#pragma unroll
    for (int k = 0; k < NPL; ++k) {
      T g[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) g[i] = f[i][k];
      if constexpr (SHIFT) to_row_reference(g, urd, urc, uru, bot, top);
      if (zhtop) zou_he_top<T, SHIFT>(g, uwg, urc, fx);
      if (SHIFT || zhtop) {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i][k] = g[i];
      }
      moments<T>(g, sd[k], mx[k], my[k]);
      u[k] = u_tilde<T, SHIFT>(sd[k], mx[k], my[k], fx, urc);
    }
    // side lanes 6..14 / 15..23 hold populations 0,1,3,2,5,6,4,7,8
    T l[9], r[9];
    l[0] = lane_value(R.side, 6);
    l[1] = lane_value(R.side, 7);
    l[3] = lane_value(R.side, 8);
    l[2] = lane_value(R.side, 9);
    l[5] = lane_value(R.side, 10);
    l[6] = lane_value(R.side, 11);
    l[4] = lane_value(R.side, 12);
    l[7] = lane_value(R.side, 13);
    l[8] = lane_value(R.side, 14);
    r[0] = lane_value(R.side, 15);
    r[1] = lane_value(R.side, 16);
    r[3] = lane_value(R.side, 17);
    r[2] = lane_value(R.side, 18);
    r[5] = lane_value(R.side, 19);
    r[6] = lane_value(R.side, 20);
    r[4] = lane_value(R.side, 21);
    r[7] = lane_value(R.side, 22);
    r[8] = lane_value(R.side, 23);
    const T wc = top ? uw6 : T(0);  // a select: no branch in the row step
    l[7] -= wc;
    l[8] += wc;
    r[7] -= wc;
    r[8] += wc;
    if constexpr (SHIFT) {
      to_row_reference(l, urd, urc, uru, bot, top);
      to_row_reference(r, urd, urc, uru, bot, top);
    }
    if (zhtop) {
      zou_he_top<T, SHIFT>(l, uwg, urc, fx);
      zou_he_top<T, SHIFT>(r, uwg, urc, fx);
    }
    T s0, m0, n0;
    moments<T>(l, s0, m0, n0);
    uL = u_tilde<T, SHIFT>(s0, m0, n0, fx, urc);
    moments<T>(r, s0, m0, n0);
    uR = u_tilde<T, SHIFT>(s0, m0, n0, fx, urc);
  };
  auto clampy = [&](int y) __attribute__((always_inline)) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };

  // The march runs upwards from y0, or downwards from y1 - 1 (the step's
  // direction, reversed on flipped strips); "prev" and "next" are the rows
  // behind and ahead of the current one.
  const bool down = (a.down != 0) != (st.flip != 0);
  const int dir = down ? -1 : 1;
  const int yfirst = down ? st.y1 - 1 : st.y0;
  // Rows the ring loads: the strip and its two halo rows. Its last loads run
  // past the far halo row and are never assembled; they re-read that halo
  // row (fetched a row or two earlier, so from cache) instead of new rows.
  auto ring_row = [&](int y) __attribute__((always_inline)) {
    return clampy(y < st.y0 - 1 ? st.y0 - 1 : (y > st.y1 ? st.y1 : y));
  };
  const int nrows = st.y1 - st.y0;
  T fc[9][NPL], Pc[NPL], sdc[NPL], mxc[NPL], myc[NPL];
  U2<T> uPrev[NPL], uCur[NPL], uLc, uRc;
  T urC[3];  // reference velocities of rows y-1, y, y+1 for the current row
  T sgc[3][NPL];  // viscoelastic model: stress of the previous step, current row
  auto take_sigma = [&](const Raw &R, T sg[3][NPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int k = 0; k < NPL; ++k) sg[p][k] = VE ? R.sg[VE ? p : 0][k] : T(0);
  };
  // ring of raw rows: the row i steps ahead of the first lives in slot i mod D
  constexpr int D = NT ? LB_VEC_DEPTH_NT : LB_VEC_DEPTH;
  Raw S[D];
  {
    // every load of the prologue is issued before the first is used, so the
    // strip pays one memory latency before its first row, not three
    Raw Rp, Rf;
    const int yp = clampy(yfirst - dir);
    load_raw(yp, Rp);
    load_raw(yfirst, Rf);
#pragma unroll
    for (int k = 1; k < D; ++k) load_raw(ring_row(yfirst + dir * k), S[k]);
    T ftmp[9][NPL], Ptmp[NPL], s0[NPL], m0[NPL], n0[NPL], ur_unused[3];
    U2<T> hl, hr;
    assemble(yp, Rp, ftmp, Ptmp, s0, m0, n0, uPrev, hl, hr, ur_unused);
    assemble(yfirst, Rf, fc, Pc, sdc, mxc, myc, uCur, uLc, uRc, urC);
    take_sigma(Rf, sgc);
  }

  // Row y: start the loads of the row D ahead, assemble the next row (loaded
  // D - 1 rows earlier), update and store row y.
  auto row_step = [&](int y, Raw &Rload, const Raw &Rasm) __attribute__((always_inline)) {
    load_raw(ring_row(y + dir * D), Rload);  // unconditional: a branch here costs more than the loads
    T fn[9][NPL], Pn[NPL], sdn[NPL], mxn[NPL], myn[NPL], urN[3];
    U2<T> uNext[NPL], uLn, uRn;
    assemble(clampy(y + dir), Rasm, fn, Pn, sdn, mxn, myn, uNext, uLn, uRn, urN);
    T sgn[3][NPL], sgo[3][NPL];
    take_sigma(Rasm, sgn);

    T out[9][NPL], trT[NPL];
    double obs[OF_COUNT];
    if constexpr (OBS) {
#pragma unroll
      for (int f = 0; f < OF_COUNT; ++f) obs[f] = 0.0;
    }
    // the row's reference and its share of d_y u_x (ghost rows mirrored)
    const T urc = urC[1];
    T kref = T(0);
    if constexpr (SHIFT) {
      const T urd = (y == 0) ? -urc : urC[0];
      const T uru = (y == ny - 1) ? T(2) * uwg - (c.zh ? urd : urc) : urC[2];
      kref = T(0.5) * (uru - urd);
    }
    // the top row's own stored 5 and 6 (what it emitted upwards), for the
    // momentum a Zou-He wall took (observation only)
    V a5{}, a6{};
    if constexpr (OBS && ZH) {
      if (c.zh && y == ny - 1) {
        a5 = vrun(y, 5);
        a6 = vrun(y, 6);
      }
    }
#pragma unroll
    for (int k = 0; k < NPL; ++k) {
      U2<T> lf, rt;
      if (k == 0) {
        lf = U2<T>{shift_up(uLc.x, uCur[NPL - 1].x), shift_up(uLc.y, uCur[NPL - 1].y)};
      } else {
        lf = uCur[k - 1];
      }
      if (k == NPL - 1) {
        rt = U2<T>{shift_down(uRc.x, uCur[0].x), shift_down(uRc.y, uCur[0].y)};
      } else {
        rt = uCur[k + 1];
      }
      U2<T> dn = down ? uNext[k] : uPrev[k], up = down ? uPrev[k] : uNext[k];
      // no-slip ghosts behind the half-way walls, or behind a Zou-He node
      // wall mirrored through the wall row
      if (y == 0) dn = U2<T>{-uCur[k].x, -uCur[k].y};
      if (y == ny - 1) {
        const U2<T> m = c.zh ? dn : uCur[k];
        up = U2<T>{(SHIFT ? T(0) : T(2) * uwg) - m.x, -m.y};
      }
      T g[9], o[9], tr;
#pragma unroll
      for (int i = 0; i < 9; ++i) g[i] = fc[i][k];
      double ob[OF_COUNT];
      const T sp[3] = {sgc[0][k], sgc[1][k], sgc[2][k]};
      T sn[3];
      node_update<T, SHIFT, OBS, VE>(g, sdc[k], mxc[k], myc[k], Pc[k], fx, lf, rt, dn, up, urc, kref, q, c.nnp, sp,
                                     sn, o, tr, ob);
      if constexpr (VE) {
#pragma unroll
        for (int p = 0; p < 3; ++p) sgo[p][k] = sn[p];
      }
      if constexpr (OBS) {
        ob[OF_DRAG] = wall_drag<T>(g, y, ny, uw6, c.zh, zh_drag<T>(a5[k], a6[k], g));
#pragma unroll
        for (int f = 0; f < OF_COUNT; ++f) obs[f] += ob[f];
      } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) out[i][k] = o[i];
        trT[k] = tr;
      }
    }
    if constexpr (OBS) {
#pragma unroll
      for (int f = 0; f < OF_COUNT; ++f) obs[f] = group_sum<64>(obs[f]);
      if (lane == 0) {
        const long long pr = (long long)c.poff + (long long)y * c.nxs + st.x0 / (64 * NPL);
        double *dst = a.part + pr * OF_COUNT;
#pragma unroll
        for (int f = 0; f < OF_COUNT; ++f) dst[f] = obs[f];
      }
    } else {
      T *w = B + tile(y, xt + lt) * (kPlanes * F) + lo;
      V v[kPlanes];
#pragma unroll
      for (int k = 0; k < NPL; ++k) {
#pragma unroll
        for (int i = 0; i < 9; ++i) v[i][k] = out[i][k];
        v[9][k] = trT[k];
      }
      if constexpr (NT) {
#pragma unroll
        for (int i = 0; i < kPlanes; ++i) __builtin_nontemporal_store(v[i], reinterpret_cast<V *>(w + i * F));
      } else {
#pragma unroll
        for (int i = 0; i < kPlanes; ++i) *reinterpret_cast<V *>(w + i * F) = v[i];
      }
      if constexpr (VE) {
        T *ws = SB + tile(y, xt + lt) * (kStressPlanes * F) + lo;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          V vs;
#pragma unroll
          for (int k = 0; k < NPL; ++k) vs[k] = sgo[p][k];
          if constexpr (NT) __builtin_nontemporal_store(vs, reinterpret_cast<V *>(ws + p * F));
          else *reinterpret_cast<V *>(ws + p * F) = vs;
        }
      }
    }

    uLc = uLn;
    uRc = uRn;
    urC[0] = urN[0];
    urC[1] = urN[1];
    urC[2] = urN[2];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int k = 0; k < NPL; ++k) sgc[p][k] = sgn[p][k];
#pragma unroll
    for (int k = 0; k < NPL; ++k) {
      uPrev[k] = uCur[k];
      uCur[k] = uNext[k];
      Pc[k] = Pn[k];
      sdc[k] = sdn[k];
      mxc[k] = mxn[k];
      myc[k] = myn[k];
#pragma unroll
      for (int i = 0; i < 9; ++i) fc[i][k] = fn[i][k];
    }
  };

  // unrolled D times so that the ring slots are fixed registers
#pragma unroll 1
  for (int i = 0; i < nrows; i += D) {
#pragma unroll
    for (int j = 0; j < D; ++j)
      if (j == 0 || i + j < nrows) row_step(yfirst + dir * (i + j), S[j], S[(j + 1) % D]);
  }
}

// ---------------------------------------------------------------------------
// Two steps per launch for vector-class channels without the pressure
// drive (either stress model, any top wall; FP32 storage relative to the
// row references or plain FP64). One workgroup of two wavefronts takes an
// output strip of columns [x0, x1) and rows [y0, y1) through steps t and
// t+1 without writing step t to memory; each lane holds NPL adjacent nodes
// of a row:
//  * the window is the 64 NPL columns starting HL NPL columns left of x0
//    (HL = ceil(4 / NPL) lanes, wrapped periodically). A step's pull and its
//    stencil each need one more column on either side, so the window loses
//    two columns per step and the HL outermost lanes store nothing; no
//    columns beside the window are read;
//  * wavefront 0 runs stage A (step t): the vector sweep's row machine over
//    the window for rows max(y0-2, 0) .. min(y1+2, ny)-1, read from the
//    state; each row's post-collision populations and trace (and with the
//    time-integrated model the stress sigma(t)) go into a ring of four rows
//    in LDS instead of memory;
//  * wavefront 1 runs stage B (step t+1): the same machine reading its rows
//    from that ring, three rows behind stage A, and stores rows y0 .. y1-1
//    of lanes HL .. 63-HL to the other buffer.
// Each wavefront runs its own loop with one barrier per row, the same number
// in both. Splitting the stages over two wavefronts halves what each keeps in
// registers, so that more wavefronts fit a SIMD and one's arithmetic covers
// the other's waits. What a row's reference adds to its pulled populations
// (FP32) is formed once per launch, a lane per row, and read from LDS.
// Every stored node saw only values of the exact step-t state, and per node
// the arithmetic is the vector sweep's (same helpers, same pull, reference
// shifts and collision). A moving top wall takes each stage's own step's
// velocity.
//
// Bound by the memory path. On 4096 x 1024 (us per step; in brackets the same
// kernel with the node update left out): FP32 41.0 (39.2), time-integrated
// FP32 50.0 (52.6 before its bands marched in pairs), FP64 70.4 (68.9 to 75 with the alignment of its stores),
// time-integrated FP64 91.8; 16 x 8192 x 2048 FP32 2580 (2510). Before, with
// the columns beside the window read for stage A, row references formed per
// row and stage A's loads issued at the end of an iteration: 50.3, 60.7, 77.3,
// 108.5, 2790. What moved it: no side columns (the FP32 kernel 150 -> 130
// VGPRs, 22% fewer vector instructions), loads issued before the update
// (44.5 -> 42.6), every other launch marching downwards, so that it starts on
// the rows written last, the likeliest to sit in the last-level cache (42.6
// -> 41.4, time-integrated 62.7 -> 56.1), strips that end on whole lines
// (two_step_unit), and neighbouring bands that march against each other
// (time-integrated 52.0 -> 50.0, see add_two_step_strips). Not kept: loads two rows ahead (spills), one node per lane
// in FP64 (86), touching lines some rows ahead (47), four wavefronts per SIMD
// in FP32 (42.9), four nodes per lane for cached FP32 states (43.2).
constexpr int kV2Ring = 4;
// The row table (FP32): shifts of the pulled populations 2, 5, 6, 4, 7, 8,
// the row's reference, its share of d_y u_x (a fixed wall behind wall rows),
// and the reference below (mirrored at the bottom wall).
constexpr int kV2Tab = 9;

// LDS of a workgroup: the ring of step-t rows, populations and trace, and
// with VE the stress sigma(t) (sizeof(T) x NPL x 2.5 KB, x 3.25 KB with VE),
// and the row table.
template <typename T>
struct V2Rows {};
template <>
struct V2Rows<float> {
  float rtab[64][kV2Tab];
};
template <typename T, int NPL, bool VE>
struct V2Shared : V2Rows<T> {
  static constexpr int RP = kPlanes + (VE ? kStressPlanes : 0);
  typename Vec<T, NPL>::type ring[kV2Ring][RP][64];
};

// One strip, marched downwards or upwards.
template <typename T, int NPL, bool NT, bool VE, bool WALL, bool DOWN>
__device__ __forceinline__ void two_step_strip(const SweepArgs &a, const Strip &st, V2Shared<T, NPL, VE> &shared) {
  // FP32: storage relative to the row references; FP64: plain storage
  constexpr bool SHIFT = sizeof(T) == 4;
  constexpr int HL = (kTwoStepMargin + NPL - 1) / NPL;  // lanes per side that store nothing
  typedef typename Vec<T, NPL>::type V;
  constexpr int RP = V2Shared<T, NPL, VE>::RP;
  auto &ring = shared.ring;
  const int lane = threadIdx.x & 63;
  // wave 0 runs stage A, wave 1 stage B of the same strip
  const bool isA = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0;
  const ChanDev c = a.ch[st.ch];
  const T *__restrict__ A = static_cast<const T *>(a.A);
  T *__restrict__ B = static_cast<T *>(a.B);
  const int nx = c.nx, ny = c.ny;
  const long long ts = c.t + a.k + (isA ? 0 : 1);  // this stage's step
  const T fx = uniform((ts < c.t_startup) ? T(c.g) : T(0));
  // WALL: a moving top wall at this stage's step: its velocity (stencil
  // ghost) and, for the half-way wall, u_w/6 of step ts - 1, whose reflected
  // links step ts pulls; or the Zou-He completion of the top row
  const T uwg = uniform((WALL && ts < c.t_startup) ? T(c.uw) : T(0));
  const T uw6 = uniform((WALL && !c.zh && ts >= 1 && ts - 1 < c.t_startup) ? T(c.uw / 6.0) : T(0));
  const Coef<T> q(c);
  constexpr int F = kTile;
  const int tiles_row = nx >> 6;
  const long long row_stride = (long long)tiles_row * kPlanes * F, srow_stride = (long long)tiles_row * kStressPlanes * F;
  const T *const A0p = A + c.off * kPlanes;
  // this lane's first column, wrapped, as an element offset inside a row
  int col = st.x0 - HL * NPL + NPL * lane;
  col += (col < 0) ? nx : 0;
  col -= (col >= nx) ? nx : 0;
  const unsigned lcol = (unsigned)(col >> 6) * (kPlanes * F) + (col & 63);
  const unsigned scol = (unsigned)(col >> 6) * (kStressPlanes * F) + (col & 63);
  auto clampy = [&](int y) __attribute__((always_inline)) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };

  // ---- rows of the two stages
  const int A0 = st.y0 - 2 < 0 ? 0 : st.y0 - 2, A1 = st.y1 + 2 > ny ? ny : st.y1 + 2;
  // the march: rows first, first + step, ...; stage A's nA rows, stage B's
  // start from the row before its first (or its first, at the wall); the
  // iterations whose barriers both stages pass
  constexpr int step = DOWN ? -1 : 1;
  const int firstA = DOWN ? A1 - 1 : A0, nA = A1 - A0;
  const int firstB = DOWN ? st.y1 - 1 : st.y0, nB = st.y1 - st.y0;
  const int nIter = (DOWN ? A1 - 1 - st.y0 : st.y1 - 1 - A0) + 4;
  // stage B's stores: lanes whose columns lie in [x0, x1)
  const bool store_lane = lane >= HL && NPL * (lane - HL) < st.x1 - st.x0;
  // FP32: the table of rows A0-1 .. A0+62 (clamped; strips have at most 56
  // rows, so rows A0-1 .. A1 fit)
  if constexpr (SHIFT) {
    if (isA) {
      const int y = clampy(A0 - 1 + lane);
      const float *ur = a.uref + c.row_off;
      const bool bot = y == 0, top = y == ny - 1;
      const T urc = ur[y], urd = ur[bot ? y : y - 1], uru = ur[top ? y : y + 1];
      T sh[9] = {T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0)};
      to_row_reference(sh, urd, urc, uru, bot, top);
      T *w = shared.rtab[lane];
      w[0] = sh[2];
      w[1] = sh[5];
      w[2] = sh[6];
      w[3] = sh[4];
      w[4] = sh[7];
      w[5] = sh[8];
      w[6] = urc;
      const T d = bot ? -urc : urd;
      w[7] = T(0.5) * ((top ? -urc : uru) - d);
      w[8] = d;
    }
    __syncthreads();
  }

  // a row's values: pulled populations, P and the previous stress, moments
  // and u~ of the window's columns, and the row's reference
  struct Row {
    T f[9][NPL], P[NPL], sd[NPL], mx[NPL], my[NPL], sg[VE ? 3 : 1][NPL];
    T urc;
  };
  struct Raw {
    V r[10];
    V sg[VE ? 3 : 1];
  };
  // stage A: a row of the state (its pull's source rows, unshifted)
  auto load_raw = [&](int y, Raw &R) __attribute__((always_inline)) {
    const bool bot = (y == 0), top = (y == ny - 1);
    const T *rc = A0p + (long long)y * row_stride;
    const T *rd = bot ? rc : rc - row_stride, *ru = top ? rc : rc + row_stride;
    auto run = [&](const T *base, int p) __attribute__((always_inline)) {
      return *reinterpret_cast<const V *>(base + p * F + lcol);
    };
    R.r[0] = run(rc, 0);
    R.r[1] = run(rc, 1);
    R.r[3] = run(rc, 3);
    R.r[9] = run(rc, 9);
    R.r[2] = run(rd, bot ? 4 : 2);
    R.r[5] = run(rd, bot ? 7 : 5);
    R.r[6] = run(rd, bot ? 8 : 6);
    R.r[4] = run(ru, top ? 2 : 4);
    R.r[7] = run(ru, top ? 5 : 7);
    R.r[8] = run(ru, top ? 6 : 8);
    if constexpr (VE) {
      const T *sr = static_cast<const T *>(a.SA) + c.off * kStressPlanes + (long long)y * srow_stride;
#pragma unroll
      for (int p = 0; p < 3; ++p) R.sg[p] = *reinterpret_cast<const V *>(sr + p * F + scol);
    }
  };
  // stage B: the same row from the LDS ring of step-t rows
  auto load_lds = [&](int y, Raw &R) __attribute__((always_inline)) {
    const bool bot = (y == 0), top = (y == ny - 1);
    const int sc = y & (kV2Ring - 1), sd = bot ? sc : ((y - 1) & (kV2Ring - 1)), su = top ? sc : ((y + 1) & (kV2Ring - 1));
    R.r[0] = ring[sc][0][lane];
    R.r[1] = ring[sc][1][lane];
    R.r[3] = ring[sc][3][lane];
    R.r[9] = ring[sc][9][lane];
    R.r[2] = ring[sd][bot ? 4 : 2][lane];
    R.r[5] = ring[sd][bot ? 7 : 5][lane];
    R.r[6] = ring[sd][bot ? 8 : 6][lane];
    R.r[4] = ring[su][top ? 2 : 4][lane];
    R.r[7] = ring[su][top ? 5 : 7][lane];
    R.r[8] = ring[su][top ? 6 : 8][lane];
    if constexpr (VE) {
#pragma unroll
      for (int p = 0; p < 3; ++p) R.sg[p] = ring[sc][kPlanes + p][lane];
    }
  };

  // Row y from its raw values.
  auto assemble = [&](int y, const Raw &R, Row &w, U2<T> u[NPL]) __attribute__((always_inline)) {
    const bool bot = (y == 0), top = (y == ny - 1);
    auto from_left = [&](const V &r, T out[NPL]) __attribute__((always_inline)) {
      out[0] = shift_in_up(r[NPL - 1]);
#pragma unroll
      for (int k = 1; k < NPL; ++k) out[k] = r[k - 1];
    };
    auto from_right = [&](const V &r, T out[NPL]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NPL - 1; ++k) out[k] = r[k + 1];
      out[NPL - 1] = shift_in_down(r[0]);
    };
    auto split = [&](const V &r, T out[NPL]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NPL; ++k) out[k] = r[k];
    };
    T sh[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
    w.urc = T(0);
    if constexpr (SHIFT) {
      const T *tab = shared.rtab[y - (A0 - 1)];
#pragma unroll
      for (int j = 0; j < 6; ++j) sh[j] = tab[j];
      w.urc = tab[6];
    }
    split(R.r[0], w.f[0]);
    from_left(R.r[1], w.f[1]);
    from_right(R.r[3], w.f[3]);
    split(R.r[9], w.P);
    split(R.r[2], w.f[2]);
    split(R.r[4], w.f[4]);
    if (bot) {
      split(R.r[5], w.f[5]);
      split(R.r[6], w.f[6]);
    } else {
      from_left(R.r[5], w.f[5]);
      from_right(R.r[6], w.f[6]);
    }
    if (top) {
      split(R.r[7], w.f[7]);
      split(R.r[8], w.f[8]);
      if constexpr (WALL) {
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
          w.f[7][k] -= uw6;
          w.f[8][k] += uw6;
        }
      }
    } else {
      from_right(R.r[7], w.f[7]);
      from_left(R.r[8], w.f[8]);
    }
    const bool zhtop = WALL && top && c.zh;
#pragma unroll
    for (int k = 0; k < NPL; ++k) {
      T g[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) g[i] = w.f[i][k];
      if constexpr (SHIFT) {
#pragma clang fp contract(off)
        g[2] += sh[0];
        g[5] += sh[1];
        g[6] += sh[2];
        g[4] += sh[3];
        g[7] += sh[4];
        g[8] += sh[5];
      }
      if (zhtop) zou_he_top<T, SHIFT>(g, uwg, w.urc, fx);
#pragma unroll
      for (int i = 0; i < 9; ++i) w.f[i][k] = g[i];
      moments<T>(g, w.sd[k], w.mx[k], w.my[k]);
      u[k] = u_tilde<T, SHIFT>(w.sd[k], w.mx[k], w.my[k], fx, w.urc);
    }
#pragma unroll
    for (int p = 0; p < (VE ? 3 : 1); ++p)
#pragma unroll
      for (int k = 0; k < NPL; ++k) w.sg[p][k] = VE ? R.sg[p][k] : T(0);
  };

  // Update of row y from its assembled values and u~ of the rows below, at
  // and above it; out receives the new populations, trace (and stress).
  auto update = [&](int y, const Row &w, const U2<T> uPrev[NPL], const U2<T> uCur[NPL], const U2<T> uNext[NPL],
                    V out[RP]) __attribute__((always_inline)) {
    T kref = T(0);
    if constexpr (SHIFT) {
      const T *tab = shared.rtab[y - (A0 - 1)];
      kref = tab[7];
      if (WALL && y == ny - 1) {
        const T urd = tab[8];
        kref = T(0.5) * ((T(2) * uwg - (c.zh ? urd : w.urc)) - urd);
      }
    }
#pragma unroll
    for (int k = 0; k < NPL; ++k) {
      U2<T> lf, rt;
      if (k == 0) lf = U2<T>{shift_in_up(uCur[NPL - 1].x), shift_in_up(uCur[NPL - 1].y)};
      else lf = uCur[k - 1];
      if (k == NPL - 1) rt = U2<T>{shift_in_down(uCur[0].x), shift_in_down(uCur[0].y)};
      else rt = uCur[k + 1];
      U2<T> dn = DOWN ? uNext[k] : uPrev[k], up = DOWN ? uPrev[k] : uNext[k];
      if (y == 0) dn = U2<T>{-uCur[k].x, -uCur[k].y};
      // no-slip ghosts behind the half-way walls (moving at u_w above), or
      // behind a Zou-He node wall mirrored through the wall row
      if (y == ny - 1) {
        const U2<T> m = (WALL && c.zh) ? dn : uCur[k];
        up = U2<T>{(SHIFT ? T(0) : T(2) * uwg) - m.x, -m.y};
      }
      T g[9], o[9], tr, sn[3];
#pragma unroll
      for (int i = 0; i < 9; ++i) g[i] = w.f[i][k];
      const T sp[3] = {VE ? w.sg[0][k] : T(0), VE ? w.sg[VE ? 1 : 0][k] : T(0), VE ? w.sg[VE ? 2 : 0][k] : T(0)};
      double ob[OF_COUNT];
      node_update<T, SHIFT, false, VE>(g, w.sd[k], w.mx[k], w.my[k], w.P[k], fx, lf, rt, dn, up, w.urc, kref, q, c.nnp,
                                       sp, sn, o, tr, ob);
#pragma unroll
      for (int i = 0; i < 9; ++i) out[i][k] = o[i];
      out[9][k] = tr;
      if constexpr (VE) {
#pragma unroll
        for (int p = 0; p < 3; ++p) out[kPlanes + p][k] = sn[p];
      }
    }
  };
  auto copy_u = [&](U2<T> to[NPL], const U2<T> from[NPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < NPL; ++k) to[k] = from[k];
  };

  Row wa, wb;
  U2<T> uPrev[NPL], uCur[NPL], uNext[NPL];
  Raw R;
  if (isA) {
    // Iteration j, row y: assembles the next row from the loads issued in the
    // previous iteration, issues those of the row after it (rows clamped to
    // the lattice), in flight during the update and across the barrier, and
    // updates row y into ring slot y mod 4.
    {
      Raw Rp;
      const int yp = clampy(firstA - step);
      load_raw(yp, Rp);
      load_raw(firstA, R);
      assemble(yp, Rp, wb, uPrev);
      assemble(firstA, R, wa, uCur);
      load_raw(clampy(firstA + step), R);
    }
    auto iteration = [&](int y, const Row &cur, Row &next) __attribute__((always_inline)) {
      assemble(clampy(y + step), R, next, uNext);
      load_raw(clampy(y + 2 * step), R);
      V out[RP];
      update(y, cur, uPrev, uCur, uNext, out);
      const int slot = y & (kV2Ring - 1);
#pragma unroll
      for (int p = 0; p < RP; ++p) ring[slot][p][lane] = out[p];
      copy_u(uPrev, uCur);
      copy_u(uCur, uNext);
      __syncthreads();
    };
#pragma unroll 1
    for (int j = 0; j < nA; j += 2) {
      iteration(firstA + step * j, wa, wb);
      if (j + 1 >= nA) break;
      iteration(firstA + step * (j + 1), wb, wa);
    }
    for (int j = nA; j < nIter; ++j) __syncthreads();
  } else {
    // Three iterations behind stage A: in iteration j it assembles the row two
    // before stage A's row from the ring and updates the one before that.
    // Stage A writes its row meanwhile, so the barriers order its writes
    // before these reads and these before a slot is written again.
    const int start = clampy(firstB - step);
    for (int j = (start - firstA) * step + 2; j > 0; --j) __syncthreads();
    load_lds(start, R);
    assemble(start, R, wa, uCur);
    __syncthreads();
    if (start != firstB) {
      copy_u(uPrev, uCur);
      load_lds(firstB, R);
      assemble(firstB, R, wa, uCur);
      __syncthreads();
    }
    T *w = B + c.off * kPlanes + (long long)firstB * row_stride;
    T *ws = VE ? static_cast<T *>(a.SB) + c.off * kStressPlanes + (long long)firstB * srow_stride : nullptr;
    auto iteration = [&](int y, const Row &cur, Row &next) __attribute__((always_inline)) {
      const int yn = clampy(y + step);
      load_lds(yn, R);
      assemble(yn, R, next, uNext);
      V out[RP];
      update(y, cur, uPrev, uCur, uNext, out);
      if (store_lane) {
#pragma unroll
        for (int p = 0; p < kPlanes; ++p) {
          V *d = reinterpret_cast<V *>(w + p * F + lcol);
          if constexpr (NT) __builtin_nontemporal_store(out[p], d);
          else *d = out[p];
        }
        if constexpr (VE) {
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            V *d = reinterpret_cast<V *>(ws + p * F + scol);
            if constexpr (NT) __builtin_nontemporal_store(out[kPlanes + p], d);
            else *d = out[kPlanes + p];
          }
        }
      }
      w += step * row_stride;
      if constexpr (VE) ws += step * srow_stride;
      copy_u(uPrev, uCur);
      copy_u(uCur, uNext);
      __syncthreads();
    };
#pragma unroll 1
    for (int j = 0; j < nB; j += 2) {
      iteration(firstB + step * j, wa, wb);
      if (j + 1 >= nB) break;
      iteration(firstB + step * (j + 1), wb, wa);
    }
  }
}

template <typename T, int NPL, bool NT, bool VE, bool WALL>
__global__ void __launch_bounds__(64 * kTwoStepWaves, two_step_waves_per_simd(sizeof(T) == 4, NPL, VE))
    sweep_vec2_kernel(SweepArgs a) {
  __shared__ V2Shared<T, NPL, VE> shared;
  const int sidx = xcd_item(blockIdx.x, a.n_wg, a.down);
  if (sidx >= a.n_strips) return;  // the whole workgroup, before any barrier
  const Strip st = a.strips[sidx];
  if (st.flip != a.down) two_step_strip<T, NPL, NT, VE, WALL, true>(a, st, shared);
  else two_step_strip<T, NPL, NT, VE, WALL, false>(a, st, shared);
}

__global__ void __launch_bounds__(256) reduce_kernel(const ChanDev *ch, const double *part,
                                                     double *prof, double *prev_ux, double *scal,
                                                     const float *uref, int update_residual,
                                                     int steps_since) {
  const ChanDev c = ch[blockIdx.x];
  __shared__ double red[7][256];
  double mass = 0, momx = 0, flux = 0, drag = 0, umax = 0, dmax = 0, bad = 0;
  for (int y = threadIdx.x; y < c.ny; y += blockDim.x) {
    double rs[OF_COUNT];
#pragma unroll
    for (int f = 0; f < OF_COUNT; ++f) rs[f] = 0.0;
    for (int xs = 0; xs < c.nxs; ++xs) {
      const double *src = part + ((long long)c.poff + (long long)y * c.nxs + xs) * OF_COUNT;
#pragma unroll
      for (int f = 0; f < OF_COUNT; ++f) rs[f] += src[f];
    }
    // FP32 storage: the row's reference velocity, left out of the node
    // values of u_x, j_x and the wall momentum (0 for FP64)
    const double ur = (double)uref[c.row_off + y];
    rs[OF_UX] += c.nx * ur;
    rs[OF_MOMX] += c.nx * ur;
    if (y == 0) rs[OF_DRAG] -= c.nx * ur / 3.0;
    if (y == c.ny - 1) rs[OF_DRAG] -= c.nx * ur / (c.zh ? 6.0 : 3.0);
    double *dst = prof + ((long long)c.row_off + y) * OF_COUNT;
#pragma unroll
    for (int f = 0; f < OF_COUNT; ++f) {
      dst[f] = rs[f] / c.nx;
      if (!isfinite(rs[f])) bad = 1;
    }
    mass += rs[OF_MASS_DEV];
    momx += rs[OF_MOMX];
    flux += rs[OF_UX];
    drag += rs[OF_DRAG];
    const double ub = rs[OF_UX] / c.nx;
    umax = fmax(umax, fabs(ub));
    const double pv = prev_ux[c.row_off + y];
    const double d = fabs(ub - pv);
    dmax = (d != d) ? INFINITY : fmax(dmax, d);
    if (update_residual) prev_ux[c.row_off + y] = ub;
  }
  red[0][threadIdx.x] = mass;
  red[1][threadIdx.x] = momx;
  red[2][threadIdx.x] = flux;
  red[3][threadIdx.x] = drag;
  red[4][threadIdx.x] = umax;
  red[5][threadIdx.x] = dmax;
  red[6][threadIdx.x] = bad;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
      for (int k = 4; k < 7; ++k) red[k][threadIdx.x] = fmax(red[k][threadIdx.x], red[k][threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double *o = scal + (long long)blockIdx.x * CS_COUNT;
    o[CS_MASS_DEV] = red[0][0];
    o[CS_MOMX] = red[1][0];
    o[CS_FLUX] = red[2][0];
    o[CS_DRAG] = red[3][0];
    const double *pr = prof + (long long)c.row_off * OF_COUNT;
    const double um = (c.ny & 1) ? pr[(c.ny / 2) * OF_COUNT + OF_UX]
                                 : 0.5 * (pr[(c.ny / 2 - 1) * OF_COUNT + OF_UX] + pr[(c.ny / 2) * OF_COUNT + OF_UX]);
    o[CS_UMID] = um;
    o[CS_UMAX] = red[4][0];
    const bool nan = red[6][0] > 0;
    o[CS_NAN] = nan ? 1.0 : 0.0;
    if (update_residual) {
      // R = max_y |ubar(t) - ubar(t - K)| / (K max_y |ubar(t)|); +inf when a
      // previous profile is missing or the data are not finite
      const double dm = red[5][0], um2 = red[4][0];
      double R;
      if (nan || !(dm < INFINITY)) R = INFINITY;
      else if (um2 == 0.0) R = (dm == 0.0) ? 0.0 : INFINITY;
      else R = dm / ((double)steps_since * um2);
      o[CS_RESIDUAL] = R;
    }
  }
}

// The generalised periodic boundaries (gpbc_change) as a pass over the state
// a step has just written, for the channels that do not step in boxes
// (column_pass_takes). One workgroup per channel; the column means are taken
// before anything is changed.
//
// Bound by latency: one row of a column per thread, the inlet column in the
// first 256 threads and the outlet column in the others, so that all loads of
// both columns are in flight together and a row's populations stay in
// registers for the change (columns of up to 256 rows read memory once). In a
// tall column the lines count: there one thread takes both nodes of a row, the
// inlet node of a row lying beside the outlet node of the row before. us per
// step with the columns apart and together, FP32: 30 x 30000 1382 / 1041, 12 x
// 20000 367 / 319; FP64 12 x 20000 764 / 638, 5 x 50000 815 / 753; but FP32 30 x
// 3000 84.7 / 88.4, 18 x 5336 105 / 111, 4 x 30000 260 / 270, FP64 3 x 80000 792 /
// 865.
constexpr int kGpbcRows = 256;      // rows of a column taken at once
constexpr int kGpbcTall = 8192;     // rows above which a thread takes both nodes,
constexpr int kGpbcRowBytes = 40;   // if a row of a plane has as many bytes
template <typename T, bool SHIFT>
__global__ void __launch_bounds__(2 * kGpbcRows) gpbc_kernel(T *B, const ChanDev *ch, int k, const float *uref,
                                                             bool boxed) {
  const ChanDev c = ch[blockIdx.x];
  if (!column_pass_takes(c, boxed)) return;
  const long long t = c.t + k;
  const double dp = (t < c.t_startup) ? c.pd : 0.0;
  const int nx = c.nx, ny = c.ny;
  const int l = threadIdx.x & (kGpbcRows - 1);
  struct Node {
    double f[9], rho;
  };
  auto node = [&](int y, bool outlet) { return B + slot(0, c.off + (long long)y * nx + (outlet ? nx - 1 : 0)); };
  auto load9 = [&](int y, bool outlet, Node &q) {
    const T *b = node(y, outlet);
    double s = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) q.f[i] = (double)b[i * kTile];
#pragma unroll
    for (int i = 0; i < 9; ++i) s += q.f[i];
    q.rho = SHIFT ? 1.0 + s : s;
  };
  __shared__ double red[2][kGpbcRows];
  auto reduce = [&]() {
    __syncthreads();
    for (int st = kGpbcRows / 2; st > 0; st >>= 1) {
      if (l < st) red[threadIdx.x / kGpbcRows][l] += red[threadIdx.x / kGpbcRows][l + st];
      __syncthreads();
    }
  };
  auto fix = [&](int y, bool outlet, const Node &q) {
    // links leaving the outlet enter the inlet, and the other way round
    const double d = outlet ? 1.0 + 1.5 * dp - red[1][0] / ny : 1.0 - 1.5 * dp - red[0][0] / ny;
    T *b = node(y, outlet);
    gpbc_change<SHIFT>(q.f, SHIFT ? (double)uref[c.row_off + y] : 0.0, d, outlet, y, ny,
                       [&](int i, double v) { b[i * kTile] = (T)v; });
  };
  if (ny <= kGpbcTall || nx * (int)sizeof(T) < kGpbcRowBytes) {
    const bool outlet = __builtin_amdgcn_readfirstlane(threadIdx.x / kGpbcRows) != 0;
    Node first;
    double sum = 0;
    if (l < ny) {
      load9(l, outlet, first);
      sum = first.rho;
    }
    for (int y = l + kGpbcRows; y < ny; y += kGpbcRows) {
      Node q;
      load9(y, outlet, q);
      sum += q.rho;
    }
    red[outlet][l] = sum;
    reduce();
    if (l < ny) fix(l, outlet, first);
    for (int y = l + kGpbcRows; y < ny; y += kGpbcRows) {
      Node q;
      load9(y, outlet, q);
      fix(y, outlet, q);
    }
    return;
  }
  if (threadIdx.x < kGpbcRows) {
    double in = 0, out = 0;
#pragma unroll 2
    for (int y = l; y < ny; y += kGpbcRows) {
      Node q;
      load9(y, false, q);
      in += q.rho;
      load9(y, true, q);
      out += q.rho;
    }
    red[0][l] = in;
    red[1][l] = out;
  }
  reduce();
  for (int y = threadIdx.x; y < ny; y += 2 * kGpbcRows) {
    Node in, out;
    load9(y, false, in);
    load9(y, true, out);
    fix(y, false, in);
    fix(y, true, out);
  }
}

// FP32 storage: moves the reference velocity of every row of the active
// channels to the row's current x-averaged u_x (prof, from the last
// observation) and restates the stored populations of the row: a value
// stored relative to E_i(uo) becomes one relative to E_i(un) by adding
// E_i(uo) - E_i(un), formed as a difference. One workgroup per row.
__global__ void __launch_bounds__(256) rereference_kernel(float *A, const ChanDev *ch, int n_ch,
                                                          const double *prof, float *uref) {
  const int r = blockIdx.x;  // row over all channels
  int lo = 0, hi = n_ch - 1;
  while (lo < hi) {  // the channel holding row r: last one with row_off <= r
    const int mid = (lo + hi + 1) / 2;
    if (ch[mid].row_off <= r) lo = mid;
    else hi = mid - 1;
  }
  const ChanDev c = ch[lo];
  if (!c.active) return;
  const float uo = uref[r];
  const double unx = prof[(long long)r * OF_COUNT + OF_UX];
  if (!(unx == unx) || fabs(unx) > 1.0) return;  // not finite or not a velocity: keep the old one
  const float un = (float)unx;
  float d[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const float cx = (i == 1 || i == 5 || i == 8) ? 1.f : ((i == 3 || i == 6 || i == 7) ? -1.f : 0.f);
    d[i] = ref_shift(weight<float>(i), cx, uo, un);
  }
  const int y = r - c.row_off;
  for (int x = threadIdx.x; x < c.nx; x += blockDim.x) {
    const long long n = c.off + (long long)y * c.nx + x;
#pragma unroll
    for (int i = 0; i < 9; ++i) A[slot(i, n)] += d[i];
  }
  __syncthreads();
  if (threadIdx.x == 0) uref[r] = un;
}

// ---------------------------------------------------------------------------
// Stress as a force density (FP64, instantaneous model): the divergence of
// the non-Newtonian stress enters as an external force in Eq. (ns), the
// alternative Sec. II.C names. A step forms u~ at every node, Sigma^nN from
// the neighbours' u~, then collides with the force f = rho0 g + div Sigma^nN
// (central differences, ghost rows extrapolated linearly through the walls)
// in the body-force terms of the forcing. The step runs as one fused kernel
// over tiles (saf_fused_kernel), on small lattices many steps at a time in
// boxes (sweep_block_kernel); observation runs the same stages as
// node-wise passes over every channel, with scratch U (u~_x, u~_y) and T
// (Sigma^nN xx, xy, yy), plane-major over the nodes of the buffer.

// Channel holding node n (channels are laid out by increasing offset).
__device__ __forceinline__ int channel_of_node(const ChanDev *ch, int n_ch, long long n) {
  int lo = 0, hi = n_ch - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (ch[mid].off <= n) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

struct SafNode {
  ChanDev c;
  int x, y;
  long long t;
};

// Decodes node n; false for padding nodes and (unless all) frozen channels.
__device__ __forceinline__ bool saf_node(const ChanDev *ch, int n_ch, long long n, int k, bool all, SafNode &s) {
  s.c = ch[channel_of_node(ch, n_ch, n)];
  const long long loc = n - s.c.off;
  if (loc < 0 || loc >= (long long)s.c.nx * s.c.ny) return false;
  if (!all && !s.c.active) return false;
  s.y = (int)(loc / s.c.nx);
  s.x = (int)(loc - (long long)s.y * s.c.nx);
  s.t = s.c.t + k;
  return true;
}

// x and y neighbours' values of a node field F (plane-major, plane nodes),
// with the ghost rule of the caller.
__global__ void __launch_bounds__(256) saf_u_kernel(const double *__restrict__ A, const ChanDev *ch, int n_ch,
                                                    long long plane, int k, int all, double *__restrict__ U) {
  for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < plane;
       n += (long long)gridDim.x * blockDim.x) {
    SafNode q;
    if (!saf_node(ch, n_ch, n, k, all, q)) continue;
    const double g = (q.t < q.c.t_startup) ? q.c.g : 0.0;
    const double uw6 = (q.t >= 1 && q.t - 1 < q.c.t_startup) ? q.c.uw / 6.0 : 0.0;
    double f[9], sd, mx, my;
    pull<double>(A, q.c.off + (long long)q.y * q.c.nx, q.c.nx, q.c.ny, q.x, q.y, uw6, f);
    moments<double>(f, sd, mx, my);
    U[n] = (mx + 0.5 * g) / sd;
    U[plane + n] = my / sd;
  }
}

// kappa_ab = d_b u~_a of a node by central differences (x periodic; wall
// ghosts -u~ below, 2 u_w - u~ above for x, -u~ for y).
__device__ __forceinline__ void saf_kappa(const double *__restrict__ U, long long plane, const SafNode &q,
                                          double &kxx, double &kxy, double &kyx, double &kyy) {
  const ChanDev &c = q.c;
  const long long row = c.off + (long long)q.y * c.nx;
  const long long n = row + q.x;
  const int xm = (q.x == 0) ? c.nx - 1 : q.x - 1, xp = (q.x == c.nx - 1) ? 0 : q.x + 1;
  const double uwg = (q.t < c.t_startup) ? c.uw : 0.0;
  const double ux = U[n], uy = U[plane + n];
  const double uxd = (q.y > 0) ? U[n - c.nx] : -ux, uyd = (q.y > 0) ? U[plane + n - c.nx] : -uy;
  const double uxu = (q.y < c.ny - 1) ? U[n + c.nx] : 2.0 * uwg - ux;
  const double uyu = (q.y < c.ny - 1) ? U[plane + n + c.nx] : -uy;
  kxx = 0.5 * (U[row + xp] - U[row + xm]);
  kxy = 0.5 * (uxu - uxd);
  kyx = 0.5 * (U[plane + row + xp] - U[plane + row + xm]);
  kyy = 0.5 * (uyu - uyd);
}

__global__ void __launch_bounds__(256) saf_stress_kernel(const ChanDev *ch, int n_ch, long long plane, int k,
                                                         int all, const double *__restrict__ U,
                                                         double *__restrict__ Tn) {
  for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < plane;
       n += (long long)gridDim.x * blockDim.x) {
    SafNode q;
    if (!saf_node(ch, n_ch, n, k, all, q)) continue;
    double kxx, kxy, kyx, kyy;
    saf_kappa(U, plane, q, kxx, kxy, kyx, kyy);
    const Coef<double> cf(q.c);
    double sxx = 0, sxy = 0, syy = 0;
    if (cf.stress_on) inlm_stress<double>(kxx, kxy, kyx, kyy, cf, sxx, sxy, syy);
    Tn[n] = sxx - cf.lgt * 2.0 * kxx;
    Tn[plane + n] = sxy - cf.lgt * (kxy + kyx);
    Tn[2 * plane + n] = syy - cf.lgt * 2.0 * kyy;
  }
}

// f_Sigma = div Sigma^nN at a node: central differences, x periodic, ghost
// rows Sigma(-1) = 2 Sigma(0) - Sigma(1), Sigma(ny) = 2 Sigma(ny-1) -
// Sigma(ny-2) (one row: zero gradient).
__device__ __forceinline__ void saf_force(const double *__restrict__ Tn, long long plane, const SafNode &q,
                                          double &fsx, double &fsy) {
  const ChanDev &c = q.c;
  const long long row = c.off + (long long)q.y * c.nx;
  const long long n = row + q.x;
  const int xm = (q.x == 0) ? c.nx - 1 : q.x - 1, xp = (q.x == c.nx - 1) ? 0 : q.x + 1;
  double dn[3], up[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double *P = Tn + p * plane;
    if (c.ny == 1) {
      dn[p] = up[p] = P[n];
    } else {
      dn[p] = (q.y > 0) ? P[n - c.nx] : 2.0 * P[n] - P[n + c.nx];
      up[p] = (q.y < c.ny - 1) ? P[n + c.nx] : 2.0 * P[n] - P[n - c.nx];
    }
  }
  fsx = 0.5 * (Tn[row + xp] - Tn[row + xm]) + 0.5 * (up[1] - dn[1]);
  fsy = 0.5 * (Tn[plane + row + xp] - Tn[plane + row + xm]) + 0.5 * (up[2] - dn[2]);
}

// One step of the stress-force path fused in one kernel, one workgroup per
// tile of kSafTX x kSafTY output nodes, each thread taking a column of
// kSafNPT of them (kSafRows rows apart): the taller tile repeats less of
// the ring work per node than one node per thread would, at the same
// number of wavefronts per CU. Each XCD takes a contiguous run of the tile
// list, which the host orders so that a run is a block of neighbouring
// tiles: adjacent tiles share the halo populations they pull and then find
// them in that XCD's L2. Each thread pulls its nodes and keeps the
// populations; u~ of the tile and of a ring of two nodes around it go to
// LDS, then Sigma^nN of the tile and a ring of one node, then each thread
// collides its nodes with div Sigma^nN from LDS. Columns wrap (x periodic;
// narrow channels repeat columns); rows outside the channel are the wall
// ghosts of saf_kappa and saf_force. The arithmetic is that of the three
// separate passes. 4096 x 1024: 124 us, 5.5 TB/s, what a large copy reaches.
constexpr int kSafTX = kSafTileX, kSafTY = kSafTileY;
constexpr int kSafRows = kSafThreads / kSafTX;            // rows of threads
constexpr int kSafNPT = kSafTY / kSafRows;                // output nodes per thread
constexpr int kSafUX = kSafTX + 4, kSafUY = kSafTY + 4;  // u~ region
constexpr int kSafSX = kSafTX + 2, kSafSY = kSafTY + 2;  // Sigma^nN region
constexpr int kSafRing = 4 * kSafUX + 4 * kSafTY;       // u~ region minus the tile
static_assert(kSafRows * kSafTX == kSafThreads && kSafNPT * kSafRows == kSafTY,
              "a whole column of output nodes per thread");
static_assert(kSafRing <= kSafThreads, "at most one ring node per thread");

template <bool NT>
__global__ void __launch_bounds__(kSafThreads) saf_fused_kernel(const double *__restrict__ A,
                                                                double *__restrict__ B, const ChanDev *ch,
                                                                const Strip *tiles, int k, int down) {
  __shared__ double su[2][kSafUY][kSafUX];
  __shared__ double sT[3][kSafSY][kSafSX];
  const int item = xcd_item(blockIdx.x, gridDim.x, down);
  const Strip tl = tiles[item];
  const ChanDev c = ch[tl.ch];
  if (!c.active) return;  // frozen channel (uniform over the workgroup)
  const int nx = c.nx, ny = c.ny;
  const long long t = c.t + k;
  const double g = (t < c.t_startup) ? c.g : 0.0;
  const double uwg = (t < c.t_startup) ? c.uw : 0.0;
  const double uw6 = (!c.zh && t >= 1 && t - 1 < c.t_startup) ? c.uw / 6.0 : 0.0;
  const Coef<double> cf(c);
  const double *__restrict__ Ac = A + c.off * kPlanes;
  double *__restrict__ Bc = B + c.off * kPlanes;
  const bool wide = nx >= kSafTX + 4;  // then halo columns wrap at most once
  auto wrapx = [&](int x) {
    if (wide) return x < 0 ? x + nx : (x >= nx ? x - nx : x);
    const int r = x % nx;
    return r < 0 ? r + nx : r;
  };
  auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
  // This thread's nodes (a column of kSafNPT, kSafRows rows apart), whose
  // populations it keeps to the collision, and (threads below kSafRing) one
  // node of the ring of two around the tile: two rows below, two above, two
  // columns on either side. All are pulled before any is used, so that
  // their loads overlap; rows outside the channel pull a row inside and
  // store nothing.
  const int jo = threadIdx.x / kSafTX, io = threadIdx.x - jo * kSafTX;
  const int xo = tl.x0 + io, xw = wrapx(xo);
  const int h = threadIdx.x;
  int hj, hi;
  if (h < 2 * kSafUX) {
    hj = h / kSafUX;
    hi = h - hj * kSafUX;
  } else if (h < 4 * kSafUX) {
    const int r = h - 2 * kSafUX;
    hj = kSafTY + 2 + r / kSafUX;
    hi = r % kSafUX;
  } else {
    const int r = h - 4 * kSafUX, side = r & 3;
    hj = 2 + (r >> 2);
    hi = side < 2 ? side : kSafUX - 4 + side;
  }
  const int hy = tl.y0 - 2 + hj;
  const bool ring = h < kSafRing;
  double f[kSafNPT][9], fh[9], Pc[kSafNPT];
  unsigned m[kSafNPT];
#pragma unroll
  for (int s = 0; s < kSafNPT; ++s) {
    const int yc = clampy(tl.y0 + jo + s * kSafRows);
    m[s] = (unsigned)yc * nx + xw;
    pull_local(Ac, nx, ny, xw, yc, uw6, f[s]);
    Pc[s] = Ac[lslot(9, m[s])];
  }
  if (ring) pull_local(Ac, nx, ny, wrapx(tl.x0 - 2 + hi), clampy(hy), uw6, fh);
  double sd[kSafNPT], mx[kSafNPT], my[kSafNPT], inv[kSafNPT];
#pragma unroll
  for (int s = 0; s < kSafNPT; ++s) {
    moments<double>(f[s], sd[s], mx[s], my[s]);
    inv[s] = recip<double>(sd[s]);  // shared with the collision
    if (tl.y0 + jo + s * kSafRows < ny) {
      const U2<double> u = u_tilde<double, false>(sd[s], mx[s], my[s], g, 0.0);
      su[0][jo + s * kSafRows + 2][io + 2] = u.x;
      su[1][jo + s * kSafRows + 2][io + 2] = u.y;
    }
  }
  if (ring && hy >= 0 && hy < ny) {
    double hs, hx, hv;
    moments<double>(fh, hs, hx, hv);
    const U2<double> u = u_tilde<double, false>(hs, hx, hv, g, 0.0);
    su[0][hj][hi] = u.x;
    su[1][hj][hi] = u.y;
  }
  __syncthreads();
  // Sigma^nN of the tile and a ring of one node (kappa with the wall ghosts)
  for (int i = threadIdx.x; i < kSafSX * kSafSY; i += kSafThreads) {
    const int j = i / kSafSX, ii = i - j * kSafSX;
    const int y = tl.y0 - 1 + j;
    if (y < 0 || y >= ny) continue;
    const int ju = j + 1, iu = ii + 1;
    const double ux = su[0][ju][iu], uy = su[1][ju][iu];
    const double uxd = (y > 0) ? su[0][ju - 1][iu] : -ux, uyd = (y > 0) ? su[1][ju - 1][iu] : -uy;
    const double uxu = (y < ny - 1) ? su[0][ju + 1][iu] : 2.0 * uwg - ux;
    const double uyu = (y < ny - 1) ? su[1][ju + 1][iu] : -uy;
    const double kxx = 0.5 * (su[0][ju][iu + 1] - su[0][ju][iu - 1]);
    const double kxy = 0.5 * (uxu - uxd);
    const double kyx = 0.5 * (su[1][ju][iu + 1] - su[1][ju][iu - 1]);
    const double kyy = 0.5 * (uyu - uyd);
    double sxx = 0, sxy = 0, syy = 0;
    if (cf.stress_on) inlm_stress<double>(kxx, kxy, kyx, kyy, cf, sxx, sxy, syy);
    sT[0][j][ii] = sxx - cf.lgt * 2.0 * kxx;
    sT[1][j][ii] = sxy - cf.lgt * (kxy + kyx);
    sT[2][j][ii] = syy - cf.lgt * 2.0 * kyy;
  }
  __syncthreads();
  // collide and stream this thread's nodes
  if (xo >= nx) return;
#pragma unroll
  for (int s = 0; s < kSafNPT; ++s) {
    const int yo = tl.y0 + jo + s * kSafRows;
    if (yo >= tl.y1) continue;
    const int n = (jo + s * kSafRows + 1) * kSafSX + io + 1;
    saf_collide(f[s], sd[s], inv[s], mx[s], my[s], g, c.omega, c.kf, &sT[0][0][0], kSafSX * kSafSY, n, n - 1, n + 1,
                -kSafSX, kSafSX, yo, ny, [&](int q, double v) __attribute__((always_inline)) {
                  if constexpr (NT) __builtin_nontemporal_store(v, &Bc[lslot(q, m[s])]);
                  else Bc[lslot(q, m[s])] = v;
                });
    if constexpr (NT) __builtin_nontemporal_store(Pc[s], &Bc[lslot(9, m[s])]);
    else Bc[lslot(9, m[s])] = Pc[s];
  }
}

// Observation of the stress-force path: one workgroup per row of every
// channel; the row sums go to the row's first x-strip partial (the others
// are zeroed) for reduce_kernel.
__global__ void __launch_bounds__(256) saf_observe_kernel(const double *__restrict__ A, const ChanDev *ch,
                                                          int n_ch, long long plane, const double *__restrict__ U,
                                                          const double *__restrict__ Tn, double *part) {
  __shared__ double red[OF_COUNT][256];
  const int r = blockIdx.x;
  int lo = 0, hi = n_ch - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (ch[mid].row_off <= r) lo = mid;
    else hi = mid - 1;
  }
  const ChanDev c = ch[lo];
  SafNode q;
  q.c = c;
  q.y = r - c.row_off;
  q.t = c.t;
  double acc[OF_COUNT];
#pragma unroll
  for (int f = 0; f < OF_COUNT; ++f) acc[f] = 0.0;
  const double g = (q.t < c.t_startup) ? c.g : 0.0;
  const double uw6 = (q.t >= 1 && q.t - 1 < c.t_startup) ? c.uw / 6.0 : 0.0;
  const Coef<double> cf(c);
  for (int x = threadIdx.x; x < c.nx; x += blockDim.x) {
    q.x = x;
    const long long n = c.off + (long long)q.y * c.nx + x;
    double f[9], sd, mx, my;
    pull<double>(A, c.off + (long long)q.y * c.nx, c.nx, c.ny, x, q.y, uw6, f);
    moments<double>(f, sd, mx, my);
    double kxx, kxy, kyx, kyy, fsx, fsy;
    saf_kappa(U, plane, q, kxx, kxy, kyx, kyy);
    saf_force(Tn, plane, q, fsx, fsy);
    double sxx = 0, sxy = 0, syy = 0;
    if (cf.stress_on) inlm_stress<double>(kxx, kxy, kyx, kyy, cf, sxx, sxy, syy);
    acc[OF_UX] += (mx + 0.5 * (g + fsx)) / sd;
    acc[OF_UY] += (my + 0.5 * fsy) / sd;
    acc[OF_SXX] += sxx;
    acc[OF_SXY] += sxy;
    acc[OF_SYY] += syy;
    acc[OF_RHOE_DEV] += sd - 1.0;
    acc[OF_MASS_DEV] += sd - 1.0;
    acc[OF_MOMX] += mx;
    acc[OF_KXY] += kxy;
    acc[OF_TRT] += Tn[n] + Tn[2 * plane + n];
    acc[OF_DRAG] += wall_drag<double>(f, q.y, c.ny, uw6, false, 0.0);
    acc[OF_KXX] += kxx;
  }
#pragma unroll
  for (int f = 0; f < OF_COUNT; ++f) red[f][threadIdx.x] = acc[f];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int f = 0; f < OF_COUNT; ++f) red[f][threadIdx.x] += red[f][threadIdx.x + st];
    __syncthreads();
  }
  double *dst = part + ((long long)c.poff + (long long)q.y * c.nxs) * OF_COUNT;
  for (int i = threadIdx.x; i < c.nxs * OF_COUNT; i += blockDim.x) dst[i] = (i < OF_COUNT) ? red[i][0] : 0.0;
}

__global__ void advance_kernel(ChanDev *ch, int n_ch, int steps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_ch && ch[i].active) ch[i].t += steps;
}

template <typename T, bool SHIFT, int TXW, bool WIDE, bool VE>
hipError_t launch_cls(bool observe, const SweepArgs &a, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  dim3 grid(a.n_wg), block(64 * LB_WG_WAVES);
  if (observe)
    hipLaunchKernelGGL((sweep_kernel<T, SHIFT, TXW, WIDE, true, VE>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((sweep_kernel<T, SHIFT, TXW, WIDE, false, VE>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <typename T, bool SHIFT, bool VE>
hipError_t launch_wide64(bool observe, const SweepArgs &a, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  dim3 grid(a.n_wg), block(64 * LB_WG_WAVES);
  if (observe)
    hipLaunchKernelGGL((sweep_wide64_kernel<T, SHIFT, true, VE>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((sweep_wide64_kernel<T, SHIFT, false, VE>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <typename T, bool SHIFT, bool VE>
hipError_t launch_vec(bool observe, const SweepArgs &a, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  constexpr int NPL = sizeof(T) == 4 ? LB_VEC_NPL32 : LB_VEC_NPL64;
  dim3 grid(a.n_wg), block(64 * LB_WG_WAVES);
  if (observe)
    hipLaunchKernelGGL((sweep_vec_kernel<T, SHIFT, true, NPL, false, VE, true>), grid, block, 0, s, a);
  else if (a.zh && a.nt)
    hipLaunchKernelGGL((sweep_vec_kernel<T, SHIFT, false, NPL, true, VE, true>), grid, block, 0, s, a);
  else if (a.zh)
    hipLaunchKernelGGL((sweep_vec_kernel<T, SHIFT, false, NPL, false, VE, true>), grid, block, 0, s, a);
  else if (a.nt)
    hipLaunchKernelGGL((sweep_vec_kernel<T, SHIFT, false, NPL, true, VE, false>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((sweep_vec_kernel<T, SHIFT, false, NPL, false, VE, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <typename T, bool SHIFT, bool VE>
hipError_t launch_model(int cls, bool observe, const SweepArgs &a, hipStream_t s) {
  switch (cls) {
    case 0: return launch_cls<T, SHIFT, 1, false, VE>(observe, a, s);
    case 1: return launch_cls<T, SHIFT, 2, false, VE>(observe, a, s);
    case 2: return launch_cls<T, SHIFT, 4, false, VE>(observe, a, s);
    case 3: return launch_cls<T, SHIFT, 8, false, VE>(observe, a, s);
    case 4: return launch_cls<T, SHIFT, 16, false, VE>(observe, a, s);
    case 5: return launch_cls<T, SHIFT, 32, false, VE>(observe, a, s);
    case 6: return launch_cls<T, SHIFT, 64, false, VE>(observe, a, s);
    case kWide64Class: return launch_wide64<T, SHIFT, VE>(observe, a, s);
    case kVecClass: return launch_vec<T, SHIFT, VE>(observe, a, s);
    default: return launch_cls<T, SHIFT, 64, true, VE>(observe, a, s);
  }
}

template <typename T, bool SHIFT>
hipError_t launch_prec(int cls, bool observe, const SweepArgs &a, hipStream_t s) {
  if (a.ve) {
    if (!a.SA || !a.SB) return hipErrorInvalidValue;
    return launch_model<T, SHIFT, true>(cls, observe, a, s);
  }
  return launch_model<T, SHIFT, false>(cls, observe, a, s);
}

}  // namespace

hipError_t launch_sweep(int fp32, int cls, bool observe, const SweepArgs &a, hipStream_t s) {
  return fp32 ? launch_prec<float, true>(cls, observe, a, s)
              : launch_prec<double, false>(cls, observe, a, s);
}

hipError_t launch_tiles(const SweepArgs &a, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  const dim3 grid(a.n_strips), block(kMainThreads);
  if (a.ve) {
    if (a.nt) hipLaunchKernelGGL((sweep_tile_kernel<true, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sweep_tile_kernel<true, false>), grid, block, 0, s, a);
  } else {
    if (a.nt) hipLaunchKernelGGL((sweep_tile_kernel<false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sweep_tile_kernel<false, false>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

template <typename T, bool VE, bool GP, bool SAF>
hipError_t launch_block_t(int threads, const SweepArgs &a, int S, hipStream_t s) {
  const dim3 grid(a.n_wg), block(threads);
  switch (threads) {
    case 256: hipLaunchKernelGGL((sweep_block_kernel<T, VE, GP, SAF, 256>), grid, block, 0, s, a, S); break;
    case 512: hipLaunchKernelGGL((sweep_block_kernel<T, VE, GP, SAF, 512>), grid, block, 0, s, a, S); break;
    case 1024: hipLaunchKernelGGL((sweep_block_kernel<T, VE, GP, SAF, 1024>), grid, block, 0, s, a, S); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_blocks(bool fp32, bool gpbc, bool stress_force, int threads, const SweepArgs &a, int S, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  if (a.ve && (!a.SA || !a.SB)) return hipErrorInvalidValue;
  if (stress_force)
    return fp32 || gpbc || a.ve ? hipErrorInvalidValue : launch_block_t<double, false, false, true>(threads, a, S, s);
#define LB_BLOCKS(VE, GP)                                       \
  (fp32 ? launch_block_t<float, VE, GP, false>(threads, a, S, s) \
        : launch_block_t<double, VE, GP, false>(threads, a, S, s))
  if (gpbc) return a.ve ? LB_BLOCKS(true, true) : LB_BLOCKS(false, true);
  return a.ve ? LB_BLOCKS(true, false) : LB_BLOCKS(false, false);
#undef LB_BLOCKS
}

hipError_t launch_reduce(const ChanDev *ch, int n_ch, const double *part, double *prof,
                         double *prev_ux, double *scal, const float *uref, int update_residual,
                         int steps_since, hipStream_t s) {
  if (n_ch == 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_kernel, dim3(n_ch), dim3(256), 0, s, ch, part, prof, prev_ux, scal, uref,
                     update_residual, steps_since);
  return hipGetLastError();
}

hipError_t launch_gpbc(int fp32, void *B, const ChanDev *ch, int n_ch, int k, const float *uref, bool boxed,
                       hipStream_t s) {
  if (n_ch == 0) return hipSuccess;
  if (fp32)
    hipLaunchKernelGGL((gpbc_kernel<float, true>), dim3(n_ch), dim3(2 * kGpbcRows), 0, s, static_cast<float *>(B),
                       ch, k, uref, boxed);
  else
    hipLaunchKernelGGL((gpbc_kernel<double, false>), dim3(n_ch), dim3(2 * kGpbcRows), 0, s,
                       static_cast<double *>(B), ch, k, uref, boxed);
  return hipGetLastError();
}

template <typename T, int NPL, bool VE, bool WALL>
void launch_two_step_w(const SweepArgs &a, hipStream_t s) {
  const dim3 grid(a.n_wg), block(64 * kTwoStepWaves);
  if (a.nt) hipLaunchKernelGGL((sweep_vec2_kernel<T, NPL, true, VE, WALL>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sweep_vec2_kernel<T, NPL, false, VE, WALL>), grid, block, 0, s, a);
}
template <typename T, int NPL, bool VE>
void launch_two_step_t(const SweepArgs &a, hipStream_t s) {
  if (a.wall) launch_two_step_w<T, NPL, VE, true>(a, s);
  else launch_two_step_w<T, NPL, VE, false>(a, s);
}

hipError_t launch_narrow_two_step(bool fp32, int nx, const SweepArgs &a, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  const dim3 grid(a.n_wg), block(128);
#define LB_N2(TT, SH, W) hipLaunchKernelGGL((sweep_narrow2_kernel<TT, SH, W>), grid, block, 0, s, a)
#define LB_N2_ALL(TT, SH)  \
  switch (nx) {            \
    case 32: LB_N2(TT, SH, 32); break; \
    case 64: LB_N2(TT, SH, 64); break; \
    default: return hipErrorInvalidValue; \
  }
  if (fp32) {
    LB_N2_ALL(float, true)
  } else {
    LB_N2_ALL(double, false)
  }
#undef LB_N2_ALL
#undef LB_N2
  return hipGetLastError();
}

template <typename T, bool SH>
int narrow2_blocks_per_cu() {
  int lo = 1 << 30;
  auto q = [&](const void *f) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 128, 0) == hipSuccess && n > 0) lo = std::min(lo, n);
  };
  q(reinterpret_cast<const void *>(sweep_narrow2_kernel<T, SH, 32>));
  q(reinterpret_cast<const void *>(sweep_narrow2_kernel<T, SH, 64>));
  return lo == (1 << 30) ? 1 : lo;
}

int narrow_two_step_blocks_per_cu(bool fp32) {
  return fp32 ? narrow2_blocks_per_cu<float, true>() : narrow2_blocks_per_cu<double, false>();
}

hipError_t launch_two_step(bool fp32, const SweepArgs &a, hipStream_t s) {
  if (a.n_strips == 0) return hipSuccess;
  if (a.ve && (!a.SA || !a.SB)) return hipErrorInvalidValue;
  const int npl = two_step_npl(fp32, a.nt, a.ve);
  if (fp32 && npl == 4) {
    launch_two_step_t<float, 4, false>(a, s);
  } else if (fp32) {
    if (a.ve) launch_two_step_t<float, 2, true>(a, s);
    else launch_two_step_t<float, 2, false>(a, s);
  } else {
    if (a.ve) launch_two_step_t<double, 2, true>(a, s);
    else launch_two_step_t<double, 2, false>(a, s);
  }
  return hipGetLastError();
}

int two_step_blocks_per_cu(bool fp32, bool nt, bool ve) {
  int n = 0;
  constexpr int b = 64 * kTwoStepWaves;
  hipError_t e;
  if (fp32 && two_step_npl(fp32, nt, ve) == 4)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_vec2_kernel<float, 4, true, false, false>, b, 0);
  else if (fp32)
    e = ve ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_vec2_kernel<float, 2, false, true, false>, b, 0)
           : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_vec2_kernel<float, 2, false, false, false>, b, 0);
  else
    e = ve ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_vec2_kernel<double, 2, false, true, false>, b, 0)
           : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sweep_vec2_kernel<double, 2, false, false, false>, b, 0);
  return (e == hipSuccess && n > 0) ? n : 1;
}

hipError_t launch_rereference(float *A, const ChanDev *ch, int n_ch, int total_rows, const double *prof,
                              float *uref, hipStream_t s) {
  if (n_ch == 0 || total_rows == 0) return hipSuccess;
  hipLaunchKernelGGL(rereference_kernel, dim3(total_rows), dim3(256), 0, s, A, ch, n_ch, prof, uref);
  return hipGetLastError();
}

static int saf_blocks(long long plane) {
  const long long b = (plane + 255) / 256;
  return (int)(b < 16384 ? b : 16384);
}

hipError_t launch_saf_fused(const double *A, double *B, const ChanDev *ch, const Strip *tiles, int n_tiles, int k,
                            int nt, int down, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  if (nt) hipLaunchKernelGGL(saf_fused_kernel<true>, dim3(n_tiles), dim3(kSafThreads), 0, s, A, B, ch, tiles, k,
                             down);
  else hipLaunchKernelGGL(saf_fused_kernel<false>, dim3(n_tiles), dim3(kSafThreads), 0, s, A, B, ch, tiles, k, down);
  return hipGetLastError();
}

hipError_t launch_saf_observe(const double *A, const ChanDev *ch, int n_ch, long long plane, int total_rows,
                              double *U, double *Tn, double *part, hipStream_t s) {
  if (n_ch == 0 || plane == 0 || total_rows == 0) return hipSuccess;
  const int nb = saf_blocks(plane);
  hipLaunchKernelGGL(saf_u_kernel, dim3(nb), dim3(256), 0, s, A, ch, n_ch, plane, 0, 1, U);
  hipLaunchKernelGGL(saf_stress_kernel, dim3(nb), dim3(256), 0, s, ch, n_ch, plane, 0, 1, U, Tn);
  hipLaunchKernelGGL(saf_observe_kernel, dim3(total_rows), dim3(256), 0, s, A, ch, n_ch, plane, U, Tn, part);
  return hipGetLastError();
}

hipError_t launch_advance(ChanDev *ch, int n_ch, int steps, hipStream_t s) {
  if (n_ch == 0 || steps == 0) return hipSuccess;
  hipLaunchKernelGGL(advance_kernel, dim3((n_ch + 255) / 256), dim3(256), 0, s, ch, n_ch, steps);
  return hipGetLastError();
}

}  // namespace lbnlm
