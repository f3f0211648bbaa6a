// Time step of the moment state for tau = tau_g = 1 (arXiv:2109.12565, Sec. 2),
// FP64, FP32 and 16-bit FP16 storage, solid cells allowed, flat walls at rest or moving along x.
//
// At tau = tau_g = 1 the BGK collision (Eqs. (2), (16)) returns the
// equilibria (Eqs. (3), (18)), so the post-collision populations of time t
// are functions of five values per node, the moments of the pulled
// populations f(t): rho_A, rho_B, the total momentum j and T. (The velocity
// shift of Eq. (6) and u^H need the forces, which are functions of the
// densities of the 5 x 5 neighbourhood.) The state kept in memory is those
// five planes: 40 bytes per node and step in FP32 instead of 216 for the 27
// populations read and written.
//
// One step, for the columns of one wavefront and a chunk of rows, marching
// upwards one row per iteration (newest row r, q = r - 2, d = r - 3):
//
//   row r    five loads (issued some rows ahead), psi of both components
//            (Eq. (12)) and its x-differences;
//   row q    forces (Eqs. (7), (10), (11), (22)), velocities, the 27
//            equilibria in registers;
//   row d    moments of the populations pulled from rows d - 1, d and d + 1
//            (bounce-back and anti-bounce-back at solid links, Sec. 2.2):
//            five stores.
//
// Every wavefront works on its own: 64 consecutive (periodic) columns of
// which the middle 58 are stored, neighbouring columns read from the
// neighbouring lane inside the arithmetic instructions (DPP wavefront
// shifts), rows kept in registers (rings of five, renamed by unrolling). No
// LDS and no barrier, so nothing but the loads is waited for, and the
// occupancy is set by the registers alone.
//
// Bound and measurements (4096 x 2048, posts along the bottom wall, average of
// a run): FP32 119 to 127 us a step on different boards (a pair's first step
// 122, its second 132 under the profiler), 336 MB = 2.6 to 2.8 TB/s; 376 vector
// instructions a row of 64 columns (the two-step kernel: 638 a node) of 4.4 to
// 4.9 cycles each on a SIMD, so the instruction issue; a variant of 272
// instructions that rounds differently (see kSameRounding) takes 97. FP64 176
// us, 671 MB = 3.8 TB/s. FP16 storage 124 to 130, the rounding adding a tenth to
// the FP32 instructions. Two-step kernel: 266, 668 and 248 us a step; single
// steps in FP32 and FP64 377 and 752. Smaller lattices: FP32 14.6 us at 1024 x
// 512 (25.3 in the two-step kernel), 6.0 at 128 x 64 (12); FP64 17.0 at 1000 x
// 500 (47.6) and 6.0 at 128 x 64 (16.4).
//
// FP64 results differ in rounding from population steps: 1 / rho from the
// hardware's reciprocal and two Newton steps (1 ulp), psi from a series of its
// own, sums in another order. Both stay at rounding level from a 64-bit
// reference (after 100 to 200 steps 4.9e-15 / 6.0e-15 population / moment steps
// in a gradient, 7.2e-14 / 7.7e-14 in a sheared flow).
#pragma once

#include <utility>

#include "lb_kernels.hpp"
#include "moment_tiles.hpp"

namespace tlbk {

// What a launch does with the rows (one of these, with kModeSolid,
// kModeMoving and, for steps, kModeTopRow).
enum : unsigned {
  kMomStep = 1u << 16,    // M(t) -> M(t+1)
  kMomObserve = 2u << 16, // observable sums of time t into partials
  kMomFields = 4u << 16,  // fields of time t
  kMomExport = 8u << 16,  // f*(t) as doubles [27][ly][lx], zero at solid nodes
  kMomShear = 16u << 16,  // with kMomStep: the xy moments of the populations of
                          // f_A and f_B pulled at time t + 1, two planes, in
                          // place of M(t + 1)
  kMomSplit = 32u << 16,  // FP32 steps: populations rounded as between the two
                          // levels of a fused launch (see equilibria_same)
  kMomStress = 64u << 16  // with kMomFields: u_x and the xy stress of time t
                          // (field planes 2, 5 and 6) from M(t) and the xy
                          // moments of f(t)
};

// Columns of a wavefront that only feed the others, on each side: a stored
// column needs equilibria within 1, whose forces need psi within 2 more.
constexpr int kMomHalo = 3;
constexpr int kMomStrip = 64 - 2 * kMomHalo;

template <typename C>
struct MomentArgs {
  StepArgs<C> s;  // src, dst: moment planes [5][pop_stride] (kMomShear: dst
                  // [2][pop_stride]); partials; fields
  double* out;    // kMomExport: [27][ly][lx]
  const C* shear; // kMomStress: the xy moments, [2][pop_stride]
  int strip;      // stored columns per wavefront (at most kMomStrip)
  const MomentTile* tiles;  // steps with solid cells: the wavefronts' tiles,
  int ntiles, nlinked;      // the nlinked first ones hold solid links
  bool src_full;    // deviation storages: src holds full values (see equilibria_stored)
  bool round_wall;  // kSameRounding: 2 w T_w rounded before a population is taken off
  // stencil weights ga w(|c|^2) + gr p(|c|^2) of the self forces, per
  // component, for offsets of 1 (g) and times the offset 2 (h); g12 w(2) /
  // rho0^2 of the cross force
  C g1[2], g2[2], g5[2], h4[2], h5[2], h8[2];
  C x2;
};

// Value of the lane holding the next column on the left (x - 1) and on the
// right (x + 1); the lanes at the ends of the wavefront read 0.
template <int kCtrl>
__device__ inline float lane_shift(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, true));
}
template <int kCtrl>
__device__ inline double lane_shift(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), kCtrl, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <typename C> __device__ inline C from_left(C v) { return lane_shift<0x138>(v); }   // wave_shr:1
template <typename C> __device__ inline C from_right(C v) { return lane_shift<0x130>(v); }  // wave_shl:1

// 1 / v from the hardware reciprocal and Newton steps, without the scaling of
// the IEEE division: densities are far from the ends of the exponent range.
// FP32: one step, the IEEE quotient for every mantissa; FP64: two, within 1
// ulp.
__device__ inline float recip_newton(float v) {
  const float r = __builtin_amdgcn_rcpf(v);
  return fmaf(r, fmaf(-v, r, 1.0f), r);
}
__device__ inline double recip_newton(double v) {
  double r = __builtin_amdgcn_rcp(v);
  r = fma(r, fma(-v, r, 1.0), r);
  return fma(r, fma(-v, r, 1.0), r);
}

// As the storage's population kernels have it (16-bit: the hardware's).
template <class St>
__device__ inline typename St::C recip_moment(typename St::C v) {
  if constexpr (St::kFast) return recip<St>(v);
  else return recip_newton(v);
}

// psi_s = rho0 (1 - e^x), x = -rho / rho0 (Eq. (12)), as -rho0 (2^k (e^f - 1) +
// 2^k - 1) with x = k ln 2 + f, |f| <= ln 2 / 2, so that small rho keeps its
// relative precision (then k = 0). e^f - 1 = f + f^2 q(f), q the Taylor sum to
// f^14 / 14! (4e-18). The library expm1 takes 53 instructions a value, this
// 26, of a row's 370 in all. Below k = -1100, 2^k is zero and psi = rho0, at any
// density. A clamp drops NaN, so it is k's copy for the exponent that is kept
// in range, and f carries the NaN of a density into psi.
__device__ inline double psi_moment(double rho, double rho0, double inv_rho0) {
  const double x = -rho * inv_rho0;
  const double k = __builtin_rint(x * 1.44269504088896340736);
  double f = fma(k, -0.693147180559945286, x);
  f = fma(k, -2.31904681384629956e-17, f);
  double q = fma(f, 1.0 / 87178291200.0, 1.0 / 6227020800.0);
  q = fma(f, q, 1.0 / 479001600.0);
  q = fma(f, q, 1.0 / 39916800.0);
  q = fma(f, q, 1.0 / 3628800.0);
  q = fma(f, q, 1.0 / 362880.0);
  q = fma(f, q, 1.0 / 40320.0);
  q = fma(f, q, 1.0 / 5040.0);
  q = fma(f, q, 1.0 / 720.0);
  q = fma(f, q, 1.0 / 120.0);
  q = fma(f, q, 1.0 / 24.0);
  q = fma(f, q, 1.0 / 6.0);
  q = fma(f, q, 0.5);
  const double e = fma(f * f, q, f);
  const double s = __builtin_ldexp(-rho0, (int)fmax(k, -1100.0));
  return fma(s, e, s + rho0);
}

// Scaled velocities t = sqrt(4.5) u make the even part of the equilibria a
// plain square: f_{i, opp i} = w_i rho (1 - |t|^2 / 3 + (c_i.t)^2) +- odd, odd =
// 3 w_i rho (c_i.t) / sqrt(4.5). (FP64: in FP32 the rounded constants would
// act on the momentum of every step, in one direction.)
constexpr double kVelScale = 2.12132034355964257;
constexpr double kOddAxis = 0.157134840263677228;  // 1 / (3 sqrt(4.5))
constexpr double kOddDiagonal = 0.25 * kOddAxis;

// The nine equilibrium populations of (rho, u) (Eqs. (3), (18)), u scaled; the
// rest one is the remainder of the zeroth moment.
__device__ inline void equilibria(double rho, double tx, double ty, double (&f)[9]) {
#pragma clang fp contract(off)
  const double xx = tx * tx;
  const double c = fma(fma(ty, ty, xx), -1.0 / 3.0, 1.0);
  const double r9 = rho * w_c2<double>(1), r36 = rho * w_c2<double>(2);
  const double o9 = rho * kOddAxis, o36 = rho * kOddDiagonal;
  const double tp = tx + ty, tm = ty - tx;
  const double s1 = r9 * (c + xx), s2 = r9 * fma(ty, ty, c);
  const double s5 = r36 * fma(tp, tp, c), s6 = r36 * fma(tm, tm, c);
  f[1] = fma(o9, tx, s1);
  f[2] = fma(o9, ty, s2);
  f[5] = fma(o36, tp, s5);
  f[6] = fma(o36, tm, s6);
  // the opposite ones as complements: a pair adds up to 2 S as it stands, so
  // the remainder needs the even parts only
  f[3] = fma(2.0, s1, -f[1]);
  f[4] = fma(2.0, s2, -f[2]);
  f[7] = fma(2.0, s5, -f[5]);
  f[8] = fma(2.0, s6, -f[6]);
  f[0] = fma(-2.0, (s1 + s2) + (s5 + s6), rho);
}

// FP32 evaluates every value of a step with the operations of the population
// kernels, one by one, multiply-adds fused as in them, walls at rest or moving:
// a run gives bit for bit the state of the launches it replaces, and a chaotic
// flow (coalescing droplets amplify a rounding a thousandfold within 300 steps)
// the same events. FP64 has no such need at 1e-13 and takes the shorter forms
// above.
template <typename C> constexpr bool kSameRounding = sizeof(C) == 4;

// The FP16 deviation storage keeps its moments in FP32: what its populations,
// rounded to 16 bits where a launch of the population kernels would have stored
// them, add up to. They are rounded in registers, after
// every step but the first of a pair (kMomSplit: the second one's start), so a
// run gives the results of 16-bit populations while 40 bytes a node move
// instead of 120. Moments of rounded populations are deviations from the
// references (rho - rho_ref, T - t_ref, exact sums), those of the others full
// values, as the fused kernel has them.

// The nine populations of a 16-bit storage as it stores them, in stored form:
// deviations w rho q - w ref +- D rounded to 16 bits, the rest population the
// remainder of `dev`, the node's deviation.
template <class St>
__device__ inline void equilibria_stored(float rho, float dev, float ref, float ux, float uy,
                                         float (&f)[9]) {
#pragma clang fp contract(off)
  const float u2 = fma(ux, ux, uy * uy);
  float sum = 0;
  auto pair = [&](auto ic, float cu) {
    constexpr int I = decltype(ic)::value, J = Dir<I>::opp;
    constexpr float w = w_dir<float>(I);
    const float wr = w * rho, q = fma(-1.5f, u2, fma(cu, 4.5f * cu, 1.0f));
    const float even = fma(wr, q, -(w * ref)), d = (3.0f * w) * rho;
    f[I] = St::stored(fma(d, cu, even));
    f[J] = St::stored(fma(-d, cu, even));
    sum = I == 1 ? f[I] + f[J] : sum + (f[I] + f[J]);
  };
  pair(std::integral_constant<int, 1>{}, ux);
  pair(std::integral_constant<int, 2>{}, uy);
  pair(std::integral_constant<int, 5>{}, ux + uy);
  pair(std::integral_constant<int, 6>{}, uy - ux);
  f[0] = dev - sum;
}

// The nine equilibria in the population kernels' operations: opposite ones
// w rho q +- D with one rounding each, the rest population the remainder of
// their sum. kSplit: as the fused kernel's second level pulls them from the
// moments between its two steps, w rho q rounded before D is added (the
// remainder is formed from the others).
template <bool kSplit, typename C>
__device__ inline void equilibria_same(C rho, C ux, C uy, C (&f)[9]) {
#pragma clang fp contract(off)
  const C u2 = fma(ux, ux, uy * uy);
  C sum = 0;
  auto pair = [&](auto ic, C cu) {
    constexpr int I = decltype(ic)::value, J = Dir<I>::opp;
    constexpr C w = w_dir<C>(I);
    const C wr = w * rho, q = fma(C(-1.5), u2, fma(cu, C(4.5) * cu, C(1)));
    const C d = (C(3) * w) * rho * cu;
    const C hi = fma(wr, q, d), lo = fma(wr, q, -d);
    sum = I == 1 ? hi + lo : sum + (hi + lo);
    f[I] = kSplit ? wr * q + d : hi;
    f[J] = kSplit ? wr * q - d : lo;
  };
  pair(std::integral_constant<int, 1>{}, ux);
  pair(std::integral_constant<int, 2>{}, uy);
  pair(std::integral_constant<int, 5>{}, ux + uy);
  pair(std::integral_constant<int, 6>{}, uy - ux);
  f[0] = rho - sum;
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <class F, int... K>
__device__ __forceinline__ void unroll_list(F&& f, std::integer_sequence<int, K...>) {
  (f(std::integral_constant<int, K>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
  unroll_list(f, std::make_integer_sequence<int, N>{});
}

// Rows of the register rings: five in use, two of them with loads in flight.
constexpr int kMomRing = 5;

// The rows y0 .. y1 - 1 of one strip, by one wavefront. kModeSolid: link masks
// are read (steps: a linked tile).
template <class St, unsigned kMode>
__device__ __forceinline__ void moment_rows(const MomentArgs<typename St::C>& ma, int strip, int y0,
                                            int y1, int lin) {
  // Multiply-adds are written out and no others formed, so that every variant
  // of this body (edge and inner rows, linked tiles, steps of a taped run)
  // rounds alike and a column's result does not depend on which one took it.
#pragma clang fp contract(off)
  using C = typename St::C;
  constexpr unsigned kFlags = kMode & 0xffffu;  // kModeSolid, kModeMoving, kModeTopRow
  constexpr bool kSolid = (kMode & kModeSolid) != 0;
  constexpr bool kStep = (kMode & kMomStep) != 0;
  constexpr bool kTop = (kMode & kModeTopRow) != 0;
  constexpr bool kShear = (kMode & kMomShear) != 0, kStress = (kMode & kMomStress) != 0;
  const StepArgs<C>& a = ma.s;
  const int lx = a.lx, ly = a.ly;
  const int lane = threadIdx.x;
  const int xl = strip * ma.strip - kMomHalo + lane;
  const int xw = ((xl % lx) + lx) % lx;
  const bool out_lane = lane >= kMomHalo && lane < kMomHalo + ma.strip && xl < lx;

  // the five planes through a buffer resource: plane and row are scalar
  // offsets, the column the lane's
  const uint32_t row_b = (uint32_t)a.pitch * sizeof(C);
  const uint32_t plane_b = (uint32_t)a.pop_stride * sizeof(C);
  // 16-bit storages: what a loaded density or temperature misses to the full
  // value, and to the deviation
  constexpr bool kDev = St::kDev;
  [[maybe_unused]] const C ref[3] = {a.ref_a, a.ref_b, a.ref_t};
  [[maybe_unused]] C to_full[3] = {0, 0, 0}, to_dev[3] = {0, 0, 0};
  if constexpr (kDev) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      to_full[k] = ma.src_full ? C(0) : ref[k];
      to_dev[k] = ma.src_full ? -ref[k] : C(0);
    }
  }
  const PopMem<Store<C>, 0> msrc(a.src, (uint64_t)plane_b * 5);
  const uint32_t vcol = (uint32_t)xw * sizeof(C);
  // Lanes that store nothing get an offset beyond the five planes (which are
  // below 2 GiB, as tlb.hip asserts), where the buffer's range check drops the
  // store: no branch around the stores.
  const PopMem<Store<C>, 0> mdst(a.dst, (uint64_t)plane_b * 5);
  const uint32_t vout = out_lane ? vcol : 0x80000000u;

  // Rings over rows, slot = iteration mod R (row r is slot S of its stage):
  // the rows that the forces of row q = r - 2 need; the loads of rows r + 1 and
  // r + kAhead are in flight in the slots of r - 4 and r - 3, whose moments are
  // spent (psi and its differences have arrays of their own).
  constexpr int R = kMomRing, kAhead = R - 3;
  C rho[R][2], mx[R], my[R], tt[R];   // loaded moments
  [[maybe_unused]] C raw[R][2];       // kDev: densities as loaded
  C psi[R][2], dpx[R][2], drx[R][2];  // psi and the x-differences of psi and rho
  constexpr bool kSame = kSameRounding<C>, kSplit = (kMode & kMomSplit) != 0;
  [[maybe_unused]] C dp2[R][2];       // kSame, kStress: psi(x + 2) - psi(x - 2)
  C v1[2] = {0, 0};                  // rho(q + 1) - rho(q - 1)
  // Carried from row q - 1 (= d), per field (f_A, f_B, g): what row d has
  // pulled from rows d - 1 and d, before the shift between lanes: from the
  // same column (pc), from the left (pl: c_x = +1) and from the right (pr); the
  // upward populations of row d on their way to row d + 1 (up: directions 2, 5,
  // 6), and, for the differences of opposite directions in j_y, those of row
  // d - 1: um2 direction 2 of each fluid, um5 and um6 of both. jx_own:
  // momentum bounced back at row d (the y part is in um2).
  C pc[3] = {0, 0, 0}, pl[3] = {0, 0, 0}, pr[3] = {0, 0, 0};
  C up[3][3] = {}, um2[2] = {0, 0}, um5 = 0, um6 = 0, jx_own = 0;
  // The same in kSame and kShear, where sums keep the population kernels' order: cp the
  // sum of directions 0..3 pulled at row d, c2, c5, c6 its upward ones, e13 the
  // difference of 1 and 3; up holds the shifted raw ones.
  [[maybe_unused]] C cp[3] = {0, 0, 0}, c2[2] = {0, 0}, c5[3] = {0, 0, 0}, c6[3] = {0, 0, 0};
  [[maybe_unused]] C e13[2] = {0, 0}, top_rho[2] = {0, 0};
  uint32_t lm_d = 0;
  [[maybe_unused]] double acc[kObsSums] = {0, 0, 0, 0, 0, 0};
  [[maybe_unused]] double top_sum = 0.0;

  auto load_row = [&](auto slot, auto inside, int r) {
    constexpr int S = decltype(slot)::value;
    if (decltype(inside)::value || (r >= 0 && r < ly)) {
      const uint32_t s = (uint32_t)r * row_b;
      (kDev ? raw : rho)[S][0] = msrc.ld(s, vcol);
      (kDev ? raw : rho)[S][1] = msrc.ld(s + plane_b, vcol);
      mx[S] = msrc.ld(s + 2 * plane_b, vcol);
      my[S] = msrc.ld(s + 3 * plane_b, vcol);
      tt[S] = msrc.ld(s + 4 * plane_b, vcol);
    } else {
      (kDev ? raw : rho)[S][0] = a.rho_wall0 - to_full[0];
      (kDev ? raw : rho)[S][1] = a.rho_wall1 - to_full[1];
    }
  };

  const int first = y0 - (kStep ? 3 : 2);
  const int last = kStep ? min(y1 + 2, ly + 1) : y1 + 1;

  // moments of row d
  [[maybe_unused]] auto put_row = [&](int d, const C (&n)[3], C jx, C jy) {
    const bool solid = kSolid && (lm_d & kSelfSolid) != 0;
    const uint32_t o = (uint32_t)d * row_b;
    // solid nodes hold the wetting densities and nothing else
    const C off0 = kDev && !kSplit ? ref[0] : C(0), off1 = kDev && !kSplit ? ref[1] : C(0);
    mdst.put(o, vout, solid ? a.rho_wall0 - off0 : n[0]);
    mdst.put(o + plane_b, vout, solid ? a.rho_wall1 - off1 : n[1]);
    mdst.put(o + 2 * plane_b, vout, solid ? C(0) : jx);
    mdst.put(o + 3 * plane_b, vout, solid ? C(0) : jy);
    mdst.put(o + 4 * plane_b, vout, solid ? C(0) : n[2]);
  };

  // xy moments of row d's populations (nothing reads those of solid nodes)
  [[maybe_unused]] auto put_shear = [&](int d, const C (&pi)[2]) {
    const uint32_t o = (uint32_t)d * row_b;
    mdst.put(o, vout, pi[0]);
    mdst.put(o + plane_b, vout, pi[1]);
  };

  // One iteration. kPsi: only row r's own part (the first four rows of a
  // chunk); kInner: rows r + kAhead .. d inside the lattice and the chunk and no
  // solid link in rows q and d, so no test of a row or a link is left and the
  // body is one straight line; kEdge: any row.
  enum Kind { kPsi, kEdge, kInner };
  auto stage = [&](auto slot, auto kind, int r) {
    constexpr int S = decltype(slot)::value;          // row r
    constexpr bool kIn = decltype(kind)::value == kInner;
    constexpr int S1 = (S + R - 1) % R, Q = (S + R - 2) % R;   // rows r - 1, q = r - 2
    constexpr int S3 = (S + R - 3) % R, S4 = (S + R - 4) % R;  // rows r - 3, r - 4
    // row r + kAhead into the slot of row r - 3, whose moments are spent
    if (kIn || r + kAhead <= last)
      load_row(std::integral_constant<int, S3>{}, std::integral_constant<bool, kIn>{}, r + kAhead);
    C v1n[2];
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      if constexpr (kDev) rho[S][l] = raw[S][l] + to_full[l];
      if constexpr (kSame) {
        psi[S][l] = psi_of<St>(rho[S][l], a.rho0, a.inv_rho0);
        const C left = from_left(psi[S][l]), right = from_right(psi[S][l]);
        dpx[S][l] = right - left;
        dp2[S][l] = from_right(right) - from_left(left);
      } else {
        psi[S][l] = psi_moment(rho[S][l], a.rho0, a.inv_rho0);
        const C left = from_left(psi[S][l]), right = from_right(psi[S][l]);
        dpx[S][l] = right - left;
        if constexpr (kStress) dp2[S][l] = from_right(right) - from_left(left);
      }
      drx[S1][l] = from_right(rho[S1][l]) - from_left(rho[S1][l]);
      v1n[l] = rho[S][l] - rho[Q][l];
    }
    const int q = r - 2;
    if (decltype(kind)::value == kPsi || (!kIn && (q < 0 || q >= ly))) {
      v1[0] = v1n[0];
      v1[1] = v1n[1];
      return;
    }
    uint32_t lq = 0;
    const C ra = rho[Q][0], rb = rho[Q][1], temp = kDev ? tt[Q] + to_full[2] : tt[Q];
    C vx[3], vy[3];  // velocities (scaled unless kSame) of the three equilibria at row q
    {
      if constexpr (!kIn) lq = link_mask<kFlags>(a, xw, q);
      // ---- forces. x-derivative: differences across the column, weighted
      // over the five rows (psi(x+2) - psi(x-2) as the neighbours' sum);
      // y-derivative: differences between rows, weighted over five columns.
      // The cross force's weights are 4 : 1, its factor g12 w_2 / rho0^2.
      C FA[2], FB[2];
      [[maybe_unused]] const C buoyancy = a.alpha_g * temp;
#pragma unroll
      for (int l = 0; l < 2; ++l) {
        C* F = l == 0 ? FA : FB;
        const int m = 1 - l;
        if constexpr (kSame) {
          constexpr C p1 = p_c2<C>(1), p2 = p_c2<C>(2), p4 = p_c2<C>(4) * C(2);
          constexpr C p5 = p_c2<C>(5), p52 = p_c2<C>(5) * C(2), p8 = p_c2<C>(8) * C(2);
          constexpr C n1 = w_c2<C>(1), n2 = w_c2<C>(2);
          const C ga = l == 0 ? a.ga0 : a.ga1, gr = l == 0 ? a.gr0 : a.gr1;
          // differences of rows -2 .. 2 across one and two columns
          C q = fma(p8, dp2[S4][l], p5 * dpx[S4][l]);
          q = fma(p52, dp2[S3][l], fma(p2, dpx[S3][l], q));
          q = fma(p4, dp2[Q][l], fma(p1, dpx[Q][l], q));
          q = fma(p52, dp2[S1][l], fma(p2, dpx[S1][l], q));
          q = fma(p8, dp2[S][l], fma(p5, dpx[S][l], q));
          C n = fma(n2, dpx[S1][l], fma(n1, dpx[Q][l], n2 * dpx[S3][l]));
          const C gx = fma(ga, n, gr * q);
          // differences of columns -2 .. 2 across one and two rows
          const C a1 = psi[S1][l] - psi[S3][l], a2 = psi[S][l] - psi[S4][l];
          const C a1l = from_left(a1), a2l = from_left(a2), a1r = from_right(a1), a2r = from_right(a2);
          q = fma(p8, from_left(a2l), p5 * from_left(a1l));
          q = fma(p52, a2l, fma(p2, a1l, q));
          q = fma(p4, a2, fma(p1, a1, q));
          q = fma(p52, a2r, fma(p2, a1r, q));
          q = fma(p8, from_right(a2r), fma(p5, from_right(a1r), q));
          n = fma(n2, a1r, fma(n1, a1, n2 * a1l));
          const C gy = fma(ga, n, gr * q);
          const C sx = fma(n2, drx[S1][m], fma(n1, drx[Q][m], n2 * drx[S3][m]));
          const C sy = fma(n2, from_right(v1[m]), fma(n1, v1[m], n2 * from_left(v1[m])));
          const C pre = -a.g12 * rho[Q][l] * a.inv_rho0 * a.inv_rho0;
          F[0] = fma(pre, sx, -(psi[Q][l] * gx));
          F[1] = fma(a.alpha_g * rho[Q][l], temp, fma(pre, sy, -(psi[Q][l] * gy)));
        } else {
          const C e1 = dpx[S1][l] + dpx[S3][l], e2 = dpx[S][l] + dpx[S4][l];
          const C w1 = fma(ma.g1[l], dpx[Q][l], fma(ma.g2[l], e1, ma.g5[l] * e2));
          const C w2 = fma(ma.h4[l], dpx[Q][l], fma(ma.h5[l], e1, ma.h8[l] * e2));
          const C qx = w1 + (from_left(w2) + from_right(w2));
          const C a1 = psi[S1][l] - psi[S3][l], a2 = psi[S][l] - psi[S4][l];
          const C b0 = fma(ma.g1[l], a1, ma.h4[l] * a2);
          const C b1 = fma(ma.g2[l], a1, ma.h5[l] * a2);
          const C b2 = fma(ma.g5[l], a1, ma.h8[l] * a2);
          const C qy = b0 + (from_left(b1 + from_left(b2)) + from_right(b1 + from_right(b2)));
          const C sx = fma(C(4), drx[Q][m], drx[S1][m] + drx[S3][m]);
          const C sy = fma(C(4), v1[m], from_left(v1[m]) + from_right(v1[m]));
          const C cross = rho[Q][l] * ma.x2;
          F[0] = -fma(psi[Q][l], qx, cross * sx);
          F[1] = fma(rho[Q][l], buoyancy, -fma(psi[Q][l], qy, cross * sy));
        }
      }
      // ---- velocities (u and u^H of the observables; scaled ones below)
      const C inv_rho = recip_moment<St>(ra + rb);
      const C Fx = FA[0] + FB[0], Fy = FA[1] + FB[1];
      if constexpr ((kMode & (kMomObserve | kMomFields)) != 0) {
        if (out_lane && q < y1) {
          const bool solid = kSolid && !kIn && (lq & kSelfSolid) != 0;
          C hx, hy;
          if constexpr (kSame && (kMode & kMomFields) != 0) {
            hx = fma(mx[Q], inv_rho, C(0.5) * Fx * inv_rho);
            hy = fma(my[Q], inv_rho, C(0.5) * Fy * inv_rho);
          } else if constexpr (kSame) {
            hx = fma(C(0.5) * Fx, inv_rho, mx[Q] * inv_rho);
            hy = fma(C(0.5) * Fy, inv_rho, my[Q] * inv_rho);
          } else {
            hx = fma(C(0.5), Fx, mx[Q]) * inv_rho;
            hy = fma(C(0.5), Fy, my[Q]) * inv_rho;
          }
          // (deviations: the reference added in double)
          const double da = kDev ? (double)ref[0] + (double)(raw[Q][0] + to_dev[0]) : (double)ra;
          const double db = kDev ? (double)ref[1] + (double)(raw[Q][1] + to_dev[1]) : (double)rb;
          const double dt = kDev ? (double)ref[2] + (double)(tt[Q] + to_dev[2]) : (double)temp;
          if constexpr ((kMode & kMomObserve) != 0) {
            if (!solid) {
              acc[0] += da;
              acc[1] += db;
              acc[2] += dt;
              acc[3] += (double)hy * dt;
              acc[4] += (double)hx * (double)hx + (double)hy * (double)hy;
              if (q == ly - 1) acc[5] += dt - (double)a.t_top;
            }
          } else if constexpr (kStress) {
            // -(1 - 1/(2 tau)) (sum c_x c_y f - rho u_x u_y) of both components,
            // and the interaction pressure: nodes at +-c share c_x c_y, so
            // differences across columns, differenced over the rows
            const size_t nn = (size_t)lx * ly, o = (size_t)q * lx + xl;
            const C* pi = ma.shear + (size_t)q * a.pitch + xl;
            const C ux = mx[Q] * inv_rho, uy = my[Q] * inv_rho;
            C visc = 0, pint = 0;
#pragma unroll
            for (int l = 0; l < 2; ++l) {
              const C* F = l == 0 ? FA : FB;
              const int m = 1 - l;
              const C rl = rho[Q][l], t = recip_moment<St>(rl);
              const C vx = fma(F[0], t, ux), vy = fma(F[1], t, uy);
              visc += fma(-(rl * vx), vy, pi[(size_t)l * a.pop_stride]);
              const C d1 = dpx[S1][l] - dpx[S3][l], d2 = dp2[S][l] - dp2[S4][l];
              const C d12 = (dpx[S][l] - dpx[S4][l]) + (dp2[S1][l] - dp2[S3][l]);
              const C self = fma(C(2) * ma.h8[l], d2, fma(ma.h5[l], d12, ma.g2[l] * d1));
              const C cross = w_c2<C>(2) * (drx[S1][m] - drx[S3][m]);
              const C pre = C(0.5) * a.g12 * a.inv_rho0 * a.inv_rho0 * rl;
              pint += fma(pre, cross, C(0.5) * psi[Q][l] * self);
            }
            a.fields[2 * nn + o] = solid ? 0.0 : (double)hx;
            a.fields[5 * nn + o] = solid ? 0.0 : (double)(C(-0.5) * visc);
            a.fields[6 * nn + o] = solid ? 0.0 : (double)pint;
          } else {
            const size_t nn = (size_t)lx * ly, o = (size_t)q * lx + xl;
            double tv = dt;
            if constexpr (kSolid) {
              if (solid) tv = (double)solid_temperature(a, xl, q);
            }
            a.fields[o] = solid ? (double)a.rho_wall0 : da;
            a.fields[nn + o] = solid ? (double)a.rho_wall1 : db;
            a.fields[2 * nn + o] = solid ? 0.0 : (double)hx;
            a.fields[3 * nn + o] = solid ? 0.0 : (double)hy;
            a.fields[4 * nn + o] = tv;
          }
        }
        v1[0] = v1n[0];
        v1[1] = v1n[1];
        return;
      }
      const C k = kSame ? inv_rho : inv_rho * C(kVelScale);
      const C ux = mx[Q] * k, uy = my[Q] * k;
      const C scale = kSame ? C(1) : C(kVelScale);
      const C tA = recip_moment<St>(ra) * scale, tB = recip_moment<St>(rb) * scale;
      vx[0] = fma(FA[0], tA, ux), vy[0] = fma(FA[1], tA, uy);
      vx[1] = fma(FB[0], tB, ux), vy[1] = fma(FB[1], tB, uy);
      vx[2] = fma(C(0.5) * Fx, k, ux), vy[2] = fma(C(0.5) * Fy, k, uy);
    }
    v1[0] = v1n[0];
    v1[1] = v1n[1];
    const C dens[3] = {ra, rb, temp};
    [[maybe_unused]] C dev[3] = {0, 0, 0};  // deviation storages
    if constexpr (kDev)
      dev[0] = raw[Q][0] + to_dev[0], dev[1] = raw[Q][1] + to_dev[1], dev[2] = tt[Q] + to_dev[2];
    auto populations = [&](auto kc, C (&f)[9]) {
      constexpr int k = decltype(kc)::value;
      if constexpr (kDev && !kSplit) equilibria_stored<St>(dens[k], dev[k], ref[k], vx[k], vy[k], f);
      else if constexpr (kSame) equilibria_same<kSplit>(dens[k], vx[k], vy[k], f);
      else equilibria(dens[k], vx[k], vy[k], f);
    };
    if constexpr ((kMode & kMomExport) != 0) {
      if (!out_lane || q >= y1) return;
      const bool solid = kSolid && !kIn && (lq & kSelfSolid) != 0;
      unroll<3>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        C f[9];
        populations(kc, f);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
          const double v = kDev ? fma(w_dir<double>(i), (double)ref[k], (double)f[i]) : (double)f[i];
          ma.out[((size_t)(9 * k + i) * ly + q) * lx + xl] = solid ? 0.0 : v;
        }
      });
      return;
    }
    if constexpr (kStep && (kSame || kShear)) {
      // Field by field. Row d = q - 1 pulls its downward populations from row
      // q, or, across a solid link, takes its own upward ones (opposite
      // direction; 2 w T_w minus them for g), and is complete; row q starts
      // with the upward ones of row q - 1 and its own level ones, bounced
      // alike.
      const int d = q - 1;
      const bool back_d = kSolid && !kIn && __any((lm_d & kFromAbove) != 0u);
      const bool back_q = !kIn && (kSolid ? __any((lq & kLinkBits & ~kFromAbove) != 0u) : q == 0);
      C n[3], jx = 0, jy = 0;
      [[maybe_unused]] C pi[2];
      auto field = [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr bool kG = k == 2;
        C f[9];
        populations(kc, f);
        // the value v of direction I, bounced where the link of row `row` is
        // solid: `own` is the node's population of the opposite direction
        auto bounce = [&](auto ic, C& v, C own, uint32_t links, int row) {
          constexpr int I = decltype(ic)::value;
          if (kSolid && ((links >> I) & 1u) == 0u) return;
          v = own;
          if constexpr (kG) {
            constexpr C w2 = C(2) * w_dir<C>(I);
            const C ts = source_wall_temperature<I, kFlags>(a, xw, row);
            const C even = wall_even_factor<I, kFlags>(a, row);
            const C tw = kDev && !kSplit ? fma(ts, even, -ref[2]) : ts * even;
            v = ma.round_wall ? w2 * tw - own : fma(w2, tw, -own);
          }
        };
        C d4 = f[4], d7 = from_right(f[7]), d8 = from_left(f[8]);
        if (back_d) {
          // the raw upward values of row d are shifted; shifting back gives
          // the lane's own
          const C own5 = from_right(up[k][1]), own6 = from_left(up[k][2]);
          bounce(std::integral_constant<int, 4>{}, d4, up[k][0], lm_d, d);
          bounce(std::integral_constant<int, 7>{}, d7, own5, lm_d, d);
          bounce(std::integral_constant<int, 8>{}, d8, own6, lm_d, d);
        }
        if constexpr (kShear) pi[k] = (c5[k] + d7) - (c6[k] + d8);
        n[k] = (cp[k] + ((d4 + c5[k]) + (c6[k] + d7))) + d8;
        if constexpr (!kG) {
          const C e57 = c5[k] - d7;
          jx += (e13[k] + e57) + (d8 - c6[k]);
          jy += ((c2[k] - d4) + e57) + (c6[k] - d8);
        }
        C u2 = up[k][0], u5 = up[k][1], u6 = up[k][2], l1 = from_left(f[1]), l3 = from_right(f[3]);
        if (back_q) {
          bounce(std::integral_constant<int, 2>{}, u2, f[4], lq, q);
          bounce(std::integral_constant<int, 5>{}, u5, f[7], lq, q);
          bounce(std::integral_constant<int, 6>{}, u6, f[8], lq, q);
          if constexpr (kSolid) {
            bounce(std::integral_constant<int, 1>{}, l1, f[3], lq, q);
            bounce(std::integral_constant<int, 3>{}, l3, f[1], lq, q);
          }
        }
        if constexpr ((kMode & kModeMoving) != 0 && !kG) {
          // moving flat walls (Sec. 2.2): the bounced diagonal links gain
          // +- 6 w_5 rho u_w, rho the sum of the node's populations (between
          // the levels of a fused launch the moment itself)
          if (!kIn && (q == 0 || q == ly - 1)) {
            C rw = dens[k];
            if constexpr (kSame && !kSplit) {
              rw = f[0];
#pragma unroll
              for (int i = 1; i < 9; ++i) rw += f[i];
              if constexpr (kDev) rw += ref[k];
            }
            if (q == 0) {
              const C m = C(6) * w_dir<C>(5) * a.uw0;
              u5 = fma(m, rw, u5);
              u6 = fma(-m, rw, u6);
            }
            if (q == ly - 1) top_rho[k] = rw;
          }
        }
        cp[k] = (f[0] + l1) + (u2 + l3);
        c5[k] = u5;
        c6[k] = u6;
        if constexpr (!kG) {
          c2[k] = u2;
          e13[k] = l1 - l3;
        }
        up[k][0] = f[2], up[k][1] = from_left(f[5]), up[k][2] = from_right(f[6]);
      };
      unroll<kShear ? 2 : 3>(field);
      if (kIn || d >= y0) {
        if constexpr (kShear) put_shear(d, pi);
        else put_row(d, n, jx, jy);
      }
      lm_d = lq;
    } else if constexpr (kStep) {
      // Field by field. Row d = q - 1 pulls its downward populations from row
      // q and is complete; row q starts with the upward ones of row q - 1 and
      // its own level ones. Nothing is pulled from outside the lattice or
      // from solid nodes (their populations are zeroed): a solid link of row
      // q adds the node's own opposite population (bounce-back) or 2 w T_w
      // minus it (anti-bounce-back).
      const int d = q - 1;
      const bool back = !kIn && (kSolid ? __any((lq & kLinkBits) != 0u) : q == 0 || q == ly - 1);
      C n[3], jx = jx_own, jy = 0, d7 = 0, d8 = 0, jxn = 0, jyn = 0;
      auto field = [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        constexpr bool kG = k == 2;
        C f[9];
        equilibria(dens[k], vx[k], vy[k], f);
        C own = 0;  // bounced into row q
        if (back) {
#define TLB_BACK(I)                                                                           \
  if (kSolid ? ((lq >> I) & 1u) != 0u                                                         \
             : (Dir<I>::cy > 0 && q == 0) || (Dir<I>::cy < 0 && q == ly - 1)) {               \
    C v = f[Dir<I>::opp];                                                                     \
    if constexpr (kG) {                                                                       \
      v = C(2) * w_dir<C>(I) * source_wall_temperature<I, kFlags>(a, xw, q) *                 \
              wall_even_factor<I, kFlags>(a, q) - v;                                          \
    } else {                                                                                  \
      jxn += C(Dir<I>::cx) * v;                                                               \
      jyn += C(Dir<I>::cy) * v;                                                               \
    }                                                                                         \
    own += v;                                                                                 \
  }
          TLB_BACK(2) TLB_BACK(5) TLB_BACK(6) TLB_BACK(4) TLB_BACK(7) TLB_BACK(8)
          if constexpr (kSolid) {
            TLB_BACK(1) TLB_BACK(3)
          }
#undef TLB_BACK
        }
        if constexpr (kSolid) {
          if ((lq & kSelfSolid) != 0u) {
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = C(0);
          }
        }
        // row d
        const C l = from_left(pl[k] + f[8]), rr = from_right(pr[k] + f[7]);
        n[k] = (pc[k] + f[4]) + (l + rr);
        if constexpr (!kG) {
          jx += l - rr;
          jy += um2[k] - f[4];
          d7 += f[7];
          d8 += f[8];
          um2[k] = up[k][0];
        }
        // row q
        pc[k] = up[k][0] + f[0];
        if (!kIn) pc[k] += own;
        pl[k] = up[k][1] + f[1];
        pr[k] = up[k][2] + f[3];
        up[k][0] = f[2], up[k][1] = f[5], up[k][2] = f[6];
      };
      const C up5 = up[0][1] + up[1][1], up6 = up[0][2] + up[1][2];
      field(std::integral_constant<int, 0>{});
      field(std::integral_constant<int, 1>{});
      field(std::integral_constant<int, 2>{});
      if (kIn || d >= y0) put_row(d, n, jx, jy + (from_left(um5 - d8) + from_right(um6 - d7)));
      um5 = up5;
      um6 = up6;
      if (!kIn) um2[0] += jyn;
      if constexpr ((kMode & kModeMoving) != 0) {
        // moving flat walls (Sec. 2.2): the two bounced diagonal links gain
        // +- 6 w_5 rho u_w, which cancel in the mass and add up in j_x
        constexpr C kw = C(12) * w_dir<C>(5);
        if (!kIn && q == 0) jxn += kw * a.uw0 * (ra + rb);
        if (!kIn && q == ly - 1) jxn += kw * a.uw1 * (ra + rb);
      }
      jx_own = jxn;
      lm_d = lq;
    }
  };

  using Psi = std::integral_constant<Kind, kPsi>;
  using Edge = std::integral_constant<Kind, kEdge>;
  using Inner = std::integral_constant<Kind, kInner>;
#pragma unroll
  for (int s = 0; s < R; ++s) {
    mx[s] = my[s] = tt[s] = C(0);
#pragma unroll
    for (int l = 0; l < 2; ++l) raw[s][l] = rho[s][l] = psi[s][l] = dpx[s][l] = dp2[s][l] = drx[s][l] = C(0);
  }
  unroll<kAhead>([&](auto k) { load_row(k, std::false_type{}, first + decltype(k)::value); });
  unroll<4>([&](auto k) { stage(k, Psi{}, first + decltype(k)::value); });
  int r = first + 4;
  stage(std::integral_constant<int, 4 % R>{}, Edge{}, r++);
  if (r <= last) stage(std::integral_constant<int, 5 % R>{}, Edge{}, r++);
  // R rows at a time: inner where the last one's load exists, d is in the
  // chunk and q is not at a flat wall.
  if constexpr (!kSolid) {
    const int inner = min(last, ly - 1) - kAhead - (R - 1);
    if (r >= 3)
      for (; r <= inner; r += R)
        unroll<R>([&](auto k) {
          constexpr int K = decltype(k)::value;
          stage(std::integral_constant<int, (6 + K) % R>{}, Inner{}, r + K);
        });
  }
  while (r <= last)
    unroll<R>([&](auto k) {
      if (r <= last) stage(std::integral_constant<int, (6 + decltype(k)::value) % R>{}, Edge{}, r++);
    });

  if constexpr (kStep) {
    if (y1 == ly) {  // the top row is complete: nothing comes down to it
      C n[3], jx = 0, jy = 0;
      [[maybe_unused]] C pi[2];
      if constexpr (kSame || kShear) {
#pragma unroll
        for (int k = 0; k < (kShear ? 2 : 3); ++k) {
          C d4 = up[k][0], d7 = from_right(up[k][1]), d8 = from_left(up[k][2]);
          if (k == 2) {
            constexpr C wa = C(2) * w_dir<C>(4), wd = C(2) * w_dir<C>(7);
            const C e4 = wall_even_factor<4, kFlags>(a, ly - 1), e7 = wall_even_factor<7, kFlags>(a, ly - 1);
            const C t4 = kDev && !kSplit ? fma(a.t_top, e4, -ref[2]) : a.t_top * e4;
            const C t7 = kDev && !kSplit ? fma(a.t_top, e7, -ref[2]) : a.t_top * e7;
            d4 = ma.round_wall ? wa * t4 - d4 : fma(wa, t4, -d4);
            d7 = ma.round_wall ? wd * t7 - d7 : fma(wd, t7, -d7);
            d8 = ma.round_wall ? wd * t7 - d8 : fma(wd, t7, -d8);
          } else if constexpr ((kMode & kModeMoving) != 0) {
            const C m = C(6) * w_dir<C>(8) * a.uw1;
            d8 = fma(m, top_rho[k], d8);
            d7 = fma(-m, top_rho[k], d7);
          }
          if constexpr (kShear) pi[k] = (c5[k] + d7) - (c6[k] + d8);
          n[k] = (cp[k] + ((d4 + c5[k]) + (c6[k] + d7))) + d8;
          if (k < 2) {
            const C e57 = c5[k] - d7;
            jx += (e13[k] + e57) + (d8 - c6[k]);
            jy += ((c2[k] - d4) + e57) + (c6[k] - d8);
          }
        }
      } else {
        jx = jx_own;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const C l = from_left(pl[k]), rr = from_right(pr[k]);
          n[k] = pc[k] + (l + rr);
          if (k < 2) jx += l - rr;
        }
        jy = (um2[0] + um2[1]) + (from_left(um5) + from_right(um6));
      }
      if constexpr (kShear) put_shear(ly - 1, pi);
      else put_row(ly - 1, n, jx, jy);
      if (kTop && out_lane) top_sum = (double)n[2] - (double)a.t_top;
    }
  }
  if constexpr ((kMode & kMomObserve) != 0) {
    // fixed-order sums of the wavefront
#pragma unroll
    for (int j = 0; j < kObsSums; ++j) {
      double v = acc[j];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
      if (lane == 0) a.partials[(size_t)lin * kObsSums + j] = v;
    }
  }
  if constexpr (kTop) {
    if (y1 == ly) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) top_sum += __shfl_down(top_sum, o, 64);
      if (lane == 0) a.partials[strip] = top_sum;
    }
  }
}

// Wavefronts per SIMD the registers are limited for. FP32 steps take 143 to 168
// VGPRs; held to the 128 of four wavefronts they spill (a body of 140 ran 17%
// slower there), and at the 168 of three only a pair's second step with solid
// cells does (10, 31 with moving walls). Limited to two, nothing spills, and 4096
// x 2048 takes 123 us a step (119), 174 with posts over the lower third (157).
// FP16 spills more at three: 4 to 9 on flat walls, 84 to 108 with solid cells,
// where two would be faster (lower third 180 us, 198 at three; posts along the
// bottom only 125, 124; 333 x 129 8.6, 14.8). FP64, with twice the registers per
// value, spills 14 to 62 at the 256 of two wavefronts, and runs as fast as
// unspilled with one (171 us a step of 4096 x 2048 either way).
template <typename C>
constexpr int kMomWaves = sizeof(C) == 4 ? 3 : 2;

template <class St, unsigned kMode>
__global__ __launch_bounds__(64, kMomWaves<typename St::C>) void lb_moment_kernel(
    MomentArgs<typename St::C> ma) {
  // Workgroups go to the eight XCDs round-robin; the remap gives each XCD,
  // and so its L2, a contiguous run of n tiles (strip fastest).
  auto xcd_run = [](int lin, int n) {
    constexpr int kXcds = 8;
    const int xcd = lin % kXcds;
    return xcd * (n / kXcds) + min(xcd, n % kXcds) + lin / kXcds;
  };
  if constexpr ((kMode & kMomStep) != 0 && (kMode & kModeSolid) != 0) {
    // Linked tiles first: they take longer, are cut shorter, and start
    // together on all XCDs. The others run the flat walls' body, so solid
    // cells cost registers and tests only where they are.
    const int lin = blockIdx.x;
    const int t = lin < ma.nlinked ? lin
                                   : ma.nlinked + xcd_run(lin - ma.nlinked, ma.ntiles - ma.nlinked);
    const MomentTile tile = ma.tiles[t];
    if (tile.linked) moment_rows<St, kMode>(ma, tile.strip, tile.y0, tile.y1, lin);
    else moment_rows<St, kMode & ~kModeSolid>(ma, tile.strip, tile.y0, tile.y1, lin);
  } else {
    const int nbx = gridDim.x;
    const int lin = blockIdx.y * nbx + blockIdx.x;
    const int t = xcd_run(lin, nbx * (int)gridDim.y);
    const int chunk = t / nbx;
    const int y0 = chunk * ma.s.rows_per_block;
    moment_rows<St, kMode>(ma, t - chunk * nbx, y0, min(y0 + ma.s.rows_per_block, ma.s.ly), lin);
  }
}

// M(0): the moments of the equilibrium start populations f(0) as the
// population path stores them (solid nodes hold the wetting densities), and the
// xy moments of f_A(0) and f_B(0) into the two planes `shear`.
template <class St>
__global__ __launch_bounds__(256) void lb_moment_init(
    typename St::C* __restrict__ dst, typename St::C* __restrict__ shear,
    const double* __restrict__ rho_a,
    const double* __restrict__ rho_b, const double* __restrict__ temp,
    const double* __restrict__ ux0, const double* __restrict__ uy0,
    const uint8_t* __restrict__ solid, int lx, int pitch, long long pop_stride,
    typename St::C rho_wall0, typename St::C rho_wall1, typename St::C ref_a,
    typename St::C ref_b, typename St::C ref_t) {
#pragma clang fp contract(off)
  using C = typename St::C;
  const int x = blockIdx.x * 256 + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= lx) return;
  const size_t q = (size_t)y * lx + x, ps = (size_t)pop_stride;
  C* m = dst + (size_t)y * pitch + x;
  C* xy = shear + (size_t)y * pitch + x;
  const C ref[3] = {St::kDev ? ref_a : C(0), St::kDev ? ref_b : C(0), St::kDev ? ref_t : C(0)};
  if (solid[q] != 0) {
    m[0] = rho_wall0 - ref[0];
    m[ps] = rho_wall1 - ref[1];
    m[2 * ps] = m[3 * ps] = m[4 * ps] = xy[0] = xy[ps] = C(0);
    return;
  }
  const C ux = ux0 ? (C)ux0[q] : C(0), uy = uy0 ? (C)uy0[q] : C(0);
  const C u2 = fma(ux, ux, uy * uy);
  const C dens[3] = {(C)rho_a[q], (C)rho_b[q], (C)temp[q]};
  C f[3][9], sum[3] = {C(0), C(0), C(0)};
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const C cu = C(dir_cx(i)) * ux + C(dir_cy(i)) * uy;
    const C shape = w_dir<C>(i) * fma(C(-1.5), u2, fma(cu, C(4.5) * cu, fma(cu, C(3), C(1))));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if constexpr (St::kDev) {
        f[k][i] = St::stored(fma(dens[k], shape, -(w_dir<C>(i) * ref[k])));
        sum[k] += f[k][i];
      } else {
        f[k][i] = dens[k] * shape;
        sum[k] = fma(shape, dens[k], sum[k]);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) f[k][0] = (dens[k] - ref[k]) - sum[k];
  m[0] = sum9(f[0]);
  m[ps] = sum9(f[1]);
  m[2 * ps] = momentum_x(f[0], f[1]);
  m[3 * ps] = momentum_y(f[0], f[1]);
  m[4 * ps] = sum9(f[2]);
#pragma unroll
  for (int k = 0; k < 2; ++k) xy[k * ps] = (f[k][5] + f[k][7]) - (f[k][6] + f[k][8]);
}

}  // namespace tlbk
