// Definitions of the launch interface, included once per storage type.
#pragma once

#include "launch.hpp"
#include "lb_kernels.hpp"
#include "lb_moment.hpp"
#include "lb_step2.hpp"

namespace tlbh {

static_assert(kMomentStrip == tlbk::kMomStrip, "columns of a moment wavefront");

namespace detail {

template <typename C>
tlbk::StepArgs<C> make_args(const Device& d, const void* src, void* dst) {
  tlbk::StepArgs<C> a{};
  const tlb_params& p = *d.p;
  a.src = src;
  a.dst = dst;
  a.link = d.link;
  a.solid = d.solid;
  a.t_bottom = static_cast<const C*>(d.t_bottom);
  a.partials = d.partials;
  a.fields = d.fields;
  a.lx = p.lx;
  a.ly = p.ly;
  a.pitch = d.pitch;
  a.rows_per_block = d.geo.rows;
  a.pop_stride = d.pop_stride;
  a.inv_tau = C(1.0 / p.tau);
  a.inv_tau_g = C(1.0 / p.tau_g);
  a.tau = C(p.tau);
  a.rho0 = C(p.rho0);
  a.inv_rho0 = C(1.0 / p.rho0);
  a.g12 = C(p.g12);
  a.ga0 = C(p.g_a[0]);
  a.ga1 = C(p.g_a[1]);
  a.gr0 = C(p.g_r[0]);
  a.gr1 = C(p.g_r[1]);
  a.alpha_g = C(p.alpha_g);
  a.t_top = C(p.t_top);
  a.rho_wall0 = C(p.rho_wall[0]);
  a.rho_wall1 = C(p.rho_wall[1]);
  a.ref_a = C(p.rho_ref[0]);
  a.ref_b = C(p.rho_ref[1]);
  a.ref_t = C(p.t_ref);
  a.uw0 = C(p.u_wall[0]);
  a.uw1 = C(p.u_wall[1]);
  return a;
}

template <class St, int BX, unsigned kMode>
void launch(const Device& d, const tlbk::StepArgs<typename St::C>& a) {
  hipLaunchKernelGGL((tlbk::lb_step_kernel<St, BX, kMode>), d.geo.grid, dim3(BX), 0, d.stream, a);
}

// Dispatch on offset width and block width (the 64-bit offset variant
// always runs 256-wide blocks).
template <class St, unsigned kMode>
void launch_geometry(const Device& d, const tlbk::StepArgs<typename St::C>& a) {
  if (d.geo.wide) launch<St, 256, kMode | tlbk::kModeWide>(d, a);
  else if (d.geo.bx == 256) launch<St, 256, kMode>(d, a);
  else launch<St, 64, kMode>(d, a);
}

// Dispatch on solid cells and on the tau = tau_g = 1 path (never for the
// stress pass, which needs the pulled populations themselves).
template <class St, unsigned kMode>
void launch_solid_tau(const Device& d, const tlbk::StepArgs<typename St::C>& a) {
  constexpr unsigned S = tlbk::kModeSolid, T1 = tlbk::kModeTauOne;
  if constexpr ((kMode & tlbk::kModeStress) != 0) {
    if (d.has_solid) launch_geometry<St, kMode | S>(d, a);
    else launch_geometry<St, kMode>(d, a);
  } else if (d.has_solid) {
    if (d.tau_one) launch_geometry<St, kMode | S | T1>(d, a);
    else launch_geometry<St, kMode | S>(d, a);
  } else {
    if (d.tau_one) launch_geometry<St, kMode | T1>(d, a);
    else launch_geometry<St, kMode>(d, a);
  }
}

// Dispatch on moving walls (a separate kernel, so walls at rest pay nothing
// for it; passes that read f(0) in place pull nothing and need no variant).
template <class St, unsigned kMode>
void launch_mode(const Device& d, const void* src, void* dst) {
  const auto a = make_args<typename St::C>(d, src, dst);
  if constexpr ((kMode & tlbk::kModeInit) == 0) {
    if (d.moving) {
      launch_solid_tau<St, kMode | tlbk::kModeMoving>(d, a);
      return;
    }
  }
  launch_solid_tau<St, kMode>(d, a);
}

template <class St, int BX, unsigned kMode>
int occupancy() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, tlbk::lb_step_kernel<St, BX, kMode>, BX, 0) !=
          hipSuccess ||
      n < 1)
    n = 1;
  return n;
}

template <class St, unsigned kMode>
int occupancy_geometry(int bx, bool wide) {
  if (wide) return occupancy<St, 256, kMode | tlbk::kModeWide>();
  if (bx == 256) return occupancy<St, 256, kMode>();
  return occupancy<St, 64, kMode>();
}

template <class St, unsigned kMode>
void launch_step2_kernel(const Device& d, const tlbk::StepArgs<typename St::C>& a) {
  if (d.geo.lanes2 == kStep2LanesNarrow)
    hipLaunchKernelGGL((tlbk::lb_step2_kernel<St, kStep2LanesNarrow, kMode>), d.geo.grid2,
                       dim3(kStep2LanesNarrow), 0, d.stream, a, d.geo.strip2);
  else
    hipLaunchKernelGGL((tlbk::lb_step2_kernel<St, kStep2Lanes, kMode>), d.geo.grid2,
                       dim3(kStep2Lanes), 0, d.stream, a, d.geo.strip2);
}

// Storages with a two-step kernel: FP64, FP32 and the 16-bit floating
// deviations (FP32 rest planes); not the fixed-point one, whose exact
// mass needs every intermediate value on its grid.
template <class St>
constexpr bool kHasStep2 = !St::kFix && (!St::kDev || St::kRest32);

// Storages with the adjoint (FP64, FP32).
template <class St>
constexpr bool kHasAdjoint = !St::kFix && !St::kDev;

template <class St>
void launch_step2(const Device& d, const void* src, void* dst, Pass pass, void* moments) {
  if constexpr (kHasStep2<St>) {
    auto a = make_args<typename St::C>(d, src, dst);
    a.rows_per_block = d.geo.rows2;
    a.moments = moments;
    constexpr unsigned M = tlbk::kModeStore | tlbk::kModeTauOne;
    constexpr unsigned S = tlbk::kModeSolid, V = tlbk::kModeMoving;
    // the adjoint's variants: flat walls at rest only
    if (pass == Pass::kStep2TopRow) {
      if (!d.moving && !d.has_solid) launch_step2_kernel<St, M | tlbk::kModeTopRow>(d, a);
      return;
    }
    if (pass == Pass::kStep2Moments || pass == Pass::kStep2MomentsTopRow) {
      if constexpr (kHasAdjoint<St>) {
        constexpr unsigned MM = M | tlbk::kModeMoments;
        if (d.moving || d.has_solid) return;
        if (pass == Pass::kStep2Moments) launch_step2_kernel<St, MM>(d, a);
        else launch_step2_kernel<St, MM | tlbk::kModeTopRow>(d, a);
      }
      return;
    }
    if (d.moving) {
      if (d.has_solid) launch_step2_kernel<St, M | S | V>(d, a);
      else launch_step2_kernel<St, M | V>(d, a);
    } else {
      if (d.has_solid) launch_step2_kernel<St, M | S>(d, a);
      else launch_step2_kernel<St, M>(d, a);
    }
  }
}

// Storages with the moment state. Not the fixed-point one, whose 27 planes have
// no room for three sets of FP32 moments, and not BF16, whose population
// kernels are compiled to roundings that equilibria_stored does not repeat at
// every node (a flip of 2^-8 of a deviation now and then).
template <class St>
constexpr bool kHasMoments = !St::kFix && !std::is_same_v<St, tlbk::StoreBF16Dev>;

template <class St, unsigned kMode>
void launch_moment_kernel(const Device& d, const tlbk::MomentArgs<typename St::C>& a) {
  constexpr bool kList = (kMode & tlbk::kMomStep) != 0 && (kMode & tlbk::kModeSolid) != 0;
  hipLaunchKernelGGL((tlbk::lb_moment_kernel<St, kMode>), kList ? dim3(d.ntiles) : d.geo.grid_m,
                     dim3(64), 0, d.stream, a);
}

// Passes that only read the time level: the walls' motion plays no part.
template <class St, unsigned kMode>
void launch_moment_solid(const Device& d, const tlbk::MomentArgs<typename St::C>& a) {
  if (d.has_solid) launch_moment_kernel<St, kMode | tlbk::kModeSolid>(d, a);
  else launch_moment_kernel<St, kMode>(d, a);
}

template <class St, unsigned kMode>
void launch_moment_split(const Device& d, const tlbk::MomentArgs<typename St::C>& a) {
  if constexpr (tlbk::kSameRounding<typename St::C> && (kMode & tlbk::kMomShear) == 0) {
    if (d.pair_second) {
      launch_moment_kernel<St, kMode | tlbk::kMomSplit>(d, a);
      return;
    }
  }
  launch_moment_kernel<St, kMode>(d, a);
}

template <class St, unsigned M>
void launch_moment_walls(const Device& d, const tlbk::MomentArgs<typename St::C>& a) {
  constexpr unsigned S = tlbk::kModeSolid, V = tlbk::kModeMoving;
  if (d.moving) {
    if (d.has_solid) launch_moment_split<St, M | S | V>(d, a);
    else launch_moment_split<St, M | V>(d, a);
  } else {
    if (d.has_solid) launch_moment_split<St, M | S>(d, a);
    else launch_moment_split<St, M>(d, a);
  }
}

template <class St>
void launch_moment(const Device& d, MomentPass pass, const void* src, void* dst) {
  using namespace tlbk;
  using C = typename St::C;
  MomentArgs<C> a{};
  a.s = make_args<C>(d, src, dst);
  a.s.rows_per_block = d.geo.rows_m;
  a.strip = d.geo.strip_m;
  a.tiles = static_cast<const MomentTile*>(d.tiles);
  a.ntiles = d.ntiles;
  a.nlinked = d.nlinked;
  a.src_full = d.src_full;
  // (the fused kernel without solid cells, at rest, loads T_w, and with it 2 w
  // T_w, in a block of its own at both levels, the others at the second)
  a.round_wall = d.pair_second || (d.pair_first && !d.has_solid && !d.moving && !St::kDev);
  a.out = static_cast<double*>(dst);
  const tlb_params& p = *d.p;
  // combined from the constants as the population kernels round them, so
  // that both evaluate the same forces
  auto w = [](int c2) { return (double)w_c2<C>(c2); };
  auto q = [](int c2) { return (double)p_c2<C>(c2); };
  for (int l = 0; l < 2; ++l) {
    const double ga = (double)C(p.g_a[l]), gr = (double)C(p.g_r[l]);
    a.g1[l] = C(ga * w(1) + gr * q(1));
    a.g2[l] = C(ga * w(2) + gr * q(2));
    a.g5[l] = C(gr * q(5));
    a.h4[l] = C(2 * gr * q(4));
    a.h5[l] = C(2 * gr * q(5));
    a.h8[l] = C(2 * gr * q(8));
  }
  a.x2 = C((double)a.s.g12 * w(2) * (double)a.s.inv_rho0 * (double)a.s.inv_rho0);
  switch (pass) {
    case MomentPass::kStep: launch_moment_walls<St, kMomStep>(d, a); break;
    case MomentPass::kStepTopRow:  // the adjoint's
      if constexpr (kHasAdjoint<St>) launch_moment_split<St, kMomStep | kModeTopRow>(d, a);
      break;
    case MomentPass::kObserve: launch_moment_solid<St, kMomObserve>(d, a); break;
    case MomentPass::kFields: launch_moment_solid<St, kMomFields>(d, a); break;
    case MomentPass::kExport: launch_moment_solid<St, kMomExport>(d, a); break;
    case MomentPass::kShear: launch_moment_walls<St, kMomStep | kMomShear>(d, a); break;
    case MomentPass::kStress:
      a.shear = static_cast<const C*>(dst);
      launch_moment_solid<St, kMomFields | kMomStress>(d, a);
      break;
  }
}

template <class St, int BT, unsigned kMode>
int step2_occupancy() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, tlbk::lb_step2_kernel<St, BT, kMode>, BT,
                                                   0) != hipSuccess ||
      n < 1)
    n = 1;
  return n;
}

template <class St, unsigned kMode>
int step2_occupancy_lanes(int lanes) {
  return lanes == kStep2LanesNarrow ? step2_occupancy<St, kStep2LanesNarrow, kMode>()
                                    : step2_occupancy<St, kStep2Lanes, kMode>();
}

}  // namespace detail

template <class St>
int Launcher<St>::step2_blocks_per_cu(bool solid, int lanes) {
  if constexpr (detail::kHasStep2<St>) {
    constexpr unsigned M = tlbk::kModeStore | tlbk::kModeTauOne;
    return solid ? detail::step2_occupancy_lanes<St, M | tlbk::kModeSolid>(lanes)
                 : detail::step2_occupancy_lanes<St, M>(lanes);
  } else {
    (void)solid;
    (void)lanes;
    return 0;
  }
}

template <class St>
int Launcher<St>::blocks_per_cu(int bx, bool wide, bool solid, bool tau_one) {
  using namespace tlbk;
  constexpr unsigned S = kModeStore;
  if (solid) {
    return tau_one ? detail::occupancy_geometry<St, S | kModeSolid | kModeTauOne>(bx, wide)
                   : detail::occupancy_geometry<St, S | kModeSolid>(bx, wide);
  }
  return tau_one ? detail::occupancy_geometry<St, S | kModeTauOne>(bx, wide)
                 : detail::occupancy_geometry<St, S>(bx, wide);
}

template <class St>
void Launcher<St>::step(const Device& d, Pass pass, const void* src, void* dst, void* moments) {
  using namespace tlbk;
  switch (pass) {
    case Pass::kStep: detail::launch_mode<St, kModeStore>(d, src, dst); break;
    case Pass::kStepObserve: detail::launch_mode<St, kModeStore | kModeObserve>(d, src, dst); break;
    case Pass::kInitStep:
      detail::launch_mode<St, kModeStore | kModeInit | kModeObserve>(d, src, dst);
      break;
    case Pass::kObserve: detail::launch_mode<St, kModeObserve>(d, src, dst); break;
    case Pass::kObserveInit: detail::launch_mode<St, kModeObserve | kModeInit>(d, src, dst); break;
    case Pass::kFields: detail::launch_mode<St, kModeFields>(d, src, dst); break;
    case Pass::kFieldsInit: detail::launch_mode<St, kModeFields | kModeInit>(d, src, dst); break;
    case Pass::kStress: detail::launch_mode<St, kModeFields | kModeStress>(d, src, dst); break;
    case Pass::kStressInit:
      detail::launch_mode<St, kModeFields | kModeStress | kModeInit>(d, src, dst);
      break;
    case Pass::kStepMoments:
      if constexpr (detail::kHasAdjoint<St>) {
        if (d.tau_one && !d.moving && !d.has_solid) {
          auto a = detail::make_args<typename St::C>(d, src, dst);
          a.moments = moments;
          detail::launch_geometry<St, kModeStore | kModeTauOne | kModeMoments>(d, a);
        }
      }
      break;
    case Pass::kStep2:
    case Pass::kStep2TopRow:
    case Pass::kStep2Moments:
    case Pass::kStep2MomentsTopRow: detail::launch_step2<St>(d, src, dst, pass, moments); break;
  }
}

template <class St>
void Launcher<St>::init_equilibrium(const Device& d, void* buf, const double* rho_a,
                                    const double* rho_b, const double* temp, const double* ux0,
                                    const double* uy0) {
  using C = typename St::C;
  const tlb_params& p = *d.p;
  dim3 grid((p.lx + 255) / 256, p.ly, 1);
  hipLaunchKernelGGL(tlbk::lb_init_equilibrium<St>, grid, dim3(256), 0, d.stream,
                     static_cast<typename St::T*>(buf), rho_a, rho_b, temp, ux0, uy0, d.solid, p.lx,
                     p.ly, d.pitch, d.pop_stride, C(p.rho_ref[0]), C(p.rho_ref[1]), C(p.t_ref));
}

template <class St>
void Launcher<St>::moment(const Device& d, MomentPass pass, const void* src, void* dst) {
  if constexpr (detail::kHasMoments<St>) detail::launch_moment<St>(d, pass, src, dst);
}

template <class St>
void Launcher<St>::init_moments(const Device& d, void* dst, void* shear, const double* rho_a,
                                const double* rho_b, const double* temp, const double* ux0,
                                const double* uy0) {
  if constexpr (detail::kHasMoments<St>) {
    using C = typename St::C;
    const tlb_params& p = *d.p;
    dim3 grid((p.lx + 255) / 256, p.ly, 1);
    hipLaunchKernelGGL(tlbk::lb_moment_init<St>, grid, dim3(256), 0, d.stream,
                       static_cast<C*>(dst), static_cast<C*>(shear), rho_a, rho_b, temp, ux0, uy0,
                       d.solid, p.lx, d.pitch, d.pop_stride, C(p.rho_wall[0]), C(p.rho_wall[1]), C(p.rho_ref[0]),
                       C(p.rho_ref[1]), C(p.t_ref));
  }
}

template <class St>
void Launcher<St>::export_populations(const Device& d, const void* buf, double* out) {
  using C = typename St::C;
  const tlb_params& p = *d.p;
  dim3 grid((p.lx + 255) / 256, p.ly, 27);
  hipLaunchKernelGGL(tlbk::lb_export_populations<St>, grid, dim3(256), 0, d.stream,
                     static_cast<const typename St::T*>(buf), out, d.solid, p.lx, p.ly, d.pitch,
                     d.pop_stride, C(p.rho_ref[0]), C(p.rho_ref[1]), C(p.t_ref));
}

}  // namespace tlbh
