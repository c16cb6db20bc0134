// Plane passes (x and y transforms of a plane in one workgroup) and, with
// LSH_P_ROWS, the x passes over blocks of rows: instances of one element type
// (LSH_P_TYPE) and part (LSH_P_PART: 0 and 1 forward, 2 and 3 inverse, for
// scalar and elastic fields).
#include "plane.hpp"

#include "dispatch.hpp"

#ifndef LSH_P_TYPE
#error "define LSH_P_TYPE and LSH_P_PART"
#endif

namespace lsh {

#ifndef LSH_P_ROWS
// Threads and vectors per thread of a square plane of nvec 16-byte vectors:
// about four a thread, and above LIM vectors 1024 threads.  The forward pass
// of conjugate gradients and the plain one take LIM = 4608 (FP32 up to 128 x
// 128, FP64 up to 96 x 96 with 512 threads; CG forward at 128 x 128 scalar FP32
// 88 us with 512 threads, 94 with 1024), the inverse passes and the refinement
// LIM = 2560 (CG inverse there 79 us and 69).
template <typename T, int N, int LIM> constexpr int sq_nt() {
  constexpr int nvec = N * N * (int)sizeof(T) / 16;
  return nvec <= 512 ? 128 : nvec <= 1024 ? 256 : nvec <= LIM ? 512 : 1024;
}

// Planes with an instance: squares of the cubic grids' lengths with every
// index at compile time, and any other plane of at most 3072 (FP32) or 2048
// (FP64) vectors with run-time lengths, where larger ones lose to the separate
// passes (applications, FP32: 16 x 32 x 256 1.2 times as fast, 32 x 96 x 192
// 0.9 times; FP64: 64 x 8 x 256 1.2 to 1.35 times, 8 x 128 x 64 0.83 times).
template <typename T, int LIM, typename F>
static int plane_config(const PlaneGeo& p, F&& f) {
  using std::integral_constant;
  if (p.nx == p.ny) {
    auto sq = [&](auto n_) {
      constexpr int N = decltype(n_)::value, NT = sq_nt<T, N, LIM>();
      constexpr int K = (PlaneSq<T, N>::nvec + NT - 1) / NT;
      return f(integral_constant<int, NT>{}, integral_constant<int, K>{}, PlaneSq<T, N>{});
    };
    switch (p.nx) {
      case 16: return sq(integral_constant<int, 16>{});
      case 32: return sq(integral_constant<int, 32>{});
      case 48: return sq(integral_constant<int, 48>{});
      case 64: return sq(integral_constant<int, 64>{});
      case 80: return sq(integral_constant<int, 80>{});
      case 96: return sq(integral_constant<int, 96>{});
      case 128: return sq(integral_constant<int, 128>{});
      case 160:
        if constexpr (sizeof(T) == 4) return sq(integral_constant<int, 160>{});
        break;
      default: break;
    }
  }
  if (p.nvec <= 512) return f(integral_constant<int, 128>{}, integral_constant<int, 4>{}, PlaneGeo{});
  if (p.nvec <= 1024) return f(integral_constant<int, 256>{}, integral_constant<int, 4>{}, PlaneGeo{});
  if (p.nvec <= 2048) return f(integral_constant<int, 512>{}, integral_constant<int, 4>{}, PlaneGeo{});
  if constexpr (sizeof(T) == 4) {
    if (p.nvec <= 3072) return f(integral_constant<int, 512>{}, integral_constant<int, 6>{}, PlaneGeo{});
  }
  return -1;
}
#else

template <typename T, int LIM, typename F>
static int plane_config(const PlaneGeo& p, F&& f) {
  using std::integral_constant;
  auto rb = [&](auto n_) {
    constexpr int N = decltype(n_)::value;
    auto go = [&](auto small_) {
      constexpr int RB = rows_per_block<T>(N, decltype(small_)::value);
      using G = PlaneFix<T, N, RB, false>;
      constexpr int NT = (G::nvec / 4 + 63) / 64 * 64, K = (G::nvec + NT - 1) / NT;
      if (p.ny % RB != 0) return -1;   // p.ny: all rows of a component
      return f(integral_constant<int, NT>{}, integral_constant<int, K>{}, G{});
    };
    return p.nvec == 2 ? go(std::true_type{}) : go(std::false_type{});
  };
  switch (p.nx) {
    case 48: return rb(integral_constant<int, 48>{});
    case 64: return rb(integral_constant<int, 64>{});
    case 80: return rb(integral_constant<int, 80>{});
    case 96: return rb(integral_constant<int, 96>{});
    case 128: return rb(integral_constant<int, 128>{});
    case 160: return rb(integral_constant<int, 160>{});
    case 192: return rb(integral_constant<int, 192>{});
    case 256: return rb(integral_constant<int, 256>{});
    case 512: return rb(integral_constant<int, 512>{});
    case 1024: return rb(integral_constant<int, 1024>{});
    default: return -1;
  }
}

#define launch_pf launch_rf
#define launch_pf6 launch_rf6
#define launch_pi launch_ri
#define launch_pi6 launch_ri6
#endif

// grid and dynamic LDS of an instance: planes or row blocks, times components
template <typename T, typename P>
static int plane_blocks(const Geo& g) {
  if constexpr (P::kY) return g.nz * g.c;
  else return (int)((long long)g.nz * g.ny / P::ny) * g.c;
}
template <typename T, typename P>
static size_t plane_lds_of(const PlaneGeo& p) {
  if constexpr (P::kStatic) return plane_lds_bytes<T>(P::nx, P::ny, P::pitch);
  else return plane_lds_bytes<T>(p.nx, p.ny, p.pitch);
}

template <typename T, bool EL, int XF>
static int pf_inst(hipStream_t s, const PlaneFwdArgs<T>& a, int nload) {
  return plane_config<T, (XF == XF_IRX ? 2560 : 4608)>(a.p, [&](auto nt_, auto k_, auto geo_) {
    constexpr int NT = decltype(nt_)::value, K = decltype(k_)::value;
    using P = decltype(geo_);
    const int nb = plane_blocks<T, P>(a.g);
    const size_t lds = plane_lds_of<T, P>(a.p);
    hipLaunchKernelGGL((k_pf<T, NT, K, EL, XF, P>), dim3(nb, nload), dim3(NT), lds, s, a);
    return nb;
  });
}

template <typename T, bool EL, int MODE>
static int pi_inst(hipStream_t s, const PlaneInvArgs<T>& a, int nload) {
  return plane_config<T, 2560>(a.p, [&](auto nt_, auto k_, auto geo_) {
    constexpr int NT = decltype(nt_)::value, K = decltype(k_)::value;
    using P = decltype(geo_);
    const int nb = plane_blocks<T, P>(a.g);
    const size_t lds = plane_lds_of<T, P>(a.p);
    hipLaunchKernelGGL((k_pi<T, NT, K, EL, MODE, P>), dim3(nb, nload), dim3(NT), lds, s, a);
    return nb;
  });
}

#if LSH_P_PART == 0
template <typename T>
int launch_pf(hipStream_t s, const PlaneFwdArgs<T>& a, int mode, int nload) {
  if (mode == XF_CG && a.g.c == 6) return launch_pf6<T>(s, a, nload);
  switch (mode) {
    case XF_PLAIN: return pf_inst<T, false, XF_PLAIN>(s, a, nload);
    case XF_CG: return pf_inst<T, false, XF_CG>(s, a, nload);
    case XF_IRX:
      if constexpr (sizeof(T) == 8) return pf_inst<T, false, XF_IRX>(s, a, nload);
      return -1;
    default: return -1;
  }
}
template int launch_pf<LSH_P_TYPE>(hipStream_t, const PlaneFwdArgs<LSH_P_TYPE>&, int, int);
#elif LSH_P_PART == 1
template <typename T>
int launch_pf6(hipStream_t s, const PlaneFwdArgs<T>& a, int nload) {
  return pf_inst<T, true, XF_CG>(s, a, nload);
}
template int launch_pf6<LSH_P_TYPE>(hipStream_t, const PlaneFwdArgs<LSH_P_TYPE>&, int);
#else
#if LSH_P_PART == 2
constexpr bool kEl = false;
#else
constexpr bool kEl = true;
#endif
template <typename T>
static int pi_mode(hipStream_t s, const PlaneInvArgs<T>& a, int mode, int nload) {
  switch (mode) {
    case XI_APPLY:
    case XI_CG: return pi_inst<T, kEl, XI_APPLY>(s, a, nload);
    case XI_CGR: return pi_inst<T, kEl, XI_CGR>(s, a, nload);
    default: break;
  }
  if constexpr (sizeof(T) == 8) {
    switch (mode) {
      case XI_IRRES: return pi_inst<T, kEl, XI_IRRES>(s, a, nload);
      case XI_RESNORM: return pi_inst<T, kEl, XI_RESNORM>(s, a, nload);
      case XI_STRAIN:
        if constexpr (!kEl) return pi_inst<T, false, XI_STRAIN>(s, a, nload);
        break;
      default: break;
    }
  }
  return -1;
}
#if LSH_P_PART == 2
template <typename T>
int launch_pi(hipStream_t s, const PlaneInvArgs<T>& a, int mode, int nload) {
  if (mode != XI_STRAIN && a.g.c == 6) return launch_pi6<T>(s, a, mode, nload);
  return pi_mode<T>(s, a, mode, nload);
}
template int launch_pi<LSH_P_TYPE>(hipStream_t, const PlaneInvArgs<LSH_P_TYPE>&, int, int);
#else
template <typename T>
int launch_pi6(hipStream_t s, const PlaneInvArgs<T>& a, int mode, int nload) {
  return pi_mode<T>(s, a, mode, nload);
}
template int launch_pi6<LSH_P_TYPE>(hipStream_t, const PlaneInvArgs<LSH_P_TYPE>&, int, int);
#endif
#endif

}  // namespace lsh
