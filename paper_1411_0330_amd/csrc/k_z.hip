// z pass fused with the Green operator; instances for one element type
// (LSH_Z_TYPE) so that FP32 and FP64 compile in parallel.  Built twice per
// type: without LSH_Z_STORED the operator is formed on the fly (launch_zg);
// with it, from the stored table (launch_zg_stored, three- and
// six-component 3D fields), in a unit of its own so both compile in parallel;
// and with LSH_Z_FLAT the pass of 2D grids (launch_zg_flat).
#include "dispatch.hpp"

namespace lsh {

#ifdef LSH_Z_STORED
constexpr bool kGS = true;
#else
constexpr bool kGS = false;
#endif

template <typename T, int NZ, int C, int TX, int P, bool PR = false>
static int z_inst(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
                  cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps) {
  constexpr int NT = TX * (NZ / P);
  const int xtiles = (g.mx + TX - 1) / TX;
  const int main_tiles = g.ny * xtiles;
  const int nyq_tiles = (g.ny + TX - 1) / TX;
  // stored operator: one workgroup per (tile, load), the loads of a tile adjacent on one XCD
  const dim3 grid = kGS ? dim3((main_tiles + nyq_tiles) * nload, 1) : dim3(main_tiles + nyq_tiles, nload);
  hipLaunchKernelGGL((k_zg<T, NZ, P, TX, C, kGS, PR>), grid, dim3(NT), 0, s, g, gp, tb, zmode, sm, sn, tw, st,
                     main_tiles, qp, ps, nload);
  return main_tiles + nyq_tiles;
}

#ifdef LSH_Z_FLAT
// 2D: the y transforms, Gamma and the inverse y transforms in one pass, as the
// last axis of an nx x 1 x ny grid.  A 2D grid has few pencils, so the pass is
// bounded by the chain of one pencil, not by memory: few points a thread (4, or
// twice the odd factor) and the fewest pencils that fill a wave, at least two.
// Two loads of a square FP64 grid, with 8 or 12 points and 64-byte row segments
// and now: 64^2 11.2 and 9.1 us, 128^2 12.9 and 9.9, 192^2 16.0 and 13.2, 256^2
// 14.0 and 11.0, 512^2 18.1 and 17.2, 1024^2 48.2 and 38.6 (the three separate
// passes at 512^2: 10.2 + 9.6 + 10.2).  FP32 at 1024 points keeps 8 points and
// four pencils (26 us; with 4 points 31 to 35).
template <typename T, int NL>
static int z2(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
              cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps) {
  constexpr bool wide = sizeof(T) == 4 && NL >= 1024;
  constexpr int P = odd_part(NL) > 1 ? p_odd<T>(NL, 2) : cmin(wide ? 8 : 4, NL);
  constexpr int TX = cmin(64, cmax(wide ? 4 : 2, 64 * P / NL));
  return z_inst<T, NL, 2, TX, P>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
}

template <typename T>
int launch_zg_flat(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
                   cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps) {
  if (g.ny != 1) return -1;
  switch (g.nz) {
#define LSH_Z2(N) \
  case N: return z2<T, N>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps)
    LSH_Z2(2);
    LSH_Z2(4);
    LSH_Z2(8);
    LSH_Z2(16);
    LSH_Z2(32);
    LSH_Z2(64);
    LSH_Z2(128);
    LSH_Z2(256);
    LSH_Z2(512);
    LSH_Z2(1024);
    LSH_Z2(48);
    LSH_Z2(96);
    LSH_Z2(192);
    LSH_Z2(80);
    LSH_Z2(160);
#undef LSH_Z2
    default: return -1;
  }
}
#else

template <typename T, int NZ, int C>
static int zm_inst(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, cpx<T>* sm,
                   cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps) {
  constexpr int P = p_zm<T, C>(NZ);
  constexpr int TX = tx_zm<T>(NZ, P);
  constexpr int NT = TX * (NZ / P);
  const int xtiles = (g.mx + TX - 1) / TX;
  const int main_tiles = g.ny * xtiles;
  const int nyq_tiles = (g.ny + TX - 1) / TX;
  hipLaunchKernelGGL((k_zgm<T, NZ, P, TX, C>), dim3(main_tiles + nyq_tiles, 1), dim3(NT), 0, s, g, gp, tb, sm, sn,
                     tw, st, main_tiles, nload, qp, ps);
  return main_tiles + nyq_tiles;
}

template <typename T, int NZ, int C, int V>
static int z_var(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
                 cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps) {
  constexpr int P0 = p_z<T, C>(NZ);
  constexpr int TX0 = tx_strided<T>(NZ, P0);
  constexpr int TXV = sv_tx<T>(NZ, P0, V), PV = sv_p(P0, V);
  if constexpr (V != 0 && sv_ok<T>(NZ, TXV, PV))
    return z_inst<T, NZ, C, TXV, PV>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
  else
    return z_inst<T, NZ, C, TX0, P0>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
}

template <typename T, int NZ, int C>
static int z_one(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
                 cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps, int variant = 0) {
  if constexpr (!kGS && sizeof(T) == 4 && (NZ == 128 || NZ == 256) && C != 2) {
    if (variant == 4 && zmode == Z_GAMMA && gp.variant != kGreenFD)
      return zm_inst<T, NZ, C>(s, g, gp, tb, sm, sn, tw, st, nload, qp, ps);
  }
  if constexpr (NZ == 128 || NZ == 256) {
    switch (variant) {
      case 1: return z_var<T, NZ, C, 1>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
      case 2: return z_var<T, NZ, C, 2>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
      case 3: return z_var<T, NZ, C, 3>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
      default: break;
    }
  }
  if constexpr (kGS && zs_ok<T, C>(NZ)) {
    constexpr int P = p_zs<T, C>(NZ), TX = tx_zs<T, C>(NZ);
    if constexpr (sizeof(T) == 4 && TX / 2 * (NZ / P) >= 64) {
      if (g.mx % TX != 0 && g.mx % (TX / 2) == 0)
        return z_inst<T, NZ, C, TX / 2, P>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    }
    return z_inst<T, NZ, C, TX, P>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
  } else {
    return z_var<T, NZ, C, 0>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
  }
}

template <typename T, int C>
static int z_c(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
               cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, int v, double* qp, int ps) {
  switch (g.nz) {
    case 2: return z_one<T, 2, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 4: return z_one<T, 4, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 8: return z_one<T, 8, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 16: return z_one<T, 16, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 32: return z_one<T, 32, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 64: return z_one<T, 64, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 128: return z_one<T, 128, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps, v);
    case 256: return z_one<T, 256, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps, v);
    case 512: return z_one<T, 512, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 1024: return z_one<T, 1024, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 48: return z_one<T, 48, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 96: return z_one<T, 96, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 192: return z_one<T, 192, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 80: return z_one<T, 80, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    case 160: return z_one<T, 160, C>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
    default: return -1;
  }
}

#ifdef LSH_Z_STORED
template <typename T>
int launch_zg_stored(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, cpx<T>* sm,
                     cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, int v, double* qp, int ps) {
  if (g.nz == 1 || tb.st == nullptr) return -1;
  if (g.c == 3) return z_c<T, 3>(s, g, gp, tb, Z_GAMMA, sm, sn, tw, st, nload, v, qp, ps);
  if (g.c == 6) return z_c<T, 6>(s, g, gp, tb, Z_GAMMA, sm, sn, tw, st, nload, v, qp, ps);
  return -1;
}

// 8-pencil tiles of the component-paired layout: two workgroups per compute
// unit, every access a whole 128-byte line
template <typename T>
int launch_zg_paired(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, cpx<T>* sp,
                     cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, double* qp, int ps) {
  if constexpr (sizeof(T) == 4) {
    if (g.c != 6 || tb.st == nullptr) return -1;
    if (g.nz == 128)
      return z_inst<T, 128, 6, 8, p_z<T, 6>(128), true>(s, g, gp, tb, Z_GAMMA, sp, sn, tw, st, nload, qp, ps);
    if (g.nz == 256)
      return z_inst<T, 256, 6, 8, p_z<T, 6>(256), true>(s, g, gp, tb, Z_GAMMA, sp, sn, tw, st, nload, qp, ps);
  }
  return -1;
}
#else
template <typename T>
int launch_zg(hipStream_t s, const Geo& g, const GreenParams& gp, const GreenTabs<T>& tb, int zmode, cpx<T>* sm,
              cpx<T>* sn, const cpx<T>* tw, const LoadState* st, int nload, int v, double* qp, int ps) {
  if (g.c == 2) return launch_zg_flat<T>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, qp, ps);
  // the stored operator (where bound) serves the Green pass of every shape
  // except the multi-load one (4), which forms its matrices itself
  if (zmode == Z_GAMMA && tb.st != nullptr && g.nz > 1 && v != 4)
    return launch_zg_stored<T>(s, g, gp, tb, sm, sn, tw, st, nload, v, qp, ps);
  if (g.c == 3) return z_c<T, 3>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, v, qp, ps);
  if (g.c == 6) return z_c<T, 6>(s, g, gp, tb, zmode, sm, sn, tw, st, nload, v, qp, ps);
  return -1;
}
#endif
#endif  // LSH_Z_FLAT

#ifndef LSH_Z_TYPE
#error "define LSH_Z_TYPE"
#endif
#ifdef LSH_Z_FLAT
template int launch_zg_flat<LSH_Z_TYPE>(hipStream_t, const Geo&, const GreenParams&, const GreenTabs<LSH_Z_TYPE>&, int,
                                        cpx<LSH_Z_TYPE>*, cpx<LSH_Z_TYPE>*, const cpx<LSH_Z_TYPE>*, const LoadState*,
                                        int, double*, int);
#elif defined(LSH_Z_STORED)
template int launch_zg_stored<LSH_Z_TYPE>(hipStream_t, const Geo&, const GreenParams&, const GreenTabs<LSH_Z_TYPE>&,
                                          cpx<LSH_Z_TYPE>*, cpx<LSH_Z_TYPE>*, const cpx<LSH_Z_TYPE>*,
                                          const LoadState*, int, int, double*, int);
template int launch_zg_paired<LSH_Z_TYPE>(hipStream_t, const Geo&, const GreenParams&, const GreenTabs<LSH_Z_TYPE>&,
                                          cpx<LSH_Z_TYPE>*, cpx<LSH_Z_TYPE>*, const cpx<LSH_Z_TYPE>*,
                                          const LoadState*, int, double*, int);
#else
template int launch_zg<LSH_Z_TYPE>(hipStream_t, const Geo&, const GreenParams&, const GreenTabs<LSH_Z_TYPE>&, int,
                                   cpx<LSH_Z_TYPE>*, cpx<LSH_Z_TYPE>*, const cpx<LSH_Z_TYPE>*, const LoadState*,
                                   int, int, double*, int);
#endif

}  // namespace lsh
