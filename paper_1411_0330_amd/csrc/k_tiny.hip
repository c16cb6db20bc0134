// Persistent CG for small grids; instances for one element type (LSH_TINY_TYPE).
#include "dispatch.hpp"
#include "tiny.hpp"

namespace lsh {

// Threads by the radix-8 butterflies of a sweep (W).  512 is the most: with
// 1024 the fields in registers spill (64^2 FP64 17 -> 22 us an iteration, 16^3
// FP64 34 -> 43; FP32 within 3%).  From 96 butterflies 256 threads (32^2 FP64
// 19 us with 128 threads, 8.3 with 256), below it 128.
template <typename T, int NX, int NY, int NZ, int C>
static int tiny_inst(hipStream_t s, const TinyArgs<T>& a, int nload) {
  constexpr int W = C * NX * NY * NZ / 16;
  constexpr int NT = W >= 512 ? 512 : W >= 96 ? 256 : 128;
  if ((a.vcoef == nullptr && a.iso == 0) || a.gp.variant == kGreenFD)
    hipLaunchKernelGGL((k_tiny_cg<T, NX, NY, NZ, C, NT, true>), dim3(nload), dim3(NT), 0, s, a);
  else
    hipLaunchKernelGGL((k_tiny_cg<T, NX, NY, NZ, C, NT, false>), dim3(nload), dim3(NT), 0, s, a);
  return nload;
}

// grids of tiny_grid(): squares 8..64 (2D), cubes of 8 and (scalar) 16
template <typename T>
int launch_tiny_cg(hipStream_t s, const TinyArgs<T>& a, int nload) {
  const Geo& g = a.g;
  if (g.nz == 1 && g.c == 2 && g.nx == g.ny) {
    switch (g.nx) {
      case 8: return tiny_inst<T, 8, 8, 1, 2>(s, a, nload);
      case 16: return tiny_inst<T, 16, 16, 1, 2>(s, a, nload);
      case 32: return tiny_inst<T, 32, 32, 1, 2>(s, a, nload);
      case 64: return tiny_inst<T, 64, 64, 1, 2>(s, a, nload);
      default: return -1;
    }
  }
  if (g.nz > 1 && g.nx == g.ny && g.ny == g.nz) {
    if (g.nx == 8 && g.c == 3) return tiny_inst<T, 8, 8, 8, 3>(s, a, nload);
    if (g.nx == 8 && g.c == 6) return tiny_inst<T, 8, 8, 8, 6>(s, a, nload);
    if (g.nx == 16 && g.c == 3) return tiny_inst<T, 16, 16, 16, 3>(s, a, nload);
  }
  return -1;
}

#ifndef LSH_TINY_TYPE
#error "define LSH_TINY_TYPE"
#endif
template int launch_tiny_cg<LSH_TINY_TYPE>(hipStream_t, const TinyArgs<LSH_TINY_TYPE>&, int);

}  // namespace lsh
