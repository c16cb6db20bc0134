// Plane passes: the x and y transforms of one z-plane of one component in one
// workgroup, the half spectrum of the plane held in LDS.
//
//   k_pf  forward: real plane (with the solver's epilogue of the x pass) ->
//         x R2C -> y, written in the plain spectrum layout;
//   k_pi  inverse: spectrum plane -> y -> x C2R -> local term and epilogue.
//
// They replace the separate x and y passes (and one spectrum write and read
// per direction) where a plane fits in LDS.  What bounds them is the traffic
// of the fields: a plane is read in one burst of 16-byte accesses, transformed
// in LDS while other workgroups of the CU read theirs, and written in one
// burst.  Transforms run in place in LDS (decimation in frequency forward,
// natural order in, digit-reversed out; decimation in time inverse), one lane
// per row of the x transforms and one lane per column of the y transforms, so
// the lanes of a wave read consecutive columns, or rows an odd pitch apart
// (no bank conflicts), and registers hold one butterfly at a time: occupancy
// is bounded by LDS alone.  Axis lengths are run-time values: radices 3 or 5
// first, then powers of two, so every later span is a power of two.
//
// Without the y transform (blocks of rows instead of planes) the same kernels
// are the x passes of larger grids: 192^3 elastic FP64 x 2 loads 824 and 592 us
// a pass in registers (280 and 356 of them, one wave per SIMD), 716 and 542
// here; 160^3 scalar FP64 353 and 317 -> 277 and 219 us.
//
// Measured against the separate passes, x + y forward and y + x inverse in CG:
// 64^3 elastic FP32 x 6 loads 41.5 + 21.3 and 21.3 + 36.0 us -> 40.3 and 39.7;
// 128^3 scalar FP32 x 3 82 + 31 and 31 + 65 -> 88 and 68; 96^3 elastic FP32 x 6
// 177 + 50 and 50 + 141 -> 150 and 115 (the y pass comes free forward; the
// inverse is left waiting for its spectrum and field reads, 4.5 TB/s).
//
// The half spectrum of a row is mx = nx/2 columns: column 0 carries the kx = 0
// value in its real part and the kx = nx/2 value in its imaginary part (both
// real for a real row); its y transform is separated into the kx = 0 column and
// the Nyquist plane by symmetry when it leaves LDS.
//
// The local term couples components only through the trace of the three normal
// ones (isotropic phases and per-voxel moduli), so a workgroup takes one
// component; in elasticity those of the normal components read the other two
// again for the trace (from cache, the planes are read side by side).
#pragma once

#include "kernels.hpp"

namespace lsh {

constexpr int kPlaneStages = 6;

// q = n / d for n d < 2^32: m = ceil(2^32 / d), d >= 2
struct FDiv {
  unsigned m, d;
};
__device__ __forceinline__ int fdiv(const int n, const FDiv& f) { return (int)__umulhi((unsigned)n, f.m); }

// Radices of one axis, odd one first, and the span (block length) each acts on.
struct PlaneAxis {
  int n, ns;
  int r[kPlaneStages];
  int l[kPlaneStages];    // block length L of the stage
  int sl[kPlaneStages];   // log2 of L / R (a power of two)
};

struct PlaneGeo {
  static constexpr bool kStatic = false, kY = true;
  int nx, ny, mx, pitch, nvec, pad;   // nvec: 16-byte vectors of one real plane (= of its half spectrum)
  FDiv by_nx, by_mx, by_ny;
  PlaneAxis ax, ay;                   // ax: the mx-point transform of the packed rows
  __device__ __forceinline__ int div_nx(int n) const { return fdiv(n, by_nx); }
  __device__ __forceinline__ int div_mx(int n) const { return fdiv(n, by_mx); }
  __device__ __forceinline__ int div_ny(int n) const { return fdiv(n, by_ny); }
};

inline FDiv make_fdiv(int d) { return FDiv{(unsigned)(((1ull << 32) + (unsigned)d - 1) / (unsigned)d), (unsigned)d}; }

// radices: the odd factor, then powers of two of at most `rmax` (16 or 8)
constexpr PlaneAxis make_axis(int n, int rmax) {
  PlaneAxis a{};
  a.n = n;
  int p = 1;
  while (n % (2 * p) == 0) p *= 2;
  int odd = n / p, m = 0;
  while ((1 << m) < p) ++m;
  if (odd > 1) a.r[a.ns++] = odd;
  const int lg = rmax == 16 ? 4 : 3;
  const int parts = (m + lg - 1) / lg;
  for (int i = 0; i < parts; ++i) {
    const int e = (m + (parts - i) - 1) / (parts - i);   // even split, larger radices first
    a.r[a.ns++] = 1 << e;
    m -= e;
  }
  int L = n;
  for (int s = 0; s < a.ns; ++s) {
    a.l[s] = L;
    L /= a.r[s];
    int lgS = 0;
    while ((1 << lgS) < L) ++lgS;
    a.sl[s] = lgS;
  }
  return a;
}

// The same with the axis lengths at compile time (every index and span a
// constant): square planes of the lengths that cubic grids have
// (Y), or blocks of NY whole rows whose y transform is left to the y pass.
template <typename T, int NX, int NY, bool Y>
struct PlaneFix {
  static constexpr bool kStatic = true, kY = Y;
  static constexpr int nx = NX, ny = NY, mx = NX / 2, pitch = mx | 1, nvec = NX * NY * (int)sizeof(T) / 16;
  static constexpr PlaneAxis ax = make_axis(mx, sizeof(T) == 4 ? 16 : 8), ay = make_axis(ny, sizeof(T) == 4 ? 16 : 8);
  __device__ __forceinline__ int div_nx(int n) const { return n / nx; }
  __device__ __forceinline__ int div_mx(int n) const { return n / mx; }
  __device__ __forceinline__ int div_ny(int n) const { return n / ny; }
};

// Row blocks: lengths with an instance, and rows per workgroup: 1024 16-byte
// vectors (768 or 1280 of lengths 3 and 5 times a power of two), or a quarter of
// them where that leaves fewer than 256 workgroups per load.
constexpr bool row_length(int n) {
  return n == 48 || n == 64 || n == 80 || n == 96 || n == 128 || n == 160 || n == 192 || n == 256 || n == 512 || n == 1024;
}
template <typename T> constexpr int rows_per_block(int n, bool small) {
  int r = 1;
  while (r * 2 * n * (int)sizeof(T) / 16 <= 1280 || (r * n * (int)sizeof(T) / 16) % 256 != 0) r *= 2;
  return small ? (r >= 4 ? r / 4 : 1) : r;
}
inline bool rows_small(const Geo& g, int rb) { return (long long)g.nz * g.ny / rb * g.c < 256; }
// workgroups per load
template <typename T> inline long long row_blocks(const Geo& g) {
  if (!row_length(g.nx)) return 0;
  return (long long)g.nz * g.ny * g.c / rows_per_block<T>(g.nx, rows_small(g, rows_per_block<T>(g.nx, false)));
}

template <typename T, int N> using PlaneSq = PlaneFix<T, N, N, true>;

template <typename P>
__device__ __forceinline__ decltype(auto) plane_geo(const PlaneGeo& p) {
  if constexpr (P::kStatic) return P{};
  else return (p);
}

// ---------------------------------------------------------------------------
// in-place transforms of every line of a plane in LDS
// ---------------------------------------------------------------------------
// element e of line i at buf[i ls + e es]; one butterfly per lane and step.
// X: lines are rows (y), else columns (kx positions).
template <int R, int DIR, bool X, typename T, int NT, typename P>
__device__ __forceinline__ void plane_stage(cpx<T>* buf, const P& p, const int L, const int sl, const cpx<T>* tw) {
  const int nline = X ? p.ny : p.mx, ls = X ? p.pitch : 1, es = X ? 1 : p.pitch;
  const int n = X ? p.mx : p.ny;
  const int S = 1 << sl;
  const int nb = nline * (n / R);
  const int tstep = (n / L) * (X ? 2 : 1);   // table step of W_L (the x table is of the row length 2 mx)
  const int rs = S * es;
#pragma unroll 1
  for (int idx = threadIdx.x; idx < nb; idx += NT) {
    const int b = X ? p.div_ny(idx) : p.div_mx(idx);
    const int line = idx - b * nline;
    const int j = b & (S - 1), blk = b >> sl;
    cpx<T>* q = buf + line * ls + (blk * L + j) * es;
    cpx<T> u[R];
    static_for<0, R>([&](auto r_) { u[decltype(r_)::value] = q[decltype(r_)::value * rs]; });
    if (DIR > 0 && S > 1) {
      static_for<1, R>([&](auto r_) {
        constexpr int r = decltype(r_)::value;
        u[r] = cmulc(u[r], tw[r * j * tstep]);
      });
    }
    dft<R, DIR>(u);
    if (DIR < 0 && S > 1) {
      static_for<1, R>([&](auto r_) {
        constexpr int r = decltype(r_)::value;
        u[r] = cmul(u[r], tw[r * j * tstep]);
      });
    }
    static_for<0, R>([&](auto r_) { q[decltype(r_)::value * rs] = u[decltype(r_)::value]; });
  }
}

template <int DIR, bool X, typename T, int NT, typename P>
__device__ __forceinline__ void plane_fft(cpx<T>* buf, const P& p, const cpx<T>* tw) {
  if constexpr (P::kStatic) {
    constexpr int ns = X ? P::ax.ns : P::ay.ns;
    static_for<0, ns>([&](auto i_) {
      constexpr int i = decltype(i_)::value, s = DIR < 0 ? i : ns - 1 - i;
      constexpr int R = X ? P::ax.r[s] : P::ay.r[s], L = X ? P::ax.l[s] : P::ay.l[s], sl = X ? P::ax.sl[s] : P::ay.sl[s];
      plane_stage<R, DIR, X, T, NT>(buf, p, L, sl, tw);
      __syncthreads();
    });
  } else {
    const PlaneAxis& a = X ? p.ax : p.ay;
    for (int i = 0; i < a.ns; ++i) {
      const int s = DIR < 0 ? i : a.ns - 1 - i;
      const int L = a.l[s], sl = a.sl[s];
      switch (a.r[s]) {
        case 2: plane_stage<2, DIR, X, T, NT>(buf, p, L, sl, tw); break;
        case 3: plane_stage<3, DIR, X, T, NT>(buf, p, L, sl, tw); break;
        case 4: plane_stage<4, DIR, X, T, NT>(buf, p, L, sl, tw); break;
        case 5: plane_stage<5, DIR, X, T, NT>(buf, p, L, sl, tw); break;
        case 8: plane_stage<8, DIR, X, T, NT>(buf, p, L, sl, tw); break;
        default:
          if constexpr (sizeof(T) == 4) plane_stage<16, DIR, X, T, NT>(buf, p, L, sl, tw);
          break;
      }
      __syncthreads();
    }
  }
}

// LDS position of frequency k of an axis (digit reversal of the radices)
__device__ __forceinline__ int plane_pos(const PlaneAxis& a, int k) {
  int pos = 0;
  for (int s = 0; s < a.ns; ++s) {
    const int q = k / a.r[s];
    pos += (k - q * a.r[s]) << a.sl[s];
    k = q;
  }
  return pos;
}

// the shared memory of a plane: spectrum, twiddles of both axes, positions
template <typename T>
struct PlaneLds {
  cpx<T>* buf;
  cpx<T>* twx;
  cpx<T>* twy;
  T* tab;            // per phase: in-I0 flag, a, b
  double* red;
  uint16_t* px;
  uint16_t* py;
};

template <typename T>
__host__ __device__ inline size_t plane_lds_bytes(int nx, int ny, int pitch) {
  const size_t b = sizeof(cpx<T>) * ((size_t)ny * pitch + nx + ny) + sizeof(T) * 3 * kMaxPhases + 16 * sizeof(double) +
                   sizeof(uint16_t) * (size_t)(nx / 2 + ny);
  return (b + 15) / 16 * 16;
}

template <typename T, typename P>
__device__ __forceinline__ PlaneLds<T> plane_lds(char* base, const P& p) {
  PlaneLds<T> s;
  s.red = reinterpret_cast<double*>(base);
  s.buf = reinterpret_cast<cpx<T>*>(s.red + 16);
  s.twx = s.buf + p.ny * p.pitch;
  s.twy = s.twx + p.nx;
  s.tab = reinterpret_cast<T*>(s.twy + p.ny);
  s.px = reinterpret_cast<uint16_t*>(s.tab + 3 * kMaxPhases);
  s.py = s.px + p.mx;
  return s;
}

template <typename T, int NT, typename P>
__device__ __forceinline__ void plane_tables(const PlaneLds<T>& s, const P& p, const cpx<T>* twx,
                                             const cpx<T>* twy) {
  for (int i = threadIdx.x; i < p.nx; i += NT) s.twx[i] = twx[i];
  if constexpr (P::kY) {
    for (int i = threadIdx.x; i < p.ny; i += NT) s.twy[i] = twy[i];
  }
  for (int i = threadIdx.x; i < p.mx; i += NT) s.px[i] = (uint16_t)plane_pos(p.ax, i);
  if constexpr (P::kY) {
    for (int i = threadIdx.x; i < p.ny; i += NT) s.py[i] = (uint16_t)plane_pos(p.ay, i);
  }
}

// (in-I0 flag, a, b) of each phase's short form a Id + b m m^T
template <typename T, int NT>
__device__ __forceinline__ void plane_phase_tab(T* tab, const T* ptab, const int nphase, const int c) {
  const int w = 2 * c * c + 5;
  for (int i = threadIdx.x; i < nphase; i += NT) {
    tab[3 * i] = ptab[(long long)i * w + 2 * c * c];
    tab[3 * i + 1] = ptab[(long long)i * w + 2 * c * c + 1];
    tab[3 * i + 2] = ptab[(long long)i * w + 2 * c * c + 2];
  }
}

// 16 bytes of reals
template <typename T> struct alignas(16) PVec { T v[16 / sizeof(T)]; };
template <typename T> __device__ __forceinline__ PVec<T> pv_load(const T* p) { return *reinterpret_cast<const PVec<T>*>(p); }
template <typename T> __device__ __forceinline__ void pv_store(T* p, const PVec<T>& v) { *reinterpret_cast<PVec<T>*>(p) = v; }

// 16-byte vector q of a real plane <-> the packed rows in LDS
template <typename T, typename P>
__device__ __forceinline__ void plane_put(cpx<T>* buf, const P& p, const int q, const PVec<T>& v) {
  constexpr int VEC = 16 / sizeof(T);
  const int e = q * VEC;
  const int y = p.div_nx(e);
  cpx<T>* b = buf + y * p.pitch + ((e - y * p.nx) >> 1);
#pragma unroll
  for (int i = 0; i < VEC / 2; ++i) b[i] = cpx<T>{v.v[2 * i], v.v[2 * i + 1]};
}
template <typename T, typename P>
__device__ __forceinline__ PVec<T> plane_get(const cpx<T>* buf, const P& p, const int q) {
  constexpr int VEC = 16 / sizeof(T);
  const int e = q * VEC;
  const int y = p.div_nx(e);
  const cpx<T>* b = buf + y * p.pitch + ((e - y * p.nx) >> 1);
  PVec<T> v;
#pragma unroll
  for (int i = 0; i < VEC / 2; ++i) {
    const cpx<T> z = b[i];
    v.v[2 * i] = z.x;
    v.v[2 * i + 1] = z.y;
  }
  return v;
}

// coefficients of (A - A0)^{-1} at the VEC voxels from `vox`: I0 flag, a and b
template <typename T> struct PCoef { PVec<T> in, a, b; };
template <bool WANT_B, typename T>
__device__ __forceinline__ PCoef<T> plane_coef(const uint8_t* phase, const T* vcoef, const T* tab,
                                               const long long nvox, const long long vox) {
  constexpr int VEC = 16 / sizeof(T);
  PCoef<T> c;
  if (vcoef != nullptr) {
    c.a = pv_load(vcoef + vox);
    if constexpr (WANT_B) c.b = pv_load(vcoef + nvox + vox);
#pragma unroll
    for (int i = 0; i < VEC; ++i) c.in.v[i] = c.a.v[i] != T(0) ? T(1) : T(0);
  } else {
    uint32_t ph;
    if constexpr (VEC == 4) ph = *reinterpret_cast<const uint32_t*>(phase + vox);
    else ph = *reinterpret_cast<const uint16_t*>(phase + vox);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      const int t = 3 * ((ph >> (8 * i)) & 0xff);
      c.in.v[i] = tab[t];
      c.a.v[i] = tab[t + 1];
      if constexpr (WANT_B) c.b.v[i] = tab[t + 2];
    }
  }
  return c;
}

template <typename T>
struct PlaneFwdArgs {
  Geo g;
  PlaneGeo p;
  const T* src;       // field (plain), residual r (CG)
  const T* pin;       // CG: p_{k-1}
  T* pout;            // CG: p_k (holds p_{k-2} on entry); IRX: x
  T* x;               // CG: solution
  const float* dsrc;  // IRX: correction
  cpx<T>* smain;
  cpx<T>* snyq;
  const cpx<T>* twx;
  const cpx<T>* twy;
  const LoadState* st;
  const T* ptab;
  const uint8_t* phase;
  const T* vcoef;
  double* partials;
  int pstride, nphase;
  IrxFold fold;
  unsigned long long* prog;
};

// Workgroup id -> (plane or row block, component): the components of a plane go
// to one XCD (ids are dealt round-robin to the 8 XCDs), one after another, so
// that the trace's second reads come from its L2.
__device__ __forceinline__ void plane_block(const int id, const int nblk, const int c, int& z, int& j) {
  const int full = nblk / 8 * 8 * c;
  if (id < full) {
    const int r = id % (8 * c);
    z = id / (8 * c) * 8 + r % 8;
    j = r / 8;
  } else {
    z = id / c;
    j = id % c;
  }
}

template <int NT>
__device__ __forceinline__ double plane_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  double s = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NW; ++i) s += red[i];
  return s;
}

// The real plane sits in LDS rows: transform x, unpack, transform y, and write
// the spectrum rows (and the Nyquist column) of spectrum row 0 at `so` / `no`.
template <typename T, int NT, int K, typename P>
__device__ __forceinline__ void plane_forward(const PlaneLds<T>& s, const P& p, cpx<T>* so, cpx<T>* no) {
  plane_fft<-1, true, T, NT>(s.buf, p, s.twx);
  // X[k] = E + W^k O, X[M-k] = conj(E - W^k O); column 0: (X[0], X[M])
  const int h = p.mx / 2;
  for (int idx = threadIdx.x; idx < (h + 1) * p.ny; idx += NT) {
    const int k = p.div_ny(idx);
    cpx<T>* row = s.buf + (idx - k * p.ny) * p.pitch;
    if (k == 0) {
      const cpx<T> z = row[0];
      row[0] = cpx<T>{z.x + z.y, z.x - z.y};
    } else {
      const int a = s.px[k], b = s.px[p.mx - k];
      const cpx<T> z = row[a], zm = row[b];
      const cpx<T> e = cpx<T>{T(0.5) * (z.x + zm.x), T(0.5) * (z.y - zm.y)};
      const cpx<T> d = cpx<T>{T(0.5) * (z.x - zm.x), T(0.5) * (z.y + zm.y)};
      const cpx<T> o = cmul(s.twx[k], mul_neg_i(d));
      row[a] = cadd(e, o);
      if (k != h) row[b] = cpx<T>{e.x - o.x, o.y - e.y};
    }
  }
  __syncthreads();
  if constexpr (P::kY) plane_fft<-1, false, T, NT>(s.buf, p, s.twy);
  constexpr int CV = 16 / sizeof(cpx<T>);   // complex values per 16 bytes
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int q = k * NT + (int)threadIdx.x;
    if (q < p.nvec) {
      const int e = q * CV;
      const int ky = p.div_mx(e);
      const int kx = e - ky * p.mx;
      const cpx<T>* row = s.buf + (P::kY ? s.py[ky] : ky) * p.pitch;
      cpx<T> o[CV];
#pragma unroll
      for (int i = 0; i < CV; ++i) o[i] = row[s.px[kx + i]];
      if (!P::kY && kx == 0) {
        no[ky] = cpx<T>{o[0].y, T(0)};
        o[0].y = T(0);
      }
      if (P::kY && kx == 0) {
        const cpx<T> c = o[0], m = s.buf[s.py[ky == 0 ? 0 : p.ny - ky] * p.pitch];
        o[0] = cpx<T>{T(0.5) * (c.x + m.x), T(0.5) * (c.y - m.y)};
        no[ky] = cpx<T>{T(0.5) * (c.y + m.y), T(0.5) * (m.x - c.x)};
      }
      if constexpr (CV == 2) *reinterpret_cast<float4*>(so + e) = float4{o[0].x, o[0].y, o[1].x, o[1].y};
      else so[e] = o[0];
    }
  }
}

// XF: XF_PLAIN, XF_CG (fused step: p_k, pending solution updates, local form)
// or XF_IRX.  One component of one plane per workgroup; with EL (elasticity)
// the workgroup of component 2 also forms the trace term of the local form,
// from the other two normal components' residuals and directions.
template <typename T, int NT, int K, bool EL, int XF, typename P>
__global__ __launch_bounds__(NT) void k_pf(const PlaneFwdArgs<T> a) {
  constexpr int VEC = 16 / sizeof(T);
  extern __shared__ __align__(16) char plane_mem[];
  decltype(auto) p = plane_geo<P>(a.p);
  const Geo& g = a.g;
  const int l = blockIdx.y, tid = threadIdx.x;
  const int nblk = (int)gridDim.x / g.c;
  int z, j;
  plane_block((int)blockIdx.x, nblk, g.c, z, j);
  const long long plane = (long long)p.nx * p.ny;
  const long long fo = (long long)l * field_elems(g) + (long long)z * plane;   // component 0 of this plane
  const long long co = fo + (long long)j * g.nvox;
  if (a.st != nullptr) progress_push(a.prog, l, a.st[l]);
  if (a.st != nullptr && !a.st[l].active) {
    // a load that is not refined still gets its zero start written (x was not zeroed)
    if (XF == XF_IRX && a.fold.xzero) {
      for (int q = tid; q < p.nvec; q += NT) pv_store(a.pout + co + (long long)q * VEC, PVec<T>{});
    }
    return;
  }
  const PlaneLds<T> s = plane_lds<T>(plane_mem, p);
  double part = 0.0;
  if constexpr (XF == XF_CG) {
    const bool first = a.st[l].first != 0;
    const bool pair = a.st[l].pending == 2;
    const T beta = static_cast<T>(a.st[l].beta);
    const T alpha = static_cast<T>(a.st[l].alpha);
    const T alpha2 = static_cast<T>(a.st[l].alpha2);
    const bool trace = EL && j == 2;
    plane_tables<T, NT>(s, p, a.twx, a.twy);
    if (a.vcoef == nullptr) plane_phase_tab<T, NT>(s.tab, a.ptab, a.nphase, g.c);
    // at most four vectors of each field at a time: the reads of a group are in
    // flight together, and the registers stay within 128 at 1024 threads
    constexpr int KG = K < 4 ? K : 4;
#pragma unroll 1
    for (int k0 = 0; k0 < K; k0 += KG) {
      PVec<T> pv[KG], po[KG];
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        const int q = (k0 + k) * NT + tid;
        if (k0 + k < K && q < p.nvec) {
          pv[k] = pv_load(a.src + co + (long long)q * VEC);
          if (!first) po[k] = pv_load(a.pin + co + (long long)q * VEC);
        }
      }
      if (k0 == 0) __syncthreads();   // the phase table
      if (!first) {
#pragma unroll
        for (int k = 0; k < KG; ++k)
#pragma unroll
          for (int i = 0; i < VEC; ++i) pv[k].v[i] += beta * po[k].v[i];
        if (pair) {
#pragma unroll
          for (int k = 0; k < KG; ++k) {
            const int q = (k0 + k) * NT + tid;
            if (k0 + k < K && q < p.nvec) {
              const PVec<T> pp = pv_load(a.pout + co + (long long)q * VEC);
              PVec<T> xv = pv_load(a.x + co + (long long)q * VEC);
#pragma unroll
              for (int i = 0; i < VEC; ++i) xv.v[i] = xv.v[i] + alpha2 * pp.v[i] + alpha * po[k].v[i];
              pv_store(a.x + co + (long long)q * VEC, xv);
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        const int q = (k0 + k) * NT + tid;
        if (k0 + k < K && q < p.nvec) {
          pv_store(a.pout + co + (long long)q * VEC, pv[k]);
          plane_put<T>(s.buf, p, q, pv[k]);
          const long long vox = (long long)z * plane + (long long)q * VEC;
          const PCoef<T> c = plane_coef<EL, T>(a.phase, a.vcoef, s.tab, g.nvox, vox);
#pragma unroll
          for (int i = 0; i < VEC; ++i) part += (double)(c.in.v[i] * c.a.v[i] * pv[k].v[i] * pv[k].v[i]);
          if constexpr (EL) {
            if (trace) {
              PVec<T> t = pv[k];
#pragma unroll
              for (int m = 0; m < 2; ++m) {
                const long long e = fo + (long long)m * g.nvox + (long long)q * VEC;
                const PVec<T> rv = pv_load(a.src + e);
                PVec<T> pm{};
                if (!first) pm = pv_load(a.pin + e);
#pragma unroll
                for (int i = 0; i < VEC; ++i) t.v[i] += rv.v[i] + beta * pm.v[i];
              }
#pragma unroll
              for (int i = 0; i < VEC; ++i) part += (double)(c.in.v[i] * c.b.v[i] * t.v[i] * t.v[i]);
            }
          }
        }
      }
    }
  } else if constexpr (XF == XF_IRX) {
    // x += d + the inner solve's pending steps (summed in FP32), or x = that
    plane_tables<T, NT>(s, p, a.twx, a.twy);
    const int np = a.fold.sti != nullptr ? a.fold.sti[l].pending : 0;
    const float al = np > 0 ? static_cast<float>(a.fold.sti[l].alpha) : 0.0f;
    const float al2 = np == 2 ? static_cast<float>(a.fold.sti[l].alpha2) : 0.0f;
    const bool nb1 = np > 0 && a.fold.pb != nullptr && a.fold.sti[l].pbuf != 0;
    const float* pn = np > 0 ? (nb1 ? a.fold.pb : a.fold.pa) : nullptr;
    const float* po = np == 2 ? (nb1 ? a.fold.pa : a.fold.pb) : nullptr;
    struct alignas(4 * VEC) FV { float v[VEC]; };
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int q = k * NT + tid;
      if (q < p.nvec) {
        const long long e = co + (long long)q * VEC;
        FV d = *reinterpret_cast<const FV*>(a.dsrc + e);
        if (np > 0) {
          const FV v1 = *reinterpret_cast<const FV*>(pn + e);
#pragma unroll
          for (int i = 0; i < VEC; ++i) d.v[i] += al * v1.v[i];
          if (np == 2) {
            const FV v2 = *reinterpret_cast<const FV*>(po + e);
#pragma unroll
            for (int i = 0; i < VEC; ++i) d.v[i] += al2 * v2.v[i];
          }
        }
        PVec<T> xv{};
        if (!a.fold.xzero) xv = pv_load(a.pout + e);
#pragma unroll
        for (int i = 0; i < VEC; ++i) xv.v[i] += static_cast<T>(d.v[i]);
        pv_store(a.pout + e, xv);
        plane_put<T>(s.buf, p, q, xv);
      }
    }
  } else {
    PVec<T> v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int q = k * NT + tid;
      if (q < p.nvec) v[k] = pv_load(a.src + co + (long long)q * VEC);
    }
    plane_tables<T, NT>(s, p, a.twx, a.twy);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int q = k * NT + tid;
      if (q < p.nvec) plane_put<T>(s.buf, p, q, v[k]);
    }
  }
  __syncthreads();
  plane_forward<T, NT, K>(s, p,
                          a.smain + (long long)l * main_cpx(g) + ((long long)j * nblk + z) * p.ny * p.mx,
                          a.snyq + (long long)l * nyq_cpx(g) + ((long long)j * nblk + z) * p.ny);
  if constexpr (XF == XF_CG) {
    const double sum = plane_sum<NT>(part, s.red);
    if (tid == 0) a.partials[(long long)l * a.pstride + blockIdx.x] = sum;
  }
}

template <typename T>
struct PlaneInvArgs {
  Geo g;
  PlaneGeo p;
  const cpx<T>* smain;
  const cpx<T>* snyq;
  const cpx<T>* twx;
  const cpx<T>* twy;
  const T* tau;
  T* out;
  const T* rin;
  float* rout;
  const T* ptab;
  const uint8_t* phase;
  const T* vcoef;
  const double* loads;
  const LoadState* st;
  double* partials;
  int pstride, nphase;
  T scale;
};

// MODE: XI_APPLY (also q = Lv with its partial v.q), XI_CGR, XI_IRRES,
// XI_RESNORM or XI_STRAIN.  With EL the workgroups of the normal components
// read all three for the trace of the local term.
// FP32 registers are held to what lets two workgroups of 1024 threads share a
// CU where LDS does (128 x 128 elastic CG: 259 us a pass against 326).
template <typename T, int NT, typename P>
constexpr int plane_waves() {
  if constexpr (!P::kStatic || sizeof(T) == 8 || NT < 1024) {
    return 1;
  } else {
    constexpr int lds = (int)sizeof(cpx<T>) * (P::ny * P::pitch + 2 * P::nx) + 1024;
    return (160 * 1024 / lds >= 2) ? 8 : 4;
  }
}

template <typename T, int NT, int K, bool EL, int MODE, typename P>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(plane_waves<T, NT, P>()))) void k_pi(const PlaneInvArgs<T> a) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int CV = 16 / sizeof(cpx<T>);
  constexpr bool LOCAL = MODE != XI_STRAIN;
  extern __shared__ __align__(16) char plane_mem[];
  decltype(auto) p = plane_geo<P>(a.p);
  const Geo& g = a.g;
  const int l = blockIdx.y, tid = threadIdx.x;
  if (a.st != nullptr && !a.st[l].active) return;
  const int nblk = (int)gridDim.x / g.c;
  int z, j;
  plane_block((int)blockIdx.x, nblk, g.c, z, j);
  const long long plane = (long long)p.nx * p.ny;
  const long long fo = (long long)l * field_elems(g) + (long long)z * plane;
  const long long co = fo + (long long)j * g.nvox;
  const PlaneLds<T> s = plane_lds<T>(plane_mem, p);
  const cpx<T>* so = a.smain + (long long)l * main_cpx(g) + ((long long)j * nblk + z) * p.ny * p.mx;
  const cpx<T>* no = a.snyq + (long long)l * nyq_cpx(g) + ((long long)j * nblk + z) * p.ny;
  PVec<T> sp[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int q = k * NT + tid;
    if (q < p.nvec) sp[k] = pv_load(reinterpret_cast<const T*>(so) + (long long)q * VEC);
  }
  plane_tables<T, NT>(s, p, a.twx, a.twy);
  if (LOCAL && a.vcoef == nullptr) plane_phase_tab<T, NT>(s.tab, a.ptab, a.nphase, g.c);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int q = k * NT + tid;
    if (q < p.nvec) {
      const int e = q * CV;
      const int ky = p.div_mx(e);
      const int kx = e - ky * p.mx;
      cpx<T>* row = s.buf + (P::kY ? s.py[ky] : ky) * p.pitch;
      cpx<T> o[CV];
#pragma unroll
      for (int i = 0; i < CV; ++i) o[i] = cpx<T>{sp[k].v[2 * i], sp[k].v[2 * i + 1]};
      if (kx == 0) {
        // kx = 0 and Nyquist columns as one: Y0 + i YN
        const cpx<T> n = no[ky];
        o[0] = cpx<T>{o[0].x - n.y, o[0].y + n.x};
      }
#pragma unroll
      for (int i = 0; i < CV; ++i) row[s.px[kx + i]] = o[i];
    }
  }
  __syncthreads();
  if constexpr (P::kY) plane_fft<1, false, T, NT>(s.buf, p, s.twy);
  // 2Z[k] = 2E + i 2O, 2Z[M-k] = conj(2E) + i conj(2O)
  const int h = p.mx / 2;
  for (int idx = tid; idx < (h + 1) * p.ny; idx += NT) {
    const int k = p.div_ny(idx);
    cpx<T>* row = s.buf + (idx - k * p.ny) * p.pitch;
    if (k == 0) {
      const cpx<T> z0 = row[0];   // (X[0], X[M])
      row[0] = cpx<T>{z0.x + z0.y, z0.x - z0.y};
    } else {
      const int ia = s.px[k], ib = s.px[p.mx - k];
      const cpx<T> xk = row[ia], xm = row[ib];
      const cpx<T> e = cpx<T>{xk.x + xm.x, xk.y - xm.y};
      const cpx<T> d = cpx<T>{xk.x - xm.x, xk.y + xm.y};
      const cpx<T> o = cmulc(d, s.twx[k]);
      row[ia] = cpx<T>{e.x - o.y, e.y + o.x};
      if (k != h) row[ib] = cpx<T>{e.x + o.y, o.x - e.y};
    }
  }
  __syncthreads();
  plane_fft<1, true, T, NT>(s.buf, p, s.twx);
  const T pl = static_cast<T>(a.loads[l * g.c + j]);
  const T al = MODE == XI_CGR ? static_cast<T>(a.st[l].alpha) : T(0);
  const bool normal = EL && j < 3;
  double part = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int q = k * NT + tid;
    if (q < p.nvec) {
      const long long e = co + (long long)q * VEC;
      PVec<T> tv, rv, res;
      if constexpr (LOCAL) tv = pv_load(a.tau + e);
      if constexpr (MODE == XI_CGR) rv = pv_load(a.rin + e);
      const PVec<T> gv = plane_get<T>(s.buf, p, q);
      if constexpr (LOCAL) {
        const PCoef<T> c =
            plane_coef<EL, T>(a.phase, a.vcoef, s.tab, g.nvox, (long long)z * plane + (long long)q * VEC);
        PVec<T> loc;
#pragma unroll
        for (int i = 0; i < VEC; ++i) loc.v[i] = c.a.v[i] * tv.v[i];
        if constexpr (EL) {
          if (normal) {
            const T* t = a.tau + fo + (long long)q * VEC;
            const PVec<T> t0 = pv_load(t), t1 = pv_load(t + g.nvox), t2 = pv_load(t + 2 * g.nvox);
#pragma unroll
            for (int i = 0; i < VEC; ++i) loc.v[i] += c.b.v[i] * (t0.v[i] + t1.v[i] + t2.v[i]);
          }
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          const T ga = gv.v[i] * a.scale;
          if constexpr (MODE == XI_CGR) {
            res.v[i] = rv.v[i] - al * (c.in.v[i] * (loc.v[i] + ga));
            part += (double)res.v[i] * res.v[i];
          } else if constexpr (MODE == XI_IRRES || MODE == XI_RESNORM) {
            res.v[i] = c.in.v[i] * (pl - loc.v[i] - ga);
            part += (double)res.v[i] * res.v[i];
          } else {
            res.v[i] = c.in.v[i] * (loc.v[i] + ga);
            part += (double)tv.v[i] * res.v[i];
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) res.v[i] = pl - gv.v[i] * a.scale;
      }
      if constexpr (MODE == XI_IRRES) {
        struct alignas(4 * VEC) FV { float v[VEC]; };
        FV f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) f.v[i] = static_cast<float>(res.v[i]);
        *reinterpret_cast<FV*>(a.rout + e) = f;
      } else if constexpr (MODE != XI_RESNORM) {
        pv_store(a.out + e, res);
      }
    }
  }
  if (a.partials != nullptr) {
    const double sum = plane_sum<NT>(part, s.red);
    if (tid == 0) a.partials[(long long)l * a.pstride + blockIdx.x] = sum;
  }
}

}  // namespace lsh
