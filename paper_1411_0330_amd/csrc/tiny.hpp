// Persistent conjugate gradients for small grids: one workgroup per load runs
// every iteration of its load in a single launch, on chip.  The residual and
// the direction stay in registers (voxel pairs of a thread, every component),
// the spectrum and the local coefficients in LDS, the operator matrices of a
// thread's wave-vectors in registers; the solution (registers in 2D, else the
// cache-resident workspace) is all that an iteration touches in memory.
//
// An iteration is the fused CG step: p = r + beta p with its local form, x, y
// (and z) transforms in place in LDS (plane.hpp: decimation in frequency, then
// in time, one butterfly per thread and step, lanes along rows or columns),
// the Green operator with p.Gamma p (Parseval), the way back, r -= alpha Lp
// with ||r||^2.  It is bounded by LDS traffic and the latency of its
// barrier-separated sweeps over the spectrum, by the stages of the axes 9 (8^2)
// to 13 (32^2 and 64^2) in 2D, 11 (8^3) and 15 (16^3); the loop that it replaced
// passed through memory between them.  One iteration of two loads, before and
// now: FP64 64^2 34 and 15.5 us, 32^2 22 and 8.3, 8^2 18 and 5.5, scalar 8^3 24
// and 7.6, scalar 16^3 81 and 34 (40 with one kernel per pass), elastic 8^3 51
// and 8.5; FP32 within the mixed solve 30 and 15 (64^2), 62 and 25 (16^3).
//
// Column 0 of the spectrum carries the kx = 0 values and, as its imaginary part
// before the y transform, the kx = nx/2 ones; the Green step takes its
// wave-vectors k and -k together and separates the two by symmetry.  Scalars
// live in registers of every thread, from LDS reductions in a fixed order.  The
// loop ends at convergence, breakdown, non-finite values or maxit, the same in
// every thread of the workgroup, so no workgroup waits on another.
#pragma once

#include <limits>

#include "plane.hpp"

namespace lsh {

template <typename T>
struct TinyArgs {
  Geo g;
  GreenParams gp;
  GreenTabs<T> tb;
  T* x;
  const T* r;     // initial residual
  const cpx<T>* tw[3];
  int iso;
  const T* ptab;
  const uint8_t* phase;
  const T* vcoef;
  LoadState* st;
  int maxit;
  double guard;   // CG breakdown when |p.Lp| <= guard r.r (see k_scal)
  HistRef hist;   // residual history (see hist_push)
};

// Workgroup sum of one double, returned to every thread (fixed order).  Lanes
// add by DPP moves: a serial chain of cross-lane LDS permutes was 1 us a sum.
template <int NT>
__device__ __forceinline__ double block_allsum(double v, double* red) {
  v = wave_total(v);
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 63) red[w] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) s += red[i];
  return s;
}

// Spectrum of a small grid in LDS: row (j, z, y) of pitch mx | 1.
template <int NX, int NY, int NZ, int C>
struct TinyGrid {
  static constexpr int MX = NX / 2, PITCH = MX | 1, ROWS = NY * NZ, NV = NX * ROWS;
  static constexpr PlaneAxis AX = make_axis(MX, 8), AY = make_axis(NY, 8), AZ = make_axis(NZ, 8);
  static constexpr PlaneAxis axis(int a) { return a == 0 ? AX : a == 1 ? AY : AZ; }
};

// One stage of the transforms along axis A of every component: up to U
// butterflies of a thread at once, all their loads before the first store.
template <int R, int DIR, int A, typename T, int NT, typename G, int C>
__device__ __forceinline__ void tiny_stage(cpx<T>* buf, const int L, const int sl, const cpx<T>* tw) {
  constexpr int n = G::axis(A).n;
  constexpr int NYv = G::AY.n, NZv = G::AZ.n;
  constexpr int es = A == 0 ? 1 : A == 1 ? G::PITCH : NYv * G::PITCH;
  constexpr int nline = A == 0 ? C * G::ROWS : A == 1 ? C * NZv * G::MX : C * NYv * G::MX;
  constexpr int nb = nline * (n / R);
  constexpr int NB = (nb + NT - 1) / NT;
  constexpr int LIM = sizeof(T) == 4 ? 16 : 8;
  constexpr int U = NB * R <= LIM ? NB : R < LIM ? LIM / R : 1;
  const int S = 1 << sl;
  const int ts = (n / L) * (A == 0 ? 2 : 1);
#pragma unroll 1
  for (int g = 0; g < NB; g += U) {
    cpx<T> u[U][R];
    cpx<T>* p[U];
    int tj[U];
    bool on[U];
    static_for<0, U>([&](auto q_) {
      constexpr int q = decltype(q_)::value;
      const int idx = (g + q) * NT + (int)threadIdx.x;
      on[q] = nb % (NT * U) == 0 || idx < nb;
      const int b = idx / nline, line = idx - b * nline;
      int base;
      if constexpr (A == 0) {
        base = line * G::PITCH;
      } else if constexpr (A == 1) {
        const int s = line / G::MX;
        base = s * NYv * G::PITCH + (line - s * G::MX);
      } else {
        const int r = line / G::MX, j = r / NYv;
        base = (j * NZv * NYv + (r - j * NYv)) * G::PITCH + (line - r * G::MX);
      }
      const int j = b & (S - 1), blk = b >> sl;
      tj[q] = j * ts;
      p[q] = buf + base + (blk * L + j) * es;
      if (on[q]) static_for<0, R>([&](auto r_) { u[q][decltype(r_)::value] = p[q][decltype(r_)::value * S * es]; });
    });
    static_for<0, U>([&](auto q_) {
      constexpr int q = decltype(q_)::value;
      if (on[q]) {
        if (DIR > 0 && S > 1) {
          static_for<1, R>([&](auto r_) {
            constexpr int r = decltype(r_)::value;
            u[q][r] = cmulc(u[q][r], tw[r * tj[q]]);
          });
        }
        dft<R, DIR>(u[q]);
        if (DIR < 0 && S > 1) {
          static_for<1, R>([&](auto r_) {
            constexpr int r = decltype(r_)::value;
            u[q][r] = cmul(u[q][r], tw[r * tj[q]]);
          });
        }
        static_for<0, R>([&](auto r_) { p[q][decltype(r_)::value * S * es] = u[q][decltype(r_)::value]; });
      }
    });
  }
}

template <int DIR, int A, typename T, int NT, typename G, int C>
__device__ __forceinline__ void tiny_fft(cpx<T>* buf, const cpx<T>* tw) {
  constexpr PlaneAxis ax = G::axis(A);
  static_for<0, ax.ns>([&](auto i_) {
    constexpr int i = decltype(i_)::value;
    constexpr PlaneAxis a = G::axis(A);
    constexpr int s = DIR < 0 ? i : a.ns - 1 - i;
    tiny_stage<a.r[s], DIR, A, T, NT, G, C>(buf, a.l[s], a.sl[s], tw);
    __syncthreads();
  });
}

// LDS position of a frequency along axis A
template <int A, typename G>
__device__ __forceinline__ int tiny_pos(int k) {
  constexpr PlaneAxis a = G::axis(A);
  int pos = 0;
  static_for<0, a.ns>([&](auto s_) {
    constexpr int s = decltype(s_)::value;
    constexpr PlaneAxis b = G::axis(A);
    pos += (k % b.r[s]) << b.sl[s];
    k /= b.r[s];
  });
  return pos;
}

// The real-split step of every row: f(row[k], row[M-k], W^k) for k = 1..H (at
// k = H = M/2 the two are one element, written as row[k] last), sum and
// difference in column 0.
template <typename T, int NT, int H, int NROW, typename F>
__device__ __forceinline__ void tiny_rows(cpx<T>* buf, const int pitch, const uint16_t* px, const int M,
                                          const cpx<T>* tw, F f) {
  constexpr int N = H * NROW, NB = (N + NT - 1) / NT;
  constexpr int LIM = sizeof(T) == 4 ? 4 : 2, U = NB < LIM ? NB : LIM;
  if ((int)threadIdx.x < NROW) {
    for (int i = threadIdx.x; i < NROW; i += NT) {
      const cpx<T> z = buf[i * pitch];
      buf[i * pitch] = cpx<T>{z.x + z.y, z.x - z.y};
    }
  }
#pragma unroll 1
  for (int g = 0; g < NB; g += U) {
    cpx<T> z[U], zm[U], w[U];
    int ia[U], ib[U];
    static_for<0, U>([&](auto q_) {
      constexpr int q = decltype(q_)::value;
      const int idx = (g + q) * NT + (int)threadIdx.x;
      if (N % (NT * U) == 0 || idx < N) {
        const int k = 1 + idx / NROW, row = (idx % NROW) * pitch;
        ia[q] = row + px[k];
        ib[q] = row + px[M - k];
        z[q] = buf[ia[q]];
        zm[q] = buf[ib[q]];
        w[q] = tw[k];
      }
    });
    static_for<0, U>([&](auto q_) {
      constexpr int q = decltype(q_)::value;
      const int idx = (g + q) * NT + (int)threadIdx.x;
      if (N % (NT * U) == 0 || idx < N) {
        f(z[q], zm[q], w[q]);
        buf[ib[q]] = zm[q];
        buf[ia[q]] = z[q];
      }
    });
  }
}

// GEN: with phases that need full matrices, or the finite-difference operator
template <typename T, int NX, int NY, int NZ, int C, int NT, bool GEN>
__global__ __launch_bounds__(NT) void k_tiny_cg(const TinyArgs<T> a) {
  using G = TinyGrid<NX, NY, NZ, C>;
  constexpr int MX = G::MX, PITCH = G::PITCH, ROWS = G::ROWS, H = MX / 2;
  constexpr int VP = (MX * ROWS + NT - 1) / NT;              // voxel pairs per thread
  constexpr int MT = ((MX - 1) * ROWS + NT - 1) / NT;        // wave-vectors with 0 < kx < nx/2 per thread
  constexpr int CT = (ROWS + NT - 1) / NT;                   // (ky, kz) of the kx = 0 and nx/2 planes per thread
  constexpr int NE = C * (C + 1) / 2;
  constexpr int TABW = 2 * C * C + 5;
  constexpr int CST = ROWS * PITCH;                          // LDS stride of a component
  constexpr bool XREG = C == 2;
  __shared__ cpx<T> buf[C * CST];
  __shared__ cpx<T> tw0[NX];
  __shared__ cpx<T> tw1[NY];
  __shared__ cpx<T> tw2[NZ];
  __shared__ T la[G::NV];                 // short form of (A - A0)^{-1}: a, zero outside I0 ...
  __shared__ T lb[C == 6 ? G::NV : 1];    // ... and b
  __shared__ uint16_t px[MX];
  __shared__ double red[NT / 64];

  const Geo& g = a.g;
  const int l = blockIdx.x;
  const int tid = threadIdx.x;
  LoadState* st = a.st + l;
  if (!st->active) return;
  for (int i = tid; i < NX; i += NT) tw0[i] = a.tw[0][i];
  for (int i = tid; i < NY; i += NT) tw1[i] = a.tw[1][i];
  for (int i = tid; i < NZ; i += NT) tw2[i] = a.tw[2][i];
  for (int i = tid; i < MX; i += NT) px[i] = (uint16_t)tiny_pos<0, G>(i);
  const bool vm = a.vcoef != nullptr;
  const bool full = GEN && !vm && a.iso == 0;    // phases without the short form: matrices from the table
  for (int i = tid; i < G::NV; i += NT) {
    if (vm) {
      la[i] = a.vcoef[i];
      if constexpr (C == 6) lb[i] = a.vcoef[G::NV + i];
    } else {
      const T* t = a.ptab + (int)a.phase[i] * TABW + 2 * C * C;
      la[i] = full || t[0] == T(0) ? t[0] : t[1] != T(0) ? t[1] : std::numeric_limits<T>::denorm_min();
      if constexpr (C == 6) lb[i] = t[2];
    }
  }
  const long long F = field_elems(g);
  T* x = a.x + (long long)l * F;
  const T* r0 = a.r + (long long)l * F;

  // the operator at this thread's wave-vectors (the finite-difference one,
  // complex, is formed at every application)
  const bool fd = GEN && a.gp.variant == kGreenFD;
  T Gm[MT][NE], G0[CT][NE], GN[CT][NE];
  if (!fd) {
    static_for<0, MT>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int q = k * NT + tid;
      if (q < (MX - 1) * ROWS) {
        const int m = q / (MX - 1), kx = 1 + q % (MX - 1), kz = m / NY, ky = m % NY;
        const int kk[3] = {kx, ky, kz};
        green_matrix<T, C>(a.gp, a.tb, kk, (long long)m * MX + kx, Gm[k]);
      }
    });
    static_for<0, CT>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int m = k * NT + tid;
      if (m < ROWS) {
        const int kz = m / NY, ky = m % NY;
        const int k0[3] = {0, ky, kz}, kn[3] = {MX, ky, kz};
        green_matrix<T, C>(a.gp, a.tb, k0, (long long)m * MX, G0[k]);
        green_matrix<T, C>(a.gp, a.tb, kn, (long long)ROWS * MX + m, GN[k]);
      }
    });
  }

  cpx<T> r[VP][C], p[VP][C], xr[XREG ? VP : 1][C];
  static_for<0, VP>([&](auto k_) {
    constexpr int k = decltype(k_)::value;
    const int q = k * NT + tid;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      r[k][j].x = r[k][j].y = p[k][j].x = p[k][j].y = T(0);
      if (q < MX * ROWS) {
        const T* rp = r0 + (long long)j * G::NV + 2 * q;
        r[k][j].x = rp[0];
        r[k][j].y = rp[1];
        if constexpr (XREG) {
          const T* xp = x + (long long)j * G::NV + 2 * q;
          xr[k][j].x = xp[0];
          xr[k][j].y = xp[1];
        }
      }
    }
  });
  const double tol2 = st->tol2;
  double rr = st->rr;
  double alpha = 0.0, beta = 0.0;
  bool first = true;
  int iters = st->iters, status = kStatusOk;
  bool done = false;
  __syncthreads();

  // row j of (A - A0)^{-1} at one voxel, times the field (v) there
  auto local_row = [&](const int vox, const int j, const T (&v)[C]) -> T {
    if (full) {
      const T* M = a.ptab + (int)a.phase[vox] * TABW + j * C;
      T s = 0;
#pragma unroll
      for (int m = 0; m < C; ++m) s += M[m] * v[m];
      return la[vox] * s;
    }
    T s = la[vox] * v[j];
    if constexpr (C == 6) {
      if (j < 3) s += lb[vox] * (v[0] + v[1] + v[2]);
    }
    return s;
  };

  for (int it = 0; it < a.maxit; ++it) {
    double part = 0.0;
    // p = r + beta p, its local form, and the rows into LDS
    static_for<0, VP>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int q = k * NT + tid;
      if (q < MX * ROWS) {
        T p0[C], p1[C];
        const int row = q / MX, n = q % MX;
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const T be = static_cast<T>(beta);
          p0[j] = p[k][j].x = first ? r[k][j].x : r[k][j].x + be * p[k][j].x;
          p1[j] = p[k][j].y = first ? r[k][j].y : r[k][j].y + be * p[k][j].y;
          buf[j * CST + row * PITCH + n] = cpx<T>{p0[j], p1[j]};
        }
        T q0 = 0, q1 = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) {
          q0 += p0[j] * local_row(2 * q, j, p0);
          q1 += p1[j] * local_row(2 * q + 1, j, p1);
        }
        part += (double)q0 + (double)q1;
      }
    });
    __syncthreads();
    tiny_fft<-1, 0, T, NT, G, C>(buf, tw0);
    // X[k] = E + W^k O, X[M-k] = conj(E - W^k O); column 0: (X[0], X[M])
    tiny_rows<T, NT, H, C * ROWS>(buf, PITCH, px, MX, tw0, [](cpx<T>& z, cpx<T>& zm, const cpx<T> w) {
      const cpx<T> e = cpx<T>{T(0.5) * (z.x + zm.x), T(0.5) * (z.y - zm.y)};
      const cpx<T> d = cpx<T>{T(0.5) * (z.x - zm.x), T(0.5) * (z.y + zm.y)};
      const cpx<T> o = cmul(w, mul_neg_i(d));
      z = cadd(e, o);
      zm = cpx<T>{e.x - o.x, o.y - e.y};
    });
    __syncthreads();
    tiny_fft<-1, 1, T, NT, G, C>(buf, tw1);
    if constexpr (NZ > 1) tiny_fft<-1, 2, T, NT, G, C>(buf, tw2);
    // Gamma and tau_hat . Gamma tau_hat (weights 2 and, on the kx = 0 and nx/2 planes, 1)
    double quad = 0.0;
    static_for<0, MT>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int q = k * NT + tid;
      if (q < (MX - 1) * ROWS) {
        const int m = q / (MX - 1), kx = 1 + q % (MX - 1), kz = m / NY, ky = m % NY;
        cpx<T>* e = buf + (tiny_pos<2, G>(kz) * NY + tiny_pos<1, G>(ky)) * PITCH + px[kx];
        cpx<T> v[C], w[C];
#pragma unroll
        for (int j = 0; j < C; ++j) w[j] = v[j] = e[j * CST];
        if (fd) {
          const int kk[3] = {kx, ky, kz};
          green_apply<T, C>(a.gp, a.tb, kk, 0, w);
        } else {
          sym_apply<T, C>(Gm[k], w);
        }
        double d = 0.0;
#pragma unroll
        for (int j = 0; j < C; ++j) {
          d += (double)v[j].x * w[j].x + (double)v[j].y * w[j].y;
          e[j * CST] = w[j];
        }
        quad += 2.0 * d;
      }
    });
    static_for<0, CT>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int m = k * NT + tid;
      if (m < ROWS) {
        const int kz = m / NY, ky = m % NY;
        const int nz_ = kz == 0 ? 0 : NZ - kz, ny_ = ky == 0 ? 0 : NY - ky;
        const int mm = nz_ * NY + ny_;   // -k
        if (m <= mm) {
          cpx<T>* e = buf + (tiny_pos<2, G>(kz) * NY + tiny_pos<1, G>(ky)) * PITCH;
          cpx<T>* f = buf + (tiny_pos<2, G>(nz_) * NY + tiny_pos<1, G>(ny_)) * PITCH;
          cpx<T> v0[C], vn[C], w0[C], wn[C];
#pragma unroll
          for (int j = 0; j < C; ++j) {
            const cpx<T> c = e[j * CST], d = f[j * CST];
            w0[j] = v0[j] = cpx<T>{T(0.5) * (c.x + d.x), T(0.5) * (c.y - d.y)};
            wn[j] = vn[j] = cpx<T>{T(0.5) * (c.y + d.y), T(0.5) * (d.x - c.x)};
          }
          if (fd) {
            const int k0[3] = {0, ky, kz}, kn[3] = {MX, ky, kz};
            green_apply<T, C>(a.gp, a.tb, k0, 0, w0);
            green_apply<T, C>(a.gp, a.tb, kn, 0, wn);
          } else {
            sym_apply<T, C>(G0[k], w0);
            sym_apply<T, C>(GN[k], wn);
          }
          double d = 0.0;
#pragma unroll
          for (int j = 0; j < C; ++j) {
            d += (double)v0[j].x * w0[j].x + (double)v0[j].y * w0[j].y + (double)vn[j].x * wn[j].x +
                 (double)vn[j].y * wn[j].y;
            // Y0 + i YN at k, conj(Y0) + i conj(YN) at -k
            e[j * CST] = cpx<T>{w0[j].x - wn[j].y, w0[j].y + wn[j].x};
            if (mm != m) f[j * CST] = cpx<T>{w0[j].x + wn[j].y, wn[j].x - w0[j].y};
          }
          quad += mm != m ? 2.0 * d : d;
        }
      }
    });
    part += quad / (double)G::NV;
    const double pq = block_allsum<NT>(part, red);
    if (!isfinite(pq)) {
      status = kStatusNumeric;
      break;
    }
    if (fabs(pq) <= a.guard * rr) {
      status = kStatusBreakdown;
      break;
    }
    alpha = rr / pq;
    first = false;
    // the way back (block_allsum's barriers stand between the Green step and this)
    if constexpr (NZ > 1) tiny_fft<1, 2, T, NT, G, C>(buf, tw2);
    tiny_fft<1, 1, T, NT, G, C>(buf, tw1);
    tiny_rows<T, NT, H, C * ROWS>(buf, PITCH, px, MX, tw0, [](cpx<T>& x0, cpx<T>& xm, const cpx<T> w) {
      const cpx<T> e = cpx<T>{x0.x + xm.x, x0.y - xm.y};
      const cpx<T> d = cpx<T>{x0.x - xm.x, x0.y + xm.y};
      const cpx<T> o = cmulc(d, w);
      x0 = cpx<T>{e.x - o.y, e.y + o.x};
      xm = cpx<T>{e.x + o.y, o.x - e.y};
    });
    __syncthreads();
    tiny_fft<1, 0, T, NT, G, C>(buf, tw0);
    // r -= alpha L p on I0, ||r||^2
    part = 0.0;
    const T al = static_cast<T>(alpha);
    const T sc = static_cast<T>(1.0 / (double)G::NV);
    static_for<0, VP>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int q = k * NT + tid;
      if (q < MX * ROWS) {
        const int row = q / MX, n = q % MX;
        const T in0 = la[2 * q] != T(0) ? T(1) : T(0), in1 = la[2 * q + 1] != T(0) ? T(1) : T(0);
        T p0[C], p1[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
          p0[j] = p[k][j].x;
          p1[j] = p[k][j].y;
        }
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const cpx<T> gv = buf[j * CST + row * PITCH + n];
          const T q0 = in0 * (local_row(2 * q, j, p0) + gv.x * sc);
          const T q1 = in1 * (local_row(2 * q + 1, j, p1) + gv.y * sc);
          r[k][j].x -= al * q0;
          r[k][j].y -= al * q1;
          part += (double)r[k][j].x * r[k][j].x + (double)r[k][j].y * r[k][j].y;
        }
      }
    });
    const double rr_new = block_allsum<NT>(part, red);
    ++iters;
    if (!isfinite(rr_new)) {
      status = kStatusNumeric;
      break;
    }
    // x += alpha p
    static_for<0, VP>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int q = k * NT + tid;
      if (q < MX * ROWS) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          if constexpr (XREG) {
            xr[k][j].x += al * p[k][j].x;
            xr[k][j].y += al * p[k][j].y;
          } else {
            cpx<T>* xp = reinterpret_cast<cpx<T>*>(x + (long long)j * G::NV + 2 * q);
            const cpx<T> xo = *xp;
            *xp = cpx<T>{xo.x + al * p[k][j].x, xo.y + al * p[k][j].y};
          }
        }
      }
    });
    beta = rr_new / rr;
    rr = rr_new;
    if (tid == 0) hist_push(a.hist, l, rr / st->bb, hist_count(a.hist, l));
    if (rr <= tol2) {
      done = true;
      break;
    }
  }
  if constexpr (XREG) {
    static_for<0, VP>([&](auto k_) {
      constexpr int k = decltype(k_)::value;
      const int q = k * NT + tid;
      if (q < MX * ROWS) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          T* xp = x + (long long)j * G::NV + 2 * q;
          xp[0] = xr[k][j].x;
          xp[1] = xr[k][j].y;
        }
      }
    });
  }
  if (tid == 0) {
    st->rr = rr;
    st->res2 = rr;
    st->alpha = alpha;
    st->beta = beta;
    st->iters = iters;
    st->status = status;
    st->pending = 0;
    st->first = first ? 1 : 0;
    st->active = (done || status != kStatusOk) ? 0 : 1;
  }
}

}  // namespace lsh
