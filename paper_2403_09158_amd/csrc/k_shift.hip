// k_shift.hip - energies of a stored defect type translated by the shift
// theorem (Sec. 3.3, eq. shift).
//
// A defect type's eigenstrain spectrum eps*_hat_0 (and stress spectrum
// sigma_hat_0) is stored once for its reference centre X0.  The type translated
// by d = X - X0 has the spectrum phi_d(xi) eps*_hat_0(xi), and its energy with a
// stress field sigma follows from Parseval's identity on the half spectrum:
//   sum_x eps*_d(x) : sigma(x) = (1/N) sum_k w(k_x) Re[phi_d(k) eps*_hat_0(k) : conj(sigma_hat(k))],
// w = 1 on the planes k_x = 0 and (even n) k_x = n/2, which hold their own
// Hermitian partners, and 2 elsewhere; the contraction weighs the shear
// components twice.  phi_d is exp(-i xi . d) with the centred labels of
// Sec. 3.4; at a bin with even-n Nyquist components it is the mean of the
// factors of the -n/2 and +n/2 representatives, which is the transform of the
// real part of the translated field.  With an excluded mover at offset d'
// (its own stress, translated, taken out of sigma) the contraction is with
// conj(sigma_hat - phi_d' sigma_hat_0).
//
// One pass over the three spectra serves up to TYPE_NP positions; each block
// leaves one FP64 partial sum per position and the partials are added in a
// fixed order, so results do not depend on scheduling.
#include "ec_internal.h"

namespace ec {

namespace {

constexpr int TT = 256;

__device__ __forceinline__ double2 cmul2(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Phase tables: the factor exp(-2 pi i l u) of axis a at bin k for entry p (u the
// offset along the axis over the cell side, l the centred label, -n/2 at an even
// n's Nyquist bin) stands at tab[phase_at(p, a, k, n)]: rows of k for x and y,
// the entries of a kz side by side for z (read together by scalar loads);
// nyq[p * 3 + a] is the factor of the +n/2 representative.  Entries are the np
// positions and, at TYPE_NP, the excluded mover (offset np).
__host__ __device__ inline size_t phase_at(int p, int a, int k, int n) {
  return a < 2 ? ((size_t)p * 2 + a) * n + k : (size_t)(TYPE_NP + 1) * (2 * n + k) + p;
}

__global__ __launch_bounds__(TT) void k_type_tables(TypeOffsets off, int rows, int np, int n,
                                                    double2* __restrict__ tab, double2* __restrict__ nyq) {
  const int t = blockIdx.x * TT + threadIdx.x;
  if (t >= rows * (n + 1)) return;
  const int r = t / (n + 1), q = t % (n + 1);
  const int l = q == n ? n / 2 : (q <= (n - 1) / 2 ? q : q - n);
  double v = (double)l * off.u[r];
  v -= floor(v);
  double sn, cs;
  sincospi(2.0 * v, &sn, &cs);
  const int p = r / 3 == np ? TYPE_NP : r / 3, a = r % 3;
  if (q == n)
    nyq[3 * p + a] = make_double2(cs, -sn);
  else
    tab[phase_at(p, a, q, n)] = make_double2(cs, -sn);
}

// One thread per column (kx, ky) and chunk of kz.  A column's phase is the
// product of its x and y factors, formed once per thread (at a Nyquist kx or ky
// the mean of the two representatives' products, which the z factor multiplies
// alike), and the z factor, the same for all lanes: a bin costs each position
// one complex product and two multiply-adds, where three table reads and two
// products per bin and position had bound the pass (128^3 FP32, 16 positions:
// 95 us against 26 for the spectra's 152 MB; now 57).  At the Nyquist plane of
// an even n the two representatives have z factors of their own.
template <typename S, bool EXCL>
__global__ __launch_bounds__(TT) void k_type_energy(const typename Cplx<S>::T* __restrict__ sig,
                                                    const typename Cplx<S>::T* __restrict__ te,
                                                    const typename Cplx<S>::T* __restrict__ ts, int n, int P,
                                                    int chunk, const double2* __restrict__ tab,
                                                    const double2* __restrict__ nyq, int np,
                                                    double* __restrict__ partial) {
  constexpr int NX = TYPE_NP + (EXCL ? 1 : 0);  // phases: the positions' and the excluded mover's
  __shared__ double red[TYPE_NP][TT / 64];
  const int NH = n / 2 + 1;
  const bool even = (n & 1) == 0;
  const int ncol = (n * NH + TT - 1) / TT;  // workgroups over the columns
  const int col = (int)(blockIdx.x % ncol) * TT + threadIdx.x;
  const int z0 = (int)(blockIdx.x / ncol) * chunk, z1 = min(n, z0 + chunk);
  const bool live = col < n * NH;
  const int kx = live ? col % NH : 0, ky = live ? col / NH : 0;
  const bool nx = even && kx == n / 2, ny = even && ky == n / 2;
  auto xy = [&](int e, bool second) {
    const double2 a = second && nx ? nyq[3 * e] : tab[phase_at(e, 0, kx, n)];
    const double2 b = second && ny ? nyq[3 * e + 1] : tab[phase_at(e, 1, ky, n)];
    return cmul2(a, b);
  };
  double2 f[NX];
#pragma unroll
  for (int j = 0; j < NX; ++j) {
    f[j] = make_double2(0.0, 0.0);
    if (j < np || j == TYPE_NP) {
      f[j] = xy(j, false);
      if (nx || ny) {
        const double2 g = xy(j, true);
        f[j] = make_double2(0.5 * (f[j].x + g.x), 0.5 * (f[j].y + g.y));
      }
    }
  }
  const double wx = (kx == 0 || nx) ? 1.0 : 2.0;
  double acc[TYPE_NP];
#pragma unroll
  for (int p = 0; p < TYPE_NP; ++p) acc[p] = 0.0;
  struct Bin {
    typename Cplx<S>::T e[6], s[6], q[EXCL ? 6 : 1];
  };
  auto load = [&](int kz, Bin& v) {
    const size_t o = spec_at(kz, ky, kx, 0, n, P);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      v.e[c] = te[o + c];
      v.s[c] = sig[o + c];
      if constexpr (EXCL) v.q[c] = ts[o + c];
    }
  };
  auto add = [&](const Bin& v, auto&& phase) {
    // A = eps*_hat_0 : conj(sigma_hat), B = eps*_hat_0 : conj(sigma_hat_0)
    double2 A = make_double2(0.0, 0.0), B = make_double2(0.0, 0.0);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const double w = c < 3 ? 1.0 : 2.0;
      const double2 e = ld2(&v.e[c]), s = ld2(&v.s[c]);
      A.x += w * (e.x * s.x + e.y * s.y);
      A.y += w * (e.y * s.x - e.x * s.y);
      if constexpr (EXCL) {
        const double2 q = ld2(&v.q[c]);
        B.x += w * (e.x * q.x + e.y * q.y);
        B.y += w * (e.y * q.x - e.x * q.y);
      }
    }
    if constexpr (EXCL) {  // D = A - B conj(phi_d')
      const double2 g = phase(TYPE_NP);
      A.x -= B.x * g.x + B.y * g.y;
      A.y -= B.y * g.x - B.x * g.y;
    }
    A.x *= wx;
    A.y *= wx;
#pragma unroll
    for (int p = 0; p < TYPE_NP; ++p) {
      if (p < np) {
        const double2 g = phase(p);
        acc[p] += g.x * A.x - g.y * A.y;
      }
    }
  };
  // the next plane's values are loaded while this one's are added; an even n's
  // Nyquist plane comes last, by itself
  const int zn = even ? n / 2 : -1;
  auto after = [&](int kz) { return kz + 1 == zn ? kz + 2 : kz + 1; };
  Bin v, w;
  int kz = z0 == zn ? z0 + 1 : z0;
  if (kz < z1) load(kz, v);
  while (kz < z1) {
    const int kn = after(kz);
    load(kn < z1 ? kn : kz, w);
    add(v, [&](int j) { return cmul2(f[j], tab[phase_at(j, 2, kz, n)]); });
    v = w;
    kz = kn;
  }
  if (z0 <= zn && zn < z1) {
    load(zn, v);
    add(v, [&](int j) {
      const double2 m0 = cmul2(xy(j, false), tab[phase_at(j, 2, zn, n)]), m1 = cmul2(xy(j, true), nyq[3 * j + 2]);
      return make_double2(0.5 * (m0.x + m1.x), 0.5 * (m0.y + m1.y));
    });
  }
  // block sums by a fixed tree
#pragma unroll
  for (int p = 0; p < TYPE_NP; ++p) {
    double v = live ? acc[p] : 0.0;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    if ((threadIdx.x & 63) == 0) red[p][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < np) {
    double v = red[threadIdx.x][0];
    for (int w = 1; w < TT / 64; ++w) v += red[threadIdx.x][w];
    partial[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = v;
  }
}

// E_p = scale * sum of the grid partials of position p: one workgroup per
// position, strided Neumaier sums per thread, then a fixed tree.
__global__ __launch_bounds__(256) void k_type_finish(const double* __restrict__ partial, int grid, double scale,
                                                     double* __restrict__ E) {
  __shared__ double rs[256], rc[256];
  const int p = blockIdx.x;
  double s = 0.0, c = 0.0;
  for (int b = threadIdx.x; b < grid; b += 256) {
    const double v = partial[(size_t)p * grid + b], t = s + v;
    c += fabs(s) >= fabs(v) ? (s - t) + v : (v - t) + s;
    s = t;
  }
  rs[threadIdx.x] = s;
  rc[threadIdx.x] = c;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      const double a = rs[threadIdx.x], v = rs[threadIdx.x + w], t = a + v;
      rc[threadIdx.x] += rc[threadIdx.x + w] + (fabs(a) >= fabs(v) ? (a - t) + v : (v - t) + a);
      rs[threadIdx.x] = t;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) E[p] = scale * (rs[0] + rc[0]);
}

}  // namespace

// kz planes per workgroup: eight amortise the column phases (more where a
// thousand workgroups have more), but a plane is a round trip to memory, so
// cells with fewer than 128 such workgroups split into pieces of two planes up.
// us per call, eight planes / this: 32^3 FP64, 1 position 92 / 84, 16 positions
// 114 / 97; 48^3 98 / 89 and 116 / 100; 64^3 106 / 101 and 129 / 118.  Eight stay
// from 96^3 on (FP64, 16 positions: 155, with four planes 159).
static int type_chunk(int n) {
  const int ncol = (n * (n / 2 + 1) + TT - 1) / TT;
  const int few = std::min(8, std::max(2, (n * ncol + 127) / 128));
  return std::max(few, (n * ncol + 1023) / 1024);
}

int type_energy_grid(int n) {
  const int ncol = (n * (n / 2 + 1) + TT - 1) / TT, chunk = type_chunk(n);
  return ncol * ((n + chunk - 1) / chunk);
}

hipError_t launch_type_energies(bool fp64, const void* sig, const void* te, const void* ts, SpecGeom g,
                                const TypeOffsets& off, double2* tab, double2* nyq, int np, bool excl, double* partial,
                                double scale, double* E, hipStream_t s) {
  if (np < 1 || np > TYPE_NP) return hipErrorInvalidValue;
  const int n = g.n, rows = 3 * (np + (excl ? 1 : 0));
  hipLaunchKernelGGL(k_type_tables, dim3((rows * (n + 1) + TT - 1) / TT), dim3(TT), 0, s, off, rows, np, n, tab,
                     nyq);
  const int grid = type_energy_grid(n), chunk = type_chunk(n);
  auto go = [&](auto* k, auto* sp) {
    using C2 = std::remove_pointer_t<decltype(sp)>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(TT), 0, s, (const C2*)sig, (const C2*)te, (const C2*)ts, n, g.P, chunk, tab,
                       nyq, np, partial);
  };
  if (fp64)
    go(excl ? k_type_energy<double, true> : k_type_energy<double, false>, (double2*)nullptr);
  else
    go(excl ? k_type_energy<float, true> : k_type_energy<float, false>, (float2*)nullptr);
  hipLaunchKernelGGL(k_type_finish, dim3(np), dim3(256), 0, s, partial, grid, scale, E);
  return hipGetLastError();
}

}  // namespace ec
