// k_fft.hip - FFT passes and the Green operator of the periodic eigenstrain solve.
//
// Half-spectrum layout: [kz][ky][kx][6] complex (the six components of a bin
// adjacent), kx in [0, n/2] with row pitch P (spec_pitch).  The solve runs:
//   x-forward (R2C, two real rows per complex transform), y-forward,
//   z-forward + Green operator + z-inverse, y-inverse, x-inverse (C2R) + stress.
// All butterflies, twiddles and the Green operator run in FP64 registers; the
// storage type S (float or double) only sets what is kept in HBM between passes.
#include <algorithm>

#include "ec_internal.h"
#include "fft_core.h"

namespace ec {

namespace {

constexpr int max_nb(int N, int F) {
  Plan2 p = plan_of(N);
  int m = 0;
  for (int s = 0; s < p.nstage; ++s) {
    int b = F * (N / p.r[s]);
    if (b > m) m = b;
  }
  return m;
}
// Wavefronts per SIMD to leave registers for: two with a direct radix, whose
// butterfly holds 43 operands (else the compiler takes more than half of them;
// 129^3 FP32 z pass 177 -> 150 us, both y passes 178 -> 158, x inverse 77 -> 52).
// The x forward and the accumulating or FP64 x inverse passes lose more to
// spilled operands than they gain (FP32 x forward 97 -> 143).
template <int N>
constexpr int min_waves() {
  return has_direct(plan_of(N)) ? 2 : 1;
}
constexpr int pick_T(int nb) { return nb >= 256 ? 256 : ((nb + 63) / 64) * 64; }


// ----------------------------------------------------------------- Green operator
//
// Sec. 3.2: eps_hat = Gamma(xi):(C:eps*_hat) with Gamma built from N = K^-1,
// K_ik = C_ijkl xi_j xi_l; here eps_hat = sym(xi (x) N (tau xi)), tau = C:eps*_hat,
// and the kernel returns sigma_hat = C:eps_hat - tau (the stress spectrum, so the
// inverse transform yields sigma directly).  Gamma is homogeneous of degree 0 in
// xi, so the integer labels stand in for xi = 2 pi k / L.

// tau = C:e for cubic C (components xx yy zz yz xz xy; the shear entries of
// e are tensor components, so they take 2 C44).
__device__ __forceinline__ void cubic_stress(const double2* e, const Cubic& C, double2* tau) {
  const double d = C.C11 - C.C12, c44x2 = 2.0 * C.C44;
  const double trx = e[0].x + e[1].x + e[2].x, try_ = e[0].y + e[1].y + e[2].y;
  const double ctx = C.C12 * trx, cty = C.C12 * try_;
#pragma unroll
  for (int c = 0; c < 3; ++c) tau[c] = make_double2(fma(d, e[c].x, ctx), fma(d, e[c].y, cty));
#pragma unroll
  for (int c = 3; c < 6; ++c) tau[c] = make_double2(c44x2 * e[c].x, c44x2 * e[c].y);
}

// w = wgt N(xi) (tau xi), N = K^-1 by the adjugate, K_ik = C_ijkl xi_j xi_l.
__device__ __forceinline__ void green_w(double ax, double ay, double az, const Cubic& C, const double2* tau,
                                        double wgt, double2* w) {
  const double x2 = ax * ax, y2 = ay * ay, z2 = az * az, r2 = x2 + y2 + z2;
  const double c44r2 = C.C44 * r2, dd = C.C11 - C.C44;
  const double K00 = fma(dd, x2, c44r2), K11 = fma(dd, y2, c44r2), K22 = fma(dd, z2, c44r2);
  const double cc = C.C12 + C.C44;
  const double ccx = cc * ax;
  const double K01 = ccx * ay, K02 = ccx * az, K12 = cc * ay * az;
  const double A00 = K11 * K22 - K12 * K12;
  const double A11 = K00 * K22 - K02 * K02;
  const double A22 = K00 * K11 - K01 * K01;
  const double A01 = K02 * K12 - K01 * K22;
  const double A02 = K01 * K12 - K02 * K11;
  const double A12 = K01 * K02 - K00 * K12;
  const double inv = wgt / (K00 * A00 + K01 * A01 + K02 * A02);
  // v = tau . xi (tau symmetric: xx yy zz yz xz xy)
  double2 v0, v1, v2;
  v0.x = tau[0].x * ax + tau[5].x * ay + tau[4].x * az;
  v0.y = tau[0].y * ax + tau[5].y * ay + tau[4].y * az;
  v1.x = tau[5].x * ax + tau[1].x * ay + tau[3].x * az;
  v1.y = tau[5].y * ax + tau[1].y * ay + tau[3].y * az;
  v2.x = tau[4].x * ax + tau[3].x * ay + tau[2].x * az;
  v2.y = tau[4].y * ax + tau[3].y * ay + tau[2].y * az;
  w[0].x = (A00 * v0.x + A01 * v1.x + A02 * v2.x) * inv;
  w[0].y = (A00 * v0.y + A01 * v1.y + A02 * v2.y) * inv;
  w[1].x = (A01 * v0.x + A11 * v1.x + A12 * v2.x) * inv;
  w[1].y = (A01 * v0.y + A11 * v1.y + A12 * v2.y) * inv;
  w[2].x = (A02 * v0.x + A12 * v1.x + A22 * v2.x) * inv;
  w[2].y = (A02 * v0.y + A12 * v1.y + A22 * v2.y) * inv;
}

// s = C:sym(xi (x) w) - tau (FIRST) or s += C:sym(xi (x) w), cubic C: normal
// entries C12 (xi . w) + (C11 - C12) xi_i w_i, shear entries
// C44 (xi_i w_j + xi_j w_i).
template <bool FIRST>
__device__ __forceinline__ void add_cubic_sym(double ax, double ay, double az, const Cubic& C, const double2* w,
                                              const double2* tau, double2* s) {
  const double d = C.C11 - C.C12;
  const double a[3] = {ax, ay, az};
  const double dx = ax * w[0].x + ay * w[1].x + az * w[2].x;
  const double dy = ax * w[0].y + ay * w[1].y + az * w[2].y;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double bx = FIRST ? fma(C.C12, dx, -tau[c].x) : fma(C.C12, dx, s[c].x);
    const double by = FIRST ? fma(C.C12, dy, -tau[c].y) : fma(C.C12, dy, s[c].y);
    s[c] = make_double2(fma(d, a[c] * w[c].x, bx), fma(d, a[c] * w[c].y, by));
  }
  // shear (yz, xz, xy) = pairs (1, 2), (0, 2), (0, 1)
  constexpr int P[3][2] = {{1, 2}, {0, 2}, {0, 1}};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int i = P[q][0], j = P[q][1];
    const double mx = fma(a[i], w[j].x, a[j] * w[i].x), my = fma(a[i], w[j].y, a[j] * w[i].y);
    const double bx = FIRST ? -tau[3 + q].x : s[3 + q].x, by = FIRST ? -tau[3 + q].y : s[3 + q].y;
    s[3 + q] = make_double2(fma(C.C44, mx, bx), fma(C.C44, my, by));
  }
}

// Centred integer label of DFT bin k in [0, n) (Sec. 3.4): k up to (n - 1) / 2,
// k - n above.  Only an even n has a Nyquist bin (k = n / 2), whose label the
// callers choose.
__device__ __forceinline__ int centred(int k, int n) { return k <= (n - 1) / 2 ? k : k - n; }
__device__ __forceinline__ bool nyquist(int k, int n) { return (n & 1) == 0 && k == n / 2; }

// sigma_hat at bin (kx in [0, n/2], ky, kz in [0, n)) from eps*_hat (in place).
// Even-n Nyquist rule: a bin with any index at n/2 gets the mean of the
// operators at the all -n/2 and all +n/2 labels (real part of the centred
// full-complex solution).  xi = 0: zero (the mean is added in FP64 later).
__device__ __forceinline__ void green_bin(double2* e, int kx, int ky, int kz, int n, const Cubic& C) {
  if (kx == 0 && ky == 0 && kz == 0) {
#pragma unroll
    for (int c = 0; c < 6; ++c) e[c] = make_double2(0.0, 0.0);
    return;
  }
  double2 tau[6], w[3];
  cubic_stress(e, C, tau);
  const int h = n / 2;
  const bool nx = nyquist(kx, n), ny = nyquist(ky, n), nz = nyquist(kz, n), nq = nx || ny || nz;
  const double lx = nx ? -h : kx, ly = ny ? -h : centred(ky, n), lz = nz ? -h : centred(kz, n);
  // every bin takes its (first) label; a Nyquist bin weighs it 1/2 and adds
  // the all +n/2 label, so the lanes of a wavefront part for one label only
  green_w(lx, ly, lz, C, tau, nq ? 0.5 : 1.0, w);
  add_cubic_sym<true>(lx, ly, lz, C, w, tau, e);
  if (nq) {
    const double px = nx ? h : lx, py = ny ? h : ly, pz = nz ? h : lz;
    green_w(px, py, pz, C, tau, 0.5, w);
    add_cubic_sym<false>(px, py, pz, C, w, tau, e);
  }
}

// Rotated crystal (C.frm set): the cubic operator applied in the cube frame,
// eps*_hat and the frequency labels rotated in and sigma_hat rotated back, so
// that the cell-frame operator is built from C' = A^T-rotated C without
// forming its 21 constants.
// The cubic operator on a bin whose eps*_hat is already in the cube frame, with
// the frequency label rotated there; sigma_hat stays in the cube frame.
__device__ __forceinline__ void green_core_rot(double2* ec, int kx, int ky, int kz, int n, const Cubic& C) {
  if (kx == 0 && ky == 0 && kz == 0) {
#pragma unroll
    for (int c = 0; c < 6; ++c) ec[c] = make_double2(0.0, 0.0);
    return;
  }
  const double* A = C.frm + 72;
  double2 tau[6], w[3];
  cubic_stress(ec, C, tau);
  const int h = n / 2;
  const bool nx = nyquist(kx, n), ny = nyquist(ky, n), nz = nyquist(kz, n), nq = nx || ny || nz;
  const double lx = nx ? -h : kx, ly = ny ? -h : centred(ky, n), lz = nz ? -h : centred(kz, n);
  auto label = [&](double x, double y, double z, double* r) {
    r[0] = A[0] * x + A[3] * y + A[6] * z;
    r[1] = A[1] * x + A[4] * y + A[7] * z;
    r[2] = A[2] * x + A[5] * y + A[8] * z;
  };
  double r[3];
  label(lx, ly, lz, r);
  green_w(r[0], r[1], r[2], C, tau, nq ? 0.5 : 1.0, w);
  add_cubic_sym<true>(r[0], r[1], r[2], C, w, tau, ec);
  if (nq) {
    label(nx ? h : lx, ny ? h : ly, nz ? h : lz, r);
    green_w(r[0], r[1], r[2], C, tau, 0.5, w);
    add_cubic_sym<false>(r[0], r[1], r[2], C, w, tau, ec);
  }
}

__device__ __forceinline__ void green_bin_rot(double2* e, int kx, int ky, int kz, int n, const Cubic& C) {
  double2 ec[6];
  rot6(C.frm, e, ec);
  green_core_rot(ec, kx, ky, kz, n, C);
  rot6(C.frm + 36, ec, e);
}

// Tile order of a persistent pass.  The tiles are split into eight
// contiguous ranges, one per XCD (dispatch puts workgroup b on XCD b % 8), so
// that neighbouring tiles share an L2.  With a counter per XCD (zero at
// launch) the workgroups of an XCD claim its tiles one at a time, so that one
// starting late behind other work on its CU takes fewer tiles instead of
// holding up the pass; without counters each takes every (grid / 8)-th tile
// of the range.  The tile after the current one is known an iteration ahead
// (for the prefetch): next() at the top of an iteration gives it, the claim
// for the one after it is issued then and stored before the iteration's last
// barrier.
struct TileWalk {
  int lo, hi, g8, xcd;
  uint32_t* ctr;  // nullptr: static order
  int* slot;      // two LDS entries
  __device__ TileWalk(int ntiles, uint32_t* c, int* sl) : ctr(c), slot(sl) {
    g8 = (int)gridDim.x / 8;
    const int per = (ntiles + 7) / 8;
    xcd = (int)(blockIdx.x % 8);
    lo = xcd * per;
    hi = min(ntiles, lo + per);
  }
  // the first two tiles (a barrier must follow before first())
  __device__ void claim_first() {
    if (ctr && threadIdx.x == 0) {
      slot[0] = lo + (int)atomicAdd(&ctr[xcd], 1u);
      slot[1] = lo + (int)atomicAdd(&ctr[xcd], 1u);
    }
  }
  __device__ int first() const { return ctr ? slot[0] : lo + (int)(blockIdx.x / 8); }
  __device__ int next(int t, int it) const { return ctr ? slot[(it + 1) & 1] : t + g8; }
  __device__ uint32_t claim_issue() { return (ctr && threadIdx.x == 0) ? atomicAdd(&ctr[xcd], 1u) : 0u; }
  __device__ void claim_store(int it, uint32_t v) {
    if (ctr && threadIdx.x == 0) slot[it & 1] = lo + (int)v;
  }
};

// ----------------------------------------------------------------- x forward (R2C)

// x forward pass with a two-stage plan of equal radices: each thread reads
// the twiddles of its second-stage butterfly from the global table into
// registers, and the block keeps no LDS copy of the table (more resident
// blocks for these short-lived ones; the inverse pass, which holds more
// registers, keeps the table).
template <int N>
constexpr bool x_twreg() {
  constexpr Plan2 P = plan_of(N);
  return P.nstage == 2 && P.r[0] == P.r[1];
}

template <int N, int NF, int T>
__device__ __forceinline__ auto x_twiddles(const double2* tw_lds, const double2* twg) {
  if constexpr (x_twreg<N>()) {
    constexpr int R = plan_of(N).r[1];
    return make_twreg<N, R, R, Map::Row, NF, T>(twg, threadIdx.x);
  } else {
    return tw_lds;
  }
}

// Persistent: each workgroup walks row groups (ROWS rows of one z plane) in a
// fixed order within its XCD's contiguous range, and loads the next group's
// owner links into registers while it decodes and transforms the current one,
// so the HBM latency of the owner map overlaps the work of the group before.
// The eigenstrains of the next group's single-owner voxels are loaded after
// the current group's transform and before its spectrum stores: vector memory
// operations complete in issue order as far as a wave's wait counter is
// concerned, so a load issued after the stores would wait for them to drain,
// and loads issued one voxel at a time would each wait for the one before.
// Voxels of several owners (a few per cent of the row groups) are decoded in
// place.
// DM: the input, 0 = owner lists, 1 = a dense field [6][n^3], 2 = a dense
// voxel-major field [n^3][6] (the resident stress).
template <int N, typename S, int DM>
__global__ __launch_bounds__(pick_T(max_nb(N, 3 * x_rows(N)))) void k_x_forward(
    const int32_t* __restrict__ own, const int2* __restrict__ lnk, const DevDefect* __restrict__ defs,
    const double* __restrict__ dense, typename Cplx<S>::T* __restrict__ spec, int P, const double2* __restrict__ twg,
    uint32_t* __restrict__ zero_ctr, int max_links) {
  constexpr int ROWS = x_rows(N);
  constexpr int NF = 3 * ROWS;  // (xx,yy), (zz,yz), (xz,xy) per row
  constexpr int T = pick_T(max_nb(N, NF));
  constexpr int LDN = N + N / 16 + 1;
  constexpr int NH = N / 2 + 1;
  constexpr int bpp = N / ROWS;
  constexpr int NG = N * bpp;  // row groups
  __shared__ double2 buf[NF * LDN];
  __shared__ double2 tw[x_twreg<N>() ? 1 : N];
  __shared__ int tslot[2];
  if constexpr (!x_twreg<N>())
    for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  if (zero_ctr && blockIdx.x == 0 && threadIdx.x < NTILECTR) zero_ctr[threadIdx.x] = 0u;
  const size_t n3 = (size_t)N * N * N;
  auto lds = [&](int f, int i) -> double2* { return &buf[f * LDN + i + (i >> 4)]; };
  constexpr int KV = (ROWS * N + T - 1) / T;
  // a group's voxels: ROWS consecutive rows, so ROWS * N consecutive ids
  // The loads below are issued without branches (a lane past the group reads
  // its last voxel and is skipped by the gather, one without an owner reads
  // the twiddle table and is masked), so that the compiler can count them and
  // wait for exactly the ones a use needs.
  auto load_links = [&](int grp, int32_t* lk) {
#pragma unroll
    for (int k = 0; k < KV; ++k) {
      const int i = threadIdx.x + k * T;
      if constexpr (DM == 0) {
        lk[k] = own[(size_t)grp * (ROWS * N) + min(i, ROWS * N - 1)];
      } else {
        lk[k] = -1;
      }
    }
  };
  // single-owner eigenstrains of a group's voxels (zero elsewhere)
  double2 ev[KV][3];
  auto load_vals = [&](const int32_t* lk) {
#pragma unroll
    for (int k = 0; k < KV; ++k) {
      if constexpr (DM == 0) {
        const double2* f = lk[k] >= 0 ? reinterpret_cast<const double2*>(defs[lk[k]].efd) : twg;
#pragma unroll
        for (int c = 0; c < 3; ++c) ev[k][c] = f[c];
      }
    }
  };
  TileWalk walk(NG, nullptr, tslot);
  int grp = walk.first();
  const int hi = walk.hi;
  int32_t link[KV], nlink[KV];
  if (grp < hi) {
    load_links(grp, link);
    load_vals(link);
  }
  const auto twp = x_twiddles<N, NF, T>(tw, twg);
  // Nothing loaded so far stays pending into the loop: the loop's waits are
  // then counted from its own steady state alone (with loads of the set-up
  // still in flight at entry, each wait would have to cover them, and in
  // every later pass it would also wait for the stores of the group before).
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  for (int it = 0; grp < hi; ++it) {
    const int gn = walk.next(grp, it);
    // past the range the loads repeat the current group, unused (so that no
    // branch makes their count uncertain)
    load_links(gn < hi ? gn : grp, nlink);
    const int z = grp / bpp;
    const int y0 = (grp % bpp) * ROWS;
    // gather the rows' six components into the transform inputs (xx + i yy, ...)
#pragma unroll
    for (int k = 0; k < KV; ++k) {
      const int i = threadIdx.x + k * T;
      if (i < ROWS * N) {
        const int r = i / N, x = i - r * N;
        double e[6];
        if (DM == 1) {
          const size_t v = ((size_t)z * N + y0 + r) * N + x;
#pragma unroll
          for (int c = 0; c < 6; ++c) e[c] = dense[c * n3 + v];
        } else if (DM == 2) {
          const double2* vp = reinterpret_cast<const double2*>(dense + 6 * (((size_t)z * N + y0 + r) * N + x));
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            const double2 t = vp[p];
            e[2 * p] = t.x;
            e[2 * p + 1] = t.y;
          }
        } else {  // one owner (loaded with the group before), or none; several: below
          const bool one = link[k] >= 0;
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            e[2 * p] = one ? ev[k][p].x : 0.0;
            e[2 * p + 1] = one ? ev[k][p].y : 0.0;
          }
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) st2(lds(3 * r + p, x), make_double2(e[2 * p], e[2 * p + 1]));
      }
    }
    if constexpr (DM == 0) {
      // voxels of several owners: the exact fixed-point sum over the chain
#pragma unroll
      for (int k = 0; k < KV; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < ROWS * N && link[k] < -1) {
          const int r = i / N, x = i - r * N;
          double e[6];
          decode_voxel(link[k], lnk, defs, e, max_links);
#pragma unroll
          for (int p = 0; p < 3; ++p) st2(lds(3 * r + p, x), make_double2(e[2 * p], e[2 * p + 1]));
        }
      }
    }
    __syncthreads();
    auto from_lds = [&](int f, int i) { return ld2(lds(f, i)); };
    auto to_lds = [&](int f, int i, double2 v) { st2(lds(f, i), v); };
    transform<N, false, Map::Row, NF, T, true, true>(twp, from_lds, from_lds, to_lds, to_lds);
    __syncthreads();
    load_vals(nlink);
    // Hermitian split of the three pair transforms of a row into the six
    // interleaved half-spectrum components.  FP64 storage: one output value per
    // thread, so consecutive threads write consecutive 16-byte values of the
    // row; FP32 storage: one bin (six values, 48 bytes) per thread, which
    // halves the LDS reads and index work where the narrower writes matter less.
    // The loops run over bins k < n/2; the thread of bin 0 of a row also does
    // its bin n/2 (k = n/2 is its own mirror), so no loop pass is left with two
    // busy threads.
    if constexpr (sizeof(S) == 8) {
      auto value = [&](int r, int k, int c) {
        const int p = c >> 1;
        const double2 zk = ld2(lds(3 * r + p, k));
        const double2 zc = conjd(ld2(lds(3 * r + p, k == 0 ? 0 : N - k)));
        const double2 v = (c & 1) ? make_double2(0.5 * (zk.y - zc.y), -0.5 * (zk.x - zc.x))
                                  : make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y + zc.y));
        st2(spec + spec_at(z, y0 + r, k, c, N, P), v);
      };
      for (int e = threadIdx.x; e < ROWS * (N / 2) * 6; e += T) {
        const int r = e / ((N / 2) * 6), q = e % ((N / 2) * 6), k = q / 6, c = q % 6;
        value(r, k, c);
        if (k == 0) value(r, N / 2, c);
      }
    } else {
      auto bin = [&](int r, int k) {
        typename Cplx<S>::T* const out = spec + spec_at(z, y0 + r, k, 0, N, P);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const double2 zk = ld2(lds(3 * r + p, k));
          const double2 zc = conjd(ld2(lds(3 * r + p, k == 0 ? 0 : N - k)));
          st2(out + 2 * p, make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y + zc.y)));
          st2(out + 2 * p + 1, make_double2(0.5 * (zk.y - zc.y), -0.5 * (zk.x - zc.x)));
        }
      };
      // a compile-time trip count, so that the compiler counts the stores
      // (the next group's gather then waits for its loads and leaves these
      // in flight)
      constexpr int NB = ROWS * (N / 2);
#pragma unroll
      for (int q0 = 0; q0 < (NB + T - 1) / T; ++q0) {
        const int e = threadIdx.x + q0 * T;
        if (NB % T == 0 || e < NB) {
          const int r = e / (N / 2), k = e % (N / 2);
          bin(r, k);
          if (k == 0) bin(r, N / 2);
        }
      }
    }
    __syncthreads();  // the next group rewrites the LDS rows
#pragma unroll
    for (int k = 0; k < KV; ++k) link[k] = nlink[k];
    grp = gn;
  }
}

// The x forward pass for eigenstrain fields that few voxels carry: one
// wavefront per row, a lane per kx, and the row transform summed directly,
// X(kx) = sum_x eps*(x) W^(kx x), over the row's covered voxels in ascending x.
// Each piece of 64 voxels is packed by ballot: its covered lanes leave their
// eigenstrains side by side in LDS (single owners fetched for all pieces in
// one round trip), where the sum reads them as broadcasts.  The Nyquist column
// of an even N (W^(N x / 2) = +-1) is summed beside the others.  One row per
// wavefront, not a loop over rows: a wave's memory counter completes in issue
// order, so the next row's links would wait for this row's stores.
//
// A link >= 0 names the record vals + link stride of six doubles (a defect's
// eigenstrain, or the values of a grid point of dislocation pieces).
//
// FP64 storage only: with FP32 storage a last-bit difference from the
// transforms moves the rounding of a spectrum value now and then, and the
// later passes spread that over the whole field at the level of the storage
// error.  At 129^3, 300 defects, the pass takes 19 us (transforms: 116, bound by
// the length-43 butterflies), at 256^3, 2000 defects, 222 (236; 811 MB written).
template <int N>
__global__ __launch_bounds__(256) void k_x_forward_rows(const int32_t* __restrict__ own, const int2* __restrict__ lnk,
                                                        const DevDefect* __restrict__ defs,
                                                        const double* __restrict__ vals, int stride,
                                                        double2* __restrict__ spec,
                                                        const double2* __restrict__ twg,
                                                        uint32_t* __restrict__ zero_ctr, int max_links) {
  constexpr int P = spec_pitch(N, true);
  constexpr int NC = (N + 63) / 64;                  // pieces of 64 voxels of a row
  constexpr bool EVEN = N % 2 == 0;
  constexpr int NK = EVEN ? N / 2 : N / 2 + 1;       // columns on the lanes
  constexpr int NQ = (NK + 63) / 64;                 // columns per lane
  __shared__ double2 tw[N + N / 16 + 1];
  __shared__ double2 stage_out[4][64 * 6];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // contiguous ranges of rows per XCD (workgroup b on XCD b % 8), four rows per workgroup
  constexpr int per = ((N * N + 3) / 4 + 7) / 8;
  const int row = ((int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8)) * 4 + wave;
  const bool live = (int)(blockIdx.x / 8) < per && row < N * N;
  int32_t link[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int x = 64 * j + lane;
    link[j] = live && x < N ? own[(size_t)row * N + x] : -1;
  }
  for (int i = threadIdx.x; i < N; i += 256) tw[i + (i >> 4)] = twg[i];
  if (zero_ctr && blockIdx.x == 0 && threadIdx.x < NTILECTR) zero_ctr[threadIdx.x] = 0u;
  double2 ev[NC][3];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    if (link[j] >= 0) {
      const double2* f = reinterpret_cast<const double2*>(vals + (size_t)link[j] * stride);
#pragma unroll
      for (int p = 0; p < 3; ++p) ev[j][p] = f[p];
    }
  }
  __syncthreads();
  if (!live) return;
  double2* const st = stage_out[wave];  // a piece's eigenstrains, three entries each; then a row's bins
  double2 acc[NQ][6];
  double nyq[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q][c] = make_double2(0.0, 0.0);
    nyq[c] = 0.0;
  }
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const bool in = link[j] != -1;
    uint64_t m = __ballot(in);
    if (m == 0) continue;
    if (in) {
      const int k = __popcll(m & ((1ull << lane) - 1));
      if (link[j] < -1) {  // several owners: the exact sum over the chain
        double e[6];
        decode_voxel(link[j], lnk, defs, e, max_links);
#pragma unroll
        for (int p = 0; p < 3; ++p) ev[j][p] = make_double2(e[2 * p], e[2 * p + 1]);
      }
#pragma unroll
      for (int p = 0; p < 3; ++p) st[3 * k + p] = ev[j][p];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int k = 0; m; ++k) {
      const int x = 64 * j + __ffsll((unsigned long long)m) - 1;
      m &= m - 1;
      double e[6];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const double2 v = st[3 * k + p];
        e[2 * p] = v.x;
        e[2 * p + 1] = v.y;
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int i = ((lane + 64 * q) * x) % N;
        const double2 f = tw[i + (i >> 4)];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          acc[q][c].x = fma(e[c], f.x, acc[q][c].x);
          acc[q][c].y = fma(e[c], f.y, acc[q][c].y);
        }
      }
      if constexpr (EVEN) {
#pragma unroll
        for (int c = 0; c < 6; ++c) nyq[c] += (x & 1) ? -e[c] : e[c];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // a lane's six values turned into runs of 16 bytes per lane over the wavefront
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
#pragma unroll
    for (int c = 0; c < 6; ++c) st[6 * lane + c] = acc[q][c];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int cnt = 6 * (NK - 64 * q < 64 ? NK - 64 * q : 64);
    double2* const out = spec + ((size_t)row * P + 64 * q) * 6;
#pragma unroll
    for (int i = 0; i < 6; ++i)
      if (lane + 64 * i < cnt) out[lane + 64 * i] = st[lane + 64 * i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if constexpr (EVEN) {
    if (lane == 0) {
      double2* const out = spec + ((size_t)row * P + NK) * 6;
#pragma unroll
      for (int c = 0; c < 6; ++c) out[c] = make_double2(nyq[c], 0.0);
    }
  }
}

// Update variant: the rows of the eigenstrain change
// dE = E_new chi_new - E_old chi_old (E: E_old in [0, 6), E_new in [6, 12))
// are built in LDS from the two footprint lists (new ids = old ids shifted by
// (sx, sy, sz) voxels when new_ids == nullptr), for rows y in [y_lo, y_lo+y_len),
// z in [z_lo, z_lo+z_len) (cyclic); other rows are zero and never touched.
// One row block (ROWS rows of one z plane) of one move; buf and tw are the
// caller's LDS (tw filled).
template <int N, typename S>
__device__ __forceinline__ void xfs_block(double2* buf, const double2* tw, const int32_t* __restrict__ old_ids,
                                          int old_cnt, const int32_t* __restrict__ new_ids, int new_cnt, int sx, int sy,
                                          int sz, const double* __restrict__ E, typename Cplx<S>::T* __restrict__ spec,
                                          int P, int y_lo, int y_len, int z_lo, int blk) {
  constexpr int ROWS = x_rows(N);
  constexpr int NF = 3 * ROWS;
  constexpr int T = pick_T(max_nb(N, NF));
  constexpr int LDN = N + N / 16 + 1;
  constexpr int NH = N / 2 + 1;
  if (!new_ids) new_cnt = old_cnt;
  for (int i = threadIdx.x; i < NF * LDN; i += T) buf[i] = make_double2(0.0, 0.0);
  const int rb = (y_len + ROWS - 1) / ROWS;
  const int zi = blk / rb;
  const int y0i = (blk % rb) * ROWS;
  int z = z_lo + zi;
  if (z >= N) z -= N;
  __syncthreads();
  auto lds = [&](int f, int i) -> double2& { return buf[f * LDN + i + (i >> 4)]; };
  // scatter sgn * Ev of the voxels that fall in this block's rows (one row per y)
  auto scatter = [&](int id, double sgn, const double* Ev) {
    const int x = id % N, y = (id / N) % N, zz = id / (N * N);
    if (zz != z) return;
    int yi = y - y_lo;
    if (yi < 0) yi += N;
    yi -= y0i;
    if (yi < 0 || yi >= ROWS || y0i + yi >= y_len) return;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      double2& slot = lds(3 * yi + p, x);
      slot.x += sgn * Ev[2 * p];
      slot.y += sgn * Ev[2 * p + 1];
    }
  };
  // Each voxel is owned by one thread per list pass; a voxel can sit in both
  // lists, so the two passes are separated by a barrier.
  for (int i = threadIdx.x; i < old_cnt; i += T) scatter(old_ids[i], -1.0, E);
  __syncthreads();
  for (int i = threadIdx.x; i < new_cnt; i += T) {
    int id;
    if (new_ids) {
      id = new_ids[i];
    } else {
      const int o = old_ids[i];
      int x = o % N + sx, y = (o / N) % N + sy, zz = o / (N * N) + sz;
      x = (x % N + N) % N;
      y = (y % N + N) % N;
      zz = (zz % N + N) % N;
      id = (zz * N + y) * N + x;
    }
    scatter(id, 1.0, E + 6);
  }
  __syncthreads();
  auto from_lds = [&](int f, int i) { return lds(f, i); };
  auto to_lds = [&](int f, int i, double2 v) { lds(f, i) = v; };
  transform<N, false, Map::Row, NF, T, true, true>(tw, from_lds, from_lds, to_lds, to_lds);
  __syncthreads();
  for (int e = threadIdx.x; e < ROWS * NH * 6; e += T) {
    const int yi = e / (NH * 6), q = e % (NH * 6), k = q / 6, c = q % 6, p = c >> 1;
    if (y0i + yi >= y_len) continue;
    int y = y_lo + y0i + yi;
    if (y >= N) y -= N;
    const double2 zk = lds(3 * yi + p, k);
    const double2 zc = conjd(lds(3 * yi + p, k == 0 ? 0 : N - k));
    const double2 v = (c & 1) ? make_double2(0.5 * (zk.y - zc.y), -0.5 * (zk.x - zc.x))
                              : make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y + zc.y));
    st2(spec + spec_at(z, y, k, c, N, P), v);
  }
  __syncthreads();  // the caller's next block rewrites LDS
}

template <int N, typename S>
__global__ __launch_bounds__(pick_T(max_nb(N, 3 * x_rows(N)))) void k_x_forward_sparse(
    const int32_t* __restrict__ old_ids, const int32_t* __restrict__ old_cnt_p, const int32_t* __restrict__ new_ids,
    int new_cnt, int sx, int sy, int sz, MoveStrain E, typename Cplx<S>::T* __restrict__ spec, int P,
    int y_lo, int y_len, int z_lo, const double2* __restrict__ twg, uint32_t* __restrict__ zero_ctr) {
  constexpr int NF = 3 * x_rows(N);
  constexpr int T = pick_T(max_nb(N, NF));
  constexpr int LDN = N + N / 16 + 1;
  __shared__ double2 buf[NF * LDN];
  __shared__ double2 tw[N];
  if (zero_ctr && blockIdx.x == 0 && threadIdx.x < NTILECTR) zero_ctr[threadIdx.x] = 0u;
  for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  xfs_block<N, S>(buf, tw, old_ids, *old_cnt_p, new_ids, new_cnt, sx, sy, sz, E.v, spec, P, y_lo, y_len, z_lo,
                  blockIdx.x);
}

// Batched hops: the row blocks of every job, job after job, over a fixed grid
// (a block takes every gridDim-th one).
template <int N, typename S>
__global__ __launch_bounds__(pick_T(max_nb(N, 3 * x_rows(N)))) void k_x_forward_sparse_batch(
    const HopJob* __restrict__ jobs, int njob, int P, const double2* __restrict__ twg, uint32_t* __restrict__ zero_ctr) {
  constexpr int NF = 3 * x_rows(N);
  constexpr int T = pick_T(max_nb(N, NF));
  constexpr int LDN = N + N / 16 + 1;
  __shared__ double2 buf[NF * LDN];
  __shared__ double2 tw[N];
  if (zero_ctr && blockIdx.x == 0 && threadIdx.x < NTILECTR) zero_ctr[threadIdx.x] = 0u;
  for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  int total = 0;
  for (int j = 0; j < njob; ++j) total += jobs[j].xitems;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    int j = 0, first = 0;
    while (item >= first + jobs[j].xitems) first += jobs[j++].xitems;
    const HopJob& J = jobs[j];
    xfs_block<N, S>(buf, tw, J.ids + J.slot, J.cnt[J.idx], nullptr, 0, J.sx, J.sy, J.sz, J.E12,
                    (typename Cplx<S>::T*)J.spec, P, J.ylo, J.ylen, J.zlo, item - first);
  }
}

// --------------------------------------------------------------- y / z pencils
//
// A tile is WX consecutive kx columns x all six components (6 WX transforms)
// of one z plane (y pass) or one y row (z pass), transformed along y or z.  In
// the component-interleaved layout every row of the tile is one contiguous
// run of 6 WX values; thread lane f = 6 w + c keeps its (column, component)
// across butterflies (the workgroup size is a multiple of 6 WX).  The last kx
// tile holds the n/2 column and idle lanes.

// largest radix of the pencil factorisation
template <int N>
constexpr int pencil_rmax() {
  constexpr Plan2 P = plan_of(N);
  return P.r[0] > P.r[1] ? (P.r[0] > P.r[2] ? P.r[0] : P.r[2]) : (P.r[1] > P.r[2] ? P.r[1] : P.r[2]);
}

// kx columns per tile: LDS for 6 WX transforms of N points stays at 48 KB
template <int N, typename LT>
constexpr int pencil_wx() {
  constexpr int w = sizeof(LT) == 8 ? 4 : 2;
  return N >= 512 ? w / 2 : (has_direct(plan_of(N)) ? 2 : w);
}

// Threads of a tile pass over NF transforms: one butterfly per thread in the
// widest-radix stage.  A direct radix has few butterflies and shares each out
// over seven threads (direct_split).
template <int N>
constexpr int tile_threads(int NF, int rmax) {
  return (has_direct(plan_of(N)) || has_direct(plan_fused(N)) ? 7 : 1) * NF * (N / rmax);
}

template <int N, typename LT>
constexpr int pencil_threads() {
  return tile_threads<N>(6 * pencil_wx<N, LT>(), pencil_rmax<N>());
}

// the pencil pass prefetches the next tile's operands (FP32 storage, plans
// without a direct radix)
template <int N, typename S>
constexpr bool pencil_pipe() {
  return sizeof(S) == 4 && !has_direct(plan_of(N));
}

// Tiles of a batch of hops: job j holds cnt(j) consecutive tiles; (job, local
// tile) of tile t by a walk over the (at most MAXBATCH) jobs.
template <class Count>
__device__ __forceinline__ int job_of_tile(int t, int njob, Count&& cnt, int& local) {
  int j = 0, first = 0;
  while (j + 1 < njob && t >= first + cnt(j)) first += cnt(j++);
  local = t - first;
  return j;
}

// BATCH: the tiles of njob hops of a batch (jobs), job after job: a job's
// spectrum and (y pass, PRUNE) its planes and input rows come from its record;
// spec, pr and ntiles are then unused.
template <int N, typename S, bool INV, typename LT, bool PRUNE, int AXIS, bool BATCH = false>
__global__ __launch_bounds__((pencil_threads<N, LT>())) __attribute__((amdgpu_waves_per_eu(min_waves<N>()))) void
k_pencil(typename Cplx<S>::T* __restrict__ spec,
                                                                     Prune pr, const double2* __restrict__ twg,
                                                                     int ntiles, uint32_t* __restrict__ ctr,
                                                                     const HopJob* __restrict__ jobs = nullptr,
                                                                     int njob = 0) {
  constexpr int WX = pencil_wx<N, LT>();
  constexpr int NF = 6 * WX;
  constexpr int T = pencil_threads<N, LT>();
  constexpr int NH = N / 2 + 1;
  constexpr int KB = (NH + WX - 1) / WX;
  constexpr Plan2 PL = plan_of(N);
  constexpr int R0 = PL.r[0];
  constexpr int NOP = ((NF * (N / R0) + T - 1) / T) * R0;  // first-stage operands per thread
  static_assert(T % NF == 0, "a thread must keep its column across butterflies");
  constexpr int P = spec_pitch(N, sizeof(S) == 8);
  // element stride along the transform axis; all offsets fit 32 bits
  constexpr int SI = AXIS == 1 ? 6 * P : 6 * N * P;
  static_assert(6LL * N * N * P < (1LL << 31), "32-bit element offsets");
  using C2 = typename Cplx<S>::T;
  __shared__ LT buf[N * NF];
  __shared__ double2 tw[N];
  for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  // tiles per job in a batch: the planes of its pruned range (y pass, PRUNE)
  // or all of them
  auto job_tiles = [&](int j) { return (PRUNE && AXIS == 1 ? jobs[j].zlen : N) * KB; };
  if constexpr (BATCH) {
    ntiles = 0;
    for (int j = 0; j < njob; ++j) ntiles += job_tiles(j);
  }
  // the spectrum, pruning and local tile index of tile t
  auto tile_of = [&](int t, C2*& base, Prune& p) -> int {
    if constexpr (BATCH) {
      int lt;
      const int j = job_of_tile(t, njob, job_tiles, lt);
      base = (C2*)jobs[j].spec;
      p = Prune{jobs[j].ylo, jobs[j].ylen, jobs[j].zlo, jobs[j].zlen};
      return lt;
    } else {
      base = spec;
      p = pr;
      return t;
    }
  };
  auto in_range_of = [&](const Prune& p, int i) {
    if (!PRUNE) return true;
    int d = i - p.in_lo;
    if (d < 0) d += N;
    return d < p.in_len;
  };
  // lane f's column in tile t (the base of the spectrum if the lane is idle)
  auto column = [&](int t, int f, bool& valid, Prune& p) -> C2* {
    C2* base;
    const int lt = tile_of(t, base, p);
    const int o = lt / KB, kx = (lt % KB) * WX + f / 6;
    valid = kx < NH;
    if (!valid) return base;
    if (AXIS == 1) {
      int z = p.z_lo + o;
      if (z >= N) z -= N;
      return base + (z * N * P + kx) * 6 + f % 6;
    }
    return base + (o * P + kx) * 6 + f % 6;
  };
  // FP32 storage: raw first-stage operands of the next tile are loaded while
  // the current one is transformed (rows outside the input range read row
  // in_lo, a cache hit, and are zeroed when consumed).  FP64 storage would
  // need twice the registers for them and loads each tile's operands in turn,
  // and so does a plan with a direct radix.
  constexpr bool PIPE = pencil_pipe<N, S>();
  C2 nxt[NOP];
  auto fetch = [&](int t, int tid) {
    if constexpr (!PIPE) return;
    bool v;
    Prune p;
    const C2* colp = column(t, tid % NF, v, p);
    for_operands<N, R0, Map::Pencil, NF, T>(
        [&](int, int i, int slot) { nxt[slot] = colp[(in_range_of(p, i) ? i : p.in_lo) * SI]; }, tid);
  };
  auto from_lds = [&](int f, int i) { return ld2(&buf[i * NF + f]); };
  auto to_lds = [&](int f, int i, double2 v) { st2(&buf[i * NF + f], v); };
  __shared__ int tslot[2];
  TileWalk walk(ntiles, PIPE ? ctr : nullptr, tslot);
  walk.claim_first();
  __syncthreads();
  int t = walk.first();
  const int hi = walk.hi;
  if (t < hi) fetch(t, threadIdx.x);
  __syncthreads();
  // two equal radices: the second stage gives a thread the same butterfly in
  // every tile, so its twiddles stay in registers (FP32 storage; with FP64
  // storage the extra registers would cost occupancy)
  constexpr bool TWREG = PL.nstage == 2 && PL.r[0] == PL.r[1] && NF * (N / R0) == T && sizeof(S) == 4;
  const auto twp = [&] {
    if constexpr (TWREG)
      return make_twreg<N, R0, R0, Map::Pencil, NF, T>(tw, threadIdx.x);
    else
      return (const double2*)tw;
  }();
  for (int it = 0; t < hi; ++it) {
    const int tn = walk.next(t, it);
    const uint32_t claim = walk.claim_issue();
    // laundered thread index: index arithmetic is redone per tile instead of
    // being held in registers across the loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    bool valid;
    Prune pt;
    C2* const colp = column(t, tid % NF, valid, pt);
    // a lane past the last column transforms whatever its loads returned
    // (finite spectrum values) and stores nothing
    // without the prefetch every operand is loaded (a row outside the input
    // range reads row in_lo, a cache hit) and zeroed afterwards, so that the
    // loads are issued together rather than one branch at a time
    auto load0 = [&](int, int i, int slot) -> double2 {
      const bool in = !PRUNE || (valid && in_range_of(pt, i));
      if constexpr (PIPE) return in ? ld2(&nxt[slot]) : make_double2(0.0, 0.0);
      const double2 v = ld2(colp + (in ? i : pt.in_lo) * SI);
      return in ? v : make_double2(0.0, 0.0);
    };
    auto store_last = [&](int, int i, double2 v) {
      if (valid) st2(colp + i * SI, v);
    };
    const bool more = tn < hi;
    if constexpr (PL.nstage == 1) {
      stage<N, R0, 1, INV, Map::Pencil, NF, T>(tw, load0, store_last, false, tid);
      if (more) fetch(tn, tid);
    } else {
      stage<N, R0, 1, INV, Map::Pencil, NF, T>(tw, load0, to_lds, false, tid);
      if (more) fetch(tn, tid);
      __syncthreads();
      if constexpr (PL.nstage == 2) {
        stage<N, PL.r[1], R0, INV, Map::Pencil, NF, T>(twp, from_lds, store_last, false, tid);
      } else {
        stage<N, PL.r[1], R0, INV, Map::Pencil, NF, T>(tw, from_lds, to_lds, true, tid);
        __syncthreads();
        stage<N, PL.r[2], R0 * PL.r[1], INV, Map::Pencil, NF, T>(tw, from_lds, store_last, false, tid);
      }
    }
    walk.claim_store(it, claim);
    __syncthreads();  // the next tile's first stage rewrites LDS
    t = tn;
  }
}

// ------------------------------------------- z-forward + Green + z-inverse (fused)
//
// One workgroup owns W kx columns of one ky row for all six components (6 W
// transforms of length N along z, each row of the tile one contiguous run of
// the interleaved spectrum) in one LDS tile: forward transforms, the Green
// step per bin in place, inverse transforms.  The spectrum is read and written
// once per solve instead of three times, and every stage has all six
// components' butterflies to spread over the workgroup.

template <int N>
struct FusedPlan {
  static constexpr Plan2 P = plan_fused(N);
  static constexpr int NSTG = P.nstage;
  static constexpr int R0 = P.r[0], R1 = P.r[1], R2 = P.r[2];
  static constexpr int RL = NSTG == 1 ? R0 : (NSTG == 2 ? R1 : R2);
  static constexpr int I0 = RL;
  static constexpr int I1 = NSTG == 1 ? 1 : (NSTG == 2 ? R0 : R1);
  static constexpr int I2 = NSTG == 3 ? R0 : 1;
};

// Two-column tiles without the operand prefetch and register twiddles (which
// would take their registers) for the lengths 24 .. 256: three or more
// resident workgroups per CU hide more latency than one four-column one with
// the prefetch (FP32 pass at 256^3 0.33 -> 0.27 ms, 240^3 0.33 -> 0.27, 160^3
// 0.098 -> 0.077, 128^3 0.070 -> 0.042, 64^3 0.030 -> 0.013, 48^3 0.024 ->
// 0.014, 32^3 0.013 -> 0.008).  At 512 the
// two-column tile keeps the prefetch (without it 3.6 -> 4.2 ms).  The odd 129
// takes two columns as well, 252 threads (its length-43 butterflies shared out
// over seven threads each; 129^3 FP32 pass 0.274 -> 0.150 ms).
template <int N>
constexpr bool zg_narrow() {
  return N >= 24 && N <= 256 && !has_direct(plan_fused(N));
}

// columns per tile: four, or two for the lengths above, at N = 512 (where a
// four-column tile would not fit) and with FP64 storage from N = 256 on
template <int N, typename S>
constexpr int zg_width() {
  return (N >= 512 || zg_narrow<N>() || has_direct(plan_fused(N)) || (sizeof(S) == 8 && N >= 256)) ? 2 : 4;
}

// one butterfly per thread in the widest-radix stage; a multiple of the 6 W
// transforms, so every lane keeps its transform
template <int N, typename S>
constexpr int zg_fft_threads() {
  using FP = FusedPlan<N>;
  constexpr int rmax = FP::R0 > FP::R1 ? (FP::R0 > FP::R2 ? FP::R0 : FP::R2) : (FP::R1 > FP::R2 ? FP::R1 : FP::R2);
  return tile_threads<N>(6 * zg_width<N, S>(), rmax);
}

// Workgroup size: the butterfly threads, or for the two-column tile at 256
// four whole wavefronts (the fourth idle in the transform stages, every one
// busy in the Green step): three resident workgroups then put three
// wavefronts on every SIMD, where three-wavefront groups would put three on
// one SIMD and two on the others, and every workgroup has a wavefront on the
// busiest one.
template <int N, typename S>
constexpr int zg_threads() {
  constexpr int t = zg_fft_threads<N, S>();
  return (N == 256 && zg_narrow<N>() && zg_width<N, S>() == 2) ? ((t + 255) / 256) * 256 : t;
}

template <int N, typename S>
constexpr bool zg_pipe() {
  return sizeof(S) == 4 && !zg_narrow<N>() && !has_direct(plan_fused(N));
}

// Wavefronts per SIMD the compiler must leave registers for: three for the
// two-column tiles of 64 .. 256 (three resident workgroups; at 256 twelve
// wavefronts per CU), else one (no bound beyond the workgroup size).
template <int N, typename S>
constexpr int zg_waves_per_eu() {
  return zg_narrow<N>() ? 3 : min_waves<N>();
}

// LDS row swizzle: the low three bits of the z index are XORed with the next
// three, so stride-R stores of the first stages spread over all banks.
__device__ __forceinline__ int zg_swz(int i) { return (i & ~7) | ((i ^ (i >> 3)) & 7); }

// BATCH: the tiles of njob hops of a batch, job after job (NT each), a job's
// spectrum and input planes from its record (spec and pr unused).
template <int N, typename S, bool PRUNE, bool ROT, bool BATCH = false>
__global__ __launch_bounds__((zg_threads<N, S>())) __attribute__((amdgpu_waves_per_eu(zg_waves_per_eu<N, S>())))
void k_zgreen(typename Cplx<S>::T* __restrict__ spec, Cubic C,
                                                                Prune pr, const double2* __restrict__ twg,
                                                                uint32_t* __restrict__ ctr,
                                                                const HopJob* __restrict__ jobs = nullptr,
                                                                int njob = 0) {
  using FP = FusedPlan<N>;
  constexpr int W = zg_width<N, S>();
  constexpr int T = zg_threads<N, S>();
  constexpr int NH = N / 2 + 1;
  constexpr int KB = (NH + W - 1) / W;
  constexpr int NT = N * KB;  // tiles
  constexpr int NF = 6 * W;   // transforms per tile
  constexpr int R0 = FP::R0, R1 = FP::R1, R2 = FP::R2;
  constexpr int NOP = ((NF * (N / R0) + T - 1) / T) * R0;  // first-stage operands per thread
  static_assert(FP::NSTG >= 2, "the first stage must not be the last");
  using C2 = typename Cplx<S>::T;
  // FP64 tile in both storage precisions: rounding the whole spectrum to FP32
  // next to the Green step and between stages roughly doubles the FP32-storage
  // energy error, while the extra LDS costs little here
  __shared__ double2 buf[6 * N * W];
  __shared__ double2 tw[N];
  for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  constexpr int P = spec_pitch(N, sizeof(S) == 8);
  constexpr int SI = 6 * N * P;  // kz stride; all offsets fit 32 bits
  static_assert(6LL * N * N * P < (1LL << 31), "32-bit element offsets");
  // the row swizzle permutes whole groups of eight rows; it pays for
  // four-column tiles, while with two columns its index arithmetic costs more
  // than the bank conflicts it removes (0.27 against 0.28 ms at 256^3)
  constexpr bool SWZ = N % 8 == 0 && W == 4;
  auto lds = [&](int f, int i) -> double2* { return &buf[__umul24(SWZ ? zg_swz(i) : i, NF) + f]; };
  auto from_lds = [&](int f, int i) { return ld2(lds(f, i)); };
  auto to_lds = [&](int f, int i, double2 v) { st2(lds(f, i), v); };
  // the spectrum and input planes of tile t, and its index within its job
  auto tile_of = [&](int t, C2*& base, Prune& p) -> int {
    if constexpr (BATCH) {
      const int j = t / NT;
      base = (C2*)jobs[j].spec;
      p = Prune{jobs[j].zlo, jobs[j].zlen, 0, N};
      return t - j * NT;
    } else {
      base = spec;
      p = pr;
      return t;
    }
  };
  auto in_z_of = [&](const Prune& p, int i) {
    if (!PRUNE) return true;
    int d = i - p.in_lo;
    if (d < 0) d += N;
    return d < p.in_len;
  };
  // FP32 storage: raw first-stage operands of the next tile, loaded while the
  // current one is transformed (rows outside the input range read row in_lo
  // instead, a cache hit, and are zeroed when consumed).  FP64 storage, and
  // a plan with a direct radix (whose operands already fill the registers),
  // load each tile's operands in turn.
  constexpr bool PIPE = zg_pipe<N, S>();
  C2 nxt[NOP];
  auto fetch = [&](int t, int tid) {
    if constexpr (!PIPE) return;
    C2* base;
    Prune p;
    const int lt = tile_of(t, base, p);
    const int f0 = tid % NF, kx = (lt % KB) * W + f0 / 6;
    const C2* col0 = base + (kx < NH ? ((lt / KB) * P + kx) * 6 + f0 % 6 : 0);
    for_operands<N, R0, Map::Pencil, NF, T>(
        [&](int, int i, int slot) { nxt[slot] = col0[(in_z_of(p, i) ? i : p.in_lo) * SI]; }, tid);
  };
  __shared__ int tslot[2];
  TileWalk walk(BATCH ? NT * njob : NT, PIPE ? ctr : nullptr, tslot);
  walk.claim_first();
  __syncthreads();
  int t = walk.first();
  const int hi = walk.hi;
  if (t < hi) fetch(t, threadIdx.x);
  __syncthreads();
  // two equal radices: the twiddled stage of either direction gives a thread
  // the same butterfly in every tile, so its twiddles stay in registers (with
  // the prefetch, FP32 storage; otherwise the extra registers would cost
  // occupancy)
  constexpr bool TWREG = FP::NSTG == 2 && R0 == R1 && PIPE;
  const auto twz = [&] {
    if constexpr (TWREG)
      return make_twreg<N, R1, R0, Map::Pencil, NF, T>(tw, threadIdx.x);
    else
      return (const double2*)tw;
  }();
  for (int it = 0; t < hi; ++it) {
    const int tn = walk.next(t, it);
    const uint32_t claim = walk.claim_issue();
    // the thread index is laundered per tile so that the many index
    // expressions derived from it are recomputed, not held in registers
    // across the loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    C2* tbase;
    Prune pt;
    const int lt = tile_of(t, tbase, pt);
    const int ky = lt / KB;
    const int f0 = tid % NF, w = f0 / 6;  // lane f = 6 w + c keeps its column
    const int kx = (lt % KB) * W + w;
    const bool valid = kx < NH;
    C2* const col0 = tbase + (valid ? (ky * P + kx) * 6 + f0 % 6 : 0);
    // a lane past the last column transforms whatever its loads returned
    // (finite spectrum values), takes no part in the Green step and stores
    // nothing
    // without the prefetch every operand is loaded (a plane outside the input
    // range reads plane in_lo, a cache hit) and zeroed afterwards, so that the
    // loads are issued together rather than one branch at a time
    auto load0 = [&](int, int i, int slot) -> double2 {
      const bool in = !PRUNE || (valid && in_z_of(pt, i));
      if constexpr (PIPE) return in ? ld2(&nxt[slot]) : make_double2(0.0, 0.0);
      const double2 v = ld2(col0 + (in ? i : pt.in_lo) * SI);
      return in ? v : make_double2(0.0, 0.0);
    };
    stage<N, R0, 1, false, Map::Pencil, NF, T>(tw, load0, to_lds, false, tid);
    if (tn < hi) fetch(tn, tid);
    __syncthreads();
    if constexpr (R2 == 1) {
      stage<N, R1, R0, false, Map::Pencil, NF, T>(twz, from_lds, to_lds, true, tid);
    } else {
      stage<N, R1, R0, false, Map::Pencil, NF, T>(tw, from_lds, to_lds, true, tid);
      __syncthreads();
      stage<N, R2, R0 * R1, false, Map::Pencil, NF, T>(tw, from_lds, to_lds, true, tid);
    }
    __syncthreads();
    // Green step: one bin (all six components) per iteration, in place.  For
    // a rotated crystal eps*_hat arrives in the cube frame (the rasterised
    // eigenstrain is kept there), the cubic operator takes rotated labels, and
    // a second loop over the same bins of each thread turns sigma_hat back to
    // the cell frame (one loop for both pushed the FP32 tile past 256 VGPRs).
#pragma unroll 1
    for (int b = tid; b < N * W; b += T) {
      const int bw = b % W, kz = b / W, bkx = kx - w + bw;
      if (bkx >= NH) continue;
      double2 e[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) e[c] = from_lds(bw * 6 + c, kz);
      if constexpr (ROT)
        green_core_rot(e, bkx, ky, kz, N, C);
      else
        green_bin(e, bkx, ky, kz, N, C);
#pragma unroll
      for (int c = 0; c < 6; ++c) to_lds(bw * 6 + c, kz, e[c]);
    }
    if constexpr (ROT) {
#pragma unroll 1
      for (int b = tid; b < N * W; b += T) {
        const int bw = b % W, kz = b / W;
        if (kx - w + bw >= NH) continue;
        double2 e[6], r[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) e[c] = from_lds(bw * 6 + c, kz);
        rot6(C.frm + 36, e, r);
#pragma unroll
        for (int c = 0; c < 6; ++c) to_lds(bw * 6 + c, kz, r[c]);
      }
    }
    __syncthreads();
    auto store_last = [&](int, int i, double2 v) {
      if (valid) st2(col0 + i * SI, v);
    };
    transform_plan<N, FP::I0, FP::I1, FP::I2, true, Map::Pencil, NF, T, NF, true, false>(twz, from_lds, from_lds,
                                                                                    to_lds, store_last, tid);
    walk.claim_store(it, claim);
    __syncthreads();  // the next tile's first stage rewrites the tile
    t = tn;
  }
}

// The fused pass with half the LDS: the same tile, its four exchanges (between
// the stages of either direction and around the Green step) going through LDS
// as real parts, then imaginary parts.  The pass is bound by the wavefronts in
// flight: a two-column tile at 240 takes 27 KB of LDS instead of 50, and with
// the thread's values in registers between the exchanges the kernel needs no
// scratch, so four workgroups of three wavefronts fit a CU's registers.  For
// two-stage plans whose stages give a thread at most one butterfly each.
// Measured, whole tile -> half: FP32 states 240^3 full pass 260 -> 222 us, a
// hop's pruned one 261 -> 213 (FP64 305 -> 302, 293 -> 244); 160^3 75 -> 71
// and 76 -> 71 (FP64 80 -> 73, 76 -> 73).  Below, there is little to gain (48^3
// 13.7 -> 10.4, 64^3 15.7 -> 14.0, 96^3 28.4 -> 27.4) or a loss (128^3 41 -> 44),
// so 24 to 128 keep the whole tile.  At 256, where the whole tile has four
// wavefronts a workgroup and needs no scratch either: 271 -> 255 full, 230 -> 242
// pruned, FP64 353 -> 363, so 256 keeps it; so does every rotated frame, whose
// Green step spills here (FP64 160^3 95 -> 120, 240^3 373 -> 492).  And so do the
// solves of FP32 states: the compiler fuses other multiplies and adds here, the
// stress moves by 1e-11, and stored-type energies, which round its transform to
// FP32 twice more, by 9e-10 (160^3; 6e-16 with the whole tile).
template <int N>
constexpr bool zg_half() {
  return N == 160 || N == 240;
}
template <int N>
constexpr int zh_threads() {
  using FP = FusedPlan<N>;
  return 12 * (FP::R0 < FP::R1 ? N / FP::R0 : N / FP::R1);
}

template <int N, typename S, bool PRUNE, bool BATCH = false>
__global__ __launch_bounds__((zh_threads<N>())) __attribute__((amdgpu_waves_per_eu(3)))
void k_zgreen_half(typename Cplx<S>::T* __restrict__ spec, Cubic C, Prune pr, const double2* __restrict__ twg,
                   const HopJob* __restrict__ jobs = nullptr, int njob = 0) {
  using FP = FusedPlan<N>;
  constexpr int W = 2, NF = 6 * W;
  constexpr int R0 = FP::R0, R1 = FP::R1;
  static_assert(FP::NSTG == 2 && R0 * R1 == N, "two stages");
  constexpr int T = zh_threads<N>();
  constexpr int NB0 = NF * (N / R0), NB1 = NF * (N / R1);
  static_assert(NB0 <= T && NB1 <= T && T % NF == 0, "one butterfly per thread and stage");
  constexpr int NH = N / 2 + 1;
  constexpr int KB = (NH + W - 1) / W;
  constexpr int NT = N * KB;
  constexpr int NBIN = N * W, BQ = (NBIN + T - 1) / T;
  constexpr int P = spec_pitch(N, sizeof(S) == 8);
  constexpr int SI = 6 * N * P;
  static_assert(6LL * N * N * P < (1LL << 31), "32-bit element offsets");
  using C2 = typename Cplx<S>::T;
  __shared__ double buf[NF * N];
  __shared__ double2 tw[N];
  const int ntiles = BATCH ? NT * njob : NT;
  const int per = (ntiles + 7) / 8;
  const int t = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per || t >= ntiles) return;
  C2* base = spec;
  Prune p = pr;
  int lt = t;
  if constexpr (BATCH) {
    const int j = t / NT;
    base = (C2*)jobs[j].spec;
    p = Prune{jobs[j].zlo, jobs[j].zlen, 0, N};
    lt = t - j * NT;
  }
  const int ky = lt / KB, kx0 = (lt % KB) * W;
  // The thread index is laundered in every phase, so that the index arithmetic
  // is done again there instead of being held in registers: f = tid % NF is the
  // thread's transform in every stage, j = tid / NF its butterfly.
  int tid = threadIdx.x;
  auto launder = [&]() { asm volatile("" : "+v"(tid)); };
  auto in0 = [&]() { return NB0 == T || tid < NB0; };
  auto in1 = [&]() { return NB1 == T || tid < NB1; };
  auto column = [&](bool& valid) -> C2* {
    const int f = tid % NF;
    valid = kx0 + f / 6 < NH;
    return base + (ky * P + (valid ? kx0 : 0)) * 6 + (valid ? f : 0);
  };
  // element j R + r (PUT) or j + r M (GET) of the thread's transform
  auto put = [&](auto& a, auto RC, bool im) {
    constexpr int R = decltype(RC)::value;
    launder();
    double* o = buf + (tid / NF) * (R * NF) + tid % NF;
#pragma unroll
    for (int r = 0; r < R; ++r) o[r * NF] = im ? a[r].y : a[r].x;
  };
  auto get = [&](auto& a, auto RC, auto MC, bool im) {
    constexpr int R = decltype(RC)::value, M = decltype(MC)::value;
    launder();
    const double* o = buf + tid;  // (tid / NF) NF + tid % NF
#pragma unroll
    for (int r = 0; r < R; ++r) (im ? a[r].y : a[r].x) = o[r * (M * NF)];
  };
  auto put_at = [&](auto& a, auto RC, auto MC, bool im) {
    constexpr int R = decltype(RC)::value, M = decltype(MC)::value;
    launder();
    double* o = buf + tid;
#pragma unroll
    for (int r = 0; r < R; ++r) o[r * (M * NF)] = im ? a[r].y : a[r].x;
  };
  using C0 = std::integral_constant<int, R0>;
  using C1 = std::integral_constant<int, R1>;
  double2 v[R0], u[R1];
  if (in0()) {
    bool valid;
    const C2* const col = column(valid);
    const int j = tid / NF;
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const int i = j + r * (N / R0);
      bool in = true;
      if constexpr (PRUNE) {
        int d = i - p.in_lo;
        if (d < 0) d += N;
        in = valid && d < p.in_len;
      }
      // planes outside the input range read plane in_lo (a cache hit) and are zeroed
      const double2 a = ld2(col + (in ? i : p.in_lo) * SI);
      v[r] = in ? a : make_double2(0.0, 0.0);
    }
  }
  for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  if (in0()) {
    Dft<R0, false>::run(v);
    put(v, C0{}, false);
  }
  __syncthreads();
  if (in1()) get(u, C1{}, C0{}, false);
  __syncthreads();
  if (in0()) put(v, C0{}, true);
  __syncthreads();
  if (in1()) {
    get(u, C1{}, C0{}, true);
    const int j = tid / NF;
#pragma unroll
    for (int r = 1; r < R1; ++r) u[r] = cmul(u[r], tw[j * r]);
    Dft<R1, false>::run(u);
  }
  __syncthreads();
  // Green step: bins tid + q T of the tile, all six components in registers
  double2 e[BQ][6];
  auto bins = [&](auto&& fn) {
    launder();
#pragma unroll
    for (int q = 0; q < BQ; ++q) {
      const int b = tid + q * T;
      if (NBIN % T == 0 || b < NBIN) fn(b, e[q]);
    }
  };
  if (in1()) put_at(u, C1{}, C0{}, false);
  __syncthreads();
  bins([&](int b, double2* g) {
#pragma unroll
    for (int c = 0; c < 6; ++c) g[c].x = buf[6 * b + c];
  });
  __syncthreads();
  if (in1()) put_at(u, C1{}, C0{}, true);
  __syncthreads();
  bins([&](int b, double2* g) {
#pragma unroll
    for (int c = 0; c < 6; ++c) g[c].y = buf[6 * b + c];
    const int kx = kx0 + b % W, kz = b / W;
    __builtin_amdgcn_sched_barrier(0);
    if (kx < NH) green_bin(g, kx, ky, kz, N, C);
    __builtin_amdgcn_sched_barrier(0);
  });
  __syncthreads();
  bins([&](int b, double2* g) {
#pragma unroll
    for (int c = 0; c < 6; ++c) buf[6 * b + c] = g[c].x;
  });
  __syncthreads();
  if (in1()) get(u, C1{}, C0{}, false);
  __syncthreads();
  bins([&](int b, double2* g) {
#pragma unroll
    for (int c = 0; c < 6; ++c) buf[6 * b + c] = g[c].y;
  });
  __syncthreads();
  if (in1()) {
    get(u, C1{}, C0{}, true);
    Dft<R1, true>::run(u);
  }
  __syncthreads();
  if (in1()) put(u, C1{}, false);
  __syncthreads();
  if (in0()) get(v, C0{}, C1{}, false);
  __syncthreads();
  if (in1()) put(u, C1{}, true);
  __syncthreads();
  if (in0()) {
    get(v, C0{}, C1{}, true);
    const int j = tid / NF;
#pragma unroll
    for (int r = 1; r < R0; ++r) v[r] = cmul(v[r], conjd(tw[j * r]));
    Dft<R0, true>::run(v);
    launder();
    bool valid;
    C2* const col = column(valid) + (tid / NF) * SI;
    if (valid)
#pragma unroll
      for (int r = 0; r < R0; ++r) st2(col + r * R1 * SI, v[r]);
  }
}

// Pointwise Green step over the half spectrum (one thread per bin).
template <typename S>
__global__ __launch_bounds__(256) void k_green(typename Cplx<S>::T* __restrict__ spec, int n, int P, Cubic C) {
  const int NH = n / 2 + 1;
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (size_t)n * n * NH) return;
  const int kx = (int)(t % NH);
  const size_t r = t / NH;
  const int ky = (int)(r % n), kz = (int)(r / n);
  typename Cplx<S>::T* const bin = spec + spec_at(kz, ky, kx, 0, n, P);
  double2 e[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) e[c] = ld2(bin + c);
  if (C.frm)
    green_bin_rot(e, kx, ky, kz, n, C);
  else
    green_bin(e, kx, ky, kz, n, C);
#pragma unroll
  for (int c = 0; c < 6; ++c) st2(bin + c, e[c]);
}

// --------------------------------------------------------- x inverse (C2R) + stress

// ACC: the result is added to a field of the stress's layout: add3 (a stress
// held beside the solve, such as that of dislocation loops), or sig itself when
// add3 is null.
// BG: the stress planes of dislocation lines along the axes in bg_mask
// ([3][n^2][6], FP64) are added as well.
// BATCH: njob hops of a batch, N N / ROWS blocks each, a job's spectrum and
// stress from its record (spec and sig unused).
// MASK: the stress is stored only at voxels some defect covers (own[v] & keep
// != -1), the voxels an energy reduction reads; the others keep what they
// held.  keep = 0 stores every voxel: the pass that forms the whole field runs
// this same code, so a covered voxel gets the same bits either way (separate
// code for the two could fuse multiplies and adds differently).
//
// With FP32 storage the exchange between two stages goes through half the LDS
// (transform_half): the workgroups of two or three wavefronts were limited to
// ten wavefronts per CU by their LDS (256^3 covered-voxel pass 172 -> 159 us; with
// registers for four wavefronts per SIMD, which spills at 256 and with FP64
// storage, 240^3 146 -> 123; FP64 storage loses, 256^3 244 -> 268).
template <int N, typename S>
constexpr bool xi_half() {
  return sizeof(S) == 4 && half_plan<N, 3 * x_rows(N), pick_T(max_nb(N, 3 * x_rows(N)))>();
}
template <int N, typename S, bool ACC>
constexpr int xi_waves() {
  return ACC ? 1 : xi_half<N, S>() ? (N < 256 ? 4 : 1) : sizeof(S) == 4 ? min_waves<N>() : 1;
}

// SWAP (with ACC): the stress replaces the one in sig, and the total it is part
// of is renewed with it, total = (total - old) + new.
template <int N, typename S, bool ACC, bool BG, bool BATCH = false, bool MASK = false, bool SWAP = false>
__global__ __launch_bounds__(pick_T(max_nb(N, 3 * x_rows(N))))
__attribute__((amdgpu_waves_per_eu(xi_waves<N, S, ACC>()))) void k_x_inverse(
    const typename Cplx<S>::T* __restrict__ spec, double* __restrict__ sig, const double* __restrict__ mean6,
    const double2* __restrict__ twg, const double* __restrict__ bg, int bg_mask,
    const HopJob* __restrict__ jobs = nullptr, const double* add3 = nullptr,
    const int32_t* __restrict__ own = nullptr, int32_t keep = -1, double* total = nullptr) {
  constexpr int ROWS = x_rows(N);
  constexpr int NF = 3 * ROWS;
  constexpr int T = pick_T(max_nb(N, NF));
  constexpr int LDN = N + N / 16 + 1;
  constexpr int P = spec_pitch(N, sizeof(S) == 8);
  constexpr int N3 = N * N * N;
  static_assert(6LL * N * N * P < (1LL << 31) && 6LL * N3 < (1LL << 31), "32-bit element offsets");
  constexpr bool HALF = xi_half<N, S>();
  __shared__ std::conditional_t<HALF, double, double2> buf[NF * LDN];
  __shared__ double2 tw[N];
  __shared__ double mean_s[6];
  for (int i = threadIdx.x; i < N; i += T) tw[i] = twg[i];
  if (threadIdx.x < 6) mean_s[threadIdx.x] = mean6[threadIdx.x];
  const int bpp = N / ROWS;
  int blk = blockIdx.x;
  if constexpr (BATCH) {
    const int j = blk / (N * bpp);
    blk -= j * (N * bpp);
    spec = (const typename Cplx<S>::T*)jobs[j].spec;
    sig = jobs[j].sig;
  }
  const int z = blk / bpp;
  const int y0 = (blk % bpp) * ROWS;
  const double scale = 1.0 / (double)N3;
  __syncthreads();
  auto load0 = [&](int f, int k) -> double2 {
    const int p = f % 3, y = y0 + f / 3;
    // components 2p and 2p+1 of bin k (or of its mirror n - k) are adjacent
    const typename Cplx<S>::T* a = spec + ((z * N + y) * P + (k <= N / 2 ? k : N - k)) * 6 + 2 * p;
    double2 A = ld2(a), B = ld2(a + 1);
    if (k > N / 2) {
      A = conjd(A);
      B = conjd(B);
    } else if (k == 0 || (N % 2 == 0 && k == N / 2)) {  // bins that are their own mirror
      A.y = 0.0;
      B.y = 0.0;
    }
    return make_double2(A.x - B.y, A.y + B.x);
  };
  // sigma is voxel-major, [n^3][6]: components 2p and 2p+1 of a voxel are one
  // aligned 16-byte pair, and the lanes of a store cover whole voxel records
  auto sig_at = [&](int f, int x) -> double2* {
    const int p = f % 3, y = y0 + f / 3;
    return reinterpret_cast<double2*>(sig + (6 * ((z * N + y) * N + x) + 2 * p));
  };
  auto add_at = [&](int f, int x) -> double2 {
    const int p = f % 3, y = y0 + f / 3;
    return *reinterpret_cast<const double2*>((add3 ? add3 : sig) + (6 * ((z * N + y) * N + x) + 2 * p));
  };
  // accumulate: the thread's old values of the last stage's outputs are read
  // before the transform, so their latency overlaps it
  constexpr Plan2 PLX = plan_of(N);
  constexpr int RL = PLX.r[PLX.nstage - 1];
  constexpr int NSL = PLX.nstage == 1 ? 1 : (PLX.nstage == 2 ? PLX.r[0] : PLX.r[0] * PLX.r[1]);
  constexpr int NOUT = ((NF * (N / RL) + T - 1) / T) * RL;
  double2 old[ACC ? NOUT : 1];
  static_assert(NOUT <= 64, "one bit per output");
  uint64_t covered = 0;  // bit per output: some defect covers its voxel
  if constexpr (MASK) {
    int32_t ow[NOUT];
    for_outputs<N, RL, NSL, Map::Row, NF, T>([&](int f, int x, int slot) {
      // keep = 0 (every voxel): the loads all read the map's first entry, one
      // cached line, instead of the whole map
      ow[slot] = own[((z * N + y0 + f / 3) * N + x) & keep] & keep;
    });
    for_outputs<N, RL, NSL, Map::Row, NF, T>(
        [&](int, int, int slot) { covered |= (uint64_t)(ow[slot] != -1) << slot; });
    // rows that no defect covers store nothing: their transform is skipped
    if (!__syncthreads_or(covered != 0)) return;
  }
  if constexpr (ACC)
    for_outputs<N, RL, NSL, Map::Row, NF, T>([&](int f, int x, int slot) {
      if (!MASK || (covered >> slot & 1))
      {
        old[slot] = add_at(f, x);
        if constexpr (SWAP) {  // the total without the old stress
          const int p = f % 3, y = y0 + f / 3;
          const double2 t = *reinterpret_cast<const double2*>(total + (6 * ((z * N + y) * N + x) + 2 * p));
          old[slot] = make_double2(t.x - old[slot].x, t.y - old[slot].y);
        }
      } else
        old[slot] = make_double2(0.0, 0.0);
    });
  auto store_last = [&](int f, int x, double2 v, int slot) {
    if constexpr (MASK)
      if (!(covered >> slot & 1)) return;
    const int p = f % 3, y = y0 + f / 3;
    double2* s01 = sig_at(f, x);
    double2 r = make_double2(v.x * scale + mean_s[2 * p], v.y * scale + mean_s[2 * p + 1]);
    if constexpr (SWAP) {
      const double2 o = old[slot];
      *reinterpret_cast<double2*>(total + (6 * ((z * N + y) * N + x) + 2 * p)) = make_double2(o.x + r.x, o.y + r.y);
    } else if constexpr (ACC) {
      const double2 o = old[slot];
      r.x += o.x;
      r.y += o.y;
    }
    if constexpr (BG) {
      const int v[3] = {x, y, z};
      for (int a = 0; a < 3; ++a) {
        if (!(bg_mask & (1 << a))) continue;
        const int a1 = a == 0 ? 1 : 0, a2 = a == 2 ? 1 : 2;
        const double2 o = *reinterpret_cast<const double2*>(bg + ((a * N + v[a2]) * N + v[a1]) * 6 + 2 * p);
        r.x += o.x;
        r.y += o.y;
      }
    }
    *s01 = r;
  };
  if constexpr (HALF) {
    transform_half<N, true, Map::Row, NF, T>((const double2*)tw, load0,
                                             [&](int f, int i) { return &buf[f * LDN + i + (i >> 4)]; }, store_last);
  } else {
    auto from_lds = [&](int f, int i) { return buf[f * LDN + i + (i >> 4)]; };
    auto to_lds = [&](int f, int i, double2 v) { buf[f * LDN + i + (i >> 4)] = v; };
    transform<N, true, Map::Row, NF, T>(tw, load0, from_lds, to_lds, store_last);
  }
}

// ------------------------------------------------------------------ launchers

// Grid of a tile-loop kernel, a multiple of eight.  Kernels that prefetch the
// next tile (FP32 storage) get as many workgroups as stay resident; the others
// get one tile per workgroup, so tiles overlap through the hardware scheduler.
template <class K>
int tile_grid(K kernel, int threads, int ntiles, bool prefetch) {
  if (!prefetch) return ((ntiles + 7) / 8) * 8;
  int dev = 0, ncu = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess)
    return -1;
  const int g = std::min(ncu * std::max(per_cu, 1), ntiles);
  return std::max(8, (g / 8) * 8);
}

// Grid of a kernel that prefetches its next tile, and whether it walks tiles
// claimed from counters: as many workgroups as stay resident, where each then
// has several tiles to walk; else one workgroup per tile (no counters), since
// claiming two tiles ahead leaves part of the chip idle.  Both y passes of a
// solve, us with / without walking, and tiles per resident workgroup: 64^3 51 /
// 18 (1), 96^3 95 / 27 (2), 128^3 119 / 42 (6), 160^3 125 / 72 (7), 240^3 291 / 357
// (29), 256^3 306 / 374 (33).
template <class K>
int walk_grid(K kernel, int threads, int ntiles, bool& walk) {
  const int g = tile_grid(kernel, threads, ntiles, true);
  walk = ntiles >= 16 * g;
  return g < 0 || walk ? g : ((ntiles + 7) / 8) * 8;
}

template <int N, typename S>
hipError_t go_xf(const int32_t* own, const int2* lnk, const DevDefect* defs, int ndef, const double* dense,
                 void* spec, SpecGeom g, const double2* tw, uint32_t* zero_ctr, hipStream_t s) {
  constexpr int T = pick_T(max_nb(N, 3 * x_rows(N)));
  static_assert(T >= NTILECTR, "the first block zeroes the tile counters");
  const int ngroups = N * (N / x_rows(N));
  using C2 = typename Cplx<S>::T;
  // as many workgroups as stay resident (a multiple of eight), at most one
  // per row group
  const int grid = tile_grid(k_x_forward<N, S, 0>, T, ngroups, true);
  if (grid < 0) return hipErrorInvalidValue;
  if (dense)
    hipLaunchKernelGGL((k_x_forward<N, S, 1>), dim3(grid), dim3(T), 0, s, own, lnk, defs, dense, (C2*)spec, g.P, tw,
                       zero_ctr, ndef);
  else
    hipLaunchKernelGGL((k_x_forward<N, S, 0>), dim3(grid), dim3(T), 0, s, own, lnk, defs, dense, (C2*)spec, g.P,
                       tw, zero_ctr, ndef);
  return hipGetLastError();
}

template <int N>
hipError_t go_xr(const int32_t* own, const int2* lnk, const DevDefect* defs, int ndef, const double* vals, int stride,
                 double2* spec, SpecGeom g, const double2* tw, uint32_t* zero_ctr, hipStream_t s) {
  if (g.P != spec_pitch(N, true)) return hipErrorInvalidValue;
  const int grid = (((N * N + 3) / 4 + 7) / 8) * 8;
  hipLaunchKernelGGL(k_x_forward_rows<N>, dim3(grid), dim3(256), 0, s, own, lnk, defs, vals, stride, spec, tw,
                     zero_ctr, ndef);
  return hipGetLastError();
}

template <int N, typename S>
hipError_t go_xf_vm(const double* vm, void* spec, SpecGeom g, const double2* tw, hipStream_t s) {
  constexpr int T = pick_T(max_nb(N, 3 * x_rows(N)));
  const int grid = tile_grid(k_x_forward<N, S, 2>, T, N * (N / x_rows(N)), true);
  if (grid < 0 || g.P != spec_pitch(N, sizeof(S) == 8)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_x_forward<N, S, 2>), dim3(grid), dim3(T), 0, s, (const int32_t*)nullptr,
                     (const int2*)nullptr, (const DevDefect*)nullptr, vm, (typename Cplx<S>::T*)spec, g.P, tw,
                     (uint32_t*)nullptr, 0);
  return hipGetLastError();
}

template <int N, typename S>
hipError_t go_xfs(const int32_t* oi, const int32_t* oc, const int32_t* ni, int nc, int sx, int sy, int sz,
                  const MoveStrain& E, void* spec, SpecGeom g, int ylo, int ylen, int zlo, int zlen, const double2* tw, uint32_t* zero_ctr,
                  hipStream_t s) {
  constexpr int T = pick_T(max_nb(N, 3 * x_rows(N)));
  static_assert(T >= NTILECTR, "the first block zeroes the tile counters");
  const int grid = zlen * ((ylen + x_rows(N) - 1) / x_rows(N));
  if (grid == 0) return zero_ctr ? launch_fill_i32((int32_t*)zero_ctr, NTILECTR, 0, s) : hipSuccess;
  hipLaunchKernelGGL((k_x_forward_sparse<N, S>), dim3(grid), dim3(T), 0, s, oi, oc, ni, nc, sx, sy, sz, E,
                     (typename Cplx<S>::T*)spec, g.P, ylo, ylen, zlo, tw, zero_ctr);
  return hipGetLastError();
}

// FP32 storage stages the inter-stage exchange in FP32 (half the LDS, so
// twice the columns per tile); FP64 storage keeps FP64 staging.
template <int N, typename S>
hipError_t go_pencil(bool inv, int axis, void* spec, SpecGeom g, Prune pr, const double2* tw, uint32_t* ctr,
                     hipStream_t s) {
  using LT = typename Cplx<S>::T;
  constexpr int T = pencil_threads<N, LT>();
  constexpr int KB = (N / 2 + 1 + pencil_wx<N, LT>() - 1) / pencil_wx<N, LT>();
  const int nouter = axis == 1 ? pr.z_len : N;
  const int ntiles = nouter * KB;
  using C2 = typename Cplx<S>::T;
  const bool prune = pr.in_len < N;
  if (g.P != spec_pitch(N, sizeof(S) == 8) || (axis != 1 && axis != 2)) return hipErrorInvalidValue;
  if (axis == 2 && prune) return hipErrorInvalidValue;  // z pruning runs in the fused z pass
  auto* k = axis == 1 ? (inv ? (prune ? k_pencil<N, S, true, LT, true, 1> : k_pencil<N, S, true, LT, false, 1>)
                             : (prune ? k_pencil<N, S, false, LT, true, 1> : k_pencil<N, S, false, LT, false, 1>))
                      : (inv ? k_pencil<N, S, true, LT, false, 2> : k_pencil<N, S, false, LT, false, 2>);
  bool walk = false;
  const int grid = pencil_pipe<N, S>() ? walk_grid(k, T, ntiles, walk) : tile_grid(k, T, ntiles, false);
  if (grid < 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(grid), dim3(T), 0, s, (C2*)spec, pr, tw, ntiles, walk ? ctr : nullptr,
                     (const HopJob*)nullptr, 0);
  return hipGetLastError();
}

template <int N, typename S, bool ACC, bool BG>
void go_xi_k(const void* spec, double* sig, const double* mean6, const double2* tw, const double* bg, int bg_mask,
             const double* add3, const int32_t* own, bool all, hipStream_t s) {
  constexpr int T = pick_T(max_nb(N, 3 * x_rows(N)));
  const int grid = N * (N / x_rows(N));
  using C2 = typename Cplx<S>::T;
  // with an owner map: the covered voxels, or all of them (all) by the same code
  if (own)
    hipLaunchKernelGGL((k_x_inverse<N, S, ACC, BG, false, true>), dim3(grid), dim3(T), 0, s, (const C2*)spec, sig,
                       mean6, tw, bg, BG ? bg_mask : 0, (const HopJob*)nullptr, add3, own, all ? 0 : -1);
  else
    hipLaunchKernelGGL((k_x_inverse<N, S, ACC, BG>), dim3(grid), dim3(T), 0, s, (const C2*)spec, sig, mean6, tw, bg,
                       BG ? bg_mask : 0, (const HopJob*)nullptr, add3);
}

template <int N, typename S>
hipError_t go_xi(bool acc, const void* spec, double* sig, SpecGeom g, const double* mean6, const double2* tw,
                 const double* bg, int bg_mask, const double* add3, const int32_t* own, bool all, hipStream_t s) {
  if (g.P != spec_pitch(N, sizeof(S) == 8) || (acc && add3) || (acc && own)) return hipErrorInvalidValue;
  if (add3 && bg && bg_mask)
    go_xi_k<N, S, true, true>(spec, sig, mean6, tw, bg, bg_mask, add3, own, all, s);
  else if (acc || add3)
    go_xi_k<N, S, true, false>(spec, sig, mean6, tw, bg, 0, add3, own, all, s);
  else if (bg && bg_mask)
    go_xi_k<N, S, false, true>(spec, sig, mean6, tw, bg, bg_mask, nullptr, own, all, s);
  else
    go_xi_k<N, S, false, false>(spec, sig, mean6, tw, bg, 0, nullptr, own, all, s);
  return hipGetLastError();
}

template <int N, typename S>
hipError_t go_xi_swap(const void* spec, double* part, double* total, SpecGeom g, const double* mean6,
                      const double2* tw, hipStream_t s) {
  constexpr int T = pick_T(max_nb(N, 3 * x_rows(N)));
  if (g.P != spec_pitch(N, sizeof(S) == 8)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_x_inverse<N, S, true, false, false, false, true>), dim3(N * (N / x_rows(N))), dim3(T), 0, s,
                     (const typename Cplx<S>::T*)spec, part, mean6, tw, (const double*)nullptr, 0,
                     (const HopJob*)nullptr, (const double*)nullptr, (const int32_t*)nullptr, 0, total);
  return hipGetLastError();
}

template <int N, typename S>
hipError_t go_hop_batch(const HopJob* jobs, int njob, SpecGeom g, Cubic C, const double2* tw, uint32_t* ctr,
                        const double* zero6, hipStream_t s) {
  using C2 = typename Cplx<S>::T;
  using LT = typename Cplx<S>::T;
  if (g.P != spec_pitch(N, sizeof(S) == 8) || njob < 1 || njob > MAXBATCH) return hipErrorInvalidValue;
  constexpr bool pipe = pencil_pipe<N, S>(), zpipe = zg_pipe<N, S>();
  constexpr int TX = pick_T(max_nb(N, 3 * x_rows(N)));
  // sparse x forward: a fixed grid walks the row blocks of every job
  hipLaunchKernelGGL((k_x_forward_sparse_batch<N, S>), dim3(256), dim3(TX), 0, s, jobs, njob, g.P, tw, ctr);
  // y forward (pruned planes and rows), fused z pass, y inverse: persistent
  // grids over the jobs' tiles
  constexpr int TP = pencil_threads<N, LT>();
  constexpr int KB = (N / 2 + 1 + pencil_wx<N, LT>() - 1) / pencil_wx<N, LT>();
  const Prune none{0, N, 0, N};
  {
    // the tiles of the jobs' pruned planes, few per resident workgroup, in a
    // fixed order
    auto* k = k_pencil<N, S, false, LT, true, 1, true>;
    const int grid = tile_grid(k, TP, njob * N * KB, pipe);
    if (grid < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(grid), dim3(TP), 0, s, (C2*)nullptr, none, tw, 0, (uint32_t*)nullptr, jobs, njob);
  }
  {
    bool done = false;
    if constexpr (zg_half<N>()) {
      if (!C.frm) {  // the same kernel as a single hop's pass
        const int nt = njob * N * ((N / 2 + 2) / 2);
        hipLaunchKernelGGL((k_zgreen_half<N, S, true, true>), dim3(((nt + 7) / 8) * 8), dim3(zh_threads<N>()), 0, s,
                           (C2*)nullptr, C, none, tw, jobs, njob);
        done = true;
      }
    }
    if (!done) {
      constexpr int W = zg_width<N, S>();
      constexpr int T = zg_threads<N, S>();
      constexpr int NT = N * ((N / 2 + 1 + W - 1) / W);
      auto* k = C.frm ? k_zgreen<N, S, true, true, true> : k_zgreen<N, S, true, false, true>;
      bool walk = false;
      const int grid = zpipe ? walk_grid(k, T, njob * NT, walk) : tile_grid(k, T, njob * NT, false);
      if (grid < 0) return hipErrorInvalidValue;
      hipLaunchKernelGGL(k, dim3(grid), dim3(T), 0, s, (C2*)nullptr, C, none, tw, walk ? ctr + 8 : nullptr, jobs, njob);
    }
  }
  {
    auto* k = k_pencil<N, S, true, LT, false, 1, true>;
    bool walk = false;
    const int grid = pipe ? walk_grid(k, TP, njob * N * KB, walk) : tile_grid(k, TP, njob * N * KB, false);
    if (grid < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(grid), dim3(TP), 0, s, (C2*)nullptr, none, tw, 0, walk ? ctr + 16 : nullptr, jobs,
                       njob);
  }
  // accumulating x inverse (a hop's mean-stress change is zero)
  hipLaunchKernelGGL((k_x_inverse<N, S, true, false, true>), dim3(njob * N * (N / x_rows(N))), dim3(TX), 0, s,
                     (const C2*)nullptr, (double*)nullptr, zero6, tw, (const double*)nullptr, 0, jobs);
  return hipGetLastError();
}

}  // namespace

#define EC_FOR_SIZES(X) X(8) X(16) X(24) X(32) X(45) X(48) X(64) X(96) X(128) X(129) X(160) X(240) X(256) X(512)

bool fft_supported(int n) {
  switch (n) {
#define EC_CASE(NN) case NN:
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
    return true;
    default:
      return false;
  }
}

bool direct_length(int n) { return has_direct(plan_of(n)); }

// Up to this part of the cell's voxels the direct row sums of the x forward
// pass beat its transforms.  The sums cost a fixed share per covered voxel, the
// transforms nothing more: us for the pass with rows / with transforms, at 0.5,
// 2.1 and 4.2 % covered: 256^3 188 / 222, 222 / 236, 234 / 260; at 3.2 % of
// 240^3 204 / 225; past that the transforms win (6.4 % of 160^3: 65 / 61, 21 %
// of 128^3: 50 / 42).  Where the transform has a direct large radix the sums win
// by far (129^3: 19 / 116 at 0.6 %; balls of 12 voxels: 35 / 117 at 5 % of the
// cell, 66 / 125 at 20, 98 / 137 at 40, 123 / 151 at 55, 140 / 160 at 70, 193 / 177
// at 100, overlaps counted once per ball).
double rows_limit(int n) { return direct_length(n) ? 0.5 : 0.04; }

int pencil_width(int n, bool) { return n >= 512 ? 8 : 16; }

hipError_t launch_x_forward(bool fp64, const int32_t* own, const int2* lnk, const DevDefect* defs, int ndef,
                            const double* dense, void* spec, SpecGeom g, const double2* tw, uint32_t* zero_ctr,
                            hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN)                                                                     \
  case NN:                                                                              \
    return fp64 ? go_xf<NN, double>(own, lnk, defs, ndef, dense, spec, g, tw, zero_ctr, s) \
                : go_xf<NN, float>(own, lnk, defs, ndef, dense, spec, g, tw, zero_ctr, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

static hipError_t x_rows_of(const int32_t* own, const int2* lnk, const DevDefect* defs, int ndef, const double* vals,
                            int stride, double2* spec, SpecGeom g, const double2* tw, uint32_t* zero_ctr,
                            hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN) \
  case NN:          \
    return go_xr<NN>(own, lnk, defs, ndef, vals, stride, spec, g, tw, zero_ctr, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_x_forward_rows(const int32_t* own, const int2* lnk, const DevDefect* defs, int ndef, double2* spec,
                                 SpecGeom g, const double2* tw, uint32_t* zero_ctr, hipStream_t s) {
  static_assert(sizeof(DevDefect) % 16 == 0 && offsetof(DevDefect, efd) % 16 == 0, "16-byte loads of efd");
  return x_rows_of(own, lnk, defs, ndef, reinterpret_cast<const double*>(defs) + offsetof(DevDefect, efd) / 8,
                   (int)(sizeof(DevDefect) / 8), spec, g, tw, zero_ctr, s);
}

hipError_t launch_x_forward_points(const int32_t* map, const double* vals, int stride, double2* spec, SpecGeom g,
                                   const double2* tw, hipStream_t s) {
  return x_rows_of(map, nullptr, nullptr, 0, vals, stride, spec, g, tw, nullptr, s);
}

hipError_t launch_x_forward_vm(bool fp64, const double* vm, void* spec, SpecGeom g, const double2* tw, hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN) \
  case NN:          \
    return fp64 ? go_xf_vm<NN, double>(vm, spec, g, tw, s) : go_xf_vm<NN, float>(vm, spec, g, tw, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_x_forward_sparse(bool fp64, const int32_t* old_ids, const int32_t* old_cnt, const int32_t* new_ids,
                                   int new_cnt, int sx, int sy, int sz, const MoveStrain& E, void* spec, SpecGeom g,
                                   int y_lo, int y_len, int z_lo, int z_len, const double2* tw, uint32_t* zero_ctr,
                                   hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN)                                                                                          \
  case NN:                                                                                                   \
    return fp64 ? go_xfs<NN, double>(old_ids, old_cnt, new_ids, new_cnt, sx, sy, sz, E, spec, g, y_lo, y_len, \
                                     z_lo, z_len, tw, zero_ctr, s)                                            \
                : go_xfs<NN, float>(old_ids, old_cnt, new_ids, new_cnt, sx, sy, sz, E, spec, g, y_lo, y_len,  \
                                    z_lo, z_len, tw, zero_ctr, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pencil(bool fp64, bool inv, int axis, void* spec, SpecGeom g, Prune pr, const double2* tw,
                         uint32_t* ctr, hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN)                                                        \
  case NN:                                                                 \
    return fp64 ? go_pencil<NN, double>(inv, axis, spec, g, pr, tw, ctr, s) \
                : go_pencil<NN, float>(inv, axis, spec, g, pr, tw, ctr, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_green(bool fp64, void* spec, SpecGeom g, Cubic C, hipStream_t s) {
  const size_t bins = (size_t)g.n * g.n * (g.n / 2 + 1);
  const int grid = (int)((bins + 255) / 256);
  if (fp64)
    hipLaunchKernelGGL(k_green<double>, dim3(grid), dim3(256), 0, s, (double2*)spec, g.n, g.P, C);
  else
    hipLaunchKernelGGL(k_green<float>, dim3(grid), dim3(256), 0, s, (float2*)spec, g.n, g.P, C);
  return hipGetLastError();
}

template <int N, typename S>
hipError_t go_zgreen(void* spec, SpecGeom g, Cubic C, Prune pr, const double2* tw, uint32_t* ctr, bool solve,
                     hipStream_t s) {
  constexpr int W = zg_width<N, S>();
  constexpr int T = zg_threads<N, S>();
  constexpr int NT = N * ((N / 2 + 1 + W - 1) / W);
  using C2 = typename Cplx<S>::T;
  const bool prune = pr.in_len < N;
  if (g.P != spec_pitch(N, sizeof(S) == 8)) return hipErrorInvalidValue;
  if constexpr (zg_half<N>()) {
    if (!C.frm && (sizeof(S) == 8 || !solve)) {
      constexpr int NTH = N * ((N / 2 + 2) / 2);
      auto* k = prune ? k_zgreen_half<N, S, true> : k_zgreen_half<N, S, false>;
      hipLaunchKernelGGL(k, dim3(((NTH + 7) / 8) * 8), dim3(zh_threads<N>()), 0, s, (C2*)spec, C, pr, tw,
                         (const HopJob*)nullptr, 0);
      return hipGetLastError();
    }
  }
  auto* k = C.frm ? (prune ? k_zgreen<N, S, true, true> : k_zgreen<N, S, false, true>)
                  : (prune ? k_zgreen<N, S, true, false> : k_zgreen<N, S, false, false>);
  bool walk = false;
  const int grid = zg_pipe<N, S>() ? walk_grid(k, T, NT, walk) : tile_grid(k, T, NT, false);
  if (grid < 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(grid), dim3(T), 0, s, (C2*)spec, C, pr, tw, walk ? ctr : nullptr, (const HopJob*)nullptr,
                     0);
  return hipGetLastError();
}

hipError_t launch_z_green(bool fp64, void* spec, SpecGeom g, Cubic C, Prune pr, const double2* tw, uint32_t* ctr,
                          bool solve, hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN)                                                      \
  case NN:                                                               \
    return fp64 ? go_zgreen<NN, double>(spec, g, C, pr, tw, ctr, solve, s)      \
                : go_zgreen<NN, float>(spec, g, C, pr, tw, ctr, solve, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_hop_batch_fft(bool fp64, const HopJob* jobs, int njob, SpecGeom g, Cubic C, const double2* tw,
                                uint32_t* ctr, const double* zero6, hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN)                                                                  \
  case NN:                                                                           \
    return fp64 ? go_hop_batch<NN, double>(jobs, njob, g, C, tw, ctr, zero6, s)     \
                : go_hop_batch<NN, float>(jobs, njob, g, C, tw, ctr, zero6, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_x_inverse(bool fp64, bool accum, const void* spec, double* sig, SpecGeom g, const double* mean6,
                            const double2* tw, hipStream_t s, const double* bg, int bg_mask, const double* add3,
                            const int32_t* own, bool all) {
  switch (g.n) {
#define EC_CASE(NN)                                                                              \
  case NN:                                                                                       \
    return fp64 ? go_xi<NN, double>(accum, spec, sig, g, mean6, tw, bg, bg_mask, add3, own, all, s) \
                : go_xi<NN, float>(accum, spec, sig, g, mean6, tw, bg, bg_mask, add3, own, all, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_x_inverse_swap(bool fp64, const void* spec, double* part, double* total, SpecGeom g,
                                 const double* mean6, const double2* tw, hipStream_t s) {
  switch (g.n) {
#define EC_CASE(NN)                                                              \
  case NN:                                                                       \
    return fp64 ? go_xi_swap<NN, double>(spec, part, total, g, mean6, tw, s)     \
                : go_xi_swap<NN, float>(spec, part, total, g, mean6, tw, s);
    EC_FOR_SIZES(EC_CASE)
#undef EC_CASE
  }
  return hipErrorInvalidValue;
}

// ------------------------------------------------------ dislocation lines (Sec. 3.1)
//
// A straight line along cell axis a is uniform along a, so its Nye tensor,
// plastic distortion and stress live on the plane k_a = 0 of the spectrum.
// Per bin (k1, k2) over the other two axes (a1 < a2): rho_hat of each spread
// line (bilinear weights over the four grid points around it, density 1/h^2),
// the distortion U_hat_ij = -i xi_k / xi^2 e_jkl b_i t_l rho_hat (Nyquist bins:
// the mean over the all -n/2 and all +n/2 representatives, the real part of the
// centred solution), eps*_hat = sym(U_hat) summed over the lines, then the Green
// step of the bin (the operator is even in xi, so a bin past n/2 along x uses its
// mirror in the half-spectrum indexing of green_bin).
__global__ __launch_bounds__(256) void k_disl_spectrum(const DevLine* __restrict__ lines, int nl, int axis, int n,
                                                       double L, Cubic C, double2* __restrict__ out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int nn = n * n;
  if (t >= nn) return;
  const int a1 = axis == 0 ? 1 : 0, a2 = axis == 2 ? 1 : 2;
  const int k1 = t % n, k2 = t / n;
  int kb[3];
  kb[axis] = 0;
  kb[a1] = k1;
  kb[a2] = k2;
  const int hn = n / 2;
  const double s2pi = 2.0 * M_PI / L;
  double2 e[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) e[c] = make_double2(0.0, 0.0);
  if (k1 != 0 || k2 != 0) {
    // the representatives of the bin: one, or two for a Nyquist bin
    double lab[2][3];
    bool nyq = false;
    for (int d = 0; d < 3; ++d) {
      const int k = kb[d];
      const bool ny = nyquist(k, n);
      nyq |= ny;
      lab[0][d] = ny ? -hn : centred(k, n);
      lab[1][d] = ny ? hn : lab[0][d];
    }
    const int nrep = nyq ? 2 : 1;
    const double h = L / n;
    for (int li = 0; li < nl; ++li) {
      const DevLine ln = lines[li];
      // rho_hat = sum_c w_c exp(-2 pi i (k1 i1 + k2 i2) / n) / h^2
      const double f1 = floor(ln.u1), f2 = floor(ln.u2);
      double2 rho = make_double2(0.0, 0.0);
      for (int c1 = 0; c1 < 2; ++c1)
        for (int c2 = 0; c2 < 2; ++c2) {
          const double w = (1.0 - fabs(ln.u1 - (f1 + c1))) * (1.0 - fabs(ln.u2 - (f2 + c2)));
          if (w == 0.0) continue;
          const int64_t i1 = (((int64_t)f1 + c1) % n + n) % n, i2 = (((int64_t)f2 + c2) % n + n) % n;
          const int64_t m = ((int64_t)k1 * i1 + (int64_t)k2 * i2) % n;
          double sn, cs;
          sincospi(-2.0 * (double)m / n, &sn, &cs);
          rho.x += w * cs;
          rho.y += w * sn;
        }
      rho.x /= h * h;
      rho.y /= h * h;
      // F = mean over the representatives of (xi x t) / xi^2
      double F[3] = {0.0, 0.0, 0.0};
      for (int r = 0; r < nrep; ++r) {
        const double x0 = s2pi * lab[r][0], x1 = s2pi * lab[r][1], x2 = s2pi * lab[r][2];
        const double q = 1.0 / ((x0 * x0 + x1 * x1 + x2 * x2) * nrep);
        F[0] += (x1 * ln.t[2] - x2 * ln.t[1]) * q;
        F[1] += (x2 * ln.t[0] - x0 * ln.t[2]) * q;
        F[2] += (x0 * ln.t[1] - x1 * ln.t[0]) * q;
      }
      // w = -i F rho
      double2 w[3];
      for (int j = 0; j < 3; ++j) w[j] = make_double2(F[j] * rho.y, -F[j] * rho.x);
      const double* b = ln.b;
      e[0].x += b[0] * w[0].x;
      e[0].y += b[0] * w[0].y;
      e[1].x += b[1] * w[1].x;
      e[1].y += b[1] * w[1].y;
      e[2].x += b[2] * w[2].x;
      e[2].y += b[2] * w[2].y;
      e[3].x += 0.5 * (b[1] * w[2].x + b[2] * w[1].x);
      e[3].y += 0.5 * (b[1] * w[2].y + b[2] * w[1].y);
      e[4].x += 0.5 * (b[0] * w[2].x + b[2] * w[0].x);
      e[4].y += 0.5 * (b[0] * w[2].y + b[2] * w[0].y);
      e[5].x += 0.5 * (b[0] * w[1].x + b[1] * w[0].x);
      e[5].y += 0.5 * (b[0] * w[1].y + b[1] * w[0].y);
    }
    int gx = kb[0], gy = kb[1], gz = kb[2];
    if (gx > hn) {
      gx = n - gx;
      gy = (n - gy) % n;
      gz = (n - gz) % n;
    }
    if (C.frm)
      green_bin_rot(e, gx, gy, gz, n, C);
    else
      green_bin(e, gx, gy, gz, n, C);
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) out[(size_t)c * nn + t] = e[c];
}

// One direction of the inverse 2-D transform by direct sums (exact phase
// reduction, m = k i mod n): DIM 0 over k1 (in [c][k2][k1] -> out [c][k2][i1]),
// DIM 1 over k2 with the 1/n^2 scale and the real part into plane [i2 * n + i1][c].
template <int DIM>
__global__ __launch_bounds__(256) void k_disl_idft(const double2* __restrict__ in, int n, double2* __restrict__ out,
                                                   double* __restrict__ plane) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int nn = n * n;
  if (t >= 6 * nn) return;
  const int c = t / nn, r = t % nn;
  const int i = r % n, o = r / n;  // output index along the transformed axis, the other axis
  double2 acc = make_double2(0.0, 0.0);
  for (int k = 0; k < n; ++k) {
    const double2 v = DIM == 0 ? in[(size_t)c * nn + (size_t)o * n + k] : in[(size_t)c * nn + (size_t)k * n + o];
    const int64_t m = ((int64_t)k * i) % n;
    double sn, cs;
    sincospi(2.0 * (double)m / n, &sn, &cs);
    acc.x += v.x * cs - v.y * sn;
    acc.y += v.x * sn + v.y * cs;
  }
  if (DIM == 0)
    out[(size_t)c * nn + (size_t)o * n + i] = acc;
  else
    plane[((size_t)i * n + o) * 6 + c] = acc.x / ((double)n * n);
}

__global__ __launch_bounds__(256) void k_bg_add(double* __restrict__ sig, const double* __restrict__ planes, int mask,
                                                int n, double sgn) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nn = (int64_t)n * n;
  if (v >= nn * n) return;
  const int x[3] = {(int)(v % n), (int)((v / n) % n), (int)(v / nn)};
  double add[6] = {0, 0, 0, 0, 0, 0};
  for (int a = 0; a < 3; ++a) {
    if (!(mask & (1 << a))) continue;
    const int a1 = a == 0 ? 1 : 0, a2 = a == 2 ? 1 : 2;
    const double* p = planes + ((size_t)a * nn + (size_t)x[a2] * n + x[a1]) * 6;
    for (int c = 0; c < 6; ++c) add[c] += p[c];
  }
  double* q = sig + 6 * v;
  for (int c = 0; c < 6; ++c) q[c] += sgn * add[c];
}

// Dislocation paths in any direction (Sec. 3.1): sigma_hat (in e) of a bin of the
// half spectrum from the nine components alpha_hat_il of its Nye tensor,
// U_hat_ij = -i e_jkl xi_k alpha_hat_il / |xi|^2 (at an even n's Nyquist bins the
// mean over the all -n/2 and all +n/2 representatives), eps*_hat = sym(U_hat) and
// the Green step; zero at xi = 0.
__device__ __forceinline__ void path_bin(const double2* al, int kx, int ky, int kz, int n, double L, const Cubic& C,
                                         double2* e) {
#pragma unroll
  for (int c = 0; c < 6; ++c) e[c] = make_double2(0.0, 0.0);
  const int k[3] = {kx, ky, kz};
  if (kx != 0 || ky != 0 || kz != 0) {
    const bool nyq = nyquist(kx, n) || nyquist(ky, n) || nyquist(kz, n);
    const int nrep = nyq ? 2 : 1;
    const double s2pi = 2.0 * M_PI / L;
    double2 U[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) U[i][j] = make_double2(0.0, 0.0);
    for (int rep = 0; rep < nrep; ++rep) {
      double x[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int h = n / 2;
        x[a] = s2pi * (nyquist(k[a], n) ? (rep == 0 ? -h : h) : centred(k[a], n));
      }
      const double q = 1.0 / ((x[0] * x[0] + x[1] * x[1] + x[2] * x[2]) * nrep);
      // U_ij += -i (xi x alpha_i.)_j / |xi|^2, alpha_i. the row i of alpha_hat
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const double2 a0 = al[3 * i], a1 = al[3 * i + 1], a2 = al[3 * i + 2];
        const double2 c0 = make_double2(x[1] * a2.x - x[2] * a1.x, x[1] * a2.y - x[2] * a1.y);
        const double2 c1 = make_double2(x[2] * a0.x - x[0] * a2.x, x[2] * a0.y - x[0] * a2.y);
        const double2 c2 = make_double2(x[0] * a1.x - x[1] * a0.x, x[0] * a1.y - x[1] * a0.y);
        // -i c = (c.y, -c.x)
        U[i][0].x += q * c0.y;
        U[i][0].y -= q * c0.x;
        U[i][1].x += q * c1.y;
        U[i][1].y -= q * c1.x;
        U[i][2].x += q * c2.y;
        U[i][2].y -= q * c2.x;
      }
    }
    e[0] = U[0][0];
    e[1] = U[1][1];
    e[2] = U[2][2];
    e[3] = make_double2(0.5 * (U[1][2].x + U[2][1].x), 0.5 * (U[1][2].y + U[2][1].y));
    e[4] = make_double2(0.5 * (U[0][2].x + U[2][0].x), 0.5 * (U[0][2].y + U[2][0].y));
    e[5] = make_double2(0.5 * (U[0][1].x + U[1][0].x), 0.5 * (U[0][1].y + U[1][0].y));
    if (C.frm)
      green_bin_rot(e, kx, ky, kz, n, C);
    else
      green_bin(e, kx, ky, kz, n, C);
  }
}

// alpha_hat summed over the pieces at every bin, sum of M_il rho_hat with the
// trilinear spread of a piece separable per axis,
//   rho_hat = prod_a e^{-2 pi i k_a f_a / n} ((1 - fr_a) + fr_a e^{-2 pi i k_a / n}),
// the exponents reduced exactly (k_a f_a mod n) and read from the twiddle table.
// Pieces are staged in LDS in chunks; one thread per bin.
constexpr int PATH_CHUNK = 128;

template <typename S>
__global__ __launch_bounds__(256) void k_path_spectrum(const DevPiece* __restrict__ pieces, int np, int n, int P,
                                                       double L, Cubic C, const double2* __restrict__ tw,
                                                       typename Cplx<S>::T* __restrict__ spec) {
  __shared__ DevPiece sp[PATH_CHUNK];
  const int NH = n / 2 + 1;
  const int64_t bins = (int64_t)n * n * NH;
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = b < bins;
  const int kx = live ? (int)(b % NH) : 0;
  const int64_t r = live ? b / NH : 0;
  const int ky = (int)(r % n), kz = (int)(r / n);
  const int k[3] = {kx, ky, kz};
  double2 e1[3];  // e^{-2 pi i k_a / n}
#pragma unroll
  for (int a = 0; a < 3; ++a) e1[a] = tw[k[a]];
  double2 al[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) al[c] = make_double2(0.0, 0.0);
  for (int p0 = 0; p0 < np; p0 += PATH_CHUNK) {
    const int m = min(PATH_CHUNK, np - p0);
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += blockDim.x) sp[i] = pieces[p0 + i];
    __syncthreads();
    if (!live) continue;
    for (int i = 0; i < m; ++i) {
      const DevPiece& q = sp[i];
      double2 rho = make_double2(1.0, 0.0);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double2 ph = tw[(k[a] * q.f[a]) % n];
        const double w = q.fr[a];
        const double2 f = make_double2((1.0 - w) + w * e1[a].x, w * e1[a].y);
        const double2 t = make_double2(ph.x * f.x - ph.y * f.y, ph.x * f.y + ph.y * f.x);
        rho = make_double2(rho.x * t.x - rho.y * t.y, rho.x * t.y + rho.y * t.x);
      }
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        al[c].x += q.M[c] * rho.x;
        al[c].y += q.M[c] * rho.y;
      }
    }
  }
  if (!live) return;
  double2 e[6];
  path_bin(al, kx, ky, kz, n, L, C, e);
  typename Cplx<S>::T* const out = spec + spec_at(kz, ky, kx, 0, n, P);
#pragma unroll
  for (int c = 0; c < 6; ++c) st2(out + c, e[c]);
}

// The same spectrum for many pieces (launch_path_points): the spread Nye tensor
// is formed on the grid, transformed, and taken through the operator per bin,
// instead of summed piece by piece at every bin.
//
// One thread per piece and grid point around it.  The points in use get a
// record each (map: the voxel's record, claimed by whichever comes first);
// contributions, products rounded to FP64, are added there in fixed point, 2^-61
// of the largest piece's power of two, each value's low 32 bits and the rest in
// sums of their own: the sums are exact and do not depend on the order, and are
// rounded to FP64 once.
__global__ __launch_bounds__(256) void k_piece_points(const DevPiece* __restrict__ pieces, int np, int n, double scale,
                                                      int32_t* __restrict__ map, int64_t* __restrict__ sums) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= 8 * np) return;
  const DevPiece& q = pieces[t / 8];
  int v[3];
  double w = 1.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int up = (t >> a) & 1;
    v[a] = q.f[a] + up;
    v[a] -= v[a] >= n ? n : 0;
    w *= up ? q.fr[a] : 1.0 - q.fr[a];
  }
  if (w == 0.0) return;
  const int64_t id = ((int64_t)v[2] * n + v[1]) * n + v[0];
  const int32_t prev = atomicCAS(&map[id], -1, t);
  unsigned long long* rec = reinterpret_cast<unsigned long long*>(sums + (size_t)(prev == -1 ? t : prev) * 18);
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    const int64_t f = llrint(w * q.M[c] * scale);
    atomicAdd(&rec[2 * c], (unsigned long long)(f >> 32));
    atomicAdd(&rec[2 * c + 1], (unsigned long long)(uint32_t)f);
  }
}

// The records as doubles, twelve per record (the last three zero).
__global__ __launch_bounds__(256) void k_piece_values(const int64_t* __restrict__ sums, int nrec, double inv,
                                                      double* __restrict__ vals) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= 12 * nrec) return;
  const int r = t / 12, c = t % 12;
  const int64_t* s = sums + (size_t)r * 18 + 2 * c;
  vals[t] = c < 9 ? ((double)s[0] * 0x1p32 + (double)s[1]) * inv : 0.0;
}

// One thread per bin: the nine transformed components (six in a, three in b)
// to the stress spectrum.
template <typename S>
__global__ __launch_bounds__(256) void k_path_bins(const double2* __restrict__ a, const double2* __restrict__ b, int n,
                                                   int Pd, int P, double L, Cubic C,
                                                   typename Cplx<S>::T* __restrict__ spec) {
  const int NH = n / 2 + 1;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * n * NH) return;
  const int kx = (int)(t % NH);
  const int64_t r = t / NH;
  const int ky = (int)(r % n), kz = (int)(r / n);
  const size_t o = spec_at(kz, ky, kx, 0, n, Pd);
  double2 al[9], e[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) al[c] = a[o + c];
#pragma unroll
  for (int c = 0; c < 3; ++c) al[6 + c] = b[o + c];
  path_bin(al, kx, ky, kz, n, L, C, e);
  typename Cplx<S>::T* const out = spec + spec_at(kz, ky, kx, 0, n, P);
#pragma unroll
  for (int c = 0; c < 6; ++c) st2(out + c, e[c]);
}

__global__ __launch_bounds__(256) void k_bg3_add(double* __restrict__ sig, const double* __restrict__ bg3,
                                                 int64_t count, double sgn) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) sig[i] += sgn * bg3[i];
}

hipError_t launch_path_spectrum(bool fp64, const DevPiece* pieces, int np, SpecGeom g, double L, Cubic C,
                                const double2* tw, void* spec, hipStream_t s) {
  const int64_t bins = (int64_t)g.n * g.n * (g.n / 2 + 1);
  const int grid = (int)((bins + 255) / 256);
  if (fp64)
    hipLaunchKernelGGL(k_path_spectrum<double>, dim3(grid), dim3(256), 0, s, pieces, np, g.n, g.P, L, C, tw,
                       (double2*)spec);
  else
    hipLaunchKernelGGL(k_path_spectrum<float>, dim3(grid), dim3(256), 0, s, pieces, np, g.n, g.P, L, C, tw,
                       (float2*)spec);
  return hipGetLastError();
}

hipError_t launch_path_points(bool fp64, const DevPiece* pieces, int np, double scale, SpecGeom g, double L, Cubic C,
                              const double2* tw, char* scratch, void* spec, hipStream_t s) {
  const PathScratch o = path_scratch(g.n, np);
  const SpecGeom gd{g.n, spec_pitch(g.n, true)};
  double2* const sp[2] = {(double2*)(scratch + o.a), (double2*)(scratch + o.b)};
  int32_t* const map = (int32_t*)(scratch + o.map);
  int64_t* const sums = (int64_t*)(scratch + o.sums);
  double* const vals = (double*)(scratch + o.vals);
  const int nrec = 8 * np;
  hipError_t e = launch_fill_i32(map, (int64_t)g.n * g.n * g.n, -1, s);
  if (e == hipSuccess) e = launch_fill_i32((int32_t*)sums, (int64_t)nrec * 36, 0, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_piece_points, dim3((nrec + 255) / 256), dim3(256), 0, s, pieces, np, g.n, scale, map, sums);
  hipLaunchKernelGGL(k_piece_values, dim3((12 * nrec + 255) / 256), dim3(256), 0, s, sums, nrec, 1.0 / scale, vals);
  const Prune full{0, g.n, 0, g.n};
  for (int h = 0; h < 2; ++h) {
    if ((e = launch_x_forward_points(map, vals + 6 * h, 12, sp[h], gd, tw, s)) != hipSuccess ||
        (e = launch_pencil(true, false, 1, sp[h], gd, full, tw, nullptr, s)) != hipSuccess ||
        (e = launch_pencil(true, false, 2, sp[h], gd, full, tw, nullptr, s)) != hipSuccess)
      return e;
  }
  const int64_t bins = (int64_t)g.n * g.n * (g.n / 2 + 1);
  const int grid = (int)((bins + 255) / 256);
  if (fp64)
    hipLaunchKernelGGL(k_path_bins<double>, dim3(grid), dim3(256), 0, s, sp[0], sp[1], g.n, gd.P, g.P, L, C,
                       (double2*)spec);
  else
    hipLaunchKernelGGL(k_path_bins<float>, dim3(grid), dim3(256), 0, s, sp[0], sp[1], g.n, gd.P, g.P, L, C,
                       (float2*)spec);
  return hipGetLastError();
}

hipError_t launch_bg3_add(double* sig, const double* bg3, int64_t n3, double sgn, hipStream_t s) {
  const int64_t count = 6 * n3;
  hipLaunchKernelGGL(k_bg3_add, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, sig, bg3, count, sgn);
  return hipGetLastError();
}

hipError_t launch_disl_plane(const DevLine* lines, int nl, int axis, int n, double L, Cubic C, double2* spec,
                             double2* tmp, double* plane, hipStream_t s) {
  const int nn = n * n;
  hipLaunchKernelGGL(k_disl_spectrum, dim3((nn + 255) / 256), dim3(256), 0, s, lines, nl, axis, n, L, C, spec);
  hipLaunchKernelGGL(k_disl_idft<0>, dim3((6 * nn + 255) / 256), dim3(256), 0, s, (const double2*)spec, n, tmp,
                     (double*)nullptr);
  hipLaunchKernelGGL(k_disl_idft<1>, dim3((6 * nn + 255) / 256), dim3(256), 0, s, (const double2*)tmp, n,
                     (double2*)nullptr, plane);
  return hipGetLastError();
}

hipError_t launch_bg_add(double* sig, const double* planes, int mask, int n, double sgn, hipStream_t s) {
  const int64_t n3 = (int64_t)n * n * n;
  hipLaunchKernelGGL(k_bg_add, dim3((unsigned)((n3 + 255) / 256)), dim3(256), 0, s, sig, planes, mask, n, sgn);
  return hipGetLastError();
}

}  // namespace ec
