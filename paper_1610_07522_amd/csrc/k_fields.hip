// Mean field of the Skyrme functional from the local densities, the Coulomb
// potential solved in momentum space, and the total energy.
//
// Sec. 2.2: h = kinetic + Skyrme mean field (Eq. Skyrme) + Coulomb, with the
// Coulomb problem solved by FFTs; Fig. 1 step 4b.  The fields are small
// (a few n^3 arrays): a pass over one is a few hundred waves, bound by the
// latency of its loads and by launches.  A spectral first derivative (Nyquist
// zeroed) or second derivative of a real field along one axis is a real
// circulant on each grid line, so all of them are n-tap circular convolutions
// with known taps; the Coulomb transform is a direct DFT per axis with one
// thread per output element.  The loops over a line have compile-time lengths,
// so that a batch of loads is in flight, both species share a launch, and the
// z transform, the 1/k^2 and its inverse are one kernel (32^3: 10 launches and
// 105 us, now 7 and 53).
#include <cmath>

#include "sky_kernels.h"

namespace sky {

namespace {
constexpr int E_THREADS = 256;  // threads per energy-reduction block
constexpr int NTERM = 7;        // energy terms

__device__ inline double kval(int f, int n, double kunit) {
  return kunit * double(f < n / 2 ? f : f - n);
}

// Fields of both species, picked by blockIdx.y.
struct Species {
  const double* in[2];
  double* out[2];
};

// out = [lap rho, d rho/dx, d rho/dy, d rho/dz, div J] at every point of the
// densities in = [rho, tau, Jx, Jy, Jz, ...].
template <int N>
__global__ void __launch_bounds__(256)
k_field_derivs(Species sp, FieldTaps tab, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  constexpr int N2 = N * N, N3 = N2 * N;
  __shared__ double c0[N], c1[N];
  if (threadIdx.x < N) {
    c0[threadIdx.x] = tab.c0[threadIdx.x];
    c1[threadIdx.x] = tab.c1[threadIdx.x];
  }
  __syncthreads();
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N3) return;
  const double* __restrict__ rho = sp.in[blockIdx.y];
  const double* __restrict__ Jx = rho + 2 * N3;
  const double* __restrict__ Jy = rho + 3 * N3;
  const double* __restrict__ Jz = rho + 4 * N3;
  double* __restrict__ o = sp.out[blockIdx.y];
  const int x = p % N, y = (p / N) % N, z = p / N2;
  double lap = 0.0, gx = 0.0, gy = 0.0, gz = 0.0, dj = 0.0;
  const int bx = z * N2 + y * N, by = z * N2 + x, bz = y * N + x;
#pragma unroll 8
  for (int j = 0; j < N; ++j) {
    const int dx = x - j < 0 ? x - j + N : x - j;
    const int dy = y - j < 0 ? y - j + N : y - j;
    const int dz = z - j < 0 ? z - j + N : z - j;
    const double rx = rho[bx + j], ry = rho[by + j * N], rz = rho[bz + j * N2];
    lap += c1[dx] * rx + c1[dy] * ry + c1[dz] * rz;
    gx += c0[dx] * rx;
    gy += c0[dy] * ry;
    gz += c0[dz] * rz;
    dj += c0[dx] * Jx[bx + j] + c0[dy] * Jy[by + j * N] + c0[dz] * Jz[bz + j * N2];
  }
  o[p] = lap;
  o[N3 + p] = gx;
  o[2 * N3 + p] = gy;
  o[3 * N3 + p] = gz;
  o[4 * N3 + p] = dj;
}

// One axis (x or y) of a 3D DFT: dst[.., k, ..] = s * sum_j src[.., j, ..]
// w^{+-k j} (forward e^{-2 pi i k j / n}; inverse the conjugate and s = 1/n).
// Along x the forward pass takes a real field and the inverse leaves the real
// part.
template <int N, int DIR, bool INV>
__global__ void __launch_bounds__(256)
k_dft_pass(const void* __restrict__ srcv, void* __restrict__ dstv, FieldTaps tab,
           const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  constexpr int N2 = N * N, N3 = N2 * N;
  __shared__ double twr[N], twi[N];
  if (threadIdx.x < N) {
    twr[threadIdx.x] = tab.twr[threadIdx.x];
    twi[threadIdx.x] = INV ? -tab.twi[threadIdx.x] : tab.twi[threadIdx.x];
  }
  __syncthreads();
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N3) return;
  const int x = p % N, y = (p / N) % N, z = p / N2;
  const int k = DIR == 0 ? x : y;
  const int base = DIR == 0 ? z * N2 + y * N : z * N2 + x;
  constexpr int STRIDE = DIR == 0 ? 1 : N;
  double sr = 0.0, si = 0.0;
  int t = 0;   // (k * j) mod n
#pragma unroll 8
  for (int j = 0; j < N; ++j) {
    double2 v;
    if (DIR == 0 && !INV) v = make_double2(static_cast<const double*>(srcv)[base + j * STRIDE], 0.0);
    else v = static_cast<const double2*>(srcv)[base + j * STRIDE];
    sr += v.x * twr[t] - v.y * twi[t];
    si += v.x * twi[t] + v.y * twr[t];
    t += k;
    if (t >= N) t -= N;
  }
  const double sc = INV ? 1.0 / double(N) : 1.0;
  if (DIR == 0 && INV) static_cast<double*>(dstv)[p] = sc * sr;
  else static_cast<double2*>(dstv)[p] = make_double2(sc * sr, sc * si);
}

// The z axis of the Coulomb solve, in place: forward DFT of each line, times
// 4 pi e2 / |k|^2 (zero at k = 0), inverse DFT.  A workgroup holds LB lines.
template <int N> constexpr int coulomb_lines() { return 256 / N; }
template <int N>
__global__ void __launch_bounds__(256)
k_coulomb_z(double2* __restrict__ buf, FieldTaps tab, double kunit, double e2,
            const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  constexpr int N2 = N * N, LB = coulomb_lines<N>();
  __shared__ double twr[N], twi[N];
  __shared__ double2 A[N][LB], B[N][LB];
  if (threadIdx.x < N) {
    twr[threadIdx.x] = tab.twr[threadIdx.x];
    twi[threadIdx.x] = tab.twi[threadIdx.x];
  }
  const int l = threadIdx.x % LB, k = threadIdx.x / LB;   // line, frequency or point
  const int line = blockIdx.x * LB + l;
  const bool live = k < N && line < N2;
  if (live) A[k][l] = buf[size_t(k) * N2 + line];
  __syncthreads();
  if (live) {
    double sr = 0.0, si = 0.0;
    int t = 0;
#pragma unroll 8
    for (int j = 0; j < N; ++j) {
      const double2 v = A[j][l];
      sr += v.x * twr[t] - v.y * twi[t];
      si += v.x * twi[t] + v.y * twr[t];
      t += k;
      if (t >= N) t -= N;
    }
    const double kx = kval(line % N, N, kunit), ky = kval(line / N, N, kunit), kz = kval(k, N, kunit);
    const double k2 = kx * kx + ky * ky + kz * kz;
    const double f = (line == 0 && k == 0) ? 0.0 : 4.0 * M_PI * e2 / k2;
    B[k][l] = make_double2(f * sr, f * si);
  }
  __syncthreads();
  if (!live) return;
  double sr = 0.0, si = 0.0;
  int t = 0;
#pragma unroll 8
  for (int j = 0; j < N; ++j) {
    const double2 v = B[j][l];
    sr += v.x * twr[t] + v.y * twi[t];
    si += v.y * twr[t] - v.x * twi[t];
    t += k;
    if (t >= N) t -= N;
  }
  buf[size_t(k) * N2 + line] = make_double2(sr / double(N), si / double(N));
}

// U, B, W of both species, their FP32 copies for the complex64 kernels, and
// the per-block energy partials.
// dens: [rho, tau, Jx, Jy, Jz, ...]; derived: [lap rho, drho x/y/z, div J].
__global__ void k_mean_field(Skyrme sk, int n3, double dV, const double* __restrict__ dn,
                             const double* __restrict__ dp, const double* __restrict__ gn,
                             const double* __restrict__ gp, const double* __restrict__ vc,
                             double* __restrict__ mn, double* __restrict__ mp,
                             float* __restrict__ mn32, float* __restrict__ mp32,
                             double* __restrict__ epart, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double red[NTERM][E_THREADS / 64];
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  double e[NTERM] = {0, 0, 0, 0, 0, 0, 0};
  if (r < n3) {
    const double rn = dn[r], rp = dp[r], tn = dn[n3 + r], tp = dp[n3 + r];
    const double ln = gn[r], lp = gp[r], djn = gn[4 * n3 + r], djp = gp[4 * n3 + r];
    const double rho = rn + rp, tau = tn + tp, lap = ln + lp, divJ = djn + djp;
    const double vcr = vc ? vc[r] : 0.0;
    const double rs = fmax(rho, 1e-30);
    const double ra = pow(rs, sk.alpha);
    const double sq = rn * rn + rp * rp;
    const double common = sk.b0 * rho + sk.b1 * tau - sk.b2 * lap - sk.b4 * divJ +
                          sk.b3 / 3.0 * (sk.alpha + 2.0) * ra * rs -
                          sk.b3p / 3.0 * sk.alpha * ra * (sq / rs);
    for (int q = 0; q < 2; ++q) {
      const double rq = q ? rp : rn, tq = q ? tp : tn, lq = q ? lp : ln, dq = q ? djp : djn;
      const double* gq = q ? gp : gn;
      double* m = q ? mp : mn;
      double U = common - sk.b0p * rq - sk.b1p * tq + sk.b2p * lq - sk.b4p * dq -
                 sk.b3p / 3.0 * 2.0 * ra * rq;
      if (q) U += vcr;
      float* m32 = q ? mp32 : mn32;
      auto put = [&](int f, double v) {
        m[f * n3 + r] = v;
        m32[f * n3 + r] = float(v);
      };
      put(0, U);
      put(1, (q ? sk.hb2m_p : sk.hb2m_n) + sk.b1 * rho - sk.b1p * rq);
      for (int c = 0; c < 3; ++c) {
        const double grad = gn[(1 + c) * n3 + r] + gp[(1 + c) * n3 + r];
        put(2 + c, sk.b4 * grad + sk.b4p * gq[(1 + c) * n3 + r]);
      }
    }
    e[0] = sk.hb2m_n * tn + sk.hb2m_p * tp;
    e[1] = sk.b0 / 2.0 * rho * rho - sk.b0p / 2.0 * sq;
    e[2] = sk.b3 / 3.0 * ra * rs * rs - sk.b3p / 3.0 * ra * sq;
    e[3] = sk.b1 * rho * tau - sk.b1p * (rn * tn + rp * tp);
    e[4] = -sk.b2 / 2.0 * rho * lap + sk.b2p / 2.0 * (rn * ln + rp * lp);
    e[5] = -sk.b4 * rho * divJ - sk.b4p * (rn * djn + rp * djp);
    e[6] = 0.5 * rp * vcr;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int t = 0; t < NTERM; ++t) {
    double v = e[t];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) red[t][wave] = v;
  }
  __syncthreads();
  if (threadIdx.x < NTERM) {
    double s = 0.0;
    for (int w = 0; w < E_THREADS / 64; ++w) s += red[threadIdx.x][w];
    epart[blockIdx.x * NTERM + threadIdx.x] = s * dV;
  }
}

// out[t] = sum of the block partials of term t, one wave per term (lane l
// takes blocks l, l + 64, ... in order, then a fixed butterfly); out[NTERM] =
// sum of the terms.
__global__ void __launch_bounds__(64 * NTERM)
k_energy_final(const double* __restrict__ epart, int nblk, double* __restrict__ out, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double term[NTERM];
  const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double s = 0.0;
  for (int b = lane; b < nblk; b += 64) s += epart[b * NTERM + t];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (lane == 0) {
    out[t] = s;
    term[t] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int k = 0; k < NTERM; ++k) tot += term[k];
    out[NTERM] = tot;
  }
}

template <int N>
void launch_derivatives(const Species& sp, const FieldTaps& tab, hipStream_t st) {
  hipLaunchKernelGGL(k_field_derivs<N>, dim3((N * N * N + 255) / 256, 2), dim3(256), 0, st, sp, tab,
                     g_launch_gate);
}

// Coulomb potential of the proton density: x and y forward, z forward, 1/k^2
// and back, y and x inverse.
template <int N>
void launch_coulomb(const double* rho_p, double* vc, double2* a, double2* b, const FieldTaps& tab,
                    double kunit, double e2, hipStream_t st) {
  const dim3 nb((N * N * N + 255) / 256), th(256);
  constexpr int LB = coulomb_lines<N>();
  hipLaunchKernelGGL((k_dft_pass<N, 0, false>), nb, th, 0, st, rho_p, a, tab, g_launch_gate);
  hipLaunchKernelGGL((k_dft_pass<N, 1, false>), nb, th, 0, st, a, b, tab, g_launch_gate);
  hipLaunchKernelGGL(k_coulomb_z<N>, dim3((N * N + LB - 1) / LB), th, 0, st, b, tab, kunit, e2,
                     g_launch_gate);
  hipLaunchKernelGGL((k_dft_pass<N, 1, true>), nb, th, 0, st, b, a, tab, g_launch_gate);
  hipLaunchKernelGGL((k_dft_pass<N, 0, true>), nb, th, 0, st, a, vc, tab, g_launch_gate);
}

}  // namespace

// With n even: c0[d] = (1/n) sum_k i k e^{2 pi i k d / n} over the modes but the
// Nyquist one = kunit (-1)^d cot(pi d / n) / 2, c1[d] = (1/n) sum_k -k^2
// e^{2 pi i k d / n} over all of them = -kunit^2 (-1)^d / (2 sin^2(pi d / n)), and
// -kunit^2 (n^2 + 2) / 12 at d = 0: the differentiation matrices of periodic
// spectral collocation (Trefethen, Spectral Methods in MATLAB, ch. 3).
FieldTaps field_taps(int n, double kunit) {
  // extended precision, and the two halves of an axis exact mirror images: the
  // taps' rounding errors then cancel in the derivative of a constant
  const long double pi = 3.14159265358979323846264338327950288L;
  FieldTaps t{};
  for (int d = 0; d < n; ++d) {
    const int e = d <= n / 2 ? d : n - d;   // distance along the shorter way
    const long double s = sinl(pi * e / n), c = cosl(pi * e / n), sign = e % 2 ? -1.0L : 1.0L;
    const double c0 = e && 2 * e != n ? double(0.5L * kunit * sign * c / s) : 0.0;
    t.c0[d] = d == e ? c0 : -c0;
    t.c1[d] = e ? double(-0.5L * kunit * kunit * sign / (s * s))
                : double(-(long double)kunit * kunit * (n * n + 2.0L) / 12.0L);
    t.twr[d] = double(cosl(2.0L * pi * e / n));
    const double si = 2 * e != n ? double(sinl(2.0L * pi * e / n)) : 0.0;
    t.twi[d] = d == e ? -si : si;
  }
  return t;
}

int energy_nblocks(int n) { return (n * n * n + E_THREADS - 1) / E_THREADS; }

size_t mean_field_scratch_bytes(int n) { return 2 * sizeof(double2) * size_t(n) * n * n; }

void mean_field(int n, GridArgs g, const Skyrme& sk, const FieldTaps& tab, const double* dens_n,
                const double* dens_p, double* der_n, double* der_p, double* mf_n, double* mf_p,
                float* mf32_n, float* mf32_p, double* vc, void* scratch, double* epart,
                double* energy, hipStream_t st) {
  const int n3 = n * n * n;
  double2* bufA = reinterpret_cast<double2*>(scratch);
  double2* bufB = bufA + n3;
  const Species sp{{dens_n, dens_p}, {der_n, der_p}};
  SKY_DISPATCH_N(n, launch_derivatives<NN>(sp, tab, st))
  const double* vcp = nullptr;
  if (sk.e2 != 0.0) {
    SKY_DISPATCH_N(n, launch_coulomb<NN>(dens_p, vc, bufA, bufB, tab, g.kunit, sk.e2, st))
    vcp = vc;
  } else {
    zero(vc, n3, st);
  }
  const int nblk = energy_nblocks(n);
  hipLaunchKernelGGL(k_mean_field, dim3(nblk), dim3(E_THREADS), 0, st, sk, n3, g.dV, dens_n,
                     dens_p, (const double*)der_n, (const double*)der_p, vcp, mf_n, mf_p, mf32_n,
                     mf32_p, epart, g_launch_gate);
  hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(64 * NTERM), 0, st, (const double*)epart, nblk,
                     energy, g_launch_gate);
}

}  // namespace sky
