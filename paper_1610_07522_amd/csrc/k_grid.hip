// Grid kernels on the spinor wave functions: h*psi, the damped gradient
// step, and the local densities.  All are passes over lines of one axis
// (fft_line.h); one workgroup takes LPW lines of one state (h, damping) or of
// a chunk of states (densities).
#include <algorithm>
#include <cmath>

#include "fft_line.h"
#include "sky_kernels.h"

namespace sky {

// Field value at point r in the kernel's precision: complex64 kernels read
// the FP32 copies (the same rounding as converting the FP64 value).
template <typename T> __device__ inline T fld_U(const MeanFieldPtrs& m, size_t r) {
  if constexpr (sizeof(T) == 4) return m.U32[r]; else return m.U[r];
}
template <typename T> __device__ inline T fld_B(const MeanFieldPtrs& m, size_t r) {
  if constexpr (sizeof(T) == 4) return m.B32[r]; else return m.B[r];
}
template <typename T> __device__ inline T fld_W(const MeanFieldPtrs& m, size_t r) {
  if constexpr (sizeof(T) == 4) return m.W32[r]; else return m.W[r];
}

// i (A_dir / 2) applied to the spinor (p, q), A_dir = (W x sigma)_dir; a and b
// are the halves of A_dir's two non-zero components: (-W_z, W_y) along
// (sigma_y, sigma_z) for x, (W_z, -W_x) along (sigma_x, sigma_z) for y, and
// (-W_y, W_x) along (sigma_x, sigma_y) for z.
template <int DIR, typename T> __device__ inline void half_so(T a, T b, cpx<T> p, cpx<T> q,
                                                              cpx<T>& op, cpx<T>& oq) {
  if (DIR == 0) {
    op = mk(a * q.re - b * p.im, a * q.im + b * p.re);
    oq = mk(b * q.im - a * p.re, -a * p.im - b * q.re);
  } else if (DIR == 1) {
    op = mk(-b * p.im - a * q.im, b * p.re + a * q.re);
    oq = mk(b * q.im - a * p.im, a * p.re - b * q.re);
  } else {
    op = mk(b * q.re - a * q.im, b * q.im + a * q.re);
    oq = mk(-b * p.re - a * p.im, a * p.re - b * p.im);
  }
}

// The local terms of one direction of h at grid point r: (i/2) A D psi into
// acc and g = (i/2) A psi - B D psi into d (D psi on entry).
template <typename T, int N, int DIR>
__device__ inline void h_local(const MeanFieldPtrs& mf, size_t r, cpx<T> vu, cpx<T> vd,
                               cpx<T>& du, cpx<T>& dd, cpx<T>& au, cpx<T>& ad) {
  constexpr int N3 = N * N * N;
  const T B = fld_B<T>(mf, r);
  T a, b;
  if (DIR == 0) { a = T(-0.5) * fld_W<T>(mf, 2 * N3 + r); b = T(0.5) * fld_W<T>(mf, N3 + r); }
  else if (DIR == 1) { a = T(0.5) * fld_W<T>(mf, 2 * N3 + r); b = T(-0.5) * fld_W<T>(mf, r); }
  else { a = T(-0.5) * fld_W<T>(mf, N3 + r); b = T(0.5) * fld_W<T>(mf, r); }
  cpx<T> gu, gd;
  half_so<DIR>(a, b, du, dd, au, ad);
  half_so<DIR>(a, b, vu, vd, gu, gd);
  du = gu - B * du;
  dd = gd - B * dd;
}

// Workgroup sum of one double per thread of a workgroup of THREADS threads,
// result in thread 0; red has one entry per wave.
constexpr int waves_of_threads(int threads) { return (threads + 63) / 64; }
template <int THREADS>
__device__ inline double block_sum(double v, double (&red)[waves_of_threads(THREADS)]) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    for (int w = 0; w < waves_of_threads(THREADS); ++w) s += red[w];
  }
  __syncthreads();
  return s;
}

// Largest |component| (real or imaginary part, as float) of the values this
// workgroup wrote, merged into *amax as float bits (non-negative floats
// order like their bit patterns).  Any blockDim; every thread must call it.
__device__ inline void block_amax(float v, unsigned int* amax) {
  __shared__ unsigned int smax;
  if (threadIdx.x == 0) smax = 0u;
  __syncthreads();
  atomicMax(&smax, __float_as_uint(v));
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(amax, smax);
}

template <typename T> __device__ inline float cabs_max(cpx<T> z) {
  return fmaxf(fabsf(float(z.re)), fabsf(float(z.im)));
}

// A pointer the compiler takes as new: loads through it are not merged with
// earlier ones (whose values would stay in registers across the transforms).
// The complex64 kernels read psi anew (from the L2) where the local terms need
// it: 24 registers fewer at 48^3, a wave more per SIMD.  The complex128 line
// passes, two waves per SIMD either way, hold it in registers of their own; a
// second load in the source is one in the kernel too, the barriers between
// keep the two apart (48^3, 400 states: 2420 us with it, 2220 without; 64^3,
// 150 states: 2360 and 1950).
template <typename P> __device__ inline P* reread(P* p) {
  asm volatile("" : "+s"(p));
  return p;
}

// ------------------------------------------------------------------ h * psi
// One pass adds the DIR part of h:
//   - D(B D psi) + (i/2) [A D psi + D(A psi)]  =  D g + (i/2) A D psi,
//   g = -B D psi + (i/2) A psi,
// plus U psi on the first pass.  The last pass also forms per-workgroup
// partial sums of <psi|h psi> for the Rayleigh quotients.
template <typename T, int N, int DIR, bool FIRST, bool LAST, int LP>
__global__ void __launch_bounds__((LineCfg<N, LP>::THREADS))
k_h_pass(const cpx<T>* __restrict__ psi, cpx<T>* __restrict__ hpsi, MeanFieldPtrs mf,
         GridArgs g, double* __restrict__ eps_part, double* __restrict__ nrm_part,
         unsigned int* __restrict__ amax, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = LineCfg<N, LP>;
  using F = LineFFT<T, N, 2, DIR == 0 && x_wave_local<N>()>;
  constexpr int YS = line_stride<T, N, 2, DIR>();
  constexpr int R1 = C::R1, R2 = C::R2, N3 = N * N * N;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> Ybuf[C::LPW * YS];
  __shared__ double red[waves_of_threads(C::THREADS)];

  int line, j;
  thread_role<N, DIR, LP>(threadIdx.x, line, j);
  const int L = blockIdx.x * C::LPW + line;
  int base, stride, a, b;
  line_geom<N, DIR>(L, base, stride, a, b);
  const size_t soff = size_t(blockIdx.y) * 2 * N3;
  const cpx<T>* p = psi + soff;
  cpx<T>* hp = hpsi + soff;
  cpx<T>* Y = Ybuf + line * YS;
  const T kun = T(g.kunit * (1.0 / N)), ksn = T(g.tw[DIR] * (1.0 / N));

  constexpr bool HOLD = sizeof(T) == 8;   // psi in registers through the pass (see reread)
  cpx<T> d[2][R1], v[2][HOLD ? R1 : 1];
  if (j < R2) {
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      int r = base + (j + R2 * j1) * stride;
      d[0][j1] = p[r];
      d[1][j1] = p[N3 + r];
      if constexpr (HOLD) {
        v[0][j1] = d[0][j1];
        v[1][j1] = d[1][j1];
      }
    }
  }
  load_twiddles<T, N>(tw);
  F::deriv(d, Y, j, tw, kun, ksn);

  // g (into d) and the accumulated local terms (into acc)
  cpx<T> acc[2][R1];
  if (j < R2) {
    const cpx<T>* q = reread(p);
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      int r = base + (j + R2 * j1) * stride;
      cpx<T> vu, vd;
      if constexpr (HOLD) {
        vu = v[0][j1];
        vd = v[1][j1];
      } else {
        vu = q[r];
        vd = q[N3 + r];
      }
      h_local<T, N, DIR>(mf, r, vu, vd, d[0][j1], d[1][j1], acc[0][j1], acc[1][j1]);
      if (FIRST) {
        const T U = fld_U<T>(mf, r);
        acc[0][j1] = acc[0][j1] + U * vu;
        acc[1][j1] = acc[1][j1] + U * vd;
      }
    }
  }
  F::deriv(d, Y, j, tw, kun, ksn);

  double dot = 0.0, nrm = 0.0;
  float am = 0.0f;
  if (j < R2) {
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      int r = base + (j + R2 * j1) * stride;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        cpx<T> t = acc[s][j1] + d[s][j1];
        if (!FIRST) t = t + hp[s * N3 + r];
        hp[s * N3 + r] = t;
        if (LAST) {
          acc[s][j1] = t;
          am = fmaxf(am, cabs_max(t));
        }
      }
    }
    if (LAST && (eps_part != nullptr || nrm_part != nullptr)) {
      const cpx<T>* q = reread(p);
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const cpx<T> t = acc[s][j1];
          cpx<T> w;
          if constexpr (HOLD) w = v[s][j1];
          else w = q[s * N3 + base + (j + R2 * j1) * stride];
          dot += double(w.re) * double(t.re) + double(w.im) * double(t.im);
          nrm += double(w.re) * double(w.re) + double(w.im) * double(w.im);
        }
      }
    }
  }
  if (LAST && eps_part != nullptr) {
    double sum = block_sum<C::THREADS>(dot, red);
    if (threadIdx.x == 0) eps_part[size_t(blockIdx.y) * gridDim.x + blockIdx.x] = sum * g.dV;
  }
  if (LAST && nrm_part != nullptr) {
    double sum = block_sum<C::THREADS>(nrm, red);
    if (threadIdx.x == 0) nrm_part[size_t(blockIdx.y) * gridDim.x + blockIdx.x] = sum * g.dV;
  }
  if (LAST && amax != nullptr) block_amax(am, amax);
}

// Sums of the per-workgroup partials of each state, out[s] = sum_t part[s][t]:
// one wave per state (lane t takes t, t + 64, ... in order, then a fixed
// butterfly), blockIdx.y picks one of two sets.  (One thread per state walked
// its 144 partials at 48^3 as a serial chain of loads, 9.3 us.)
__global__ void __launch_bounds__(256)
k_sum_partials(const double* __restrict__ part0, const double* __restrict__ part1, int ntile,
               int nstate, double* __restrict__ out0, double* __restrict__ out1,
               const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (s >= nstate) return;
  const double* part = blockIdx.y ? part1 : part0;
  double acc = 0.0;
  for (int t = lane; t < ntile; t += 64) acc += part[size_t(s) * ntile + t];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  if (lane == 0) (blockIdx.y ? out1 : out0)[s] = acc;
}

static void sum_partials(const double* part0, const double* part1, int ntile, int nstate,
                         double* out0, double* out1, hipStream_t st) {
  hipLaunchKernelGGL(k_sum_partials, dim3(unsigned(nstate + 3) / 4, part1 ? 2 : 1), dim3(256), 0, st,
                     part0, part1, ntile, nstate, out0, out1, g_launch_gate);
}

// Per workgroup of a grid (tiles, states): partials of Re <a|b> and <a|a> of a
// state, and the largest |component| of a and of b merged into mx[0] and
// mx[1] (b may be null: <a|a> and mx[0] only), for states whose producer did
// not form them.
__global__ void __launch_bounds__(256)
k_state_dots(const float2* __restrict__ a, const float2* __restrict__ b, long V, double dV,
             double* __restrict__ dot_part, double* __restrict__ nrm_part,
             unsigned int* __restrict__ mx, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double red[waves_of_threads(256)];
  const size_t off = size_t(blockIdx.y) * V;
  double dot = 0.0, nrm = 0.0;
  float ma = 0.0f, mb = 0.0f;
  for (long i = long(blockIdx.x) * 256 + threadIdx.x; i < V; i += long(gridDim.x) * 256) {
    const float2 x = a[off + i];
    nrm += double(x.x) * double(x.x) + double(x.y) * double(x.y);
    ma = fmaxf(ma, fmaxf(fabsf(x.x), fabsf(x.y)));
    if (b != nullptr) {
      const float2 y = b[off + i];
      dot += double(x.x) * double(y.x) + double(x.y) * double(y.y);
      mb = fmaxf(mb, fmaxf(fabsf(y.x), fabsf(y.y)));
    }
  }
  const size_t at = size_t(blockIdx.y) * gridDim.x + blockIdx.x;
  const double sn = block_sum<256>(nrm, red);
  if (threadIdx.x == 0) nrm_part[at] = sn * dV;
  block_amax(ma, mx);
  if (b == nullptr) return;
  const double sd = block_sum<256>(dot, red);
  if (threadIdx.x == 0) dot_part[at] = sd * dV;
  block_amax(mb, mx + 1);
}

void state_dots(const void* a, const void* b, int n, int nstate, double dV, double* part,
                double* dot, double* nrm, unsigned int* mx, hipStream_t st) {
  if (nstate <= 0) return;
  const long V = 2L * n * n * n;
  const int nt = std::min(grid_ntiles(n), 8);
  double* npart = part + size_t(nstate) * nt;
  hipLaunchKernelGGL(k_state_dots, dim3(nt, nstate), dim3(256), 0, st, (const float2*)a,
                     (const float2*)b, V, dV, part, npart, mx, g_launch_gate);
  if (b) sum_partials(part, npart, nt, nstate, dot, nrm, st);
  else sum_partials(npart, nullptr, nt, nstate, nrm, nullptr, st);
}

// ------------------------------------------------------------------ xy planes
// One workgroup takes a z-slice of one state (both spin components, N x N
// points) through the x lines (rows) and the y lines (columns) of a pass, so
// that x and y cost one read and one write of the state instead of two each.
// Threads: N lines x RT per line.  Slices in LDS have rows padded to N + 1.
template <int N> struct PlaneCfg {
  static constexpr int R1 = Fact<N>::R1, R2 = Fact<N>::R2;
  static constexpr int RT = R1 > R2 ? R1 : R2;
  static constexpr int THREADS = N * RT;
  static constexpr int PITCH = N + 1;
  static constexpr int SPIN = N * PITCH;   // one spin component of the slice
};

// LDS of the h slice kernel: one exchange buffer per line, for the x and the y
// lines in turn (and for a slice in between).
template <typename T, int N> constexpr int plane_buf() {
  const int x = line_stride<T, N, 2, 0>(), y = line_stride<T, N, 2, 1>();
  return N * (x > y ? x : y);
}
template <typename T, int N> constexpr bool plane_fits() {
  return PlaneCfg<N>::THREADS <= 1024 && (plane_buf<T, N>() + N) * int(sizeof(cpx<T>)) <= 80 * 1024;
}
// Waves per SIMD the h slice kernel is compiled for: the compiler's own choice
// (1: no demand), but at 48^3 complex64 five, three workgroups per CU, where
// its choice is four and two.  The registers are 96 then and six spill
// (400 states, with the z pass: 1114 to 1120 us; with four 1124 to 1131).
// Elsewhere one more does not fit the LDS (64^3: 78 KB a workgroup; 8^3 and
// 16^3 complex64) or spills more than it hides: complex64 24^3 x 200 85 us
// with eight, 74 with its own six; 32^3 x 200 208 with eight and 138 with
// six, 138 with its own five; complex128 24^3 x 100 122 with five and 79 with
// four, 74 with its own three; 32^3 x 160 320 with four, 227 with its own three.
template <typename T, int N> constexpr int plane_waves() {
  return sizeof(T) == 4 && N == 48 ? 5 : 1;
}
// The damped step's slice kernels exchange in place in the slice (no line
// buffers).  Default wherever they fit: x and y cost one read and one write
// instead of two.  Measured against the line passes (us): complex64 8^3 x 60
// 20.8 / 25.3, 16^3 x 100 28.8 / 29.5, 24^3 x 200 78 / 102, 32^3 x 200 138 / 203,
// 48^3 x 400 1038 / 1578, 64^3 x 150 929 / 1355; complex128 16^3 x 60 28.1 / 29.6,
// 24^3 x 100 74 / 90, 32^3 x 160 237 / 321, 48^3 x 100 645 / 780.
template <typename T, int N> constexpr bool damp_slices_fit() {
  return PlaneCfg<N>::THREADS <= 1024 && (2 * PlaneCfg<N>::SPIN + N) * sizeof(cpx<T>) <= 80 * 1024;
}
// The slices are the default wherever they fit.  Measured against the line
// passes (us, with <h>): complex64 8^3 x 60 12.2 / 14.2, 16^3 x 100 19.7 / 25.9,
// 24^3 x 200 73 / 88, 32^3 x 200 147 / 173, 48^3 x 400 1125 / 1236, 64^3 x 150
// 970 / 1050; complex128 16^3 x 60 21.9 / 27.0, 24^3 x 100 76 / 82, 32^3 x 160
// 241 / 278.  The tuner decides per box.

// Deterministic workgroup sum of one double per thread (any blockDim), using
// buf[blockDim.x] of LDS; the result is returned to thread 0.
__device__ inline double tree_sum(double v, double* buf) {
  buf[threadIdx.x] = v;
  __syncthreads();
  int n = blockDim.x;
  while (n > 1) {
    const int h = (n + 1) / 2;
    if (threadIdx.x < n - h) buf[threadIdx.x] += buf[threadIdx.x + h];
    __syncthreads();
    n = h;
  }
  return buf[0];
}

// x and y parts of h psi on slice z = blockIdx.x of state blockIdx.y, added to
// what hpsi holds (the z part and U psi); partial sums of <psi|h psi> and
// <psi|psi>.  HBM traffic: psi and h psi read, h psi written (with the z pass
// five state transfers, against eight by line passes).  Registers decide how
// many workgroups a CU holds, so nothing is kept that can be had again: psi is
// read anew (from the L2) where the local terms need it, and the x part goes
// to the y lines' threads through the exchange buffer, which is all the LDS
// there is.  At 48^3 complex64 it is compiled for five
// waves per SIMD (three workgroups per CU): 400 states take 739 us for these
// two directions (2.9 TB/s; vector issue busy three quarters of the cycles),
// where the kernel that kept psi in LDS and registers, two workgroups per CU,
// took 1250 us and the two line passes 900 us.
template <typename T, int N>
__global__ void __launch_bounds__(PlaneCfg<N>::THREADS, (plane_waves<T, N>()))
k_h_plane(const cpx<T>* __restrict__ psi, cpx<T>* __restrict__ hpsi, MeanFieldPtrs mf, GridArgs g,
          double* __restrict__ eps_part, double* __restrict__ nrm_part,
          unsigned int* __restrict__ amax, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = PlaneCfg<N>;
  using FX = LineFFT<T, N, 2, x_wave_local<N>()>;
  using FY = LineFFT<T, N, 2>;
  constexpr int R1 = C::R1, R2 = C::R2, RT = C::RT, PITCH = C::PITCH, SP = C::SPIN;
  constexpr int N2 = N * N, N3 = N * N2;
  constexpr int XS = line_stride<T, N, 2, 0>(), YS = line_stride<T, N, 2, 1>();
  static_assert(plane_buf<T, N>() >= 2 * SP, "a slice fits the exchange buffers");
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> E[plane_buf<T, N>()];
  const int zoff = blockIdx.x * N2;
  const size_t soff = size_t(blockIdx.y) * 2 * N3;
  const cpx<T>* p = psi + soff;
  cpx<T>* hp = hpsi + soff;
  const T kun = T(g.kunit * (1.0 / N)), kx = T(g.tw[0] * (1.0 / N)), ky = T(g.tw[1] * (1.0 / N));
  cpx<T> acc[2][R1], d[2][R1];
  {  // x lines: row ly, role jx (role fastest: consecutive threads, consecutive x)
    const int jx = threadIdx.x % RT, ly = threadIdx.x / RT;
    const int r0 = zoff + ly * N + jx;
    if (jx < R2) {
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1) {
        d[0][j1] = p[r0 + R2 * j1];
        d[1][j1] = p[N3 + r0 + R2 * j1];
      }
    }
    load_twiddles<T, N>(tw);
    FX::deriv(d, E + ly * XS, jx, tw, kun, kx);
    if (jx < R2) {
      const cpx<T>* q = reread(p);
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1) {
        const int r = r0 + R2 * j1;
        h_local<T, N, 0>(mf, r, q[r], q[N3 + r], d[0][j1], d[1][j1], acc[0][j1], acc[1][j1]);
      }
    }
    FX::deriv(d, E + ly * XS, jx, tw, kun, kx);
    __syncthreads();   // every x line is done with its buffer
    if (jx < R2) {
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1) {
        const int e = ly * PITCH + jx + R2 * j1;
        E[e] = acc[0][j1] + d[0][j1];
        E[SP + e] = acc[1][j1] + d[1][j1];
      }
    }
  }
  // y lines: column lx (line fastest: consecutive threads, consecutive x)
  const int lx = threadIdx.x % N, jy = threadIdx.x / N;
  const int r0 = zoff + jy * N + lx;
  if (jy < R2) {
    const cpx<T>* q = reread(p);
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      d[0][j1] = q[r0 + R2 * j1 * N];
      d[1][j1] = q[N3 + r0 + R2 * j1 * N];
    }
  }
  __syncthreads();
  if (jy < R2) {
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      const int e = (jy + R2 * j1) * PITCH + lx;
      acc[0][j1] = E[e];
      acc[1][j1] = E[SP + e];
    }
  }
  __syncthreads();
  FY::deriv(d, E + lx * YS, jy, tw, kun, ky);
  if (jy < R2) {
    const cpx<T>* q = reread(p);
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      const int r = r0 + R2 * j1 * N;
      cpx<T> au, ad;
      h_local<T, N, 1>(mf, r, q[r], q[N3 + r], d[0][j1], d[1][j1], au, ad);
      acc[0][j1] = acc[0][j1] + au;
      acc[1][j1] = acc[1][j1] + ad;
    }
  }
  FY::deriv(d, E + lx * YS, jy, tw, kun, ky);
  double dot = 0.0, nrm = 0.0;
  float am = 0.0f;
  if (jy < R2) {
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      const int r = r0 + R2 * j1 * N;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const cpx<T> t = acc[s][j1] + d[s][j1] + hp[s * N3 + r];
        hp[s * N3 + r] = t;
        acc[s][j1] = t;
        am = fmaxf(am, cabs_max(t));
      }
    }
    if (eps_part != nullptr || nrm_part != nullptr) {
      const cpx<T>* q = reread(p);
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const cpx<T> v = q[s * N3 + r0 + R2 * j1 * N], t = acc[s][j1];
          dot += double(v.re) * double(t.re) + double(v.im) * double(t.im);
          nrm += double(v.re) * double(v.re) + double(v.im) * double(v.im);
        }
      }
    }
  }
  if (eps_part != nullptr) {   // E again for the reductions
    __syncthreads();
    const double sum = tree_sum(dot, reinterpret_cast<double*>(E));
    if (threadIdx.x == 0) eps_part[size_t(blockIdx.y) * gridDim.x + blockIdx.x] = sum * g.dV;
  }
  if (nrm_part != nullptr) {
    __syncthreads();
    const double sum = tree_sum(nrm, reinterpret_cast<double*>(E));
    if (threadIdx.x == 0) nrm_part[size_t(blockIdx.y) * gridDim.x + blockIdx.x] = sum * g.dV;
  }
  if (amax != nullptr) block_amax(am, amax);
}

// Damped step, first half: r = h psi - eps psi on slice z of state
// blockIdx.y, forward FFTs along x and y, spectrum to out; ||r||^2 partials.
template <typename T, int N>
__global__ void __launch_bounds__(PlaneCfg<N>::THREADS)
k_damp_fwd_xy(const cpx<T>* __restrict__ psi, const cpx<T>* __restrict__ hpsi,
              const double* __restrict__ eps, cpx<T>* __restrict__ out, GridArgs g,
              double* __restrict__ r2_part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = PlaneCfg<N>;
  using F = LineFFTInPlace<T, N, 2>;
  constexpr int R1 = C::R1, R2 = C::R2, RT = C::RT, PITCH = C::PITCH, SP = C::SPIN;
  constexpr int N2 = N * N, N3 = N * N2;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> P[2 * SP];
  load_twiddles<T, N>(tw);
  const int zoff = blockIdx.x * N2;
  const size_t soff = size_t(blockIdx.y) * 2 * N3;
  const T e = T(eps[blockIdx.y]);
  double r2 = 0.0;
  constexpr int NIT = (2 * N2 + C::THREADS - 1) / C::THREADS;   // unrolled: loads go out together
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = threadIdx.x + it * C::THREADS;
    if (i < 2 * N2) {
      const int s = i / N2, q = i - s * N2;
      const size_t o = soff + s * N3 + zoff + q;
      const cpx<T> res = hpsi[o] - e * psi[o];
      r2 += double(res.re) * double(res.re) + double(res.im) * double(res.im);
      P[s * SP + (q / N) * PITCH + q % N] = res;
    }
  }
  __syncthreads();
  {  // x lines, in place (row ly; rows fastest across the lanes, whose odd
     // pitch puts a wave's accesses in distinct LDS banks)
    const int ly = threadIdx.x % N, j = threadIdx.x / N;
    cpx<T> va[2][R1], vb[2][R2];
    if (j < R2)
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
        for (int s = 0; s < 2; ++s) va[s][j1] = P[s * SP + ly * PITCH + j + R2 * j1];
    F::forward(va, vb, P + ly * PITCH, SP, 1, j, tw);
    if (j < R1)
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
        for (int s = 0; s < 2; ++s) P[s * SP + ly * PITCH + j + R1 * k2] = vb[s][k2];
  }
  __syncthreads();
  {  // y lines, in place (column lx)
    const int lx = threadIdx.x % N, j = threadIdx.x / N;
    cpx<T> va[2][R1], vb[2][R2];
    if (j < R2)
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
        for (int s = 0; s < 2; ++s) va[s][j1] = P[s * SP + (j + R2 * j1) * PITCH + lx];
    F::forward(va, vb, P + lx, SP, PITCH, j, tw);
    if (j < R1)
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
        for (int s = 0; s < 2; ++s) P[s * SP + (j + R1 * k2) * PITCH + lx] = vb[s][k2];
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = threadIdx.x + it * C::THREADS;
    if (i < 2 * N2) {
      const int s = i / N2, q = i - s * N2;
      out[soff + s * N3 + zoff + q] = P[s * SP + (q / N) * PITCH + q % N];
    }
  }
  __syncthreads();   // P is free again: reuse it for the reduction
  const double sum = tree_sum(r2, reinterpret_cast<double*>(P));
  if (threadIdx.x == 0) r2_part[size_t(blockIdx.y) * gridDim.x + blockIdx.x] = sum * g.dV;
}

// Damped step, last half: inverse FFTs along y and x of slice z of the
// filtered spectrum in buf, then phi = psi - result, in place.
template <typename T, int N>
__global__ void __launch_bounds__(PlaneCfg<N>::THREADS)
k_damp_inv_xy(const cpx<T>* __restrict__ psi, cpx<T>* __restrict__ buf,
              unsigned int* __restrict__ amax, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = PlaneCfg<N>;
  using F = LineFFTInPlace<T, N, 2>;
  constexpr int R1 = C::R1, R2 = C::R2, RT = C::RT, PITCH = C::PITCH, SP = C::SPIN;
  constexpr int N2 = N * N, N3 = N * N2;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> P[2 * SP];
  load_twiddles<T, N>(tw);
  const int zoff = blockIdx.x * N2;
  const size_t soff = size_t(blockIdx.y) * 2 * N3;
  // fixed trip counts, unrolled: each thread's loads of a loop go out together
  constexpr int NIT = (2 * N2 + C::THREADS - 1) / C::THREADS;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = threadIdx.x + it * C::THREADS;
    if (i < 2 * N2) {
      const int s = i / N2, q = i - s * N2;
      P[s * SP + (q / N) * PITCH + q % N] = buf[soff + s * N3 + zoff + q];
    }
  }
  __syncthreads();
  {  // y lines (column lx): frequencies -> positions
    const int lx = threadIdx.x % N, j = threadIdx.x / N;
    cpx<T> va[2][R1], vb[2][R2];
    if (j < R1)
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
        for (int s = 0; s < 2; ++s) vb[s][k2] = P[s * SP + (j + R1 * k2) * PITCH + lx];
    F::inverse(vb, va, P + lx, SP, PITCH, j, tw);
    if (j < R2)
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
        for (int s = 0; s < 2; ++s) P[s * SP + (j + R2 * j1) * PITCH + lx] = va[s][j1];
  }
  __syncthreads();
  {  // x lines (row ly; rows fastest across the lanes, as in the forward half)
    const int ly = threadIdx.x % N, j = threadIdx.x / N;
    cpx<T> va[2][R1], vb[2][R2];
    if (j < R1)
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
        for (int s = 0; s < 2; ++s) vb[s][k2] = P[s * SP + ly * PITCH + j + R1 * k2];
    F::inverse(vb, va, P + ly * PITCH, SP, 1, j, tw);
    if (j < R2)
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
        for (int s = 0; s < 2; ++s) P[s * SP + ly * PITCH + j + R2 * j1] = va[s][j1];
  }
  __syncthreads();
  float am = 0.0f;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int i = threadIdx.x + it * C::THREADS;
    if (i < 2 * N2) {
      const int s = i / N2, q = i - s * N2;
      const size_t o = soff + s * N3 + zoff + q;
      const cpx<T> t = psi[o] - P[s * SP + (q / N) * PITCH + q % N];
      buf[o] = t;
      am = fmaxf(am, cabs_max(t));
    }
  }
  if (amax != nullptr) block_amax(am, amax);
}

// ------------------------------------------------------------------ damping
// phi = psi - F^-1[ x0 F(h psi - eps psi) / (E0 + hb2m |k|^2) ], done as
// forward x, forward y, (forward z, filter, inverse z), inverse y, inverse x,
// in place in the phi buffer.  The first pass also forms ||r||^2 partials.
struct DampArgs {
  double x0, e0, hb2m;
};

// pass 0: r = h psi - eps psi, forward FFT along x, store spectrum.
template <typename T, int N>
__global__ void __launch_bounds__(LineCfg<N>::THREADS)
k_damp_fwd_x(const cpx<T>* __restrict__ psi, const cpx<T>* __restrict__ hpsi,
             const double* __restrict__ eps, cpx<T>* __restrict__ out, GridArgs g,
             double* __restrict__ r2_part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = LineCfg<N>;
  using F = LineFFT<T, N, 2, x_wave_local<N>()>;
  constexpr int YS = line_stride<T, N, 2, 0>();
  constexpr int R1 = C::R1, R2 = C::R2, N3 = N * N * N;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> Ybuf[C::LPW * YS];
  __shared__ double red[waves_of_threads(C::THREADS)];
  load_twiddles<T, N>(tw);
  int line, j;
  thread_role<N, 0>(threadIdx.x, line, j);
  const int L = blockIdx.x * C::LPW + line;
  int base, stride, a, b;
  line_geom<N, 0>(L, base, stride, a, b);
  const size_t soff = size_t(blockIdx.y) * 2 * N3;
  const T e = T(eps[blockIdx.y]);
  cpx<T> va[2][R1], vb[2][R2];
  double r2 = 0.0;
  if (j < R2) {
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      int r = base + (j + R2 * j1) * stride;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        cpx<T> h = hpsi[soff + s * N3 + r], p = psi[soff + s * N3 + r];
        cpx<T> res = h - e * p;
        r2 += double(res.re) * double(res.re) + double(res.im) * double(res.im);
        va[s][j1] = res;
      }
    }
  }
  F::forward(va, vb, Ybuf + line * YS, j, tw);
  if (j < R1) {
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
      int r = base + (j + R1 * k2) * stride;
      out[soff + r] = vb[0][k2];
      out[soff + N3 + r] = vb[1][k2];
    }
  }
  double sum = block_sum<C::THREADS>(r2, red);
  if (threadIdx.x == 0) r2_part[size_t(blockIdx.y) * gridDim.x + blockIdx.x] = sum * g.dV;
}

// forward (INV = false) or inverse (INV = true) FFT along y, in place.
template <typename T, int N, bool INV>
__global__ void __launch_bounds__(LineCfg<N>::THREADS)
k_damp_y(cpx<T>* __restrict__ buf, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = LineCfg<N>;
  using F = LineFFT<T, N, 2>;
  constexpr int YS = line_stride<T, N, 2, 1>();
  constexpr int R1 = C::R1, R2 = C::R2, N3 = N * N * N;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> Ybuf[C::LPW * YS];
  load_twiddles<T, N>(tw);
  int line, j;
  thread_role<N, 1>(threadIdx.x, line, j);
  const int L = blockIdx.x * C::LPW + line;
  int base, stride, a, b;
  line_geom<N, 1>(L, base, stride, a, b);
  cpx<T>* p = buf + size_t(blockIdx.y) * 2 * N3;
  cpx<T> va[2][R1], vb[2][R2];
  cpx<T>* Y = Ybuf + line * YS;
  if (!INV) {
    if (j < R2)
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
        for (int s = 0; s < 2; ++s) va[s][j1] = p[s * N3 + base + (j + R2 * j1) * stride];
    F::forward(va, vb, Y, j, tw);
    if (j < R1)
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
        for (int s = 0; s < 2; ++s) p[s * N3 + base + (j + R1 * k2) * stride] = vb[s][k2];
  } else {
    if (j < R1)
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
        for (int s = 0; s < 2; ++s) vb[s][k2] = p[s * N3 + base + (j + R1 * k2) * stride];
    F::inverse(vb, va, Y, j, tw);
    if (j < R2)
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
        for (int s = 0; s < 2; ++s) p[s * N3 + base + (j + R2 * j1) * stride] = va[s][j1];
  }
}

// forward FFT along z, multiply by x0 / (E0 + hb2m |k|^2), inverse along z.
// The line's x and y indices are frequency indices at this point.
//   MODE 0: plain damping.
//   MODE 1: read only: add the state's spectral power per |k| shell,
//           sum |F r(k)|^2 over both spinor components, to pow[state][shell].
//   MODE 2: damping times gain[state][shell(k)] (learned preconditioner, or
//           one-hot rows that restrict the step to one shell).
template <typename T, int N, int MODE>
__global__ void __launch_bounds__(LineCfg<N>::THREADS)
k_damp_z(cpx<T>* __restrict__ buf, GridArgs g, DampArgs d, const float* __restrict__ gain,
         double* __restrict__ pow, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = LineCfg<N>;
  using F = LineFFT<T, N, 2>;
  constexpr int YS = line_stride<T, N, 2, 2>();
  constexpr int R1 = C::R1, R2 = C::R2, N3 = N * N * N;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> Ybuf[C::LPW * YS];
  __shared__ double spow[PC_SHELLS];
  load_twiddles<T, N>(tw);
  if (MODE == 1 && threadIdx.x < PC_SHELLS) spow[threadIdx.x] = 0.0;
  int line, j;
  thread_role<N, 2>(threadIdx.x, line, j);
  const int L = blockIdx.x * C::LPW + line;
  int base, stride, a, b;
  line_geom<N, 2>(L, base, stride, a, b);
  cpx<T>* p = buf + size_t(blockIdx.y) * 2 * N3;
  cpx<T>* Y = Ybuf + line * YS;
  cpx<T> va[2][R1], vb[2][R2];
  if (j < R2)
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
      for (int s = 0; s < 2; ++s) va[s][j1] = p[s * N3 + base + (j + R2 * j1) * stride];
  F::forward(va, vb, Y, j, tw);
  double lpow[PC_SHELLS];
  if (MODE == 1)
#pragma unroll
    for (int s = 0; s < PC_SHELLS; ++s) lpow[s] = 0.0;
  if (j < R1) {
    const int ia = a < N / 2 ? a : a - N, ib = b < N / 2 ? b : b - N;
    double kx = g.kunit * double(ia) + g.tw[0];
    double ky = g.kunit * double(ib) + g.tw[1];
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
      int f = j + R1 * k2;
      const int ic = f < N / 2 ? f : f - N;
      double kz = g.kunit * double(ic) + g.tw[2];
      const double kk = kx * kx + ky * ky + kz * kz;
      const int m2 = ia * ia + ib * ib + ic * ic;
      if (MODE == 1) {
        const int sh = k_shell(m2, N);
        double pw = 0.0;
#pragma unroll
        for (int s = 0; s < 2; ++s)
          pw += double(vb[s][k2].re) * double(vb[s][k2].re) + double(vb[s][k2].im) * double(vb[s][k2].im);
#pragma unroll
        for (int s = 0; s < PC_SHELLS; ++s) lpow[s] += (s == sh) ? pw : 0.0;
      } else {
        // the three inverse transforms' 1/N go into the filter
        double mm = d.x0 / (double(N) * N * N) / (d.e0 + d.hb2m * kk);
        if (MODE == 2) mm *= double(gain[size_t(blockIdx.y) * PC_SHELLS + k_shell(m2, N)]);
        const T m = T(mm);
#pragma unroll
        for (int s = 0; s < 2; ++s) vb[s][k2] = m * vb[s][k2];
      }
    }
  }
  if (MODE == 1) {
    __syncthreads();
#pragma unroll
    for (int s = 0; s < PC_SHELLS; ++s) {
      double v = lpow[s];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
      if ((threadIdx.x & 63) == 0) atomicAdd(&spow[s], v);
    }
    __syncthreads();
    if (threadIdx.x < PC_SHELLS)
      atomicAdd(&pow[size_t(blockIdx.y) * PC_SHELLS + threadIdx.x], spow[threadIdx.x]);
    return;
  }
  F::inverse(vb, va, Y, j, tw);
  if (j < R2)
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
      for (int s = 0; s < 2; ++s) p[s * N3 + base + (j + R2 * j1) * stride] = va[s][j1];
}

// inverse FFT along x and phi = psi - (damped residual), in place in buf.
template <typename T, int N>
__global__ void __launch_bounds__(LineCfg<N>::THREADS)
k_damp_inv_x(const cpx<T>* __restrict__ psi, cpx<T>* __restrict__ buf,
             unsigned int* __restrict__ amax, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = LineCfg<N>;
  using F = LineFFT<T, N, 2, x_wave_local<N>()>;
  constexpr int YS = line_stride<T, N, 2, 0>();
  constexpr int R1 = C::R1, R2 = C::R2, N3 = N * N * N;
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> Ybuf[C::LPW * YS];
  load_twiddles<T, N>(tw);
  int line, j;
  thread_role<N, 0>(threadIdx.x, line, j);
  const int L = blockIdx.x * C::LPW + line;
  int base, stride, a, b;
  line_geom<N, 0>(L, base, stride, a, b);
  const size_t soff = size_t(blockIdx.y) * 2 * N3;
  cpx<T>* Y = Ybuf + line * YS;
  cpx<T> va[2][R1], vb[2][R2];
  if (j < R1)
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2)
#pragma unroll
      for (int s = 0; s < 2; ++s) vb[s][k2] = buf[soff + s * N3 + base + (j + R1 * k2) * stride];
  F::inverse(vb, va, Y, j, tw);
  float am = 0.0f;
  if (j < R2)
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        size_t r = soff + s * N3 + base + (j + R2 * j1) * stride;
        const cpx<T> t = psi[r] - va[s][j1];
        buf[r] = t;
        am = fmaxf(am, cabs_max(t));
      }
  if (amax != nullptr) block_amax(am, amax);
}

// ------------------------------------------------------------------ densities
// Pass DIR over a chunk of states accumulates, at every point, the terms of
// rho, tau, J (and the diagnostics s, j) that need d/d(DIR) psi:
//   x: rho, s_x, s_y, s_z, tau_x, j_x, J_y(x), J_z(x)          (slots 0..7)
//   y: tau_y, j_y, J_x(y), J_z(y)                              (slots 8..11)
//   z: tau_z, j_z, J_x(z), J_y(z)                              (slots 12..15)
// with J_k = sum_lm eps_klm Im(psi^dag sigma_m d_l psi).  Partial sums per
// state chunk (blockIdx.y; the first species' chunks, then the second's) go to
// part[chunk][slot][point] and are reduced in fixed order.
template <typename T, int N, int DIR>
__global__ void __launch_bounds__(LineCfg<N>::THREADS)
k_dens_pass(DensArgs grp, GridArgs g, double* __restrict__ part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using C = LineCfg<N>;
  using F = LineFFT<T, N, 2, DIR == 0 && x_wave_local<N>()>;
  constexpr int YS = line_stride<T, N, 2, DIR>();
  constexpr int R1 = C::R1, R2 = C::R2, N3 = N * N * N;
  constexpr int NS = DIR == 0 ? 8 : 4;
  constexpr int SLOT0 = DIR == 0 ? 0 : (DIR == 1 ? 8 : 12);
  __shared__ cpx<T> tw[N];
  __shared__ cpx<T> Ybuf[C::LPW * YS];
  load_twiddles<T, N>(tw);
  int line, j;
  thread_role<N, DIR>(threadIdx.x, line, j);
  const int L = blockIdx.x * C::LPW + line;
  int base, stride, a, b;
  line_geom<N, DIR>(L, base, stride, a, b);
  cpx<T>* Y = Ybuf + line * YS;

  double acc[NS][R1];
#pragma unroll
  for (int q = 0; q < NS; ++q)
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) acc[q][j1] = 0.0;

  // chunks of the flat (group, state) index: every group's states in order;
  // the next state's line is loaded into registers while this one is
  // transformed
  const bool second = int(blockIdx.y) >= grp.sp[0].nchunk;
  const DensSpecies& sp = grp.sp[second ? 1 : 0];
  const int nstate = sp.nstate;
  const int s0 = (int(blockIdx.y) - (second ? grp.sp[0].nchunk : 0)) * grp.chunk;
  const int s1 = min(nstate * grp.ngroup, s0 + grp.chunk);
  auto load_line = [&](int fs, cpx<T> (&dst)[2][R1]) {
    const int t = fs / nstate, st = fs - t * nstate;
    const cpx<T>* p = reinterpret_cast<const cpx<T>*>(sp.psi[t]) + size_t(st) * 2 * N3;
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      const int r = base + (j + R2 * j1) * stride;
      dst[0][j1] = p[r];
      dst[1][j1] = p[N3 + r];
    }
  };
  cpx<T> vn[2][R1];
  if (s0 < s1 && j < R2) load_line(s0, vn);
  for (int fs = s0; fs < s1; ++fs) {
    // derivatives in units of kunit / N: integer multipliers, exact in FP32; the
    // sums are scaled in FP64
    const T ksn = T(grp.kshift[fs / nstate][DIR]);
    cpx<T> v[2][R1], d[2][R1];
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      v[0][j1] = d[0][j1] = vn[0][j1];
      v[1][j1] = d[1][j1] = vn[1][j1];
    }
    if (fs + 1 < s1 && j < R2) load_line(fs + 1, vn);
    F::deriv(d, Y, j, tw, T(1), ksn);
    if (j < R2) {
#pragma unroll
      for (int j1 = 0; j1 < R1; ++j1) {
        cpx<T> u = v[0][j1], w = v[1][j1], du = d[0][j1], dw = d[1][j1];
        // psi^dag sigma d psi for the three Pauli matrices
        cpx<T> sx = conj(u) * dw + conj(w) * du;
        cpx<T> sy = mul_i(conj(w) * du - conj(u) * dw);
        cpx<T> sz = conj(u) * du - conj(w) * dw;
        double tau = double(norm2(du)) + double(norm2(dw));
        double cur = double((conj(u) * du).im) + double((conj(w) * dw).im);
        if (DIR == 0) {
          cpx<T> sxy = conj(u) * w;                 // psi^dag sigma psi pieces
          acc[0][j1] += double(norm2(u)) + double(norm2(w));
          acc[1][j1] += 2.0 * double(sxy.re);
          acc[2][j1] += 2.0 * double(sxy.im);
          acc[3][j1] += double(norm2(u)) - double(norm2(w));
          acc[4][j1] += tau;
          acc[5][j1] += cur;
          acc[6][j1] -= double(sz.im);             // J_y += eps_yxz Im(sz) = -Im
          acc[7][j1] += double(sy.im);             // J_z += eps_zxy Im(sy) = +Im
        } else if (DIR == 1) {
          acc[0][j1] += tau;
          acc[1][j1] += cur;
          acc[2][j1] += double(sz.im);             // J_x += eps_xyz Im(sz)
          acc[3][j1] -= double(sx.im);             // J_z += eps_zyx Im(sx)
        } else {
          acc[0][j1] += tau;
          acc[1][j1] += cur;
          acc[2][j1] -= double(sy.im);             // J_x += eps_xzy Im(sy)
          acc[3][j1] += double(sx.im);             // J_y += eps_yzx Im(sx)
        }
      }
    }
  }
  if (j < R2) {
    double* out = part + size_t(blockIdx.y) * 16 * N3;
    const double u = g.kunit * (1.0 / N);
#pragma unroll
    for (int j1 = 0; j1 < R1; ++j1) {
      int r = base + (j + R2 * j1) * stride;
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        // rho and s carry no derivative, tau two, j and J one
        constexpr int TAU = DIR == 0 ? 4 : 0;
        const double sc = q < TAU ? 1.0 : q == TAU ? u * u : u;
        out[size_t(SLOT0 + q) * N3 + r] = sc * acc[q][j1];
      }
    }
  }
}

// rho, tau, J[3], s[3], j[3] (11 fields) of species blockIdx.y from its chunk
// partials (zero without chunks).
__global__ void k_dens_reduce(const double* __restrict__ part, DensArgs grp, int n3, double scale,
                              const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n3) return;
  const DensSpecies& sp = grp.sp[blockIdx.y];
  const int c0 = blockIdx.y ? grp.sp[0].nchunk : 0;
  double q[16];
  for (int k = 0; k < 16; ++k) q[k] = 0.0;
  for (int c = c0; c < c0 + sp.nchunk; ++c) {
    const double* p = part + size_t(c) * 16 * n3 + r;
    for (int k = 0; k < 16; ++k) q[k] += p[size_t(k) * n3];
  }
  if (scale != 1.0)
    for (int k = 0; k < 16; ++k) q[k] *= scale;
  double* o = sp.dens;
  o[0 * n3 + r] = q[0];                       // rho
  o[1 * n3 + r] = q[4] + q[8] + q[12];        // tau
  o[2 * n3 + r] = q[10] + q[14];              // J_x
  o[3 * n3 + r] = q[6] + q[15];               // J_y
  o[4 * n3 + r] = q[7] + q[11];               // J_z
  o[5 * n3 + r] = q[1];                       // s_x
  o[6 * n3 + r] = q[2];                       // s_y
  o[7 * n3 + r] = q[3];                       // s_z
  o[8 * n3 + r] = q[5];                       // j_x
  o[9 * n3 + r] = q[9];                       // j_y
  o[10 * n3 + r] = q[13];                     // j_z
}

// ------------------------------------------------------------------ conversion
__global__ void k_c128_to_c64(const double2* __restrict__ a, float2* __restrict__ b, size_t n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) b[i] = make_float2(float(a[i].x), float(a[i].y));
}
__global__ void k_c64_to_c128(const float2* __restrict__ a, double2* __restrict__ b, size_t n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) b[i] = make_double2(double(a[i].x), double(a[i].y));
}

void convert_states(const void* src, int src_prec, void* dst, int dst_prec, size_t n,
                    hipStream_t st) {
  if (n == 0) return;
  const unsigned nb = unsigned((n + 255) / 256);
  if (src_prec == 0 && dst_prec == 1)
    hipLaunchKernelGGL(k_c128_to_c64, dim3(nb), dim3(256), 0, st, (const double2*)src, (float2*)dst, n, g_launch_gate);
  else if (src_prec == 1 && dst_prec == 0)
    hipLaunchKernelGGL(k_c64_to_c128, dim3(nb), dim3(256), 0, st, (const float2*)src, (double2*)dst, n, g_launch_gate);
  else
    hipMemcpyAsync(dst, src, n * (src_prec == 0 ? 16 : 8), hipMemcpyDeviceToDevice, st);
}

// ------------------------------------------------------------------ launchers
template <int N> static int ntiles() { return N * N / LineCfg<N>::LPW; }

// Pencil counts the h passes can run with: half, default and double the
// default lines per workgroup, where they tile the plane, fit 1024 threads
// and (double precision, double lines) the LDS.
template <int N> static constexpr bool lines_ok(int lp, int bytes_per_cpx) {
  return lp > 0 && (N * N) % lp == 0 && LineCfg<N>::RT * lp <= 1024 &&
         lp * (2 * Fact<N>::R1 * (Fact<N>::R2 + 1) + 1) * bytes_per_cpx <= 96 * 1024;
}

// Partial sums the last pass forms (each may be null).
struct HParts {
  double *eps, *nrm;
  unsigned int* amax;
};

template <typename T, int N, int LP>
static void launch_h_lp(const void* psi, void* hpsi, int nstate, MeanFieldPtrs mf, GridArgs g,
                        HParts pt, hipStream_t st) {
  dim3 grid(N * N / LineCfg<N, LP>::LPW, nstate), block(LineCfg<N, LP>::THREADS);
  auto p = reinterpret_cast<const cpx<T>*>(psi);
  auto h = reinterpret_cast<cpx<T>*>(hpsi);
  hipLaunchKernelGGL((k_h_pass<T, N, 0, true, false, LP>), grid, block, 0, st, p, h, mf, g, nullptr,
                     nullptr, nullptr, g_launch_gate);
  hipLaunchKernelGGL((k_h_pass<T, N, 1, false, false, LP>), grid, block, 0, st, p, h, mf, g, nullptr,
                     nullptr, nullptr, g_launch_gate);
  hipLaunchKernelGGL((k_h_pass<T, N, 2, false, true, LP>), grid, block, 0, st, p, h, mf, g, pt.eps,
                     pt.nrm, pt.amax, g_launch_gate);
}

// z pass (with U psi) by line pencils, then the x and y parts on LDS slices.
template <typename T, int N>
static void launch_h_plane(const void* psi, void* hpsi, int nstate, MeanFieldPtrs mf, GridArgs g,
                           HParts pt, hipStream_t st) {
  constexpr int D = LineCfg<N>::LPW;
  auto p = reinterpret_cast<const cpx<T>*>(psi);
  auto h = reinterpret_cast<cpx<T>*>(hpsi);
  hipLaunchKernelGGL((k_h_pass<T, N, 2, true, false, D>), dim3(N * N / D, nstate),
                     dim3(LineCfg<N>::THREADS), 0, st, p, h, mf, g, nullptr, nullptr, nullptr,
                     g_launch_gate);
  hipLaunchKernelGGL((k_h_plane<T, N>), dim3(N, nstate), dim3(PlaneCfg<N>::THREADS), 0, st, p, h,
                     mf, g, pt.eps, pt.nrm, pt.amax, g_launch_gate);
}

// lines: 0 = default, H_PLANE = x and y on LDS slices, else pencils per
// workgroup of the three line passes (one of h_pass_lines).  Returns the
// eps partials (workgroups) per state, or 0 if lines is not supported.
template <typename T, int N>
static int launch_apply_h(const void* psi, void* hpsi, int nstate, MeanFieldPtrs mf, GridArgs g,
                          HParts pt, int lines, hipStream_t st) {
  constexpr int D = LineCfg<N>::LPW;
  constexpr int H = (D / 2 > 0 && lines_ok<N>(D / 2, sizeof(cpx<T>))) ? D / 2 : D;
  constexpr int W = lines_ok<N>(2 * D, sizeof(cpx<T>)) ? 2 * D : D;
  constexpr bool PL = plane_fits<T, N>();
  if (lines == 0) lines = plane_fits<T, N>() ? H_PLANE : D;
  if (lines == H_PLANE) {
    if constexpr (PL) {
      launch_h_plane<T, N>(psi, hpsi, nstate, mf, g, pt, st);
      return N;
    }
    return 0;
  }
  if (lines == D) { launch_h_lp<T, N, D>(psi, hpsi, nstate, mf, g, pt, st); return N * N / D; }
  if (lines == H) { launch_h_lp<T, N, H>(psi, hpsi, nstate, mf, g, pt, st); return N * N / H; }
  if (lines == W) { launch_h_lp<T, N, W>(psi, hpsi, nstate, mf, g, pt, st); return N * N / W; }
  return 0;
}

// Candidates of the tuner: the slice variant (where it fits), then half,
// default and double pencils (deduplicated).  Returns the count.
template <typename T, int N> static int lines_list(int* out) {
  constexpr int D = LineCfg<N>::LPW;
  int k = 0;
  if (plane_fits<T, N>()) out[k++] = H_PLANE;
  const int c[3] = {(D / 2 > 0 && lines_ok<N>(D / 2, sizeof(cpx<T>))) ? D / 2 : D, D,
                    lines_ok<N>(2 * D, sizeof(cpx<T>)) ? 2 * D : D};
  for (int i = 0; i < 3; ++i) {
    bool dup = false;
    for (int m = 0; m < k; ++m) dup = dup || out[m] == c[i];
    if (!dup) out[k++] = c[i];
  }
  return k;
}

template <typename T, int N> static int lines_default() {
  return plane_fits<T, N>() ? H_PLANE : LineCfg<N>::LPW;
}

int grid_ntiles(int n) {
  int r = 0;
  SKY_DISPATCH_N(n, r = std::max(2 * ntiles<NN>(), NN));
  return r;   // room for the h passes at half the default pencils, or one per slice
}

int h_pass_lines(int n, int prec, int* out) {
  int k = 0;
  if (prec == 0) SKY_DISPATCH_N(n, k = (lines_list<double, NN>(out)))
  else SKY_DISPATCH_N(n, k = (lines_list<float, NN>(out)))
  return k;
}

int damp_slices_available(int n, int prec) {
  int v = 0;
  if (prec == 0) SKY_DISPATCH_N(n, v = (damp_slices_fit<double, NN>() ? 1 : 0))
  else SKY_DISPATCH_N(n, v = (damp_slices_fit<float, NN>() ? 1 : 0))
  return v;
}

int h_pass_default(int n, int prec) {
  int v = 0;
  if (prec == 0) SKY_DISPATCH_N(n, v = (lines_default<double, NN>()))
  else SKY_DISPATCH_N(n, v = (lines_default<float, NN>()))
  return v;
}

int apply_h(int n, int prec, const void* psi, void* hpsi, int nstate, MeanFieldPtrs mf,
            GridArgs g, double* eps_part, double* eps, hipStream_t st, int lines,
            unsigned int* amax, double* nrm) {
  if (nstate <= 0) return 1;
  int nt = 0;
  double* np = nrm ? eps_part + size_t(nstate) * grid_ntiles(n) : nullptr;
  const HParts pt{eps ? eps_part : nullptr, np, amax};
  if (prec == 0) SKY_DISPATCH_N(n, nt = (launch_apply_h<double, NN>(psi, hpsi, nstate, mf, g, pt, lines, st)))
  else SKY_DISPATCH_N(n, nt = (launch_apply_h<float, NN>(psi, hpsi, nstate, mf, g, pt, lines, st)))
  if (nt == 0) return 0;
  if (eps_part && eps) sum_partials(eps_part, np, nt, nstate, eps, nrm, st);
  return 1;
}

// stage 0: the whole step; 1: residual, forward x and y and (with shell_pow)
// the shell powers, leaving the partial spectrum in phi; 2: the z filter
// (with gain) and the inverse passes, continuing from stage 1.
template <typename T, int N>
static void launch_damp(const void* psi, const void* hpsi, const double* eps, void* phi,
                        int nstate, GridArgs g, DampArgs d, double* r2_part, const float* gain,
                        double* shell_pow, int stage, int xy, unsigned int* amax, hipStream_t st) {
  dim3 grid(ntiles<N>(), nstate), block(LineCfg<N>::THREADS);
  dim3 pgrid(N, nstate), pblock(PlaneCfg<N>::THREADS);
  auto p = reinterpret_cast<const cpx<T>*>(psi);
  auto h = reinterpret_cast<const cpx<T>*>(hpsi);
  auto o = reinterpret_cast<cpx<T>*>(phi);
  const bool pl = damp_slices_fit<T, N>() && xy != 0;
  if (stage != 2) {
    if (pl) {
      if constexpr (damp_slices_fit<T, N>())
        hipLaunchKernelGGL((k_damp_fwd_xy<T, N>), pgrid, pblock, 0, st, p, h, eps, o, g, r2_part, g_launch_gate);
    } else {
      hipLaunchKernelGGL((k_damp_fwd_x<T, N>), grid, block, 0, st, p, h, eps, o, g, r2_part, g_launch_gate);
      hipLaunchKernelGGL((k_damp_y<T, N, false>), grid, block, 0, st, o, g_launch_gate);
    }
    if (shell_pow)
      hipLaunchKernelGGL((k_damp_z<T, N, 1>), grid, block, 0, st, o, g, d, nullptr, shell_pow, g_launch_gate);
  }
  if (stage == 1) return;
  if (gain)
    hipLaunchKernelGGL((k_damp_z<T, N, 2>), grid, block, 0, st, o, g, d, gain, nullptr, g_launch_gate);
  else
    hipLaunchKernelGGL((k_damp_z<T, N, 0>), grid, block, 0, st, o, g, d, nullptr, nullptr, g_launch_gate);
  if (pl) {
    if constexpr (damp_slices_fit<T, N>())
      hipLaunchKernelGGL((k_damp_inv_xy<T, N>), pgrid, pblock, 0, st, p, o, amax, g_launch_gate);
  } else {
    hipLaunchKernelGGL((k_damp_y<T, N, true>), grid, block, 0, st, o, g_launch_gate);
    hipLaunchKernelGGL((k_damp_inv_x<T, N>), grid, block, 0, st, p, o, amax, g_launch_gate);
  }
}

void damped_step(int n, int prec, const void* psi, const void* hpsi, const double* eps,
                 void* phi, int nstate, GridArgs g, double x0, double e0, double hb2m,
                 double* r2_part, double* r2, hipStream_t st, const float* gain,
                 double* shell_pow, int stage, int xy, unsigned int* amax) {
  if (nstate <= 0) return;
  DampArgs d{x0, e0, hb2m};
  if (prec == 0) SKY_DISPATCH_N(n, launch_damp<double, NN>(psi, hpsi, eps, phi, nstate, g, d, r2_part, gain, shell_pow, stage, xy, amax, st))
  else SKY_DISPATCH_N(n, launch_damp<float, NN>(psi, hpsi, eps, phi, nstate, g, d, r2_part, gain, shell_pow, stage, xy, amax, st))
  if (stage == 2) return;
  int nt = 0;
  if (prec == 0)
    SKY_DISPATCH_N(n, nt = (damp_slices_fit<double, NN>() && xy != 0) ? NN : ntiles<NN>())
  else
    SKY_DISPATCH_N(n, nt = (damp_slices_fit<float, NN>() && xy != 0) ? NN : ntiles<NN>())
  if (r2) sum_partials(r2_part, nullptr, nt, nstate, r2, nullptr, st);
}

// Workgroups of a density pass that a CU holds at once, by registers (the y
// pass; where it matters, the chunk bound of the caller being larger).  A
// constant, so that the order of the sums is that of the grid and form alone.
template <typename T, int N> constexpr int dens_groups_per_cu() {
  if (sizeof(T) == 8) return N >= 48 ? 1 : N >= 24 ? 2 : 3;
  return N >= 48 ? 2 : N == 32 ? 3 : 4;
}
constexpr int CUS = 256;

// Chunks of states: each is a row of workgroups over the grid's lines, the card
// holds `rows` of them at once, and a pass takes about ceil(chunks / rows) times
// a chunk's states.  More chunks cost partial sums (16 doubles per point and
// chunk, written and read: as much as the three passes' reads of 16/3
// complex64 or 8/3 complex128 states).  The count, up to the caller's bound,
// is the one whose estimate is least: where many rows fit, as many as fill the
// card once, where few do (48^3 and 64^3), several rounds of shorter ones,
// since one round cannot be cut to fit two species.
// 640 + 160 complex64 states at 32^3: 32 chunks per species and launches of its
// own took 386 us for the passes and 62 for the sums, now 301 and 25.
// Densities and mean field by 32 chunks per species, by one round and by this
// rule (ms): complex128 48^3 x 1600 + 400 6.27, 6.72 and 5.03, x 1000 + 1000 6.32,
// 8.26 and 4.99; 64^3 x 300 + 75 3.45, 3.21 and 2.28; complex64 48^3 x 1600 + 400
// 3.14, 2.65 and 2.60, x 1000 + 1000 3.14, 2.73 and 2.58.
template <typename T, int N>
static void launch_dens(DensArgs& grp, int nspecies, int nchunk_max, GridArgs g, double* part,
                        hipStream_t st) {
  int total = 0;
  for (int q = 0; q < nspecies; ++q) total += grp.ngroup * grp.sp[q].nstate;
  auto chunks = [&](int c) {
    int k = 0;
    for (int q = 0; q < nspecies; ++q) k += (grp.ngroup * grp.sp[q].nstate + c - 1) / c;
    return k;
  };
  const double rows = double(dens_groups_per_cu<T, N>() * CUS) / ntiles<N>();
  const double sums = sizeof(T) == 8 ? 8.0 / 3.0 : 16.0 / 3.0;
  int chunk = 1;
  double best = HUGE_VAL;
  for (int want = nchunk_max; want >= nspecies; --want) {
    // the smallest chunk whose count over all species does not exceed `want`
    int c = std::max(1, (total + want - 1) / want);
    while (chunks(c) > want) ++c;
    const double cost = std::ceil(chunks(c) / rows) * c + sums * chunks(c) / rows;
    if (cost <= best) {
      best = cost;
      chunk = c;
    }
  }
  grp.chunk = chunk;
  for (int q = 0; q < nspecies; ++q)
    grp.sp[q].nchunk = (grp.ngroup * grp.sp[q].nstate + chunk - 1) / chunk;
  const int nchunk = chunks(chunk);
  if (nchunk > 0) {
    dim3 grid(ntiles<N>(), nchunk), block(LineCfg<N>::THREADS);
    hipLaunchKernelGGL((k_dens_pass<T, N, 0>), grid, block, 0, st, grp, g, part, g_launch_gate);
    hipLaunchKernelGGL((k_dens_pass<T, N, 1>), grid, block, 0, st, grp, g, part, g_launch_gate);
    hipLaunchKernelGGL((k_dens_pass<T, N, 2>), grid, block, 0, st, grp, g, part, g_launch_gate);
  }
  constexpr int n3 = N * N * N;
  hipLaunchKernelGGL(k_dens_reduce, dim3((n3 + 255) / 256, nspecies), dim3(256), 0, st,
                     (const double*)part, grp, n3, 1.0 / std::max(1, grp.ngroup), g_launch_gate);
}

int densities(int n, int prec, int nspecies, const void* const (*psi)[DENS_MAX_GROUPS],
              const int* nstate, double* const* dens, const GridArgs* g, int ngroup,
              int nchunk_max, double* part, hipStream_t st) {
  if (ngroup < 0 || ngroup > DENS_MAX_GROUPS || nspecies < 1 || nspecies > 2 || nchunk_max < nspecies)
    return 0;
  // one launch per pass over all species and groups (twists): each species'
  // flat (group, state) index is cut into chunks of consecutive states
  DensArgs grp{};
  grp.ngroup = ngroup;
  for (int t = 0; t < ngroup; ++t)
    for (int a = 0; a < 3; ++a) grp.kshift[t][a] = g[t].tw[a] / g[0].kunit;
  for (int q = 0; q < nspecies; ++q) {
    for (int t = 0; t < ngroup; ++t) grp.sp[q].psi[t] = psi[q][t];
    grp.sp[q].nstate = std::max(0, nstate[q]);
    grp.sp[q].dens = dens[q];
  }
  if (prec == 0) SKY_DISPATCH_N(n, launch_dens<double, NN>(grp, nspecies, nchunk_max, g[0], part, st))
  else SKY_DISPATCH_N(n, launch_dens<float, NN>(grp, nspecies, nchunk_max, g[0], part, st))
  return 1;
}

}  // namespace sky
