// Batched radix FFTs along one grid axis, staged through LDS.
//
// Sec. 2.2 of the paper takes every derivative of a wave function with FFTs.
// Here a line of N points (one axis of the box, all spin components) is
// transformed by a two-stage Cooley-Tukey factorisation N = R1 * R2:
//
//   stage A: thread j (< R2) holds the points j + R2*j1 (j1 < R1) in
//            registers, does a length-R1 DFT over j1 and the inter-stage
//            twiddle w_N^(j*k1);
//   exchange through a small per-line LDS buffer;
//   stage B: thread j (< R1) holds the frequencies j + R1*k2 (k2 < R2) and
//            does a length-R2 DFT over k2.
//
// A spectral multiplier is applied to the stage-B registers, and the inverse
// runs the same stages backwards, so a derivative F^-1[m(k) F psi] costs two
// LDS exchanges and returns the result to the same thread/positions that
// loaded the input.  Forward sign: X[k] = sum_n x[n] exp(-2 pi i n k / N);
// neither direction scales: the 1/N of the inverse goes into the multiplier.
//
// The complex64 passes are bound by vector issue as much as by memory (48^3:
// the z pass of h psi issues in 92% of its cycles, the slice pass in 75%), so the
// transforms are kept lean: twiddle-free and multiply-add forms of the small DFTs, no products
// by w^0, one multiplier per frequency, twiddles from a table.
#pragma once

#include "sky_common.h"

namespace sky {

// ---------------------------------------------------------------- small DFTs
template <typename T, int R, bool INV> struct DFT;

template <typename T, bool INV> struct DFT<T, 1, INV> {
  __device__ static inline void run(cpx<T>*) {}
};

template <typename T, bool INV> struct DFT<T, 2, INV> {
  __device__ static inline void run(cpx<T>* v) {
    cpx<T> a = v[0], b = v[1];
    v[0] = a + b;
    v[1] = a - b;
  }
};

template <typename T, bool INV> struct DFT<T, 3, INV> {
  __device__ static inline void run(cpx<T>* v) {
    constexpr T s3 = T(0.86602540378443864676);
    cpx<T> t1 = v[1] + v[2], t2 = v[1] - v[2];
    cpx<T> m = v[0] - T(0.5) * t1;
    cpx<T> it2 = mul_i(t2);                   // i (v1 - v2)
    v[0] = v[0] + t1;
    if (INV) { v[1] = m + s3 * it2; v[2] = m - s3 * it2; }
    else     { v[1] = m - s3 * it2; v[2] = m + s3 * it2; }
  }
};

template <typename T, bool INV> struct DFT<T, 4, INV> {
  __device__ static inline void run(cpx<T>* v) {
    cpx<T> a = v[0] + v[2], b = v[0] - v[2];
    cpx<T> c = v[1] + v[3], d = mul_i(v[1] - v[3]);
    v[0] = a + c;
    v[2] = a - c;
    if (INV) { v[1] = b + d; v[3] = b - d; }
    else     { v[1] = b - d; v[3] = b + d; }
  }
};

// 6 = 2 * 3 as a prime-factor transform: with n = 3 n1 + 2 n2 and
// k = 3 k1 + 4 k2 (mod 6) the two factors need no twiddles between them (36
// real operations; the common-factor split took 44).
template <typename T, bool INV> struct DFT<T, 6, INV> {
  __device__ static inline void run(cpx<T>* v) {
    cpx<T> s[3] = {v[0] + v[3], v[2] + v[5], v[4] + v[1]};
    cpx<T> d[3] = {v[0] - v[3], v[2] - v[5], v[4] - v[1]};
    DFT<T, 3, INV>::run(s);
    DFT<T, 3, INV>::run(d);
    v[0] = s[0]; v[4] = s[1]; v[2] = s[2];
    v[3] = d[0]; v[1] = d[1]; v[5] = d[2];
  }
};

// 8 as even and odd 4-point transforms; the eighth-turn factors
// (1 -+ i) / sqrt(2) enter the last additions as multiply-adds (52 real
// operations; with general twiddle products 60).
template <typename T, bool INV> struct DFT<T, 8, INV> {
  __device__ static inline void run(cpx<T>* v) {
    constexpr T r2 = T(0.70710678118654752440);  // 1/sqrt(2)
    cpx<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    DFT<T, 4, INV>::run(e);
    DFT<T, 4, INV>::run(o);
    // o[1] w, o[2] w^2, o[3] w^3 with w = exp(-+ i pi / 4); the first and last
    // without their 1/sqrt(2)
    const cpx<T> t1 = INV ? mk(o[1].re - o[1].im, o[1].im + o[1].re)
                          : mk(o[1].re + o[1].im, o[1].im - o[1].re);
    const cpx<T> t2 = INV ? mul_i(o[2]) : mk(o[2].im, -o[2].re);
    const cpx<T> t3 = INV ? mk(-o[3].re - o[3].im, o[3].re - o[3].im)
                          : mk(o[3].im - o[3].re, -o[3].re - o[3].im);
    v[0] = e[0] + o[0];
    v[4] = e[0] - o[0];
    v[1] = mk(e[1].re + r2 * t1.re, e[1].im + r2 * t1.im);
    v[5] = mk(e[1].re - r2 * t1.re, e[1].im - r2 * t1.im);
    v[2] = e[2] + t2;
    v[6] = e[2] - t2;
    v[3] = mk(e[3].re + r2 * t3.re, e[3].im + r2 * t3.im);
    v[7] = mk(e[3].re - r2 * t3.re, e[3].im - r2 * t3.im);
  }
};

// ---------------------------------------------------------------- line engine
// Launch shape of the line kernels for grid size N.
// Lines (pencils) per workgroup: LP = 0 picks the default, otherwise LP.
template <int N, int LP = 0> struct LineCfg {
  static constexpr int R1 = Fact<N>::R1, R2 = Fact<N>::R2;
  static constexpr int RT = R1 > R2 ? R1 : R2;          // threads per line
  static constexpr int LPW = LP ? LP : ((RT == 4) ? 64 : 32);   // lines per workgroup
  static constexpr int THREADS = RT * LPW;
  static_assert((N * N) % LPW == 0, "lines must tile the plane");
  static_assert(THREADS <= 1024, "workgroup too large");
};

// Orders a line's LDS writes before its threads' reads: a workgroup barrier, or,
// where the threads of every line belong to one wave (WL), only the order of
// that wave's own LDS operations.
template <bool WL> __device__ inline void line_barrier() {
  if (WL) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// FFT of S spinor components along one line, S in {1, 2}.
// Y is the line's LDS exchange buffer of YSIZE complex values.
//
// Each direction holds one barrier, between the writes of its first stage and
// the reads of its second.  None is needed around it: the second stage of
// forward reads the row (s, j) that the first of inverse, in the same thread,
// writes, and the second of inverse reads the column j that the first of
// forward writes, so transforms with the same (line, j) -> thread map may
// follow each other.  A caller that uses Y otherwise, or with another map,
// separates the uses itself.  WL: the lines are wave-local (line_barrier).
template <typename T, int N, int S, bool WL = false> struct LineFFT {
  static constexpr int R1 = Fact<N>::R1, R2 = Fact<N>::R2;
  static constexpr int YROW = R2 + 1;                 // padded row
  static constexpr int YSIZE = S * R1 * YROW + 1;     // odd stride between lines

  // va[s][j1] at positions j + R2*j1  ->  vb[s][k2] at frequencies j + R1*k2
  __device__ static inline void forward(cpx<T> (&va)[S][R1], cpx<T> (&vb)[S][R2],
                                        cpx<T>* Y, int j, const cpx<T>* twN) {
    if (j < R2) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        DFT<T, R1, false>::run(va[s]);
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1)
          Y[(s * R1 + k1) * YROW + j] = k1 ? va[s][k1] * twN[j * k1] : va[s][k1];
      }
    }
    line_barrier<WL>();
    if (j < R1) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) vb[s][k2] = Y[(s * R1 + j) * YROW + k2];
        DFT<T, R2, false>::run(vb[s]);
      }
    }
  }

  // vb[s][k2] at frequencies j + R1*k2  ->  va[s][j1] at positions j + R2*j1
  __device__ static inline void inverse(cpx<T> (&vb)[S][R2], cpx<T> (&va)[S][R1],
                                        cpx<T>* Y, int j, const cpx<T>* twN) {
    if (j < R1) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        DFT<T, R2, true>::run(vb[s]);
#pragma unroll
        for (int j2 = 0; j2 < R2; ++j2)
          Y[(s * R1 + j) * YROW + j2] = j2 ? vb[s][j2] * conj(twN[j2 * j]) : vb[s][j2];
      }
    }
    line_barrier<WL>();
    if (j < R2) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1) va[s][k1] = Y[(s * R1 + k1) * YROW + j];
        DFT<T, R1, true>::run(va[s]);
      }
    }
  }

  // In-place spectral derivative i*(k + kshift) along the line, Nyquist kept
  // (k = -N/2); kshift is the Bloch shift of twisted boundary conditions.  kun
  // and ksn are the wave-number unit and kshift divided by N (the inverse's
  // scale); a caller that scales the result itself passes 1 and kshift / unit.
  // R2 is even, so whether a frequency wraps depends on k2 alone.
  __device__ static inline void deriv(cpx<T> (&va)[S][R1], cpx<T>* Y, int j,
                                      const cpx<T>* twN, T kun, T ksn) {
    cpx<T> vb[S][R2];
    forward(va, vb, Y, j, twN);
    if (j < R1) {
      const T tj = T(j);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) {
        const T k = kun * (tj + T(R1 * k2 - (k2 < R2 / 2 ? 0 : N))) + ksn;
#pragma unroll
        for (int s = 0; s < S; ++s) vb[s][k2] = mul_i(k * vb[s][k2]);
      }
    }
    inverse(vb, va, Y, j, twN);
  }
};

// Whether the threads of an x line (consecutive, RT of them) share a wave.
template <int N> constexpr bool x_wave_local() { return 64 % LineCfg<N>::RT == 0; }

// Distance in LDS between the exchange buffers of consecutive lines of a
// workgroup (complex values).  Along y and z consecutive lanes hold
// consecutive lines, which the odd YSIZE spreads over the banks.  Along x a
// wave holds 64 / RT lines of RT consecutive threads; for those the strides
// below put the words of every exchange access of a wave in distinct banks,
// for 32 and for 64 banks of 4 bytes and 8- or 16-byte values (counted on
// the CPU for each access of the two stages; N = 24, whose lines straddle
// waves, takes the stride with the fewest shared banks).
template <int N, int S> constexpr int x_line_stride() {
  constexpr int one[6] = {12, 20, 38, 40, 56, 72};     // S = 1
  constexpr int two[6] = {20, 44, 70, 72, 120, 152};   // S = 2
  constexpr int i = N == 8 ? 0 : N == 16 ? 1 : N == 24 ? 2 : N == 32 ? 3 : N == 48 ? 4 : 5;
  return S == 1 ? one[i] : two[i];
}
template <typename T, int N, int S, int DIR> constexpr int line_stride() {
  constexpr int v = DIR == 0 ? x_line_stride<N, S>() : LineFFT<T, N, S>::YSIZE;
  static_assert(v >= S * Fact<N>::R1 * (Fact<N>::R2 + 1), "exchange buffer too small");
  return v;
}

// The same two-stage FFT with the exchange done in place, in the line's own
// N slots: element idx of spin component s lives at base[s * sp + idx * es]
// (es = 1 for a row, the row pitch for a column of an LDS slice).  Stage A
// of thread j writes exactly the slots it loaded (k1 * R2 + j), so only the
// stage boundaries need barriers; the inverse starts with one, since its
// stage-B writes land on slots other threads have just loaded from.  Every
// thread of the workgroup must call these (barriers).
template <typename T, int N, int S> struct LineFFTInPlace {
  static constexpr int R1 = Fact<N>::R1, R2 = Fact<N>::R2;

  // va[s][j1] at positions j + R2*j1  ->  vb[s][k2] at frequencies j + R1*k2
  __device__ static inline void forward(cpx<T> (&va)[S][R1], cpx<T> (&vb)[S][R2], cpx<T>* base,
                                        int sp, int es, int j, const cpx<T>* twN) {
    if (j < R2) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        DFT<T, R1, false>::run(va[s]);
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1)
          base[s * sp + (k1 * R2 + j) * es] = k1 ? va[s][k1] * twN[j * k1] : va[s][k1];
      }
    }
    __syncthreads();
    if (j < R1) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) vb[s][k2] = base[s * sp + (j * R2 + k2) * es];
        DFT<T, R2, false>::run(vb[s]);
      }
    }
    __syncthreads();
  }

  // vb[s][k2] at frequencies j + R1*k2  ->  va[s][j1] at positions j + R2*j1
  __device__ static inline void inverse(cpx<T> (&vb)[S][R2], cpx<T> (&va)[S][R1], cpx<T>* base,
                                        int sp, int es, int j, const cpx<T>* twN) {
    __syncthreads();
    if (j < R1) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        DFT<T, R2, true>::run(vb[s]);
#pragma unroll
        for (int j2 = 0; j2 < R2; ++j2)
          base[s * sp + (j * R2 + j2) * es] = j2 ? vb[s][j2] * conj(twN[j2 * j]) : vb[s][j2];
      }
    }
    __syncthreads();
    if (j < R2) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1) va[s][k1] = base[s * sp + (k1 * R2 + j) * es];
        DFT<T, R1, true>::run(va[s]);
      }
    }
    __syncthreads();
  }
};

// cos(2 pi m / 192), m = 0 .. 48 (192 is a multiple of every grid size).
static __device__ const double TW_COS[49] = {
    1.0, 0.99946458747636568, 0.99785892323860348, 0.99518472667219693,
    0.99144486137381038, 0.98664333208487898, 0.98078528040323043, 0.97387697927733363,
    0.96592582628906831, 0.95694033573220882, 0.94693012949510569, 0.93590592675732565,
    0.92387953251128674, 0.91086382492117579, 0.89687274153268826, 0.88192126434835505,
    0.8660254037844386, 0.84920218152657889, 0.83146961230254524, 0.81284668459161524,
    0.79335334029123517, 0.77301045336273699, 0.75183980747897738, 0.72986407269783571,
    0.70710678118654757, 0.68359230202287125, 0.65934581510006884, 0.63439328416364549,
    0.60876142900872066, 0.58247769686780215, 0.55557023301960218, 0.52806785065036799,
    0.5, 0.47139673682599764, 0.4422886902190013, 0.41270702980439472,
    0.38268343236508978, 0.35225004792123349, 0.32143946530316159, 0.29028467725446239,
    0.25881904510252074, 0.2270762630343732, 0.19509032201612828, 0.16289547339458874,
    0.1305261922200516, 0.098017140329560604, 0.065403129230143062, 0.032719082821776144,
    0.0};

// exp(-2 pi i m / N), m < N, into LDS (all threads of the block help), from
// the quarter-wave table: its loads overlap the caller's line loads, where
// the sine and cosine of each workgroup's 48 angles cost its first wave about
// 200 instructions.
template <typename T, int N> __device__ inline void load_twiddles(cpx<T>* tw) {
  static_assert(192 % N == 0, "the table holds the 192nd roots of unity");
  for (int m = threadIdx.x; m < N; m += blockDim.x) {
    const int i = m * (192 / N), q = i / 48, r = i % 48;
    const double a = TW_COS[r], b = TW_COS[48 - r];   // cos, sin of the angle past quadrant q
    const double c = q == 0 ? a : q == 1 ? -b : q == 2 ? -a : b;
    const double s = q == 0 ? b : q == 1 ? a : q == 2 ? -b : -a;
    tw[m] = mk(T(c), T(-s));
  }
  __syncthreads();
}

// Geometry of line number L along axis DIR (0 = x, 1 = y, 2 = z):
// offset of its first point and the stride between its points.
template <int N, int DIR> __device__ inline void line_geom(int L, int& base, int& stride,
                                                           int& a, int& b) {
  a = L % N;
  b = L / N;
  if (DIR == 0) { base = b * N * N + a * N; stride = 1; }          // (y, z)
  else if (DIR == 1) { base = b * N * N + a; stride = N; }         // (x, z)
  else { base = b * N + a; stride = N * N; }                       // (x, y)
}

// Thread -> (line within workgroup, role j).  Along x the role varies
// fastest so consecutive threads touch consecutive points; along y and z
// the line varies fastest so consecutive threads touch consecutive x.
template <int N, int DIR, int LP = 0> __device__ inline void thread_role(int t, int& line, int& j) {
  constexpr int RT = LineCfg<N, LP>::RT, LPW = LineCfg<N, LP>::LPW;
  if (DIR == 0) { j = t % RT; line = t / RT; }
  else { j = t / LPW; line = t % LPW; }
}

}  // namespace sky
