// Dense complex FP64 products on the FP64 matrix cores (MFMA 16x16x4).
//
// Sec. 3.3.1: the overlap I = <phi|phi> and subspace Hamiltonian
// H = <phi|h phi> are inner products of all state pairs, computed for the
// lower triangle only (Fig. 3).  Sec. 3.3.3: the orthonormalised, diagonal
// states are built with one product psi = phi (C Z) (step 3e).
//
// Every wave owns an output sub-tile of 16 x 16 blocks and loads its operands
// from L2 in the layout of the matrix instruction.  Staging 64 x 64 tiles in
// LDS moved half the operand bytes, but the matrix cores waited at its two
// barriers per chunk, and ragged orders left quarters of the tiles dead.
#include <algorithm>
#include <type_traits>

#include "mfma_f64.h"
#include "sky_kernels.h"

namespace sky {

namespace {
using mfma::GT;
using mfma::KC;
using mfma::TM;

constexpr int NXCD = 8;   // workgroups are dealt to the XCDs in turn, each has its own L2

// Lower-triangle tile pair number p -> (ta, tb), ta >= tb.
__device__ inline void tri_pair(int p, int& ta, int& tb) {
  int a = int((sqrt(8.0 * p + 1.0) - 1.0) * 0.5);
  while ((a + 1) * (a + 2) / 2 <= p) ++a;
  while (a * (a + 1) / 2 > p) --a;
  ta = a;
  tb = p - a * (a + 1) / 2;
}

// A wave's sub-tile of NB x NB blocks of 16 x 16, its operands loaded from
// L2 straight in the layout of the matrix instruction: lane (r, kq) holds row
// (or column) 16 i + r at contraction index kq of each step of four.
template <int NB>
struct Sub {
  mfma::d4 re[NB][NB], im[NB][NB];
  __device__ inline Sub() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) re[i][j] = im[i][j] = mfma::d4{0, 0, 0, 0};
  }
  // += conj(a) b^T (CONJA) or a b^T over one step
  template <bool CONJA>
  __device__ inline void step(const double2 (&a)[NB], const double2 (&b)[NB]) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const double ai = CONJA ? -a[i].y : a[i].y;
        re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, re[i][j], 0, 0, 0);
        im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].y, im[i][j], 0, 0, 0);
        re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, b[j].y, re[i][j], 0, 0, 0);
        im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, b[j].x, im[i][j], 0, 0, 0);
      }
  }
};
constexpr int KQ = KC / 4;   // steps per chunk

// ----------------------------------------------------------- overlap (lower)
// part[(z*npair + pair)*split + s][64*64] = sum over chunk s of conj(A) B^T,
// the blocks of the 64 x 64 tile pairs that hold elements of the lower triangle.
// One wave per 16 NB x 16 NB sub-tile of the triangle, split s and product z;
// the waves need neither LDS nor barriers.  The loads of a step are issued as
// soon as the step before frees their registers, three steps (of 16 matrix
// instructions) ahead.  Rows past m read the last row; their results are
// never read.  Grid (ceil(nsub / 4), split, nz), dealt out so that the
// sub-tiles and both products of one split run on one XCD and share its L2.
// Bound by the matrix cores: 150 states at 24^3, both products, 187 us with
// tiles in LDS, now 114 (60 TF over its sub-tiles); 8 states at 16^3 22.5 ->
// 10.2 us.  Sub-tiles of one block up to 16 states.
template <int NB>
__global__ void __launch_bounds__(GT)
k_overlap_lower(const double2* __restrict__ A, const double2* __restrict__ B0,
                const double2* __restrict__ B1, int m, long k, int split, double2* __restrict__ part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  constexpr int SUB = 16 * NB, PER = TM / SUB;
  int w4 = blockIdx.x, s = blockIdx.y, z = blockIdx.z;
  if (split % NXCD == 0) {
    const int ng = gridDim.x, id = w4 + ng * (s + split * z), per = ng * int(gridDim.z), idx = id / NXCD;
    s = idx / per * NXCD + id % NXCD;
    w4 = idx % per % ng;
    z = idx % per / ng;
  }
  const int nt = (m + TM - 1) / TM, npair = nt * (nt + 1) / 2, ns = (m + SUB - 1) / SUB;
  const int lane = threadIdx.x & 63, r = lane & 15, kq = lane >> 4;
  const int u = __builtin_amdgcn_readfirstlane(w4 * (GT / 64) + (threadIdx.x >> 6));
  if (u >= ns * (ns + 1) / 2) return;
  int ua, ub;
  tri_pair(u, ua, ub);
  const long nck = k / KC;
  const long c0 = nck * s / split, c1 = nck * (s + 1) / split;
  const double2* B = z ? B1 : B0;
  const double2 *pa[NB], *pb[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    pa[i] = A + size_t(min(ua * SUB + 16 * i + r, m - 1)) * k + kq;
    pb[i] = B + size_t(min(ub * SUB + 16 * i + r, m - 1)) * k + kq;
  }
  double2 a[KQ][NB], b[KQ][NB];
  auto load = [&](long c, int q) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      a[q][i] = pa[i][c * KC + 4 * q];
      b[q][i] = pb[i][c * KC + 4 * q];
    }
  };
  Sub<NB> acc;
  if (c0 < c1)
#pragma unroll
    for (int q = 0; q < KQ; ++q) load(c0, q);
  for (long c = c0; c < c1; ++c) {
    const long cn = min(c + 1, c1 - 1);
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      acc.template step<true>(a[q], b[q]);
      load(cn, q);
    }
  }
  int ta = ua / PER, tb = ub / PER;
  const int pair = ta * (ta + 1) / 2 + tb;
  double2* out = part + ((size_t(z) * npair + pair) * split + s) * TM * TM +
                 (ua % PER * SUB) * TM + ub % PER * SUB;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        out[(16 * i + 4 * e + kq) * TM + 16 * j + r] = make_double2(acc.re[i][j][e], acc.im[i][j][e]);
}

// C[a][b] = scale * sum_s part[..][s][..] in order of s on the lower
// triangle, the upper one mirrored from it and the diagonal made real.  Grid
// (npair * RB^2, nz): one 16 x 16 block of a tile pair per workgroup, one
// element per thread, eight partials in flight.  Bound by the partials' read
// once enough workgroups are in flight: with one workgroup per tile pair and
// a loop over its 4096 elements the 12 workgroups of 150 states x 64 splits
// took 274 us for 50 MB, now 6.4 us.  The mirrored block goes out through
// LDS, so that both writes are coalesced.
constexpr int RB = TM / 16;   // 16 x 16 blocks per tile side
__global__ void __launch_bounds__(256)
k_overlap_reduce(const double2* __restrict__ part, int npair, int split, int m, double scale,
                 double2* __restrict__ C0, double2* __restrict__ C1, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double2 T[16][17];
  const int pair = blockIdx.x / (RB * RB), sub = blockIdx.x % (RB * RB), z = blockIdx.y;
  double2* C = z ? C1 : C0;
  int ta, tb;
  tri_pair(pair, ta, tb);
  const int br = (sub / RB) * 16, bc = (sub % RB) * 16;
  const int row0 = ta * TM + br, col0 = tb * TM + bc;
  if (row0 >= m || col0 > row0) return;   // outside, or above the diagonal
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
  const int row = row0 + r, col = col0 + c;
  const double2* p = part + (size_t(z) * npair + pair) * split * TM * TM + (br + r) * TM + bc + c;
  double re = 0.0, im = 0.0;
  if (row < m && col <= row) {
    int s = 0;
    for (; s + 8 <= split; s += 8) {
      double2 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[size_t(s + u) * TM * TM];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        re += v[u].x;
        im += v[u].y;
      }
    }
    for (; s < split; ++s) {
      const double2 v = p[size_t(s) * TM * TM];
      re += v.x;
      im += v.y;
    }
    const double2 v = make_double2(scale * re, col == row ? 0.0 : scale * im);
    C[size_t(row) * m + col] = v;
    T[r][c] = v;
  }
  __syncthreads();
  const int mr = col0 + r, mc = row0 + c;   // mirrored element (mr, mc) = conj (mc, mr)
  if (mc < m && mr < mc) {
    const double2 v = T[c][r];
    C[size_t(mr) * m + mc] = make_double2(v.x, -v.y);
  }
}

// ----------------------------------------------------------- combine
// Y[b][v] = sum_a U[a][b] X[a][v]: M = b (rows of Y), N = v, K = a.  One wave per
// sub-tile of 32 x 32, as k_overlap_lower; grid (k / 32 / 4, row tiles of 32),
// dealt out so that the row tiles of one column tile run on one XCD and X
// is read from HBM once.  150 states at 24^3: 133 us with tiles in LDS, now 112.
constexpr int CT = 32;   // sub-tile side
__global__ void __launch_bounds__(GT)
k_combine(const double2* __restrict__ X, const double2* __restrict__ U, double2* __restrict__ Y,
          int m, long k, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  int vt = blockIdx.x, bt = blockIdx.y;
  if (gridDim.x % NXCD == 0) {
    const int id = vt + int(gridDim.x) * bt, idx = id / NXCD;
    bt = idx % int(gridDim.y);
    vt = idx / int(gridDim.y) * NXCD + id % NXCD;
  }
  const int lane = threadIdx.x & 63, lc = lane & 15, kq = lane >> 4;
  const long v0 = (long(vt) * (GT / 64) + (threadIdx.x >> 6)) * CT;
  const int b0 = bt * CT;
  double2 u[KQ][2], x[KQ][2];
  auto load = [&](int a0, int q) {
    const int a = a0 + 4 * q + kq;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int col = lc + 16 * e, b = b0 + col;
      u[q][e] = a < m ? U[size_t(a) * m + min(b, m - 1)] : make_double2(0, 0);
      x[q][e] = a < m ? X[size_t(a) * k + v0 + col] : make_double2(0, 0);
    }
  };
  Sub<2> acc;
#pragma unroll
  for (int q = 0; q < KQ; ++q) load(0, q);
  for (int a0 = 0; a0 < m; a0 += KC)
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      acc.step<false>(u[q], x[q]);
      load(a0 + KC, q);
    }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int b = b0 + 16 * i + 4 * e + kq;
        if (b < m) Y[size_t(b) * k + v0 + 16 * j + lc] = make_double2(acc.re[i][j][e], acc.im[i][j][e]);
      }
}

// ----------------------------------------------------------- square products
// C = alpha op(A) op(B) + add 1, op 0 = N, 1 = conjugate transpose; all m x m
// row-major (addp, if given, holds add).  Grid (column, row sub-tiles, products):
// one or two independent products of the same form.
// MIRROR: a product known to be Hermitian; only sub-tiles on or below the
// diagonal are computed, the upper triangle is their mirror image and the
// diagonal real.  One sub-tile of NB x NB blocks per workgroup, the contraction
// split over its waves in consecutive ranges of at least two chunks, the
// partials summed in wave order through LDS.  Operands are loaded from L2 as in
// k_overlap_lower; the last row or column is repeated past m, and the
// contraction is zero past it.  64 x 64 tiles staged in LDS, split over
// workgroups and summed by a second launch, took 13 us at 150 states where this
// takes 6, and as long at 1600.
struct SquareArgs {
  const double2 *A, *B;
  double2* C;
};
template <int NB, int QW, int OPA, int OPB, bool MIRROR>
__global__ void __launch_bounds__(64 * QW)
k_gemm_square(SquareArgs g0, SquareArgs g1, int m, double alpha, double add,
              const double* __restrict__ addp, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  if (MIRROR && blockIdx.x > blockIdx.y) return;
  const double2* __restrict__ A = blockIdx.z ? g1.A : g0.A;
  const double2* __restrict__ B = blockIdx.z ? g1.B : g0.B;
  double2* __restrict__ C = blockIdx.z ? g1.C : g0.C;
  constexpr int QT = 16 * NB, NTH = 64 * QW;
  __shared__ double red[QW][QT][QT + 1];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, kq = lane >> 4;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = blockIdx.y * QT, c0 = blockIdx.x * QT;
  const int nk = (m + KC - 1) / KC;
  const double2 *pa[NB], *pb[NB];
  const size_t sa = OPA == 0 ? 1 : m, sb = OPB == 0 ? m : 1;   // along the contraction
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    pa[i] = A + size_t(min(r0 + 16 * i + r, m - 1)) * (OPA == 0 ? m : 1);
    pb[i] = B + size_t(min(c0 + 16 * i + r, m - 1)) * (OPB == 0 ? 1 : m);
  }
  double2 a[KQ][NB], b[KQ][NB];
  auto load = [&](int kc, int q) {
    const int k = kc * KC + 4 * q + kq;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      a[q][i] = k < m ? pa[i][k * sa] : make_double2(0, 0);
      b[q][i] = k < m ? pb[i][k * sb] : make_double2(0, 0);
      if (OPB) b[q][i].y = -b[q][i].y;
    }
  };
  Sub<NB> acc;
  const int split = min(QW, max(1, nk / 2));
  const int kc0 = g < split ? nk * g / split : 0, kc1 = g < split ? nk * (g + 1) / split : 0;
#pragma unroll
  for (int q = 0; q < KQ; ++q) load(kc0, q);
  for (int kc = kc0; kc < kc1; ++kc)
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      acc.template step<OPA != 0>(a[q], b[q]);
      load(kc + 1, q);
    }
  // real parts, then imaginary parts, through LDS; element e of the thread is
  // (e / QT, e % QT) of the sub-tile
  constexpr int NV = QT * QT / NTH > 0 ? QT * QT / NTH : 1;
  double2 v[NV], w[NV];   // the element, and its mirror image's source
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    if (part) __syncthreads();
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          red[g][16 * i + 4 * e + kq][16 * j + r] = part ? acc.im[i][j][e] : acc.re[i][j][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int e = tid + q * NTH, i = e / QT, j = e % QT;
      if (e >= QT * QT) break;
      double x = red[0][i][j], y = red[0][j][i];
#pragma unroll
      for (int h = 1; h < QW; ++h) {
        x += red[h][i][j];
        y += red[h][j][i];
      }
      if (part) v[q].y = x; else v[q].x = x;
      if (part) w[q].y = y; else w[q].x = y;
    }
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int e = tid + q * NTH, i = e / QT, j = e % QT;
    if (e >= QT * QT) break;
    const bool diag = MIRROR && r0 == c0;
    double2 x = v[q];
    if (diag && i < j) x = make_double2(w[q].x, -w[q].y);
    x.x *= alpha;
    x.y *= alpha;
    if (diag && i == j) x.y = 0.0;
    if (r0 + i == c0 + j) x.x += addp ? *addp : add;
    if (r0 + i < m && c0 + j < m) C[size_t(r0 + i) * m + c0 + j] = x;
    if (MIRROR && !diag && c0 + i < m && r0 + j < m)
      C[size_t(c0 + i) * m + r0 + j] = make_double2(alpha * w[q].x, -alpha * w[q].y);
  }
}

int overlap_split(int m, long k) {
  if (m <= 0) return 1;
  const int nt = (m + TM - 1) / TM;
  const int npair = nt * (nt + 1) / 2;
  long nck = k / KC;
  int split = (2048 + 2 * npair - 1) / (2 * npair);
  if (split < 1) split = 1;
  if (split > nck) split = int(nck);
  if (split > 64) split = 64;
  return split;
}
}  // namespace

// Split-K factors tried by the autotuner: half, default and double.
int overlap_split_candidates(int m, long k, int* out) {
  const int d = overlap_split(m, k);
  const long nck = k / KC;
  int n = 0;
  for (int c : {d / 2, d, 2 * d})
    if (c >= 1 && c <= 64 && c <= nck && (n == 0 || out[n - 1] != c)) out[n++] = c;
  return n;
}

size_t overlap_scratch_bytes(int m, long k) {
  const int nt = (m + TM - 1) / TM;
  const int npair = nt * (nt + 1) / 2;
  int c[3];
  const int nc = overlap_split_candidates(m, k, c);
  int split = 1;
  for (int i = 0; i < nc; ++i) split = std::max(split, c[i]);
  return size_t(split) * 2 * npair * TM * TM * sizeof(double2);
}

void overlap_lower(const void* A, const void* B0, const void* B1, int m, long k, double scale,
                   void* C0, void* C1, void* part, hipStream_t st, hipEvent_t* ev, int split_req) {
  if (m <= 0) return;
  const int nt = (m + TM - 1) / TM;
  const int npair = nt * (nt + 1) / 2;
  const int split = split_req > 0 ? split_req : overlap_split(m, k);
  const int nz = B1 ? 2 : 1;
  if (ev) hipEventRecord(ev[0], st);
  auto launch = [&](auto kernel, int sub) {
    const int ns = (m + sub - 1) / sub, nsub = ns * (ns + 1) / 2;
    hipLaunchKernelGGL(kernel, dim3(unsigned((nsub + 3) / 4), split, nz), dim3(GT), 0, st,
                       (const double2*)A, (const double2*)B0, (const double2*)B1, m, k, split,
                       (double2*)part, g_launch_gate);
  };
  if (m <= 16) launch(k_overlap_lower<1>, 16);
  else launch(k_overlap_lower<2>, 32);
  if (ev) hipEventRecord(ev[1], st);
  overlap_reduce(part, npair, split, m, scale, C0, C1, nz, st);
}

void overlap_reduce(const void* part, int npair, int split, int m, double scale, void* C0,
                    void* C1, int nz, hipStream_t st) {
  hipLaunchKernelGGL(k_overlap_reduce, dim3(unsigned(npair * RB * RB), nz), dim3(256), 0, st,
                     (const double2*)part, npair, split, m, scale, (double2*)C0, (double2*)C1,
                     g_launch_gate);
}

void combine(const void* X, const void* U, void* Y, int m, long k, hipStream_t st) {
  if (m <= 0) return;
  dim3 grid(unsigned(k / (CT * (GT / 64))), (m + CT - 1) / CT);
  hipLaunchKernelGGL(k_combine, grid, dim3(GT), 0, st, (const double2*)X, (const double2*)U,
                     (double2*)Y, m, k, g_launch_gate);
}

// Blocks per sub-tile: one while the 32 x 32 sub-tiles would be fewer than the
// CUs (256 at 512 states; Rayleigh-Ritz of 400: 2820 us against 2910), two from
// there (1600: 10.1 ms against 10.3).
constexpr int SQ_NB1_MAX = 512;

namespace {
void square(const SquareArgs& g0, const SquareArgs& g1, int count, int opA, int opB, int m, hipStream_t st,
            int herm, double alpha, double add, const double* addp) {
  if (m <= 0) return;
  auto go = [&](auto nb, auto qw) {
    constexpr int NB = decltype(nb)::value, QW = decltype(qw)::value;
    const unsigned nt = unsigned((m + 16 * NB - 1) / (16 * NB));
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(nt, nt, unsigned(count)), dim3(64 * QW), 0, st, g0, g1, m, alpha, add,
                         addp, g_launch_gate);
    };
    if (opA == 0 && opB == 0) herm ? launch(k_gemm_square<NB, QW, 0, 0, true>) : launch(k_gemm_square<NB, QW, 0, 0, false>);
    else if (opA == 0) herm ? launch(k_gemm_square<NB, QW, 0, 1, true>) : launch(k_gemm_square<NB, QW, 0, 1, false>);
    else if (opB == 0) herm ? launch(k_gemm_square<NB, QW, 1, 0, true>) : launch(k_gemm_square<NB, QW, 1, 0, false>);
    else herm ? launch(k_gemm_square<NB, QW, 1, 1, true>) : launch(k_gemm_square<NB, QW, 1, 1, false>);
  };
  if (m <= SQ_NB1_MAX) go(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
}

SquareArgs square_args(const void* A, const void* B, void* C) {
  return SquareArgs{(const double2*)A, (const double2*)B, (double2*)C};
}
}  // namespace

void gemm_square(const void* A, int opA, const void* B, int opB, void* C, int m, hipStream_t st, int herm,
                 double add, const double* addp, double alpha) {
  const SquareArgs g = square_args(A, B, C);
  square(g, g, 1, opA, opB, m, st, herm, alpha, add, addp);
}

void gemm_square_pair(const void* A0, const void* B0, void* C0, const void* A1, const void* B1, void* C1, int m,
                      hipStream_t st) {
  square(square_args(A0, B0, C0), square_args(A1, B1, C1), 2, 0, 0, m, st, 0, 1.0, 0.0, nullptr);
}

}  // namespace sky
