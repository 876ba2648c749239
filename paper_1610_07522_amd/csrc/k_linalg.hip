// Dense FP64 Hermitian linear algebra of the subspace step (Sec. 3.3.2):
// Cholesky factor of the overlap and its inverse (the orthonormalising
// transform), and a Hermitian eigensolver for the subspace Hamiltonian.
//
// The eigensolver is a blocked two-sided Jacobi method: the matrix is cut
// into 16-wide blocks, block pairs are visited in round-robin order, each
// 32x32 pair sub-matrix is diagonalised inside one workgroup (cyclic Jacobi
// in LDS), and the resulting unitaries are applied to the whole matrix and
// to the eigenvector accumulator.  Jacobi suits this step because the
// subspace Hamiltonian is nearly diagonal after the first iterations, and
// every round is fully parallel.
#include <vector>
#include <algorithm>
#include <cmath>

#include "jacobi_rot.h"
#include "mfma_f64.h"
#include "sky_kernels.h"

namespace sky {

thread_local const int* g_launch_gate = nullptr;


namespace {
using namespace jrot;
constexpr int CB = 64;    // Cholesky block
constexpr int JB = 16;    // Jacobi block (pair sub-problem = 2*JB)
constexpr int JP = 2 * JB;
constexpr int JE = JP * JP / 256;   // pair-matrix elements per thread (256 threads)
constexpr int RV = 64;              // rows of V per workgroup in the V update
// Cyclic sweeps per pair sub-problem and round: one, since a pair meets its
// other partners before a second sweep on it pays (24^3 initialisation with
// 151 + 50 states: 9.5, 7.5 and 5.6 ms with 3, 2 and 1; 48^3 with 1600 + 400:
// 308, 276 and 249 ms).  Two blocks (m <= 32) are one pair for good: it runs to
// convergence in one launch.  The pair tolerance is 100x tighter than the
// global one so that the ~(n/32)^2/2 converged pair blocks together stay below
// the global off-diagonal bound.
constexpr int JACOBI_INNER = 1;
constexpr int JACOBI_INNER_ONE_PAIR = 12;

// ------------------------------------------------------------------ Cholesky
// Factor the kw x kw diagonal block at (k0, k0) in LDS and invert it:
// A[k0.., k0..] <- L_kk (lower), Dinv <- L_kk^-1 (CB x CB, lower).
__global__ void __launch_bounds__(256)
k_chol_diag(double2* __restrict__ A, int m, int k0, double2* __restrict__ Dinv, int* info,
            double piv_min, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double2 S[CB][CB + 1];
  __shared__ double2 X[CB][CB + 1];
  __shared__ int bad;
  const int kw = min(CB, m - k0);
  const int tid = threadIdx.x;
  if (tid == 0) bad = 0;
  for (int e = tid; e < CB * CB; e += blockDim.x) {
    int i = e / CB, j = e % CB;
    S[i][j] = (i < kw && j < kw) ? A[size_t(k0 + i) * m + k0 + j] : make_double2(0, 0);
    X[i][j] = make_double2(0, 0);
  }
  __syncthreads();
  for (int j = 0; j < kw; ++j) {
    if (tid == 0) {
      double d = S[j][j].x;
      if (!(d > piv_min)) { bad = 1; d = 1.0; }
      S[j][j] = make_double2(sqrt(d), 0.0);
    }
    __syncthreads();
    const double inv = 1.0 / S[j][j].x;
    for (int i = j + 1 + tid; i < kw; i += blockDim.x) S[i][j] = cscale(inv, S[i][j]);
    __syncthreads();
    // trailing update of the lower part: S[i][l] -= L[i][j] conj(L[l][j]), i >= l > j
    const int w = kw - j - 1;
    for (int e = tid; e < w * w; e += blockDim.x) {
      int i = j + 1 + e / w, l = j + 1 + e % w;
      if (l <= i) S[i][l] = csub(S[i][l], cmulc(S[i][j], S[l][j]));
    }
    __syncthreads();
  }
  // inverse of L by columns: X[i][c] = (delta_ic - sum_{c<=l<i} L[i][l] X[l][c]) / L[i][i]
  if (tid < kw) {
    const int c = tid;
    for (int i = c; i < kw; ++i) {
      double2 s = make_double2(i == c ? 1.0 : 0.0, 0.0);
      for (int l = c; l < i; ++l) s = csub(s, cmul(S[i][l], X[l][c]));
      X[i][c] = cscale(1.0 / S[i][i].x, s);
    }
  }
  __syncthreads();
  for (int e = tid; e < CB * CB; e += blockDim.x) {
    int i = e / CB, j = e % CB;
    if (i < kw && j < kw) {
      A[size_t(k0 + i) * m + k0 + j] = (j <= i) ? S[i][j] : make_double2(0, 0);
    }
    Dinv[e] = X[i][j];
  }
  if (tid == 0 && bad) atomicExch(info, 1);
}

// Panel below the diagonal block: L[i][k0..] = A[i][k0..] * L_kk^-H, for
// the 64-row block starting at row r0 = k0 + kw + blockIdx.x * CB.
__global__ void __launch_bounds__(256)
k_chol_panel(double2* __restrict__ A, int m, int k0, const double2* __restrict__ Dinv, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double2 P[CB][CB + 1];
  __shared__ double2 D[CB][CB + 1];
  const int kw = min(CB, m - k0);
  const int r0 = k0 + kw + blockIdx.x * CB;
  const int tid = threadIdx.x;
  for (int e = tid; e < CB * CB; e += blockDim.x) {
    int i = e / CB, j = e % CB;
    P[i][j] = (r0 + i < m && j < kw) ? A[size_t(r0 + i) * m + k0 + j] : make_double2(0, 0);
    D[i][j] = Dinv[e];
  }
  __syncthreads();
  // out[i][j] = sum_l P[i][l] conj(D[j][l])
  for (int e = tid; e < CB * CB; e += blockDim.x) {
    int i = e / CB, j = e % CB;
    if (r0 + i >= m || j >= kw) continue;
    double2 s = make_double2(0, 0);
    for (int l = 0; l <= j; ++l) s = cadd(s, cmulc(P[i][l], D[j][l]));
    A[size_t(r0 + i) * m + k0 + j] = s;
  }
}

// Trailing update A[i][j] -= sum_l L[i][k0+l] conj(L[j][k0+l]) on the lower
// tiles of the trailing matrix (tile pair number -> (ti, tj), ti >= tj).
__global__ void __launch_bounds__(256)
k_chol_update(double2* __restrict__ A, int m, int k0, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double2 Li[CB][CB + 1];
  __shared__ double2 Lj[CB][CB + 1];
  const int kw = min(CB, m - k0);
  const int t0 = k0 + kw;
  int p = blockIdx.x, a = 0;
  while ((a + 1) * (a + 2) / 2 <= p) ++a;
  const int ti = a, tj = p - a * (a + 1) / 2;
  const int i0 = t0 + ti * CB, j0 = t0 + tj * CB;
  const int tid = threadIdx.x;
  for (int e = tid; e < CB * CB; e += blockDim.x) {
    int r = e / CB, l = e % CB;
    Li[r][l] = (i0 + r < m && l < kw) ? A[size_t(i0 + r) * m + k0 + l] : make_double2(0, 0);
    Lj[r][l] = (j0 + r < m && l < kw) ? A[size_t(j0 + r) * m + k0 + l] : make_double2(0, 0);
  }
  __syncthreads();
  for (int e = tid; e < CB * CB; e += blockDim.x) {
    int r = e / CB, c = e % CB;
    int gi = i0 + r, gj = j0 + c;
    if (gi >= m || gj >= m || gj > gi) continue;
    double2 s = make_double2(0, 0);
    for (int l = 0; l < kw; ++l) s = cadd(s, cmulc(Li[r][l], Lj[c][l]));
    size_t idx = size_t(gi) * m + gj;
    A[idx] = csub(A[idx], s);
  }
}

// Block row ib of Linv (jb < ib), on the FP64 matrix cores:
//   Linv[ib][jb] = -Dinv[ib] * S,  S = sum_{kb=jb}^{ib-1} L[ib][kb] Linv[kb][jb]
// one workgroup per jb; Linv[ib][ib] = Dinv[ib] is written by jb == ib.
__global__ void __launch_bounds__(256)
k_tri_inv_row(const double2* __restrict__ L, double2* __restrict__ Linv, int m, int ib,
              const double2* __restrict__ Dinv_all, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  using namespace mfma;
  __shared__ double2 sA[TM * KP];
  __shared__ double2 sB[TM * KP];
  __shared__ double2 Ssh[CB][CB + 1];
  const int jb = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int r0 = ib * CB;
  const double2* Di = Dinv_all + size_t(ib) * CB * CB;
  if (jb == ib) {
    for (int e = tid; e < CB * CB; e += blockDim.x) {
      int r = e / CB, c = e % CB;
      if (r0 + r < m && r0 + c < m) Linv[size_t(r0 + r) * m + r0 + c] = Di[e];
    }
    return;
  }
  Acc acc;
  zero(acc);
  for (int kb = jb; kb < ib; ++kb) {
    for (int kc = 0; kc < CB; kc += KC) {
      for (int e = tid; e < TM * KC; e += GT) {
        const int t = e / KC, k = e % KC;
        const int col = kb * CB + kc + k;            // < m since kb < ib
        sA[t * KP + k] = (r0 + t < m) ? L[size_t(r0 + t) * m + col] : make_double2(0, 0);
        sB[t * KP + k] = Linv[size_t(col) * m + jb * CB + t];
      }
      __syncthreads();
      tile<false>(acc, sA, sB, wm, wn, lane);
      __syncthreads();
    }
  }
  foreach(acc, wm, wn, lane, [&](int row, int col, double re, double im) {
    Ssh[row][col] = make_double2(re, im);
  });
  __syncthreads();
  zero(acc);
  for (int kc = 0; kc < CB; kc += KC) {
    for (int e = tid; e < TM * KC; e += GT) {
      const int t = e / KC, k = e % KC;
      sA[t * KP + k] = Di[t * CB + kc + k];
      sB[t * KP + k] = Ssh[kc + k][t];
    }
    __syncthreads();
    tile<false>(acc, sA, sB, wm, wn, lane);
    __syncthreads();
  }
  foreach(acc, wm, wn, lane, [&](int row, int col, double re, double im) {
    if (r0 + row < m && jb * CB + col < m)
      Linv[size_t(r0 + row) * m + jb * CB + col] = make_double2(-re, -im);
  });
}

__global__ void k_zero_cpx(double2* __restrict__ p, size_t n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = make_double2(0, 0);
}

__global__ void k_zero(double* __restrict__ p, size_t n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

// ------------------------------------------------------------------ Loewdin series
// D = A - 1 and per-block partial sums of |D_ij|^2.
__global__ void __launch_bounds__(256)
k_minus_identity(const double2* __restrict__ A, double2* __restrict__ D, int m,
                 double* __restrict__ part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  double acc = 0.0;
  const size_t n = size_t(m) * m;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n;
       e += size_t(gridDim.x) * blockDim.x) {
    double2 a = A[e];
    if (e / m == e % m) a.x -= 1.0;
    D[e] = a;
    acc += a.x * a.x + a.y * a.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  __shared__ double red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// out[0] (and host[0], host-visible memory, if given) = sum of part[0 .. nb): lane t of one wave adds t, t + 64, ... in
// order, then a fixed butterfly (a one-thread loop over 256 partials is a
// serial chain of loads: 18 us, now 4).
__global__ void k_sum_parts(const double* __restrict__ part, int nb, double* __restrict__ out,
                            double* __restrict__ host, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  double s = 0.0;
  for (int b = threadIdx.x; b < nb; b += 64) s += part[b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (threadIdx.x == 0) {
    out[0] = s;
    if (host != nullptr) host[0] = s;
  }
}

// P = a D + c 1
__global__ void k_axpy_identity(const double2* __restrict__ D, double a, double c,
                                double2* __restrict__ P, int m, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= size_t(m) * m) return;
  const double2 d = D[e];
  P[e] = make_double2(a * d.x + ((e / m == e % m) ? c : 0.0), a * d.y);
}

// ------------------------------------------------------------------ Jacobi
// Diagonalise the 32x32 pair sub-matrix of blocks (P, Q) of A (ld = mp)
// and write its unitary J (32x32, row-major, local index l < 16 -> block P).
// A round rotates 16 disjoint index pairs at once; thread (u, v) owns the 2x2
// block of row pair u and column pair v, and two rows of J for column pair v.
// A workgroup is alone on its CU and bound by the latency of a round, so a
// round is kept to one barrier: every lane computes the rotation of its own
// column pair (the sixteen rotations once per 16 lanes, shared with the row
// pairs by a shuffle) straight from the matrix, which is written to the other
// of two buffers; the pairs of every round come from a table.  With rotations
// made by 16 threads between two barriers, divisions and index arithmetic in
// every round, a sweep of 31 rounds took 42 us, now 28 with its loads.
constexpr int JT = 256;    // threads of a pair sub-problem workgroup
__global__ void __launch_bounds__(JT)
k_jacobi_pair(const double2* __restrict__ A, int mp, const int2* __restrict__ pairs,
              double2* __restrict__ Jout, int* __restrict__ rotated, double tol, int max_inner, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  static_assert(JT == JB * JB && JB == 16, "one thread per 2x2 block, 16 pairs per quarter wave");
  __shared__ double2 S[2][JP][JP + 1];
  __shared__ double2 J[JP][JP + 1];
  __shared__ unsigned short sched[JP - 1][JB];
  __shared__ double red[JT / 64][2];
  const int2 pq = pairs[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63;
  const int u = tid / JB, v = tid % JB;
  for (int e = tid; e < JP * JP; e += JT) {
    int i = e / JP, j = e % JP;
    int gi = (i < JB ? pq.x * JB + i : pq.y * JB + i - JB);
    int gj = (j < JB ? pq.x * JB + j : pq.y * JB + j - JB);
    S[0][i][j] = A[size_t(gi) * mp + gj];
    J[i][j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  for (int e = tid; e < (JP - 1) * JB; e += JT) {
    int p, q;
    rr_pair(JP, e / JB, e % JB, p, q);
    sched[e / JB][e % JB] = (unsigned short)(p < q ? p | (q << 8) : q | (p << 8));
  }
  __syncthreads();
  int cur = 0, any_rot = 0;
  for (int sweep = 0; sweep < max_inner; ++sweep) {
    // convergence test on the sub-matrix (the same value in every thread)
    double off = 0.0, dia = 0.0;
    for (int e = tid; e < JP * JP; e += JT) {
      int i = e / JP, j = e % JP;
      const double2 x = S[cur][i][j];
      double w = x.x * x.x + x.y * x.y;
      if (i == j) dia += w; else off += w;
    }
    for (int o = 32; o > 0; o >>= 1) {
      off += __shfl_down(off, o, 64);
      dia += __shfl_down(dia, o, 64);
    }
    if (lane == 0) { red[tid >> 6][0] = off; red[tid >> 6][1] = dia; }
    __syncthreads();
    double o = 0.0, d = 0.0;
    for (int w = 0; w < JT / 64; ++w) { o += red[w][0]; d += red[w][1]; }
    if ((o <= tol * tol * d) || (o < 1e-300)) break;
    any_rot = 1;
    for (int r = 0; r < JP - 1; ++r) {
      const int cu = sched[r][u], cv = sched[r][v];
      const int pu = cu & 255, qu = cu >> 8, pv = cv & 255, qv = cv >> 8;
      const double2 (*X)[JP + 1] = S[cur];
      const double2 x00 = X[pu][pv], x01 = X[pu][qv], x10 = X[qu][pv], x11 = X[qu][qv];
      const double2 j00 = J[2 * u][pv], j01 = J[2 * u][qv];
      const double2 j10 = J[2 * u + 1][pv], j11 = J[2 * u + 1][qv];
      const Rot gv = make_rot_rsq(X[pv][pv].x, X[qv][qv].x, X[pv][qv]);
      Rot gu;
      gu.c = __shfl(gv.c, u, 64);
      gu.s = __shfl(gv.s, u, 64);
      gu.er = __shfl(gv.er, u, 64);
      gu.ei = __shfl(gv.ei, u, 64);
      const double2 epu = make_double2(gu.er, gu.ei), epv = make_double2(gv.er, gv.ei);
      // right multiply by G_v: col p' = e c col_p - s col_q ; col q' = e s col_p + c col_q
      const double2 z00 = cmul(x00, epv), z10 = cmul(x10, epv);
      const double2 y00 = csub(cscale(gv.c, z00), cscale(gv.s, x01));
      const double2 y01 = cadd(cscale(gv.s, z00), cscale(gv.c, x01));
      const double2 y10 = csub(cscale(gv.c, z10), cscale(gv.s, x11));
      const double2 y11 = cadd(cscale(gv.s, z10), cscale(gv.c, x11));
      // left multiply by G_u^H: row p' = conj(e) c row_p - s row_q ; row q' = conj(e) s row_p + c row_q
      const double2 w00 = cmulc(y00, epu), w01 = cmulc(y01, epu);
      double2 (*Y)[JP + 1] = S[cur ^ 1];
      Y[pu][pv] = csub(cscale(gu.c, w00), cscale(gu.s, y10));
      Y[pu][qv] = csub(cscale(gu.c, w01), cscale(gu.s, y11));
      Y[qu][pv] = cadd(cscale(gu.s, w00), cscale(gu.c, y10));
      Y[qu][qv] = cadd(cscale(gu.s, w01), cscale(gu.c, y11));
      // J <- J G
      const double2 k0 = cmul(j00, epv), k1 = cmul(j10, epv);
      J[2 * u][pv] = csub(cscale(gv.c, k0), cscale(gv.s, j01));
      J[2 * u][qv] = cadd(cscale(gv.s, k0), cscale(gv.c, j01));
      J[2 * u + 1][pv] = csub(cscale(gv.c, k1), cscale(gv.s, j11));
      J[2 * u + 1][qv] = cadd(cscale(gv.s, k1), cscale(gv.c, j11));
      cur ^= 1;
      __syncthreads();
    }
  }
  if (tid == 0) rotated[blockIdx.x] = any_rot;
  if (!any_rot) return;   // J = identity: the apply kernel skips this pair
  double2* out = Jout + size_t(blockIdx.x) * JP * JP;
  for (int e = tid; e < JP * JP; e += JT) out[e] = J[e / JP][e % JP];
}

// One round's unitaries applied to A and to the eigenvector accumulator V, one
// launch for both (they touch different matrices; at a few hundred states
// each is a handful of workgroups and costs a launch's latency).
//   Workgroups 0 .. np (np + 1) / 2 - 1: A[{Pu,Qu}][{Pv,Qv}] <- J_u^H A J_v for
//   the pair pairs u >= v (number -> (u, v)); the mirrored block (v, u) gets
//   the conjugate transpose, since A stays Hermitian.
//   The rest: V[rows][{P,Q}] <- V[rows][{P,Q}] J, RV rows and one pair each.
// Pairs whose J is the identity are skipped.  Each thread forms outputs of one
// column, so that an element of the unitary is read from LDS once for all of
// them (12 + 12 us in two launches at 151 states, now 10.7; at 1600 states
// 28 + 34 us before).  The product loops stay rolled: unrolled in full they
// spill.
__global__ void __launch_bounds__(256)
k_jacobi_apply(double2* __restrict__ A, double2* __restrict__ V, int mp, int np,
               const int2* __restrict__ pairs, const double2* __restrict__ Jall,
               const int* __restrict__ rotated, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double2 X[RV][JP + 1];
  __shared__ double2 M[JP][JP + 1];
  const int tid = threadIdx.x, j = tid % JP, i0 = tid / JP;   // column; rows i0 + 8 q
  auto gidx = [&](int2 p, int l) { return l < JB ? p.x * JB + l : p.y * JB + l - JB; };
  const int na = np * (np + 1) / 2;
  if (int(blockIdx.x) >= na) {
    constexpr int NQ = RV * JP / 256;
    const int nv = int(blockIdx.x) - na, v = nv % np, r0 = (nv / np) * RV;
    if (!rotated[v]) return;
    const int col = gidx(pairs[v], j);
    const double2* Jv = Jall + size_t(v) * JP * JP;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int i = i0 + 8 * q;
      X[i][j] = (r0 + i < mp) ? V[size_t(r0 + i) * mp + col] : make_double2(0, 0);
    }
    for (int e = tid; e < JP * JP; e += 256) M[e / JP][e % JP] = Jv[e];
    __syncthreads();
    double2 s[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) s[q] = make_double2(0, 0);
#pragma unroll 2
    for (int l = 0; l < JP; ++l) {
      const double2 w = M[l][j];
#pragma unroll
      for (int q = 0; q < NQ; ++q) s[q] = cadd(s[q], cmul(X[i0 + 8 * q][l], w));
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (r0 + i0 + 8 * q < mp) V[size_t(r0 + i0 + 8 * q) * mp + col] = s[q];
    return;
  }
  int u = 0;
  while ((u + 1) * (u + 2) / 2 <= int(blockIdx.x)) ++u;
  const int v = int(blockIdx.x) - u * (u + 1) / 2;
  const int ru = rotated[u], rv = rotated[v];
  if (!ru && !rv) return;
  const int2 pu = pairs[u], pv = pairs[v];
  const double2* Ju = Jall + size_t(u) * JP * JP;
  const double2* Jv = Jall + size_t(v) * JP * JP;
  const int col = gidx(pv, j);
#pragma unroll
  for (int q = 0; q < JE; ++q) {
    const int i = i0 + 8 * q;
    X[i][j] = A[size_t(gidx(pu, i)) * mp + col];
    if (rv) M[i][j] = Jv[i * JP + j];
  }
  __syncthreads();
  double2 y[JE];
  if (rv) {                               // Y = X Jv
#pragma unroll
    for (int q = 0; q < JE; ++q) y[q] = make_double2(0, 0);
#pragma unroll 2
    for (int l = 0; l < JP; ++l) {
      const double2 w = M[l][j];
#pragma unroll
      for (int q = 0; q < JE; ++q) y[q] = cadd(y[q], cmul(X[i0 + 8 * q][l], w));
    }
  } else {
#pragma unroll
    for (int q = 0; q < JE; ++q) y[q] = X[i0 + 8 * q][j];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < JE; ++q) {
    X[i0 + 8 * q][j] = y[q];
    if (ru) M[i0 + 8 * q][j] = Ju[(i0 + 8 * q) * JP + j];
  }
  __syncthreads();
  if (ru) {                               // T = Ju^H Y
#pragma unroll
    for (int q = 0; q < JE; ++q) y[q] = make_double2(0, 0);
#pragma unroll 2
    for (int l = 0; l < JP; ++l) {
      const double2 w = X[l][j];
#pragma unroll
      for (int q = 0; q < JE; ++q) y[q] = cadd(y[q], cconjmul(M[l][i0 + 8 * q], w));
    }
  }
#pragma unroll
  for (int q = 0; q < JE; ++q) {
    const int row = gidx(pu, i0 + 8 * q);
    A[size_t(row) * mp + col] = y[q];
    if (u != v) A[size_t(col) * mp + row] = make_double2(y[q].x, -y[q].y);
  }
}

// Off-diagonal and diagonal squared norms of A (mp x mp), per block partials.
__global__ void k_offnorm(const double2* __restrict__ A, int mp, double* __restrict__ part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double red[4][2];
  double off = 0.0, dia = 0.0;
  const size_t n = size_t(mp) * mp;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n;
       e += size_t(gridDim.x) * blockDim.x) {
    double2 a = A[e];
    double v = a.x * a.x + a.y * a.y;
    if (e / mp == e % mp) dia += v; else off += v;
  }
  for (int o = 32; o > 0; o >>= 1) {
    off += __shfl_down(off, o, 64);
    dia += __shfl_down(dia, o, 64);
  }
  if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6][0] = off; red[threadIdx.x >> 6][1] = dia; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double o = 0.0, d = 0.0;
    for (int w = 0; w < 4; ++w) { o += red[w][0]; d += red[w][1]; }
    part[2 * blockIdx.x] = o;
    part[2 * blockIdx.x + 1] = d;
  }
}

// Sums of the block partials, one wave, as k_sum_parts.
__global__ void k_offnorm_final(const double* __restrict__ part, int nb, double* __restrict__ out, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  double o = 0.0, d = 0.0;
  for (int b = threadIdx.x; b < nb; b += 64) { o += part[2 * b]; d += part[2 * b + 1]; }
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) {
    o += __shfl_down(o, k, 64);
    d += __shfl_down(d, k, 64);
  }
  if (threadIdx.x == 0) {
    out[0] = o;   // host-visible memory
    out[1] = d;
  }
}

// Pad-copy A (m x m) into Ap (mp x mp) with zero coupling, V = identity.
__global__ void k_jacobi_init(const double2* __restrict__ A, int m, double2* __restrict__ Ap,
                              double2* __restrict__ V, int mp, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= size_t(mp) * mp) return;
  int i = int(e / mp), j = int(e % mp);
  Ap[e] = (i < m && j < m) ? A[size_t(i) * m + j] : make_double2(0, 0);
  V[e] = make_double2(i == j ? 1.0 : 0.0, 0.0);
}

// Sort eigenvalues ascending (ties by index) and gather eigenvector columns.
__global__ void k_jacobi_sort(const double2* __restrict__ Ap, const double2* __restrict__ V,
                              int m, int mp, double* __restrict__ w, double2* __restrict__ Z, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int i = blockIdx.x;   // source column
  const double wi = Ap[size_t(i) * mp + i].x;
  __shared__ int rank_s;
  if (threadIdx.x == 0) rank_s = 0;
  __syncthreads();
  int cnt = 0;
  for (int j = threadIdx.x; j < m; j += blockDim.x) {
    double wj = Ap[size_t(j) * mp + j].x;
    if (wj < wi || (wj == wi && j < i)) ++cnt;
  }
  atomicAdd(&rank_s, cnt);
  __syncthreads();
  const int rk = rank_s;
  if (threadIdx.x == 0) w[rk] = wi;
  for (int r = threadIdx.x; r < m; r += blockDim.x) Z[size_t(r) * m + rk] = V[size_t(r) * mp + i];
}

__global__ void k_scale_columns(double2* __restrict__ X, const double* __restrict__ d, int m, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= size_t(m) * m) return;
  double s = d[e % m];
  X[e] = make_double2(s * X[e].x, s * X[e].y);
}

__global__ void k_inv_sqrt(double* __restrict__ w, int m, int* info, double floor_v, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  double v = w[i];
  if (!(v > floor_v)) { atomicExch(info, 1); v = 1.0; }
  w[i] = 1.0 / sqrt(v);
}

// The pivot k of A - diag(gap) is the least v^H (A - diag(gap)) v over v with v_k = 1
// and nothing past k; A's own v, row k of L^-1 over its last element, gives it to
// first order (the next term is gap^2 over the leading block's least eigenvalue).
// One wave per row; one read of L^-1, a launch's latency beside the factorisation.
__global__ void __launch_bounds__(256)
k_gap_pivots(const double2* __restrict__ Linv, const double* __restrict__ gap, int m, int* info,
             double floor_v, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (k >= m) return;
  const double2* u = Linv + size_t(k) * m;
  double s = 0.0;
  for (int i = lane; i <= k; i += 64) s += (u[i].x * u[i].x + u[i].y * u[i].y) * gap[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0 && !((1.0 - s) / (u[k].x * u[k].x) > floor_v)) atomicExch(info, 1);
}

// The eigenvalue k of A - diag(gap) to first order, w_k - sum_i gap_i |X_ik|^2.
// 64 columns per workgroup, every fourth row per wave: one read of X after a Jacobi solve.
__global__ void __launch_bounds__(256)
k_gap_eigenvalues(const double2* __restrict__ X, const double* __restrict__ w,
                  const double* __restrict__ gap, int m, int* info, double floor_v,
                  const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double part[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, k = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (k < m)
    for (int i = wave; i < m; i += 4) {
      const double2 x = X[size_t(i) * m + k];
      s += (x.x * x.x + x.y * x.y) * gap[i];
    }
  part[wave][lane] = s;
  __syncthreads();
  if (wave != 0 || k >= m) return;
  s = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
  if (!(w[k] - s > floor_v)) atomicExch(info, 1);
}

int jacobi_dims(int m, int& nb) {
  nb = (m + JB - 1) / JB;
  if (nb < 2) nb = 2;
  if (nb & 1) ++nb;
  return nb * JB;
}
}  // namespace

void zero(double* p, size_t n, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_zero, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p, n, g_launch_gate);
}

__global__ void k_identity(double2* __restrict__ A, int m, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= size_t(m) * m) return;
  A[e] = make_double2((e / m == e % m) ? 1.0 : 0.0, 0.0);
}

void identity(void* A, int m, hipStream_t st) {
  if (m <= 0) return;
  const size_t mm = size_t(m) * m;
  hipLaunchKernelGGL(k_identity, dim3(unsigned((mm + 255) / 256)), dim3(256), 0, st, (double2*)A, m, g_launch_gate);
}

__global__ void k_zero_f32(float* __restrict__ p, size_t n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

void zero_f32(float* p, size_t n, hipStream_t st) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_zero_f32, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p, n, g_launch_gate);
}

void cholesky_inverse(void* Av, void* Linvv, int m, void* work, int* info, hipStream_t st,
                      double piv_min) {
  if (m <= 0) return;
  auto A = (double2*)Av;
  auto Linv = (double2*)Linvv;
  auto Dinv = (double2*)work;   // nblk * CB * CB
  const int nblk = (m + CB - 1) / CB;
  for (int kb = 0; kb < nblk; ++kb) {
    const int k0 = kb * CB;
    hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(256), 0, st, A, m, k0,
                       Dinv + size_t(kb) * CB * CB, info, piv_min, g_launch_gate);
    const int rest = m - (k0 + min(CB, m - k0));
    if (rest > 0) {
      const int nb = (rest + CB - 1) / CB;
      hipLaunchKernelGGL(k_chol_panel, dim3(nb), dim3(256), 0, st, A, m, k0,
                         (const double2*)(Dinv + size_t(kb) * CB * CB), g_launch_gate);
      hipLaunchKernelGGL(k_chol_update, dim3(nb * (nb + 1) / 2), dim3(256), 0, st, A, m, k0, g_launch_gate);
    }
  }
  const size_t mm = size_t(m) * m;
  hipLaunchKernelGGL(k_zero_cpx, dim3(unsigned((mm + 255) / 256)), dim3(256), 0, st, Linv, mm, g_launch_gate);
  for (int ib = 0; ib < nblk; ++ib)
    hipLaunchKernelGGL(k_tri_inv_row, dim3(ib + 1), dim3(256), 0, st, (const double2*)A, Linv, m,
                       ib, (const double2*)Dinv, g_launch_gate);
}

size_t jacobi_scratch_bytes(int m) {
  int nb;
  const int mp = jacobi_dims(m, nb);
  size_t b = 0;
  b += 2 * size_t(mp) * mp * sizeof(double2);                 // Ap, V
  b += size_t(nb / 2) * JP * JP * sizeof(double2);            // J
  b += size_t(nb) * nb * sizeof(int2);                        // round-robin table
  b += size_t(nb) * sizeof(int) + 256;                        // rotated flags
  b += 4096 * sizeof(double);                                 // norm partials
  return b + 1024;
}

int jacobi_eigh(void* Av, int m, double* w, void* Zv, void* work, double tol, int max_sweeps,
                hipStream_t st, double* host) {
  if (m <= 0) return 0;
  int nb;
  const int mp = jacobi_dims(m, nb);
  const int np = nb / 2;
  char* wp = (char*)work;
  auto Ap = (double2*)wp; wp += size_t(mp) * mp * sizeof(double2);
  auto V = (double2*)wp; wp += size_t(mp) * mp * sizeof(double2);
  auto Jall = (double2*)wp; wp += size_t(np) * JP * JP * sizeof(double2);
  auto pairs = (int2*)wp; wp += size_t(nb) * nb * sizeof(int2);
  auto rotated = (int*)wp; wp += size_t(nb) * sizeof(int) + 256;
  auto norms = (double*)wp;
  // round-robin schedule of the block pairs, all rounds
  std::vector<int2> sched(size_t(nb - 1) * np);
  for (int r = 0; r < nb - 1; ++r)
    for (int i = 0; i < np; ++i) {
      const int n1 = nb - 1;
      int p = (i == 0) ? 0 : ((i + r - 1) % n1) + 1;
      int q = ((n1 - i + r - 1) % n1) + 1;
      sched[size_t(r) * np + i] = make_int2(std::min(p, q), std::max(p, q));
    }
  hipMemcpyAsync(pairs, sched.data(), sched.size() * sizeof(int2), hipMemcpyHostToDevice, st);
  const size_t mm = size_t(mp) * mp;
  hipLaunchKernelGGL(k_jacobi_init, dim3(unsigned((mm + 255) / 256)), dim3(256), 0, st,
                     (const double2*)Av, m, Ap, V, mp, g_launch_gate);
  const int nrb = 256;
  int sweeps = 0;
  bool done = false;
  for (; sweeps <= max_sweeps; ++sweeps) {
    hipLaunchKernelGGL(k_offnorm, dim3(nrb), dim3(256), 0, st, (const double2*)Ap, mp, norms, g_launch_gate);
    hipLaunchKernelGGL(k_offnorm_final, dim3(1), dim3(64), 0, st, (const double*)norms, nrb,
                       host, g_launch_gate);
    if (hipStreamSynchronize(st) != hipSuccess) return -2;
    if (!std::isfinite(host[0]) || !std::isfinite(host[1])) return -2;
    if (host[0] <= tol * tol * host[1] || host[0] < 1e-300) { done = true; break; }
    if (sweeps == max_sweeps) break;   // the norm after the last sweep was checked
    for (int r = 0; r < nb - 1; ++r) {
      const int2* pr = pairs + size_t(r) * np;
      hipLaunchKernelGGL(k_jacobi_pair, dim3(np), dim3(JT), 0, st, (const double2*)Ap, mp, pr,
                         Jall, rotated, tol * 1e-2, np == 1 ? JACOBI_INNER_ONE_PAIR : JACOBI_INNER,
                         g_launch_gate);
      hipLaunchKernelGGL(k_jacobi_apply, dim3(np * (np + 1) / 2 + (mp + RV - 1) / RV * np),
                         dim3(256), 0, st, Ap, V, mp, np, pr, (const double2*)Jall,
                         (const int*)rotated, g_launch_gate);
    }
  }
  hipLaunchKernelGGL(k_jacobi_sort, dim3(m), dim3(256), 0, st, (const double2*)Ap,
                     (const double2*)V, m, mp, w, (double2*)Zv, g_launch_gate);
  return done ? sweeps : -1;
}

void eig_sort(const void* D, const void* V, int m, int ld, double* w, void* Z, hipStream_t st) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_jacobi_sort, dim3(m), dim3(256), 0, st, (const double2*)D, (const double2*)V,
                     m, ld, w, (double2*)Z, g_launch_gate);
}

int loewdin_series(const void* Iv, void* Cv, void* Dv, void* Tv, int m, double max_dev,
                   double* scratch, hipStream_t st, double* host, double eps) {
  if (m <= 0) return 0;
  auto D = (double2*)Dv;
  const size_t mm = size_t(m) * m;
  const int nb = int(std::min<size_t>(256, (mm + 255) / 256));
  hipLaunchKernelGGL(k_minus_identity, dim3(nb), dim3(256), 0, st, (const double2*)Iv, D, m, scratch, g_launch_gate);
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(64), 0, st, (const double*)scratch, nb, scratch + nb, host, g_launch_gate);
  if (hipStreamSynchronize(st) != hipSuccess) return -1;
  const double f = sqrt(host[0]);
  if (!std::isfinite(f)) return -1;
  if (!(f <= max_dev)) return 0;
  // (1 + D)^-1/2 = sum_k c_k D^k, c_k = c_{k-1} (1 - 2k) / (2k); ||D||_2 <= f, so the
  // tail after p terms is below |c_{p+1}| f^{p+1} / (1 - f); stop below eps.
  double c[16];
  c[0] = 1.0;
  for (int k = 1; k < 16; ++k) c[k] = c[k - 1] * (1.0 - 2.0 * k) / (2.0 * k);
  int p = 1;
  while (p < 14 && fabs(c[p + 1]) * pow(f, p + 1) / (1.0 - f) > eps) ++p;
  // Horner: P = c_{p-1} 1 + c_p D; P <- c_k 1 + D P for k = p-2 .. 0
  auto C = (double2*)Cv, T = (double2*)Tv;
  double2* cur = (p % 2) ? C : T;   // ping-pong so that the last product lands in C
  double2* nxt = (p % 2) ? T : C;
  const unsigned ge = unsigned((mm + 255) / 256);
  hipLaunchKernelGGL(k_axpy_identity, dim3(ge), dim3(256), 0, st, (const double2*)D, c[p], c[p - 1],
                     cur, m, g_launch_gate);
  for (int k = p - 2; k >= 0; --k) {
    gemm_square(D, 0, cur, 0, nxt, m, st, 1, c[k]);   // a polynomial in D: Hermitian
    std::swap(cur, nxt);
  }
  return p;
}

// ------------------------------------------------------------------ inverse square root
// C = I^-1/2 by the coupled Newton-Schulz iteration
//   T = 1 + (1 - Z Y) / 2,  Z <- T Z,  Y <- Y T   from  Y = I / s, Z = 1
// (s >= ||I||_2 the largest absolute row sum; Z -> (I/s)^-1/2, the defect
// falls quadratically once below one) and one Newton step on C I C = 1 with
// the overlap itself.  Error of the states' overlap at condition 10, 100, 1e3
// (300 states): 2e-15, 5e-15, 4e-14 against 4e-14, 7e-14, 2e-13 by
// eigenvectors; near 1e6 the two are level, so the steps are limited to what
// overlaps to about 1e3 take.
// Two launches a step, the two updates in one, against some 40 of a Jacobi sweep:
// 151 + 50 trial states at 24^3, initialisation 4990 -> 800 us.
constexpr int NEWTON_STEPS = 13;
constexpr double NEWTON_DEFECT = 1e-8;   // of C I C before its last step: the square is below rounding
// The iteration does not see the overlap's scale, but its caller refuses an
// eigenvalue at or below 1e-10 and norms that overflow when squared.  A defect
// below 0.7 within 13 steps means that every eigenvalue of I / s grew to 0.3
// by at most 2.25 a step, so that it was above 7.9e-6: from s = NEWTON_NORM_MIN
// on none is near 1e-10.  Other overlaps go by eigenvectors, which decide.
constexpr double NEWTON_NORM_MIN = 1e-4, NEWTON_NORM_MAX = 1e150;

// rs[i] = sum_j |I_ij|, one wave per row.
__global__ void __launch_bounds__(256)
k_row_sums(const double2* __restrict__ I, int m, double* __restrict__ rs) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= m) return;
  double a = 0.0;
  for (int j = lane; j < m; j += 64) a += hypot(I[size_t(i) * m + j].x, I[size_t(i) * m + j].y);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if (lane == 0) rs[i] = a;
}

// Largest of rs[0 .. m), NaN kept; the same in every thread of 256.
__device__ inline double max_of(const double* __restrict__ rs, int m, double* red) {
  double v = 0.0;
  for (int i = threadIdx.x; i < m; i += 256) v = (rs[i] > v || rs[i] != rs[i]) ? rs[i] : v;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double t = __shfl_xor(v, o);
    v = (t > v || t != t) ? t : v;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = red[0];
  for (int w = 1; w < 4; ++w) v = (red[w] > v || red[w] != red[w]) ? red[w] : v;
  return v;
}

// Y = X / s (ROOT: X / sqrt(s)), s = max rs; host (if given, host-visible) gets s.
template <bool ROOT>
__global__ void __launch_bounds__(256)
k_scale_by_norm(const double2* __restrict__ X, const double* __restrict__ rs, int m, double2* __restrict__ Y,
                double* __restrict__ host) {
  __shared__ double red[4];
  const double s = max_of(rs, m, red), f = ROOT ? 1.0 / sqrt(s) : 1.0 / s;
  if (host != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *host = s;
  const size_t n = size_t(m) * m;
  for (size_t e = size_t(blockIdx.x) * 256 + threadIdx.x; e < n; e += size_t(gridDim.x) * 256)
    Y[e] = make_double2(f * X[e].x, f * X[e].y);
}

// T = 1 + (1 - P) / 2.
__global__ void __launch_bounds__(256)
k_newton_half(const double2* __restrict__ P, double2* __restrict__ T, int m) {
  const size_t n = size_t(m) * m;
  for (size_t e = size_t(blockIdx.x) * 256 + threadIdx.x; e < n; e += size_t(gridDim.x) * 256)
    T[e] = make_double2((e / m == e % m ? 1.5 : 0.0) - 0.5 * P[e].x, -0.5 * P[e].y);
}

bool inverse_sqrt(const void* Iv, void* Cv, void* const* work, int m, double* rs, double* scratch,
                  hipStream_t st, double* host) {
  auto I = (const double2*)Iv;
  double2* w[6];
  for (int i = 0; i < 6; ++i) w[i] = (double2*)work[i];
  double2 *Y = w[0], *Yn = w[1], *Z = w[2], *Zn = w[3], *T = w[4], *P = w[5];
  const int nb = int(std::min<size_t>(256, (size_t(m) * m + 255) / 256));
  // ||1 - Z Y||_F from t = 1 + (1 - Z Y) / 2 (d: work)
  auto norm = [&](const double2* t, double2* d) -> double {
    hipLaunchKernelGGL(k_minus_identity, dim3(nb), dim3(256), 0, st, t, d, m, scratch, (const int*)nullptr);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(64), 0, st, (const double*)scratch, nb, scratch + nb, host,
                       (const int*)nullptr);
    return hipStreamSynchronize(st) == hipSuccess ? 2.0 * sqrt(host[0]) : HUGE_VAL;
  };
  // the order of the factors and the missing symmetrisation matter: rounding
  // errors that do not commute with I then stay bounded
  auto step = [&] {
    gemm_square(Z, 0, Y, 0, T, m, st, 0, 1.5, nullptr, -0.5);
    gemm_square_pair(T, Z, Zn, Y, T, Yn, m, st);
    std::swap(Z, Zn);
    std::swap(Y, Yn);
  };
  hipLaunchKernelGGL(k_row_sums, dim3((m + 3) / 4), dim3(256), 0, st, I, m, rs);
  hipLaunchKernelGGL(k_scale_by_norm<false>, dim3(nb), dim3(256), 0, st, I, (const double*)rs, m, Y, host + 1);
  hipLaunchKernelGGL(k_newton_half, dim3(nb), dim3(256), 0, st, (const double2*)Y, Z, m);   // Z_0 = 1
  gemm_square(Y, 0, Z, 0, Yn, m, st, 1);
  std::swap(Y, Yn);
  int done = 0;
  for (int n = 7;; n = 3) {
    for (int k = 0; k < n; ++k) step();
    done += n;
    double f = norm(T, P);   // before the last step
    if (!std::isfinite(f) || !(host[1] >= NEWTON_NORM_MIN && host[1] <= NEWTON_NORM_MAX)) return false;
    if (f < 0.7) {
      // the defect goes from f to at most 3/4 f^2 + 1/4 f^3
      for (f = 0.75 * f * f + 0.25 * f * f * f; f > 1e-9; f = 0.75 * f * f + 0.25 * f * f * f) step();
      break;
    }
    if (done >= NEWTON_STEPS) return false;
  }
  hipLaunchKernelGGL(k_scale_by_norm<true>, dim3(nb), dim3(256), 0, st, (const double2*)Z, (const double*)rs, m, Zn,
                     (double*)nullptr);
  gemm_square(Zn, 0, I, 0, T, m, st);
  gemm_square(T, 0, Zn, 0, Y, m, st, 1, 1.5, nullptr, -0.5);
  gemm_square(Zn, 0, Y, 0, Cv, m, st, 1);
  return norm(Y, P) <= NEWTON_DEFECT;   // false for NaN
}

// ------------------------------------------------------------------ device-decided steps
// The kernels below make the decisions of the host-driven steps on the
// device; they are launched without a gate and read the box's flags
// themselves.
__global__ void k_set_flag(int* __restrict__ flags, int idx, int value) {
  if (threadIdx.x == 0) flags[idx] = value;
}
__global__ void k_set_double(double* __restrict__ d, int idx, double value) {
  if (threadIdx.x == 0) d[idx] = value;
}

void set_flag(int* flags, int idx, int value, hipStream_t st) {
  hipLaunchKernelGGL(k_set_flag, dim3(1), dim3(64), 0, st, flags, idx, value);
}
void set_double(double* d, int idx, double value, hipStream_t st) {
  hipLaunchKernelGGL(k_set_double, dim3(1), dim3(64), 0, st, d, idx, value);
}

constexpr int SERIES_PMAX = 14;   // terms of the series at most (as loewdin_series)

// From ||D||_F^2 (fro2): the term count p of the series and its
// coefficients (dbl[D_SERIES + 2 ..]), the gates of the Horner steps, or the
// hand-over to the host.  Same arithmetic as loewdin_series.
__global__ void k_series_plan(const double* __restrict__ fro2, double max_dev, double eps, int pcap,
                              int* __restrict__ flags, double* __restrict__ dbl, int set) {
  if (threadIdx.x != 0) return;
  const bool active = flags[F_ACTIVE] != 0;
  const double f = sqrt(*fro2);
  int p = 0;
  if (active) {
    if (!isfinite(f) || !(f <= max_dev)) {
      flags[F_HOST] = HOST_LOEWDIN;
      flags[F_HOST_SET] = set;
      flags[F_ACTIVE] = 0;
    } else {
      double c[16];
      c[0] = 1.0;
      for (int k = 1; k < 16; ++k) c[k] = c[k - 1] * (1.0 - 2.0 * k) / (2.0 * k);
      p = 1;
      while (p < pcap && fabs(c[p + 1]) * pow(f, p + 1) / (1.0 - f) > eps) ++p;
      for (int k = 0; k < 16; ++k) dbl[D_SERIES + 2 + k] = c[k];
    }
  }
  dbl[D_SERIES] = f;
  dbl[D_SERIES + 1] = double(p);
  for (int k = 0; k <= SERIES_PMAX - 2; ++k) flags[F_SERIES + k] = (active && p > 0 && k <= p - 2) ? 1 : 0;
}

// Horner start P = c_{p-1} 1 + c_p D, written to the buffer that step p-2
// reads (buf[(p-1) % 2]); gated by the box's F_ACTIVE and run only if the
// series was planned (p > 0).
__global__ void k_series_start(const double2* __restrict__ D, const double* __restrict__ dbl,
                               double2* __restrict__ buf0, double2* __restrict__ buf1, int m,
                               const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int p = int(dbl[D_SERIES + 1]);
  if (p <= 0) return;
  const double a = dbl[D_SERIES + 2 + p], c = dbl[D_SERIES + 2 + p - 1];
  double2* P = ((p - 1) % 2) ? buf1 : buf0;
  const size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= size_t(m) * m) return;
  const double2 d = D[e];
  P[e] = make_double2(a * d.x + ((e / m == e % m) ? c : 0.0), a * d.y);
}

void loewdin_series_dev(const void* Iv, void* Cv, void* Dv, void* Tv, int m, double max_dev,
                        double eps, double* scratch, hipStream_t st, int* flags, double* dbl, int set) {
  if (m <= 0) return;
  auto D = (double2*)Dv;
  const size_t mm = size_t(m) * m;
  const int nb = int(std::min<size_t>(256, (mm + 255) / 256));
  const int* active = flags + F_ACTIVE;
  {
    GateScope g(active);
    hipLaunchKernelGGL(k_minus_identity, dim3(nb), dim3(256), 0, st, (const double2*)Iv, D, m, scratch, g_launch_gate);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(64), 0, st, (const double*)scratch, nb, scratch + nb, (double*)nullptr, g_launch_gate);
  }
  // the most terms any accepted norm (f <= max_dev) can need, plus one:
  // Horner steps beyond those are never taken and are not captured
  double c[16];
  c[0] = 1.0;
  for (int k = 1; k < 16; ++k) c[k] = c[k - 1] * (1.0 - 2.0 * k) / (2.0 * k);
  int pmax = 1;
  while (pmax < SERIES_PMAX && fabs(c[pmax + 1]) * pow(max_dev, pmax + 1) / (1.0 - max_dev) > eps)
    ++pmax;
  const int pcap = std::min(pmax + 1, SERIES_PMAX);
  hipLaunchKernelGGL(k_series_plan, dim3(1), dim3(64), 0, st, (const double*)(scratch + nb), max_dev,
                     eps, pcap, flags, dbl, set);
  // buf[0] = C receives the last Horner step (k = 0), buf[1] = T
  auto C = (double2*)Cv, T = (double2*)Tv;
  double2* buf[2] = {C, T};
  const unsigned ge = unsigned((mm + 255) / 256);
  hipLaunchKernelGGL(k_series_start, dim3(ge), dim3(256), 0, st, (const double2*)D,
                     (const double*)dbl, C, T, m, active);
  for (int k = pcap - 2; k >= 0; --k) {
    GateScope g(flags + F_SERIES + k);
    gemm_square(D, 0, buf[(k + 1) % 2], 0, buf[k % 2], m, st, 1, 0.0, dbl + D_SERIES + 2 + k);
  }
}

// One workgroup of 256 threads: Delta-eps from the residual norms of the
// occupied states of every set, in a fixed order.
struct R2Sets {
  const double* r2[64];
  int nocc[64];
};
__global__ void __launch_bounds__(256)
k_iteration_end(R2Sets sets, int nset, int count, int* __restrict__ flags, double* __restrict__ dbl) {
  if (flags[F_ACTIVE] == 0) return;
  __shared__ double buf[256];
  double acc = 0.0;
  for (int s = 0; s < nset; ++s)
    for (int a = threadIdx.x; a < sets.nocc[s]; a += 256) acc += sets.r2[s][a];
  buf[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) buf[threadIdx.x] += buf[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double de = sqrt(buf[0] / double(count > 0 ? count : 1));
    dbl[D_DE] = de;
    flags[F_ITER] += 1;
    if (!isfinite(de)) {
      flags[F_HOST] = HOST_NAN;
      flags[F_HOST_SET] = 0;
      flags[F_ACTIVE] = 0;
    } else if (dbl[D_TOL] > 0.0 && de <= dbl[D_TOL]) {
      flags[F_CONV] = 1;
      flags[F_ACTIVE] = 0;
    }
  }
}

void iteration_end(const double* const* r2, const int* nocc, int nset, int count, int* flags,
                   double* dbl, hipStream_t st) {
  R2Sets sets{};
  const int ns = std::min(nset, 64);
  for (int s = 0; s < ns; ++s) {
    sets.r2[s] = r2[s];
    sets.nocc[s] = nocc[s];
  }
  hipLaunchKernelGGL(k_iteration_end, dim3(1), dim3(256), 0, st, sets, ns, count, flags, dbl);
}

// Gauge of the paper-literal update.  info[3 c .. 3 c + 2] = (start a, size k,
// offset o) of the cluster holding column c; a cluster's k x k diagonal
// block lives at packed[o ..] row-major.
__global__ void k_gauge_gather(const double2* __restrict__ Z, int m, const int* __restrict__ info,
                               double2* __restrict__ packed, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int c = blockIdx.y;
  const int a = info[3 * c], k = info[3 * c + 1], o = info[3 * c + 2];
  for (int r = threadIdx.x; r < k; r += blockDim.x)
    packed[size_t(o) + size_t(r) * k + (c - a)] = Z[size_t(a + r) * m + c];
}

// out[:, c] = sum_l Z[:, a + l] Q[l][c - a] over the cluster of column c.
__global__ void k_gauge_apply(const double2* __restrict__ Z, int m, const int* __restrict__ info,
                              const double2* __restrict__ Q, double2* __restrict__ out, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int c = blockIdx.y;
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= m) return;
  const int a = info[3 * c], k = info[3 * c + 1], o = info[3 * c + 2];
  double2 acc = make_double2(0.0, 0.0);
  for (int l = 0; l < k; ++l) acc = cadd(acc, cmul(Z[size_t(row) * m + a + l], Q[size_t(o) + size_t(l) * k + (c - a)]));
  out[size_t(row) * m + c] = acc;
}

void gauge_gather(const void* Z, int m, const int* info, void* packed, hipStream_t st) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_gauge_gather, dim3(1, m), dim3(64), 0, st, (const double2*)Z, m, info,
                     (double2*)packed, g_launch_gate);
}

void gauge_apply(const void* Z, int m, const int* info, const void* Q, void* out, hipStream_t st) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_gauge_apply, dim3((m + 255) / 256, m), dim3(256), 0, st, (const double2*)Z, m,
                     info, (const double2*)Q, (double2*)out, g_launch_gate);
}

void scale_columns(void* X, const double* d, int m, hipStream_t st) {
  const size_t mm = size_t(m) * m;
  hipLaunchKernelGGL(k_scale_columns, dim3(unsigned((mm + 255) / 256)), dim3(256), 0, st,
                     (double2*)X, d, m, g_launch_gate);
}

void gap_pivots(const void* Linv, const double* gap, int m, int* info, hipStream_t st, double floor_v) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_gap_pivots, dim3((m + 3) / 4), dim3(256), 0, st, (const double2*)Linv, gap, m, info,
                     floor_v, g_launch_gate);
}

void gap_eigenvalues(const void* X, const double* w, const double* gap, int m, int* info, hipStream_t st,
                     double floor_v) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_gap_eigenvalues, dim3((m + 63) / 64), dim3(256), 0, st, (const double2*)X, w, gap, m,
                     info, floor_v, g_launch_gate);
}

void inv_sqrt(double* w, int m, int* info, hipStream_t st, double floor_v) {
  hipLaunchKernelGGL(k_inv_sqrt, dim3((m + 255) / 256), dim3(256), 0, st, w, m, info, floor_v, g_launch_gate);
}

}  // namespace sky
