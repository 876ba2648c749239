// Subspace solves of up to SMALL_M states in one workgroup (Sec. 3.3.2, steps
// 3b-3d): Loewdin's I^-1/2 by its series, H' = C H C, the eigenvector
// refinement with its cluster solves and stop tests, the sorted eigenpairs
// and U = C Z, by the formulas of loewdin_series and refine_eigh.
//
// At these sizes a product takes a microsecond on one CU, and the general
// path's launches and host waits (some 15 launches and a wait per refinement
// step) are what a solve costs.  Here every matrix stays in LDS, the
// products run on the FP64 matrix cores of the one CU, and the host waits once
// for the outcome.  What bounds it is the latency of the serial steps: products
// of 0.5 (16 states) to 1 us (32), and the rounds of the cluster rotations.
// 16^3, FP64: an iteration of 8 + 8 states 1000 -> 413 us; overlap, solve and
// combination of 8 states 296 -> 93 us, of 32 states 385 -> 140 us.  Above 32
// states the eight matrices no longer fit LDS (32: 136 of 160 KB).
#include <cmath>

#include "jacobi_rot.h"
#include "mfma_f64.h"
#include "sky_kernels.h"

namespace sky {

namespace {
using namespace jrot;
using mfma::d4;

constexpr int SM = SMALL_M;      // largest order
constexpr int NT = 256;          // threads
constexpr int TEAM_K = 16;       // widest cluster solved by one wave

struct SmallArgs {
  const double2 *I, *H;          // overlap and Hamiltonian; I null: H is diagonalised as it is
  double2 *C, *Hp, *Z, *U;       // I^-1/2, H', eigenvectors, C Z (C, Hp, U unused without I)
  double* w;
  int m, maxit, set;
  double max_dev, eps;           // the series: largest ||I - 1||_F, remainder
  RefineTargets tg;
  double* host;                  // host-visible outcome, or null
  int* flags;                    // the box's flags (device-decided runs), or null
};

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// out = op(A) B over matrices stored to order MP (zero beyond m), op the
// conjugate transpose with CT.  HERM: the product is Hermitian; the lower
// triangle is computed and mirrored.  Order 16: one wave each for the real and
// the imaginary part; order 32: a tile per wave.  Ends with a barrier; out
// is neither A nor B.
template <int MP, bool CT, bool HERM>
__device__ inline void product(double2* __restrict__ out, const double2* A, const double2* B) {
  constexpr int LD = MP + 1;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int ti = MP == 32 ? wv >> 1 : 0, tj = MP == 32 ? wv & 1 : 0;
  const bool re = MP == 32 || wv == 0, im = MP == 32 || wv == 1;
  if ((re || im) && !(HERM && tj > ti)) {
    d4 cr{0, 0, 0, 0}, ci{0, 0, 0, 0};
    double2 a[MP / 4], b[MP / 4];
#pragma unroll
    for (int q = 0; q < MP / 4; ++q) {
      const int k = 4 * q + kq;
      b[q] = B[k * LD + 16 * tj + r];
      a[q] = CT ? A[k * LD + 16 * ti + r] : A[(16 * ti + r) * LD + k];
      if (CT) a[q].y = -a[q].y;
    }
    if (re)
#pragma unroll
      for (int q = 0; q < MP / 4; ++q) {
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].x, b[q].x, cr, 0, 0, 0);
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[q].y, b[q].y, cr, 0, 0, 0);
      }
    if (im)
#pragma unroll
      for (int q = 0; q < MP / 4; ++q) {
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].x, b[q].y, ci, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].y, b[q].x, ci, 0, 0, 0);
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 16 * ti + 4 * e + kq, j = 16 * tj + r;
      if (HERM && j > i) continue;
      if (re) out[i * LD + j].x = cr[e];
      if (im) out[i * LD + j].y = HERM && i == j ? 0.0 : ci[e];
      if (HERM && i > j) {
        if (re) out[j * LD + i].x = cr[e];
        if (im) out[j * LD + i].y = -ci[e];
      }
    }
  }
  __syncthreads();
}

// Sums of v[0 .. N) over the workgroup, the last as a maximum that keeps NaN
// when MAXLAST; the same in every thread.
template <int N, bool MAXLAST>
__device__ inline void reduce(double (&v)[N], double (*red)[3]) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const double t = __shfl_xor(v[q], o, 64);
      if (MAXLAST && q == N - 1) v[q] = (t > v[q] || t != t) ? t : v[q];
      else v[q] += t;
    }
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int q = 0; q < N; ++q) red[threadIdx.x >> 6][q] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N; ++q) {
    v[q] = red[0][q];
    for (int w = 1; w < NT / 64; ++w) {
      const double t = red[w][q];
      if (MAXLAST && q == N - 1) v[q] = (t > v[q] || t != t) ? t : v[q];
      else v[q] += t;
    }
  }
}

struct ClusterWork {
  Rot rot[4][SM / 2];
  int2 pair[4][SM / 2];
  double red[4][3];
};

// Jacobi solve of the cluster of k sorted positions from s0 (see
// k_ref_cluster_eig): W's block (rows and columns s0 ..) gets the unitary that
// diagonalises the cluster block of (1 + R/2) S (1 + R/2).  M0, M1: work, the
// same block of each.  By one wave (TEAM false) or the workgroup.  Odd k: the
// index k stands for a row and column of zeros that nothing rotates with.
template <int MP, bool TEAM>
__device__ inline void cluster_eig(const double2* S, const double2* R, const int* order, int s0, int k,
                                   double tol, double2* M0, double2* M1, double2* Wm, ClusterWork& cw) {
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tid = TEAM ? threadIdx.x : lane;
  constexpr int LD = MP + 1;
  constexpr int T = TEAM ? NT : 64;
  auto sync = [] {
    if (TEAM) __syncthreads();
    else wave_sync();
  };
  const int np = (k + 1) & ~1, nh = np / 2;
  double2* M = M0 + s0 * LD + s0;
  double2* P = M1 + s0 * LD + s0;
  double2* J = Wm + s0 * LD + s0;
  for (int e = tid; e < k * k; e += T) {
    const int i = e / k, j = e % k, oi = order[s0 + i], oj = order[s0 + j];
    const double2 a = S[oi * LD + oj], b = S[oj * LD + oi];
    M[i * LD + j] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    if (R) {
      const double2 c = R[oi * LD + oj], d = R[oj * LD + oi];
      J[i * LD + j] = make_double2(0.5 * (c.x + d.x), 0.5 * (c.y - d.y));
    }
  }
  sync();
  if (R) {
    for (int e = tid; e < k * k; e += T) {
      const int i = e / k, j = e % k;
      double2 acc = M[i * LD + j];
      for (int l = 0; l < k; ++l) acc = cadd(acc, cscale(0.5, cmul(M[i * LD + l], J[l * LD + j])));
      P[i * LD + j] = acc;
    }
    sync();
    for (int e = tid; e < k * k; e += T) {
      const int i = e / k, j = e % k;
      double2 acc = P[i * LD + j];
      for (int l = 0; l < k; ++l) acc = cadd(acc, cscale(0.5, cmul(J[i * LD + l], P[l * LD + j])));
      M[i * LD + j] = acc;
    }
    sync();
  }
  for (int e = tid; e < k * k; e += T) J[(e / k) * LD + e % k] = make_double2(e / k == e % k ? 1.0 : 0.0, 0.0);
  sync();
  const double2 zero = make_double2(0.0, 0.0);
  for (int sweep = 0; sweep < 16; ++sweep) {
    double v[2] = {0.0, 0.0};   // off-diagonal, diagonal
    for (int e = tid; e < k * k; e += T) {
      const int i = e / k, j = e % k;
      const double2 x = M[i * LD + j];
      v[i == j ? 1 : 0] += x.x * x.x + x.y * x.y;
    }
    if (TEAM) {
      reduce<2, false>(v, cw.red);
    } else {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        v[0] += __shfl_xor(v[0], o, 64);
        v[1] += __shfl_xor(v[1], o, 64);
      }
    }
    if ((v[0] <= tol * tol * v[1]) || (v[0] < 1e-300)) break;   // the same in every thread
    for (int r = 0; r < np - 1; ++r) {
      if (lane < nh) {
        int p, q;
        rr_pair(np, r, lane, p, q);
        if (p > q) { const int t = p; p = q; q = t; }
        cw.pair[wv][lane] = make_int2(p, q);
        Rot g{1.0, 0.0, 1.0, 0.0};
        if (q < k) g = make_rot(M[p * LD + p].x, M[q * LD + q].x, M[p * LD + q]);
        cw.rot[wv][lane] = g;
      }
      wave_sync();
      // M <- G^H M G on the 2x2 blocks (rotation u rows, rotation v columns)
      for (int e = tid; e < nh * nh; e += T) {
        const int u = e / nh, w = e % nh;
        const int pu = cw.pair[wv][u].x, qu = cw.pair[wv][u].y, pv = cw.pair[wv][w].x, qv = cw.pair[wv][w].y;
        const bool ru = qu < k, rv = qv < k;
        const Rot gu = cw.rot[wv][u], gv = cw.rot[wv][w];
        const double2 epu = make_double2(gu.er, gu.ei), epv = make_double2(gv.er, gv.ei);
        const double2 x00 = M[pu * LD + pv], x01 = rv ? M[pu * LD + qv] : zero;
        const double2 x10 = ru ? M[qu * LD + pv] : zero, x11 = ru && rv ? M[qu * LD + qv] : zero;
        const double2 y00 = csub(cscale(gv.c, cmul(x00, epv)), cscale(gv.s, x01));
        const double2 y01 = cadd(cscale(gv.s, cmul(x00, epv)), cscale(gv.c, x01));
        const double2 y10 = csub(cscale(gv.c, cmul(x10, epv)), cscale(gv.s, x11));
        const double2 y11 = cadd(cscale(gv.s, cmul(x10, epv)), cscale(gv.c, x11));
        P[pu * LD + pv] = csub(cscale(gu.c, cmulc(y00, epu)), cscale(gu.s, y10));
        if (rv) P[pu * LD + qv] = csub(cscale(gu.c, cmulc(y01, epu)), cscale(gu.s, y11));
        if (ru) P[qu * LD + pv] = cadd(cscale(gu.s, cmulc(y00, epu)), cscale(gu.c, y10));
        if (ru && rv) P[qu * LD + qv] = cadd(cscale(gu.s, cmulc(y01, epu)), cscale(gu.c, y11));
      }
      // J <- J G
      for (int e = tid; e < k * nh; e += T) {
        const int i = e / nh, w = e % nh;
        const int pv = cw.pair[wv][w].x, qv = cw.pair[wv][w].y;
        if (qv >= k) continue;
        const Rot gv = cw.rot[wv][w];
        const double2 epv = make_double2(gv.er, gv.ei);
        const double2 x0 = J[i * LD + pv], x1 = J[i * LD + qv];
        J[i * LD + pv] = csub(cscale(gv.c, cmul(x0, epv)), cscale(gv.s, x1));
        J[i * LD + qv] = cadd(cscale(gv.s, cmul(x0, epv)), cscale(gv.c, x1));
      }
      double2* t = M;
      M = P;
      P = t;
      sync();
    }
  }
}

template <int MP>
__global__ void __launch_bounds__(NT)
k_subspace_small(SmallArgs p, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  constexpr int LD = MP + 1;
  __shared__ double2 mat[8][MP * LD];
  __shared__ double ser[16], lam[SM], red[4][3];
  __shared__ int rank[SM], order[SM], reach[SM], cstart[SM], csize[SM], clist[SM / 2], ncl;
  __shared__ ClusterWork cw;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = p.m;
  double2 *A = mat[0], *X = mat[1], *S = mat[2], *R = mat[3], *T = mat[4], *E = mat[5], *B = mat[6],
          *Q = mat[7];
  auto load = [&](double2* d, const double2* src, bool minus1) {
    for (int e = tid; e < MP * MP; e += NT) {
      const int i = e / MP, j = e % MP;
      double2 v = make_double2(0.0, 0.0);
      if (i < m && j < m) v = src[i * m + j];
      if (minus1 && i == j && i < m) v.x -= 1.0;
      d[i * LD + j] = v;
    }
  };
  auto store = [&](double2* d, const double2* src) {
    for (int e = tid; e < m * m; e += NT) d[e] = src[(e / m) * LD + e % m];
  };
  // the outcome: series terms (-1 not finite, 0 too far from orthonormality),
  // refinement steps (-1: none that converged) and the steps taken
  auto finish = [&](int terms, int its, int taken) {
    if (p.host != nullptr && tid == 0) {
      p.host[0] = double(terms);
      p.host[1] = double(its);
    }
    if (p.flags != nullptr && tid == 0) {
      p.flags[F_REF_RUN] = 0;
      p.flags[F_REF_STEPS] = taken;
      if (terms <= 0 || its < 0) {
        p.flags[F_HOST] = terms <= 0 ? HOST_LOEWDIN : HOST_REFINE;
        p.flags[F_HOST_SET] = p.set;
        p.flags[F_ACTIVE] = 0;
      }
    }
  };
  int terms = 1;
  if (p.I != nullptr) {
    // ---- C = I^-1/2 in Horner form, H' = C H C (D in S, H in X)
    load(S, p.I, true);
    load(X, p.H, false);
    __syncthreads();
    double f2[1] = {0.0};
    for (int e = tid; e < m * m; e += NT) {
      const double2 d = S[(e / m) * LD + e % m];
      f2[0] += d.x * d.x + d.y * d.y;
    }
    reduce<1, false>(f2, red);
    const double f = sqrt(f2[0]);
    if (!isfinite(f) || !(f <= p.max_dev)) {
      finish(isfinite(f) ? 0 : -1, -1, 0);
      return;
    }
    double c[15];
    c[0] = 1.0;
#pragma unroll
    for (int k = 1; k < 15; ++k) c[k] = c[k - 1] * (1.0 - 2.0 * k) / (2.0 * k);
    double ck[2] = {c[1], c[0]};   // c_p and c_{p-1}
    double fp = f * f;             // f^(p+1)
#pragma unroll
    for (int k = 2; k < 15; ++k)
      if (terms == k - 1 && fabs(c[k]) * fp / (1.0 - f) > p.eps) {
        terms = k;
        ck[0] = c[k];
        ck[1] = c[k - 1];
        fp *= f;
      }
    if (tid == 0)
#pragma unroll
      for (int k = 0; k < 15; ++k) ser[k] = c[k];
    double2 *cur = T, *nxt = E;
    for (int e = tid; e < MP * MP; e += NT) {
      const int i = e / MP, j = e % MP;
      const double2 d = S[i * LD + j];
      cur[i * LD + j] = make_double2(ck[0] * d.x + (i == j && i < m ? ck[1] : 0.0), ck[0] * d.y);
    }
    __syncthreads();
    for (int k = terms - 2; k >= 0; --k) {
      product<MP, false, true>(nxt, S, cur);   // a polynomial in D: Hermitian
      if (tid < m) nxt[tid * LD + tid].x += ser[k];
      __syncthreads();
      double2* t = cur;
      cur = nxt;
      nxt = t;
    }
    store(p.C, cur);
    product<MP, false, false>(Q, cur, X);
    product<MP, false, true>(A, Q, cur);
    store(p.Hp, A);
  } else {
    load(A, p.H, false);
    __syncthreads();
  }
  // ---- refinement: see refine_eigh
  const double tol = p.tg.tol;
  double dia[1] = {0.0};
  if (tid < m) dia[0] = A[tid * LD + tid].x * A[tid * LD + tid].x;
  reduce<1, false>(dia, red);
  double tau = p.tg.noise * sqrt(dia[0] / m);
  if (tid < SM) order[tid] = tid;
  int its = -1, it = 0;
  for (;; ++it) {
    const double2 *Sp = A, *Rp = nullptr;
    if (it > 0) {
      product<MP, true, true>(R, X, X);
      product<MP, false, false>(T, A, X);
      product<MP, true, true>(S, X, T);
      // R <- 1 - X^H X; norms (the mirrored products are exactly Hermitian)
      double v[3] = {0.0, 0.0, 0.0};
      for (int e = tid; e < MP * MP; e += NT) {
        const int i = e / MP, j = e % MP;
        if (i >= m || j >= m || i < j) continue;
        const double2 s = S[i * LD + j], g = R[i * LD + j];
        double rg;
        if (i == j) {
          v[1] += s.x * s.x;
          R[i * LD + j] = make_double2(1.0 - g.x, 0.0);
          rg = fabs(1.0 - g.x);
        } else {
          const double s2 = s.x * s.x + s.y * s.y;
          // couplings at the noise floor of H' count as converged (not rotated)
          if (s2 > tau * tau) v[0] += 2.0 * s2;
          if (s2 != s2) v[0] = s2;
          R[i * LD + j] = make_double2(-g.x, -g.y);
          R[j * LD + i] = make_double2(-g.x, g.y);
          rg = hypot(g.x, g.y);
        }
        v[2] = (rg > v[2] || rg != rg) ? rg : v[2];
      }
      reduce<3, true>(v, red);
      if (v[0] != v[0] || v[1] != v[1] || v[2] != v[2]) break;
      if ((v[0] <= tol * tol * v[1] || v[0] < 1e-300) && v[2] <= p.tg.orth) {
        its = it;
        break;
      }
      if (it >= p.maxit) break;
      Sp = S;
      Rp = R;
      tau = p.tg.noise * sqrt(v[1] / m);
    }
    if (tid < SM) lam[tid] = tid < m ? Sp[tid * LD + tid].x / (1.0 - (Rp ? Rp[tid * LD + tid].x : 0.0)) : 0.0;
    __syncthreads();
    // ranks and reaches, one half wave per state
    for (int i = tid >> 5; i < SM; i += NT / 32) {
      const int j = lane & 31;
      const double li = lam[i], lj = lam[j];
      const bool less = i < m && j < m && (lj < li || (lj == li && j < i));
      const unsigned long long bits = __ballot(less);
      const int rk = __popc(unsigned(bits >> (lane & 32)));
      if (j == 0 && i < m) {
        rank[i] = rk;
        order[rk] = i;
      }
    }
    __syncthreads();
    for (int i = tid >> 5; i < SM; i += NT / 32) {
      const int j = lane & 31;
      int best = i < m ? rank[i] : 0;
      if (i < m && j < m && rank[j] > best) {
        const double li = lam[i], lj = lam[j];
        const double2 s = Sp[i * LD + j];
        const double2 r = Rp ? Rp[i * LD + j] : make_double2(0.0, 0.0);
        const double g1 = hypot(s.x + lj * r.x, s.y + lj * r.y);
        const double g2 = hypot(s.x + li * r.x, s.y + li * r.y);
        // couplings at the noise floor tau of H' never join a cluster
        if (fmax(g1, g2) > tau && fmax(g1, g2) > REF_THETA * fabs(lj - li)) best = rank[j];
      }
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
      if (j == 0 && i < m) reach[rank[i]] = best;
    }
    __syncthreads();
    // clusters: cuts after the positions that no strong coupling crosses
    if (wv == 0) {
      int run = lane < m ? reach[lane] : -1;
#pragma unroll
      for (int o = 1; o < SM; o <<= 1) {
        const int t = __shfl_up(run, o, 64);
        if (lane >= o) run = max(run, t);
      }
      const unsigned long long cuts = __ballot(lane < m && (run == lane || lane == m - 1));
      const unsigned long long below = lane < m ? cuts & ((1ull << lane) - 1) : 0ull;
      const int st = below ? 64 - __clzll(below) : 0;
      const int end = lane < m ? lane + __ffsll(cuts >> lane) : 0;   // one past the cluster's last
      const bool lead = lane < m && st == lane && end - st > 1;
      const unsigned long long leads = __ballot(lead);
      if (lane < m) {
        cstart[lane] = st;
        csize[lane] = end - st;
      }
      if (lead) clist[__popcll(leads & ((1ull << lane) - 1))] = lane;
      if (lane == 0) ncl = __popcll(leads);
    }
    // B = P blockdiag(W): W of the clusters in Q, work in T and E
    for (int e = tid; e < MP * LD; e += NT) B[e] = make_double2(0.0, 0.0);
    __syncthreads();
    const int nc = ncl;
    for (int c = wv; c < nc; c += NT / 64) {
      const int s0 = clist[c], k = csize[s0];
      if (k <= TEAM_K) cluster_eig<MP, false>(Sp, Rp, order, s0, k, tol * 1e-2, T, E, Q, cw);
    }
    __syncthreads();
    for (int c = 0; MP > TEAM_K && c < nc; ++c) {
      const int s0 = clist[c], k = csize[s0];
      if (k > TEAM_K) cluster_eig<MP, true>(Sp, Rp, order, s0, k, tol * 1e-2, T, E, Q, cw);
    }
    __syncthreads();
    for (int e = tid; e < MP * MP; e += NT) {
      const int a = e / MP, b = e % MP;
      if (a >= m || b >= m || cstart[a] != cstart[b]) continue;
      B[order[a] * LD + b] = csize[a] > 1 ? Q[a * LD + b] : make_double2(1.0, 0.0);
    }
    __syncthreads();
    // S2 in Q, R2 in E
    product<MP, false, false>(T, Sp, B);
    product<MP, true, false>(Q, B, T);
    if (Rp) {
      product<MP, false, false>(T, Rp, B);
      product<MP, true, false>(E, B, T);
    }
    if (tid < m) lam[tid] = Q[tid * LD + tid].x / (1.0 - (Rp ? E[tid * LD + tid].x : 0.0));
    __syncthreads();
    // the update, in place of R2
    double emax[1] = {0.0};
    for (int e = tid; e < MP * MP; e += NT) {
      const int a = e / MP, b = e % MP;
      double2 v = make_double2(0.0, 0.0);
      if (a < m && b < m) {
        const double2 s2 = Q[a * LD + b], r2 = Rp ? E[a * LD + b] : make_double2(0.0, 0.0);
        if (cstart[a] == cstart[b]) {
          v = cscale(0.5, r2);
        } else {
          const double2 gb = cadd(s2, cscale(lam[b], r2)), ga = cadd(s2, cscale(lam[a], r2));
          const double den = lam[b] - lam[a];
          if (fmax(hypot(gb.x, gb.y), hypot(ga.x, ga.y)) <= tau) {
            v = cscale(0.5, r2);   // coupling at the noise floor: orthonormality only
          } else if (den != 0.0) {
            v = cscale(1.0 / den, gb);
            const double em = hypot(v.x, v.y);
            if (em > REF_E_CLAMP) v = cscale(REF_E_CLAMP / em, v);
          }
        }
      }
      E[a * LD + b] = v;
      const double mag = hypot(v.x, v.y);
      emax[0] = (mag > emax[0] || mag != mag) ? mag : emax[0];
    }
    reduce<1, true>(emax, red);
    const bool second = !(emax[0] <= p.tg.e2skip);
    if (second) product<MP, false, false>(T, E, E);
    for (int e = tid; e < MP * MP; e += NT) {
      const int a = e / MP, b = e % MP;
      double2 q = E[a * LD + b];
      if (second) q = cadd(q, cscale(0.5, T[a * LD + b]));
      if (a == b && a < m) q.x += 1.0;
      E[a * LD + b] = q;
    }
    __syncthreads();
    if (it == 0) {
      product<MP, false, false>(X, B, E);
    } else {
      product<MP, false, false>(Q, B, E);
      product<MP, false, false>(T, X, Q);
      double2* t = X;
      X = T;
      T = t;
    }
  }
  if (its < 0) {
    finish(terms, -1, it);
    return;
  }
  // ---- eigenpairs in ascending order (Z in T), U = C Z
  if (tid < SM) lam[tid] = tid < m ? S[tid * LD + tid].x : 0.0;
  __syncthreads();
  for (int i = tid >> 5; i < SM; i += NT / 32) {
    const int j = lane & 31;
    const double li = lam[i], lj = lam[j];
    const unsigned long long bits = __ballot(i < m && j < m && (lj < li || (lj == li && j < i)));
    const int rk = __popc(unsigned(bits >> (lane & 32)));
    if (j == 0 && i < m) {
      rank[i] = rk;
      p.w[rk] = li;
    }
  }
  for (int e = tid; e < MP * LD; e += NT) T[e] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int e = tid; e < m * m; e += NT) T[(e / m) * LD + rank[e % m]] = X[(e / m) * LD + e % m];
  __syncthreads();
  store(p.Z, T);
  if (p.I != nullptr) {
    load(A, p.C, false);   // this workgroup wrote it before the barriers above
    __syncthreads();
    product<MP, false, false>(Q, A, T);
    store(p.U, Q);
  }
  finish(terms, its, its);
}

}  // namespace

bool subspace_small(const void* I, const void* H, void* C, void* Hp, void* Z, void* U, int m, double* w,
                    double max_dev, double eps, const RefineTargets& tg, int maxit, hipStream_t st,
                    double* host, int* flags, int set) {
  if (m < 1 || m > SMALL_M) return false;
  SmallArgs a{(const double2*)I, (const double2*)H, (double2*)C, (double2*)Hp, (double2*)Z, (double2*)U,
              w, m, maxit, set, max_dev, eps, tg, host, flags};
  if (m <= 16) hipLaunchKernelGGL(k_subspace_small<16>, dim3(1), dim3(NT), 0, st, a, g_launch_gate);
  else hipLaunchKernelGGL(k_subspace_small<32>, dim3(1), dim3(NT), 0, st, a, g_launch_gate);
  return true;
}

}  // namespace sky
