// Learned spectral preconditioner of the damped step (an extension of
// Eq. dampstep: the paper's damping x0 / (E0 + T_k) is fixed).
//
// The plain step is phi = psi - x0 F^-1[F r / (E0 + T_k)], r = h psi - <h> psi.
// The learned step multiplies the damping, per state alpha and |k| shell s,
// by a gain g = GMAX sigmoid(o), o = MLP(features(alpha, s)):
//   x0 = |k| at the shell centre / |k|max,   x1 = <h>_alpha / E0,
//   x2 = log10(P_s / P + 1e-12) / 6 + 1   (share of the residual's spectral
//        power in shell s),                 x3 = T_k at the shell centre / E0.
// The MLP is 4 -> 128 -> 128 -> 128 -> 1 with ReLU, BF16 weights (rounded
// from FP32 master weights, round to nearest even) and FP32 accumulation.
//
// Training targets come from the solver's own iterates.  For a sampled state,
// the step restricted to shell s is d_s = x0 F^-1[1_s F r / (E0 + T_k)]; to
// first order, with the mean field frozen, the residual after the step
// psi - sum_s g_s d_s is r - sum_s g_s w_s with w_s = (h - <h>) d_s, and the
// target gains minimise |r - sum_s g_s w_s|^2 (real g, normal equations with
// a small ridge, clamped to [0, GMAX]).  The loss is the residual-power
// weighted mean square error of the gains; training is Adam on the GPU with
// this file's forward and backward kernels.
#include <cmath>
#include <random>
#include <vector>

#include "sky_kernels.h"

namespace sky {

namespace {
constexpr int PIN = 4;
constexpr int PH = 128;
constexpr float GMAX = 4.0f;
// parameter offsets: W1[PH][PIN], b1[PH], W2[PH][PH], b2, W3[PH][PH], b3, W4[PH], b4
constexpr int OW1 = 0, OB1 = OW1 + PH * PIN, OW2 = OB1 + PH, OB2 = OW2 + PH * PH,
              OW3 = OB2 + PH, OB3 = OW3 + PH * PH, OW4 = OB3 + PH, OB4 = OW4 + PH,
              NPAR = OB4 + 1;
constexpr int NS_MAX = 32;   // sampled states per collection

__device__ inline float bf16_round(float x) {
  unsigned int u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return __uint_as_float(u & 0xFFFF0000u);
}

// Packed BF16 copies of the two 128 x 128 weights behind the rounded parameters
// (16-byte aligned): W2, W3 row-major for the forward layers, then both
// transposed for the backward ones, so that every B operand of a matrix
// instruction is one 16-byte load.
constexpr int OPACK = (NPAR + 3) / 4 * 4;          // in floats from the parameters
constexpr int WSZ = PH * PH;
__device__ inline unsigned short bf16_hi(float x) { return (unsigned short)(__float_as_uint(x) >> 16); }
__device__ inline const unsigned short* packed(const float* Pb, int layer, bool transposed) {
  return reinterpret_cast<const unsigned short*>(Pb + OPACK) + (transposed ? 2 * WSZ : 0) + layer * WSZ;
}

__global__ void k_round_params(const float* __restrict__ p, float* __restrict__ q, int n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float v = bf16_round(p[i]);
  q[i] = v;
  const int layer = (i >= OW2 && i < OB2) ? 0 : (i >= OW3 && i < OB3) ? 1 : -1;
  if (layer < 0) return;
  unsigned short* w = reinterpret_cast<unsigned short*>(q + OPACK) + layer * WSZ;
  const int o = i - (layer ? OW3 : OW2);
  w[o] = bf16_hi(v);
  w[2 * WSZ + (o % PH) * PH + o / PH] = bf16_hi(v);
}

// ---- forward pass on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16)
// A workgroup carries 16 samples through the MLP, each of its four waves a
// quarter of the neurons.  The two 128 x 128 layers are MFMA products: the
// weights are BF16 values already (the parameters are rounded by
// k_round_params), and each FP32 activation is split exactly into three BF16
// terms h = t0 + t1 + t2 (8 significant bits each, rounded to nearest at each
// step), so that every product t_i w is exact in FP32 and the layer is FP32
// activations x BF16 weights with FP32 accumulation, as the scalar form, up
// to the order of the sums.  MFMA operands: lane l supplies 8 consecutive
// contraction elements starting at 8 (l / 16) of row (A: sample) or column (B:
// neuron) l % 16; register e of lane l returns sample 4 (l / 16) + e, neuron
// l % 16.  The first (4 inputs) and last (1 output) layers are scalar.
//
// A few thousand rows are a few hundred short chains of layers: what counts is
// their latency and that they reach every CU.  Hence 16 rows per workgroup (64
// left three quarters of the CUs idle at 4099 rows), both layers' weights
// loaded before the first is needed, and activations split once, by the wave
// that makes them, into BF16 planes in LDS.  4099 rows: forward 34 -> 11.5,
// backward with the loss 45 -> 12.9.
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int FR = 16;         // samples per workgroup
constexpr int FWV = 4;         // waves per workgroup
constexpr int NJ = PH / 16 / FWV;   // 16-neuron blocks per wave
constexpr int KS = PH / 32;    // matrix instructions per block and split term
constexpr int PLP = PH + 8;    // LDS row pitch of the BF16 planes

// x = v[0][t] + v[1][t] + v[2][t] as three BF16 bit patterns (exact for
// normal FP32 x: 8 significant bits per term, rounded to nearest at each step).
__device__ inline void split3(float x, unsigned short& a, unsigned short& b, unsigned short& c) {
  const float x0 = bf16_round(x), x1 = bf16_round(x - x0), x2 = bf16_round(x - x0 - x1);
  a = bf16_hi(x0);
  b = bf16_hi(x1);
  c = bf16_hi(x2);
}

// Split planes of a workgroup's 16 x 128 activations.
struct alignas(16) Planes {
  unsigned short v[3][FR][PLP];
  __device__ void put(int s, int n, float x) { split3(x, v[0][s][n], v[1][s][n], v[2][s][n]); }
};

struct Weights {
  us8 w[NJ][KS];
};

// The wave's B operands of one layer, neurons (or inputs) 32 wv .. 32 wv + 31.
__device__ inline Weights load_weights(const unsigned short* __restrict__ W, int wv, int lane) {
  Weights r;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      r.w[j][ks] = *reinterpret_cast<const us8*>(W + ((wv * NJ + j) * 16 + (lane & 15)) * PH + ks * 32 +
                                                 (lane >> 4) * 8);
  return r;
}

__device__ inline void layer_mfma(const Planes& in, const Weights& w, f4v (&acc)[NJ], int lane) {
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const us8 a = *reinterpret_cast<const us8*>(&in.v[t][lane & 15][ks * 32 + (lane >> 4) * 8]);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a),
                                                         __builtin_bit_cast(bf8, w.w[j][ks]), acc[j], 0, 0, 0);
    }
}

// H1..H3 (all or none) keep the activations for the backward pass; O the outputs.
__global__ void __launch_bounds__(64 * FWV)
k_mlp_fwd(const float* __restrict__ P, const float* __restrict__ X, int ldx, int B,
          float* __restrict__ H1, float* __restrict__ H2, float* __restrict__ H3,
          float* __restrict__ O, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ Planes pa, pb;
  __shared__ float red[FWV][FR];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int b0 = blockIdx.x * FR;
  const Weights w2 = load_weights(packed(P, 0, false), wv, lane);
  const Weights w3 = load_weights(packed(P, 1, false), wv, lane);
  {  // layer 1: thread -> neuron, half of the samples
    const int n = tid % PH, s0 = (tid / PH) * (FR / 2);
    float w1[PIN];
#pragma unroll
    for (int i = 0; i < PIN; ++i) w1[i] = P[OW1 + n * PIN + i];
    const float bn = P[OB1 + n];
#pragma unroll
    for (int q = 0; q < FR / 2; ++q) {
      const int s = s0 + q, b = b0 + s;
      float a = bn;
      if (b < B)
#pragma unroll
        for (int i = 0; i < PIN; ++i) a += w1[i] * X[size_t(b) * ldx + i];
      a = fmaxf(a, 0.0f);
      pa.put(s, n, a);
      if (H1 && b < B) H1[size_t(b) * PH + n] = a;
    }
  }
  const int col = lane & 15, r0 = 4 * (lane >> 4);
  float bias2[NJ], bias3[NJ], w4[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = (wv * NJ + j) * 16 + col;
    bias2[j] = P[OB2 + n];
    bias3[j] = P[OB3 + n];
    w4[j] = P[OW4 + n];
  }
  __syncthreads();
  f4v acc[NJ];
  layer_mfma(pa, w2, acc, lane);
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = (wv * NJ + j) * 16 + col, b = b0 + r0 + e;
      const float v = fmaxf(acc[j][e] + bias2[j], 0.0f);
      pb.put(r0 + e, n, v);
      if (H2 && b < B) H2[size_t(b) * PH + n] = v;
    }
  __syncthreads();
  layer_mfma(pb, w3, acc, lane);
  // layer 4: the wave's neurons of each sample, lanes in a fixed order
  float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = (wv * NJ + j) * 16 + col, b = b0 + r0 + e;
      const float v = fmaxf(acc[j][e] + bias3[j], 0.0f);
      o[e] += v * w4[j];
      if (H3 && b < B) H3[size_t(b) * PH + n] = v;
    }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int k = 1; k < 16; k <<= 1) o[e] += __shfl_xor(o[e], k);
    if (col == 0) red[wv][r0 + e] = o[e];
  }
  __syncthreads();
  if (tid < FR && b0 + tid < B) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < FWV; ++w) v += red[w][tid];
    O[b0 + tid] = v + P[OB4];
  }
}

// Sum of the sample weights (column 5 of the rows), at least so that it can
// divide: one workgroup, fixed order.
__global__ void __launch_bounds__(1024)
k_pc_wsum(const float* __restrict__ S, int B, double* __restrict__ wsum, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ double red[16];
  double v = 0.0;
  for (int b = threadIdx.x; b < B; b += 1024) v += double(S[size_t(b) * 6 + 5]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < 16; ++w) s += red[w];
    *wsum = s > 0.0 ? s : 1.0;
  }
}

// Loss terms and dL/do per sample: g = GMAX sigmoid(o),
// L = sum_b w_b (g_b - t_b)^2 / sum_b w_b.  S = [x0..x3, t, w] rows.  Then
// dL/d(pre-activation) of the three hidden layers of FR samples:
// D3 = dO W4 relu'(H3), D2 = (D3 W3) relu'(H2), D1 = (D2 W2) relu'(H1), the
// products on the BF16 matrix cores as in the forward layers, with the
// transposed weights.  lpart[blockIdx.x]: the workgroup's loss terms.
__global__ void __launch_bounds__(64 * FWV)
k_mlp_bwd_act(const float* __restrict__ P, const float* __restrict__ S, const float* __restrict__ H1,
              const float* __restrict__ H2, const float* __restrict__ H3,
              const float* __restrict__ O, const double* __restrict__ wsump, int B,
              float* __restrict__ dO, float* __restrict__ D1, float* __restrict__ D2,
              float* __restrict__ D3, double* __restrict__ lpart, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ Planes pa, pb;
  __shared__ float dos[FR];
  __shared__ double ls[FR];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int b0 = blockIdx.x * FR;
  const Weights w3 = load_weights(packed(P, 1, true), wv, lane);
  const Weights w2 = load_weights(packed(P, 0, true), wv, lane);
  if (tid < FR) {
    const int b = b0 + tid;
    float d = 0.0f;
    double l = 0.0;
    if (b < B) {
      const double wsum = *wsump;
      const float t = S[size_t(b) * 6 + 4], w = S[size_t(b) * 6 + 5];
      const float sg = 1.0f / (1.0f + expf(-O[b]));
      const float g = GMAX * sg;
      const float e = g - t;
      l = double(w) * double(e) * double(e) / wsum;
      d = float(2.0 * double(w) * double(e) / wsum) * GMAX * sg * (1.0f - sg);
      dO[b] = d;
    }
    dos[tid] = d;
    ls[tid] = l;
  }
  // the masks of this wave's outputs, ahead of the products that need them
  const int col = lane & 15, r0 = 4 * (lane >> 4);
  bool on2[NJ][4], on1[NJ][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = (wv * NJ + j) * 16 + col, b = b0 + r0 + e;
      on2[j][e] = b < B && H2[size_t(b) * PH + n] > 0.0f;
      on1[j][e] = b < B && H1[size_t(b) * PH + n] > 0.0f;
    }
  __syncthreads();
  if (tid == 0) {
    double l = 0.0;
    for (int k = 0; k < FR; ++k) l += ls[k];
    lpart[blockIdx.x] = l;
  }
  {
    const int n = tid % PH, s0 = (tid / PH) * (FR / 2);
    const float w4 = P[OW4 + n];
#pragma unroll
    for (int q = 0; q < FR / 2; ++q) {
      const int s = s0 + q, b = b0 + s;
      float v = 0.0f;
      if (b < B) {
        v = H3[size_t(b) * PH + n] > 0.0f ? dos[s] * w4 : 0.0f;
        D3[size_t(b) * PH + n] = v;
      }
      pa.put(s, n, v);
    }
  }
  __syncthreads();
  f4v acc[NJ];
  layer_mfma(pa, w3, acc, lane);
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = (wv * NJ + j) * 16 + col, b = b0 + r0 + e;
      const float v = on2[j][e] ? acc[j][e] : 0.0f;
      pb.put(r0 + e, n, v);
      if (b < B) D2[size_t(b) * PH + n] = v;
    }
  __syncthreads();
  layer_mfma(pb, w2, acc, lane);
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = (wv * NJ + j) * 16 + col, b = b0 + r0 + e;
      if (b < B) D1[size_t(b) * PH + n] = on1[j][e] ? acc[j][e] : 0.0f;
    }
}

// ---- parameter gradient
constexpr int GCH = 64;    // samples per chunk of the gradient partials
constexpr int GSUB = 32;   // samples per MFMA step (the contraction of one MFMA)
constexpr int GLP = GSUB + 8;   // LDS row pitch of the transposed planes

// Eight consecutive samples of one neuron, samples past the chunk's end zero.
struct Eight {
  float v[8];
  __device__ void load(const float* __restrict__ p, int b, int c1, int n) {
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = b + t < c1 ? p[size_t(b + t) * PH + n] : 0.0f;
  }
  // the three split terms as one 16-byte store each, at [term][row][8 g ..]
  __device__ void put(unsigned short* base, int rows, int row, int g) const {
    us8 w[3];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      unsigned short a, b, c;
      split3(v[t], a, b, c);
      w[0][t] = a;
      w[1][t] = b;
      w[2][t] = c;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<us8*>(base + (k * rows + row) * GLP + 8 * g) = w[k];
  }
};

// Partial gradient of every parameter over the samples of chunk blockIdx.x:
// part[chunk][p].  The two 128 x 128 weight blocks are D^T H over the chunk
// on the BF16 matrix cores: both FP32 operands split in three BF16 terms,
// the six products t_i u_j with i + j <= 2 (the dropped ones are below
// 2^-24 of the product), FP32 accumulation.  blockIdx.y = 2 m + h takes the
// output rows 64 h .. 64 h + 63 of block m (W2: D2^T H1, W3: D3^T H2), wave w
// 16 of them, and the biases of those rows; y = 0 also W1 and b1, y = 3 W4 and
// b4, as FP32 sums over the chunk.  Four workgroups per chunk instead of one
// keep every CU busy from 4096 rows on.  Operands are split once, by the
// thread that loads them, and stored with the samples running along the rows,
// so that a fragment is one 16-byte read; the small sums are taken from the
// loaded registers (4099 rows: 36 us, now 13.6).
__global__ void __launch_bounds__(256)
k_mlp_grad_part(const float* __restrict__ S, const float* __restrict__ H1,
                const float* __restrict__ H2, const float* __restrict__ H3,
                const float* __restrict__ dO, const float* __restrict__ D1,
                const float* __restrict__ D2, const float* __restrict__ D3, int B,
                float* __restrict__ part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  __shared__ alignas(16) unsigned short dsp[3 * 64 * GLP], hsp[3 * PH * GLP];
  __shared__ float xs[GCH][PIN], dos[GCH];
  __shared__ float red[5][256];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int y = blockIdx.y, m = y >> 1, j0 = (y & 1) * 64;
  const float* __restrict__ D = m ? D3 : D2;
  const float* __restrict__ H = m ? H2 : H1;
  const float* __restrict__ E = y == 0 ? D1 : H3;
  const bool extra = y == 0 || y == 3;
  const int c0 = blockIdx.x * GCH, c1 = min(B, c0 + GCH);
  float* out = part + size_t(blockIdx.x) * NPAR;
  const int r = lane & 15, kg = (lane >> 4) * 8;
  if (tid < GCH * PIN) xs[tid / PIN][tid % PIN] = c0 + tid / PIN < c1 ? S[size_t(c0 + tid / PIN) * 6 + tid % PIN] : 0.0f;
  if (tid < GCH) dos[tid] = c0 + tid < c1 ? dO[c0 + tid] : 0.0f;
  f4v acc[PH / 16];
#pragma unroll
  for (int ib = 0; ib < PH / 16; ++ib) acc[ib] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int PI[6] = {0, 0, 1, 0, 1, 2};
  constexpr int PJ[6] = {0, 1, 0, 2, 1, 0};
  // thread -> neuron and sample groups: D nd, gd; H and E nh, gh and gh + 2
  const int nd = tid & 63, gd = tid >> 6, nh = tid & 127, gh = tid >> 7;
  float bsum = 0.0f, es[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};   // es: W1 rows and b1, or W4
  for (int s0 = c0; s0 < c1; s0 += GSUB) {
    Eight d, h[2], e[2];
    d.load(D, s0 + 8 * gd, c1, j0 + nd);
#pragma unroll
    for (int q = 0; q < 2; ++q) h[q].load(H, s0 + 8 * (gh + 2 * q), c1, nh);
    if (extra)
#pragma unroll
      for (int q = 0; q < 2; ++q) e[q].load(E, s0 + 8 * (gh + 2 * q), c1, nh);
    __syncthreads();   // the previous step's fragments are read (and xs, dos are there)
    d.put(dsp, 64, nd, gd);
#pragma unroll
    for (int q = 0; q < 2; ++q) h[q].put(hsp, PH, nh, gh + 2 * q);
#pragma unroll
    for (int t = 0; t < 8; ++t) bsum += d.v[t];
    if (extra)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int sr = s0 - c0 + 8 * (gh + 2 * q) + t;
          if (y == 0) {
#pragma unroll
            for (int i = 0; i < PIN; ++i) es[i] += e[q].v[t] * xs[sr][i];
            es[PIN] += e[q].v[t];
          } else {
            es[0] += e[q].v[t] * dos[sr];
          }
        }
    __syncthreads();
    us8 a[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      a[k] = *reinterpret_cast<const us8*>(dsp + (k * 64 + wv * 16 + r) * GLP + kg);
#pragma unroll
    for (int ib = 0; ib < PH / 16; ++ib) {
      us8 u[3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        u[k] = *reinterpret_cast<const us8*>(hsp + (k * PH + ib * 16 + r) * GLP + kg);
#pragma unroll
      for (int q = 0; q < 6; ++q)
        acc[ib] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a[PI[q]]),
                                                          __builtin_bit_cast(bf8, u[PJ[q]]), acc[ib], 0, 0, 0);
    }
  }
  // output rows j (neuron of the layer's output) and columns i (its input)
#pragma unroll
  for (int ib = 0; ib < PH / 16; ++ib)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      out[(m ? OW3 : OW2) + (j0 + wv * 16 + 4 * (lane >> 4) + e) * PH + ib * 16 + r] = acc[ib][e];
  // small sums: the sample groups of a neuron in order
  red[0][tid] = bsum;
  __syncthreads();
  if (tid < 64) out[(m ? OB3 : OB2) + j0 + tid] = red[0][tid] + red[0][tid + 64] + red[0][tid + 128] + red[0][tid + 192];
  if (!extra) return;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 5; ++i) red[i][tid] = es[i];
  __syncthreads();
  if (y == 0) {
    for (int p = tid; p < PH * PIN + PH; p += 256) {
      const int j = p < PH * PIN ? p / PIN : p - PH * PIN, i = p < PH * PIN ? p % PIN : PIN;
      out[(i < PIN ? OW1 + p : OB1 + j)] = red[i][j] + red[i][j + PH];
    }
  } else {
    if (tid < PH) out[OW4 + tid] = red[0][tid] + red[0][tid + PH];
    if (tid == PH) {
      float v = 0.0f;
      for (int s = 0; s < GCH; ++s) v += dos[s];
      out[OB4] = v;
    }
  }
}

// G[p] = sum over the chunks of part[chunk][p], in chunk order.  The workgroup
// past the parameters sums the loss terms (one wave's worth of partial sums in
// a fixed order) for the host.
__global__ void __launch_bounds__(256)
k_mlp_grad_sum(const float* __restrict__ part, int nchunk, float* __restrict__ G,
               const double* __restrict__ lpart, int nl, double* __restrict__ host,
               const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ double red[4];
    double l = 0.0;
    for (int i = threadIdx.x; i < nl; i += 256) l += lpart[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) *host = red[0] + red[1] + red[2] + red[3];
    return;
  }
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= NPAR) return;
  float v = 0.0f;
#pragma unroll 8
  for (int c = 0; c < nchunk; ++c) v += part[size_t(c) * NPAR + p];
  G[p] = v;
}

__global__ void k_adam(float* __restrict__ P, const float* __restrict__ G, float* __restrict__ M,
                       float* __restrict__ V, int n, float lr, float b1, float b2, float c1,
                       float c2, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float g = G[i];
  const float m = b1 * M[i] + (1.0f - b1) * g;
  const float v = b2 * V[i] + (1.0f - b2) * g * g;
  M[i] = m;
  V[i] = v;
  P[i] -= lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
}

// Features of (state alpha, shell s) rows: X[(a*S + s)][0..3] (row length 6).
__global__ void k_pc_features(const double* __restrict__ pow, const double* __restrict__ eps,
                              int stride, int ns, double e0, double hb2m, double kmax,
                              float* __restrict__ X, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= ns * PC_SHELLS) return;
  const int a = r / PC_SHELLS, s = r % PC_SHELLS;
  const int al = a * stride;
  double ptot = 0.0;
  for (int t = 0; t < PC_SHELLS; ++t) ptot += pow[size_t(al) * PC_SHELLS + t];
  const double frac = ptot > 0.0 ? pow[size_t(al) * PC_SHELLS + s] / ptot : 0.0;
  const double kc = (s + 0.5) / PC_SHELLS;
  float* x = X + size_t(r) * 6;
  x[0] = float(kc);
  x[1] = float(eps[al] / e0);
  x[2] = float(log10(frac + 1e-12) / 6.0 + 1.0);
  x[3] = float(hb2m * (kc * kmax) * (kc * kmax) / e0);
  x[5] = float(frac);   // sample weight: share of the residual in the shell
}

// gain[r] = GMAX sigmoid(O[r])
__global__ void k_pc_gains(const float* __restrict__ O, int n, float* __restrict__ gain, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n) gain[r] = GMAX / (1.0f + expf(-O[r]));
}

// Batch b = a*S + s of the sampled states: copies of psi, h psi, <h> and a
// one-hot gain row selecting shell s.
template <typename T>
__global__ void k_pc_gather(const T* __restrict__ psi, const T* __restrict__ hpsi,
                            const double* __restrict__ eps, const int* __restrict__ idx,
                            long V, T* __restrict__ bpsi, T* __restrict__ bh,
                            double* __restrict__ beps, float* __restrict__ onehot, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int b = blockIdx.y, a = b / PC_SHELLS, s = b % PC_SHELLS;
  const size_t src = size_t(idx[a]) * V, dst = size_t(b) * V;
  for (long e = long(blockIdx.x) * blockDim.x + threadIdx.x; e < V; e += long(gridDim.x) * blockDim.x) {
    bpsi[dst + e] = psi[src + e];
    bh[dst + e] = hpsi[src + e];
  }
  if (blockIdx.x == 0 && threadIdx.x < PC_SHELLS) {
    onehot[size_t(b) * PC_SHELLS + threadIdx.x] = threadIdx.x == s ? 1.0f : 0.0f;
    if (threadIdx.x == 0) beps[b] = eps[idx[a]];
  }
}

// d = psi - phi (in place in phi)
template <typename T>
__global__ void k_pc_dir(const T* __restrict__ bpsi, T* __restrict__ bphi, size_t n, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < n) {
    const T a = bpsi[e];
    T b = bphi[e];
    b.x = a.x - b.x;
    b.y = a.y - b.y;
    bphi[e] = b;
  }
}

// Gram partials per sampled state: w_s = h d_s - eps d_s, r = h psi - eps psi;
// part[a][blk][q] for q < S(S+1)/2 (s <= t) then S entries <w_s, r>.
constexpr int NG = PC_SHELLS * (PC_SHELLS + 1) / 2 + PC_SHELLS;
template <typename T>
__global__ void __launch_bounds__(256)
k_pc_gram(const T* __restrict__ bpsi, const T* __restrict__ bh, const T* __restrict__ bd,
          const T* __restrict__ bhd, const double* __restrict__ beps, long V,
          double* __restrict__ part, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int a = blockIdx.y;
  double acc[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) acc[q] = 0.0;
  const size_t b0 = size_t(a) * PC_SHELLS;
  const double e = beps[b0];
  for (long x = long(blockIdx.x) * blockDim.x + threadIdx.x; x < V; x += long(gridDim.x) * blockDim.x) {
    double wr[PC_SHELLS], wi[PC_SHELLS];
#pragma unroll
    for (int s = 0; s < PC_SHELLS; ++s) {
      const T d = bd[(b0 + s) * V + x], hd = bhd[(b0 + s) * V + x];
      wr[s] = double(hd.x) - e * double(d.x);
      wi[s] = double(hd.y) - e * double(d.y);
    }
    const T p = bpsi[b0 * V + x], h = bh[b0 * V + x];
    const double rr = double(h.x) - e * double(p.x), ri = double(h.y) - e * double(p.y);
    int q = 0;
#pragma unroll
    for (int s = 0; s < PC_SHELLS; ++s)
#pragma unroll
      for (int t = s; t < PC_SHELLS; ++t) acc[q++] += wr[s] * wr[t] + wi[s] * wi[t];
#pragma unroll
    for (int s = 0; s < PC_SHELLS; ++s) acc[q++] += wr[s] * rr + wi[s] * ri;
  }
  __shared__ double red[4][NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    double v = acc[q];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = v;
  }
  __syncthreads();
  if (threadIdx.x < NG)
    part[(size_t(a) * gridDim.x + blockIdx.x) * NG + threadIdx.x] =
        red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// Per sampled state: sum the Gram partials, solve (G + lam 1) g = c by
// Cholesky (FP64), clamp to [0, GMAX], write the target column t of the
// sample rows.  One thread per state.
__global__ void k_pc_solve(const double* __restrict__ part, int nblk, int ns, float* __restrict__ S, const int* __restrict__ sky_gate) {
  if (sky_gate != nullptr && *sky_gate == 0) return;
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= ns) return;
  double Gm[PC_SHELLS][PC_SHELLS], c[PC_SHELLS];
  double sum[NG];
  for (int q = 0; q < NG; ++q) sum[q] = 0.0;
  for (int k = 0; k < nblk; ++k)
    for (int q = 0; q < NG; ++q) sum[q] += part[(size_t(a) * nblk + k) * NG + q];
  int q = 0;
  for (int s = 0; s < PC_SHELLS; ++s)
    for (int t = s; t < PC_SHELLS; ++t) { Gm[s][t] = sum[q]; Gm[t][s] = sum[q]; ++q; }
  for (int s = 0; s < PC_SHELLS; ++s) c[s] = sum[q++];
  double tr = 0.0;
  for (int s = 0; s < PC_SHELLS; ++s) tr += Gm[s][s];
  const double lam = 1e-6 * tr / PC_SHELLS + 1e-300;
  for (int s = 0; s < PC_SHELLS; ++s) Gm[s][s] += lam;
  // Cholesky in place (lower)
  for (int k = 0; k < PC_SHELLS; ++k) {
    double d = Gm[k][k];
    for (int l = 0; l < k; ++l) d -= Gm[k][l] * Gm[k][l];
    d = sqrt(fmax(d, 1e-300));
    Gm[k][k] = d;
    for (int i = k + 1; i < PC_SHELLS; ++i) {
      double v = Gm[i][k];
      for (int l = 0; l < k; ++l) v -= Gm[i][l] * Gm[k][l];
      Gm[i][k] = v / d;
    }
  }
  double y[PC_SHELLS], g[PC_SHELLS];
  for (int i = 0; i < PC_SHELLS; ++i) {
    double v = c[i];
    for (int l = 0; l < i; ++l) v -= Gm[i][l] * y[l];
    y[i] = v / Gm[i][i];
  }
  for (int i = PC_SHELLS - 1; i >= 0; --i) {
    double v = y[i];
    for (int l = i + 1; l < PC_SHELLS; ++l) v -= Gm[l][i] * g[l];
    g[i] = v / Gm[i][i];
  }
  for (int s = 0; s < PC_SHELLS; ++s)
    S[(size_t(a) * PC_SHELLS + s) * 6 + 4] = float(fmin(fmax(g[s], 0.0), double(GMAX)));
}
}  // namespace

int precond_nparams() { return NPAR; }
int precond_ns_max() { return NS_MAX; }

void precond_init_params(float* P_dev, unsigned seed, hipStream_t st) {
  std::vector<float> h(NPAR, 0.0f);
  std::mt19937 rng(seed);
  auto fill = [&](int off, int fan_in, int fan_out) {
    const float a = std::sqrt(6.0f / float(fan_in + fan_out));
    std::uniform_real_distribution<float> u(-a, a);
    for (int i = 0; i < fan_in * fan_out; ++i) h[off + i] = u(rng);
  };
  fill(OW1, PIN, PH);
  fill(OW2, PH, PH);
  fill(OW3, PH, PH);
  fill(OW4, PH, 1);
  for (int j = 0; j < PH; ++j) { h[OB1 + j] = 0.01f; h[OB2 + j] = 0.01f; h[OB3 + j] = 0.01f; }
  for (int j = 0; j < PH; ++j) h[OW4 + j] *= 0.1f;
  h[OB4] = std::log(1.0f / (GMAX - 1.0f));   // gain 1 at the start: the plain damping
  hipMemcpyAsync(P_dev, h.data(), sizeof(float) * NPAR, hipMemcpyHostToDevice, st);
  hipStreamSynchronize(st);
}

void precond_round(const float* P, float* Pb, hipStream_t st) {
  hipLaunchKernelGGL(k_round_params, dim3((NPAR + 255) / 256), dim3(256), 0, st, P, Pb, NPAR, g_launch_gate);
}

void precond_forward(const float* Pb, const float* X, int B, float* H1, float* H2, float* H3,
                     float* O, hipStream_t st) {
  if (B <= 0) return;
  hipLaunchKernelGGL(k_mlp_fwd, dim3((B + FR - 1) / FR), dim3(64 * FWV), 0, st, Pb, X, 6, B, H1, H2,
                     H3, O, g_launch_gate);
}

void precond_features(const double* pow, const double* eps, int stride, int ns, double e0,
                      double hb2m, double kmax, float* X, hipStream_t st) {
  const int n = ns * PC_SHELLS;
  if (n <= 0) return;
  hipLaunchKernelGGL(k_pc_features, dim3((n + 127) / 128), dim3(128), 0, st, pow, eps, stride, ns,
                     e0, hb2m, kmax, X, g_launch_gate);
}

void precond_gains(const float* O, int n, float* gain, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_pc_gains, dim3((n + 255) / 256), dim3(256), 0, st, O, n, gain, g_launch_gate);
}

size_t precond_rounded_floats() { return OPACK + 2 * size_t(WSZ); }
size_t precond_loss_doubles(int rows) { return size_t(rows + FR - 1) / FR + 1; }

void precond_wsum(const float* S, int B, double* wsum, hipStream_t st) {
  hipLaunchKernelGGL(k_pc_wsum, dim3(1), dim3(1024), 0, st, S, B, wsum, g_launch_gate);
}

void precond_loss_grad(const float* Pb, const float* S, int B, const double* wsum, float* H1,
                       float* H2, float* H3, float* O, float* dO, float* D1, float* D2, float* D3,
                       float* G, float* gpart, double* lpart, double* host, hipStream_t st) {
  if (B <= 0) return;
  precond_forward(Pb, S, B, H1, H2, H3, O, st);
  const int nl = (B + FR - 1) / FR;
  hipLaunchKernelGGL(k_mlp_bwd_act, dim3(nl), dim3(64 * FWV), 0, st, Pb, S, (const float*)H1,
                     (const float*)H2, (const float*)H3, (const float*)O, wsum, B, dO, D1, D2, D3,
                     lpart, g_launch_gate);
  const int nchunk = (B + GCH - 1) / GCH;
  hipLaunchKernelGGL(k_mlp_grad_part, dim3(nchunk, 4), dim3(256), 0, st, S, (const float*)H1,
                     (const float*)H2, (const float*)H3, (const float*)dO, (const float*)D1,
                     (const float*)D2, (const float*)D3, B, gpart, g_launch_gate);
  hipLaunchKernelGGL(k_mlp_grad_sum, dim3((NPAR + 255) / 256 + 1), dim3(256), 0, st,
                     (const float*)gpart, nchunk, G, (const double*)lpart, nl, host, g_launch_gate);
}

void precond_adam(float* P, const float* G, float* M, float* V, int step, float lr,
                  hipStream_t st) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - std::pow(b1, float(step)), c2 = 1.0f - std::pow(b2, float(step));
  hipLaunchKernelGGL(k_adam, dim3((NPAR + 255) / 256), dim3(256), 0, st, P, G, M, V, NPAR, lr, b1,
                     b2, c1, c2, g_launch_gate);
}

void precond_gather(int prec, const void* psi, const void* hpsi, const double* eps,
                    const int* idx, int ns, long V, void* bpsi, void* bh, double* beps,
                    float* onehot, hipStream_t st) {
  dim3 grid(64, unsigned(ns * PC_SHELLS));
  if (prec == 0)
    hipLaunchKernelGGL(k_pc_gather<double2>, grid, dim3(256), 0, st, (const double2*)psi,
                       (const double2*)hpsi, eps, idx, V, (double2*)bpsi, (double2*)bh, beps, onehot, g_launch_gate);
  else
    hipLaunchKernelGGL(k_pc_gather<float2>, grid, dim3(256), 0, st, (const float2*)psi,
                       (const float2*)hpsi, eps, idx, V, (float2*)bpsi, (float2*)bh, beps, onehot, g_launch_gate);
}

void precond_dir(int prec, const void* bpsi, void* bphi, size_t n, hipStream_t st) {
  const unsigned nb = unsigned((n + 255) / 256);
  if (prec == 0)
    hipLaunchKernelGGL(k_pc_dir<double2>, dim3(nb), dim3(256), 0, st, (const double2*)bpsi,
                       (double2*)bphi, n, g_launch_gate);
  else
    hipLaunchKernelGGL(k_pc_dir<float2>, dim3(nb), dim3(256), 0, st, (const float2*)bpsi,
                       (float2*)bphi, n, g_launch_gate);
}

int precond_gram_blocks() { return 128; }

void precond_targets(int prec, const void* bpsi, const void* bh, const void* bd, const void* bhd,
                     const double* beps, int ns, long V, double* part, float* S, hipStream_t st) {
  const int nblk = precond_gram_blocks();
  dim3 grid(nblk, ns);
  if (prec == 0)
    hipLaunchKernelGGL(k_pc_gram<double2>, grid, dim3(256), 0, st, (const double2*)bpsi,
                       (const double2*)bh, (const double2*)bd, (const double2*)bhd, beps, V, part, g_launch_gate);
  else
    hipLaunchKernelGGL(k_pc_gram<float2>, grid, dim3(256), 0, st, (const float2*)bpsi,
                       (const float2*)bh, (const float2*)bd, (const float2*)bhd, beps, V, part, g_launch_gate);
  hipLaunchKernelGGL(k_pc_solve, dim3((ns + 63) / 64), dim3(64), 0, st, (const double*)part, nblk,
                     ns, S, g_launch_gate);
}

size_t precond_gpart_bytes(int rows) {
  return sizeof(float) * size_t(NPAR) * size_t((rows + GCH - 1) / GCH);
}

size_t precond_gram_bytes(int ns) { return sizeof(double) * size_t(ns) * precond_gram_blocks() * NG; }

}  // namespace sky
