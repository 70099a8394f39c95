// Universal differential equation on matrix cores: Lotka-Volterra plus a
// 2-32-32-2 tanh MLP whose weights are shared by every trajectory, FP32 with
// FP32 accumulation.  Record and reverse sweep are the ones of the explicit
// pairs (paper, Sections 2.1, 3.1 and 3.4) with Tsit5; what changes is the
// right-hand side, which is evaluated for a whole wavefront at once.
//
// MLP on MFMA (v_mfma_f32_32x32x2f32).  A wavefront holds 32 trajectories:
// lane l (half hf = l / 32, column c = l % 32) works on trajectory c, and
// both halves hold its state and take its steps alike.  Every layer is
// computed in the transposed form out[unit][trajectory] =
// W[unit][k] x[k][trajectory], so the trajectories sit on the MFMA's N
// dimension and the weights are the A operand.  In the accumulator layout a
// lane holds, for its trajectory, the 16 units
//   U(r, hf) = 8 (r / 4) + 4 hf + (r % 4),   r = 0..15.
// The next layer takes its B operand for K-step k straight from register k
// (the K index enumerates units in the order U(k, kk), kk = 0, 1), so hidden
// activations never leave registers.  Only the 2-vector output of the MLP
// crosses between the lane halves (v_permlane32_swap).
//
// What bounds these kernels is instruction time.  The FP32 matrix
// instructions do not overlap with vector instructions, neither of the same
// wavefront nor of another on the SIMD (8 MFMA take 0.22 us, 96 FMA 0.18 us,
// the two interleaved 0.42 us): a kernel lasts as long as both together.
// Why 32 trajectories a wavefront and not 64 (one per lane, two column
// blocks): with 64, 2^16 trajectories are one wavefront per SIMD, whose waits
// for LDS and memory nothing fills, and a smaller ensemble leaves SIMDs idle
// while each wavefront does twice the work.  The work on a trajectory's own
// scalars is done twice now, about a twentieth of the whole.
//
// All lanes of a wavefront must run every right-hand side together.  The
// kernels below therefore keep finished lanes in the loop (doing zero-length
// steps) until the whole wavefront is done.
//
// Weight gradient.  Per stage the contribution sum over trajectories of
// delta2 h1^T (32 x 32) is one more MFMA chain with the trajectories as the
// K dimension; delta2 and h1 are transposed through a per-wave LDS tile for
// it.  Every other weight gradient is accumulated per lane and reduced over
// the lanes at the end, in a fixed order.
#pragma once
#include <math.h>

#include "erk.h"

namespace ens {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int UDE_NP = 1218;
constexpr int UDE_OW1 = 0, UDE_OB1 = 64, UDE_OW2 = 96, UDE_OB2 = 1120, UDE_OW3 = 1152,
              UDE_OB3 = 1216;
constexpr float LV_A = 1.5f, LV_B = 1.0f, LV_G = 3.0f, LV_D = 1.0f;
constexpr int UDE_TRAJ = 32;                   // trajectories per wavefront
constexpr int UDE_WAVES = 4;                   // wavefronts per block
constexpr int UDE_BLOCK_TRAJ = UDE_TRAJ * UDE_WAVES;
// LDS row of a transposed tile: 36 floats keep the rows 16-byte aligned, and
// a lane's 16-byte write shifted by 4 banks from its neighbour's
constexpr int UDE_STRIDE = 36;
constexpr int UDE_TILE = UDE_TRAJ * UDE_STRIDE;  // one [32 trajectories][32 units] tile

// Per-lane gradient accumulators.
struct UdeGrad {
  v16f w2;          // dW2[U(r, hf)][c] (the MFMA accumulator)
  float w3[2][16];  // dW3[o][U(r, hf)]
  float b2[16];     // db2[U(r, hf)]
  float w1[2][16];  // dW1[U(r, hf)][k]
  float b1[16];     // db1[U(r, hf)]
  float b3[2];      // db3[o] (both halves hold the same sum)
};

__device__ __forceinline__ int ude_unit(int r, int hf) {
  return 8 * (r >> 2) + 4 * hf + (r & 3);
}

// The weights of the forward kernels, in registers: each lane's MFMA operands
// and the entries of its half's units (about 80 of the 256 registers that two
// wavefronts per SIMD leave).
struct UdeRegW {
  float va1;         // W1[c][hf]
  float va2f[16];    // W2[c][U(k, hf)]
  float vb1[16];     // b1[U(r, hf)]
  float vb2[16];     // b2[U(r, hf)]
  float vw3[2][16];  // W3[o][U(r, hf)]
  float vb3[2];
  __device__ __forceinline__ void load(const float* th) {
    const int l = __lane_id(), hf = l >> 5, c = l & 31;
    va1 = th[UDE_OW1 + 2 * c + hf];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int u = ude_unit(k, hf);
      va2f[k] = th[UDE_OW2 + 32 * c + u];
      vb1[k] = th[UDE_OB1 + u];
      vb2[k] = th[UDE_OB2 + u];
      vw3[0][k] = th[UDE_OW3 + u];
      vw3[1][k] = th[UDE_OW3 + 32 + u];
    }
    vb3[0] = th[UDE_OB3];
    vb3[1] = th[UDE_OB3 + 1];
  }
  __device__ __forceinline__ void reload() const {}
  __device__ __forceinline__ float a1() const { return va1; }
  __device__ __forceinline__ float a2f(int k) const { return va2f[k]; }
  __device__ __forceinline__ float b1(int r) const { return vb1[r]; }
  __device__ __forceinline__ float b2(int r) const { return vb2[r]; }
  __device__ __forceinline__ float w3(int o, int r) const { return vw3[o][r]; }
  __device__ __forceinline__ float b3(int o) const { return vb3[o]; }
};

// The weights of the reverse sweep, in LDS (its registers hold the gradient):
// the MFMA operands [slot][lane], which a wavefront reads as 64 consecutive
// floats; the per-unit entries [half][slot], which each half reads four at a
// time at one address.  9 KB, and 9 KB of tiles per wavefront.
struct UdeLds {
  float s_a1[64];        // W1[c][hf]
  float s_a2f[16][64];   // W2[c][U(k, hf)]    (forward layer 2)
  float s_a2b[16][64];   // W2[U(k, hf)][c]    (transposed, for delta h1)
  float s_b1[2][16];     // b1[U(r, hf)]
  float s_b2[2][16];     // b2[U(r, hf)]
  float s_w3[2][2][16];  // [hf][o][r]: W3[o][U(r, hf)]
  float s_w1[2][2][16];  // [hf][k][r]: W1[U(r, hf)][k]
  float s_b3[2];
  float coef[6][6];      // Tsit5, [j][0]: b_j; [j][l], l > j: a_lj
  // a wavefront's two tiles (delta2, h1); at the end its partial, along the row
  alignas(16) float tile[UDE_WAVES][2 * UDE_TILE];

  // a compiler memory barrier before each use of the layers: without it the
  // loads leave the sweep's loop, and the registers they would stay in spill
  // (560 B a lane)
  __device__ __forceinline__ void reload() const { __asm__ __volatile__("" ::: "memory"); }
  __device__ __forceinline__ float a1() const { return s_a1[__lane_id()]; }
  __device__ __forceinline__ float a2f(int k) const { return s_a2f[k][__lane_id()]; }
  __device__ __forceinline__ float a2b(int k) const { return s_a2b[k][__lane_id()]; }
  __device__ __forceinline__ float b1(int r) const { return s_b1[__lane_id() >> 5][r]; }
  __device__ __forceinline__ float b2(int r) const { return s_b2[__lane_id() >> 5][r]; }
  __device__ __forceinline__ float w3(int o, int r) const { return s_w3[__lane_id() >> 5][o][r]; }
  __device__ __forceinline__ float w1(int k, int r) const { return s_w1[__lane_id() >> 5][k][r]; }
  __device__ __forceinline__ float b3(int o) const { return s_b3[o]; }
};
static_assert(2 * UDE_TILE >= UDE_NP, "a wavefront's tiles hold its partial at the end");

// Fill the LDS image from the parameter vector (W1, b1, W2, b2, W3, b3).
__device__ __forceinline__ void ude_load_weights(UdeLds& s, const float* th) {
  for (int i = threadIdx.x; i < 64; i += blockDim.x) {
    const int hf = i >> 5, c = i & 31;
    s.s_a1[i] = th[UDE_OW1 + 2 * c + hf];
  }
  for (int i = threadIdx.x; i < 16 * 64; i += blockDim.x) {
    const int k = i >> 6, l = i & 63, hf = l >> 5, c = l & 31;
    const int u = ude_unit(k, hf);
    s.s_a2f[k][l] = th[UDE_OW2 + 32 * c + u];
    s.s_a2b[k][l] = th[UDE_OW2 + 32 * u + c];
  }
  for (int i = threadIdx.x; i < 32; i += blockDim.x) {
    const int hf = i >> 4, r = i & 15, u = ude_unit(r, hf);
    s.s_b1[hf][r] = th[UDE_OB1 + u];
    s.s_b2[hf][r] = th[UDE_OB2 + u];
    s.s_w3[hf][0][r] = th[UDE_OW3 + u];
    s.s_w3[hf][1][r] = th[UDE_OW3 + 32 + u];
    s.s_w1[hf][0][r] = th[UDE_OW1 + 2 * u];
    s.s_w1[hf][1][r] = th[UDE_OW1 + 2 * u + 1];
  }
  if (threadIdx.x < 2) s.s_b3[threadIdx.x] = th[UDE_OB3 + threadIdx.x];
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < Tsit5::SU; ++j)
#pragma unroll
      for (int l = 0; l < Tsit5::SU; ++l)
        s.coef[j][l] = l == 0 ? (float)Tsit5::B[j] : l > j ? (float)Tsit5::A[l][j] : 0.f;
  }
}

// The sum of the two halves' values, low half first, in every lane.
__device__ __forceinline__ float ude_join(float v) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// tanh in FP32 (relative error below 5e-7): for |x| < 0.55 the odd series
// x + x^3 P(x^2), P of degree 4 fitted by least squares to (tanh(x)/x - 1)/x^2
// on [0, 0.55]; above, 1 - 2 / (e^{2|x|} + 1) with the hardware exp2 and
// reciprocal (the series avoids that form's cancellation near 0).  SERIES: |x|
// is known to be below.
template <bool SERIES = false>
__device__ __forceinline__ float ude_tanh(float x) {
  const float ax = fabsf(x);
  float big = x;
  if constexpr (!SERIES) {
    const float e = __builtin_amdgcn_exp2f(ax * 2.8853900817779268f);  // 2^(2|x| / ln 2)
    big = fmaT(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
  }
  const float x2 = x * x;
  float q = -0.026664944365620613f;
  q = fmaT(q, x2, 0.03440927714109421f);
  q = fmaT(q, x2, -0.05673672631382942f);
  q = fmaT(q, x2, 0.13355417549610138f);
  q = fmaT(q, x2, -0.3333379626274109f);
  const float small = fmaT(x * x2, q, x);
  return SERIES || ax < 0.55f ? small : copysignf(big, x);
}

// tanh of a layer.  Where every |x| of the wavefront is below 0.55 (layers of
// small weights; a NaN counts as below, and gives NaN either way) the other
// branch's exp2 and reciprocal, more than half of the cost, are left out: the
// same values.
__device__ __forceinline__ void ude_tanh_layer(v16f& v) {
  float m = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) m = fmaxf(m, fabsf(v[r]));
  if (!__any(m >= 0.55f)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = ude_tanh<true>(v[r]);
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = ude_tanh(v[r]);
  }
}

__device__ __forceinline__ v16f mfma32(float a, float b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Hidden layers in the accumulator layout: h1 = tanh(W1 y + b1) ...
template <class Wt>
__device__ __forceinline__ void ude_layer1(const Wt& W, const float* y, v16f& h1) {
  const float x = (__lane_id() >> 5) ? y[1] : y[0];  // feature hf of trajectory c
  W.reload();
#pragma unroll
  for (int r = 0; r < 16; ++r) h1[r] = W.b1(r);
  h1 = mfma32(W.a1(), x, h1);
  ude_tanh_layer(h1);
}

// ... and h2 = tanh(W2 h1 + b2).
template <class Wt>
__device__ __forceinline__ void ude_layer2(const Wt& W, const v16f& h1, v16f& h2) {
  W.reload();
#pragma unroll
  for (int r = 0; r < 16; ++r) h2[r] = W.b2(r);
#pragma unroll
  for (int k = 0; k < 16; ++k) h2 = mfma32(W.a2f(k), h1[k], h2);
  ude_tanh_layer(h2);
}

// f(y) = f_LV(y) + W3 h2 + b3 for this lane's trajectory, and h2.
// Wave-uniform: every lane of the wavefront must call it.
template <class Wt>
__device__ __forceinline__ void ude_rhs(const Wt& W, const float* y, float* f, v16f& h2) {
  v16f h1;
  ude_layer1(W, y, h1);
  ude_layer2(W, h1, h2);
  W.reload();
  float p0 = 0.f, p1 = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    p0 = fmaT(W.w3(0, r), h2[r], p0);
    p1 = fmaT(W.w3(1, r), h2[r], p1);
  }
  const float n0 = ude_join(p0), n1 = ude_join(p1);
  const float xy = y[0] * y[1];
  f[0] = (n0 + W.b3(0)) + (LV_A * y[0] - LV_B * xy);
  f[1] = (n1 + W.b3(1)) + (LV_D * xy - LV_G * y[1]);
}

// The system on weights in registers or LDS (UdeRegW, UdeLds); p points to them.
template <class Wt>
struct LvUdeOn {
  static constexpr int D = 2, NP = 0, ID = 5;
  __device__ static inline void rhs(const float* y, const float* p, float* f) {
    v16f h2;
    ude_rhs(*reinterpret_cast<const Wt*>(p), y, f, h2);
  }
};

// The system as the reverse sweep evaluates it: each right-hand side of a step
// keeps its h2 for the stage's VJP, which then forms h1 alone (one matrix
// instruction instead of 17 and half the tanh).  The 6 x 16 values a lane are
// private memory (scratch, written and read whole lines at a time): registers
// and LDS are full at two wavefronts per SIMD.  p points to a UdeKeep.
struct UdeKeep {
  const UdeLds* W;
  float4 (*h2)[4];  // [stage][4 x 4 units]
  int stage;        // of the next right-hand side
};

struct LvUdeSweep {
  static constexpr int D = 2, NP = 0, ID = 5;
  __device__ static inline void rhs(const float* y, const float* p, float* f) {
    UdeKeep& K = *reinterpret_cast<UdeKeep*>(const_cast<float*>(p));
    v16f h2;
    ude_rhs(*K.W, y, f, h2);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      K.h2[K.stage][q] = make_float4(h2[4 * q], h2[4 * q + 1], h2[4 * q + 2], h2[4 * q + 3]);
    ++K.stage;
  }

  // gy = (df/dy)^T w; the weight gradient of w^T f is added to the lane's
  // accumulators g.  kept: the stage's h2.  Wave-uniform.
  __device__ static inline void vjp(const float* y, const UdeLds& W, const float4* kept,
                                    const float* w, float* gy, UdeGrad& g) {
    const int l = __lane_id(), hf = l >> 5, c = l & 31;
    const int wave = threadIdx.x >> 6;
    v16f h1, h2;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = kept[q];
      h2[4 * q] = v.x;
      h2[4 * q + 1] = v.y;
      h2[4 * q + 2] = v.z;
      h2[4 * q + 3] = v.w;
    }
    ude_layer1(W, y, h1);
    W.reload();

    // output layer: dW3 += w h2^T, db3 += w, delta2 = (W3^T w) (1 - h2^2)
    v16f d2;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      g.w3[0][r] = fmaT(w[0], h2[r], g.w3[0][r]);
      g.w3[1][r] = fmaT(w[1], h2[r], g.w3[1][r]);
      d2[r] = fmaT(W.w3(1, r), w[1], W.w3(0, r) * w[0]) * fmaT(-h2[r], h2[r], 1.f);
      g.b2[r] = g.b2[r] + d2[r];
    }
    g.b3[0] = g.b3[0] + w[0];
    g.b3[1] = g.b3[1] + w[1];

    // stage delta2 and h1 as [trajectory][unit] tiles for the weight gradient
    // (registers 4 q .. 4 q + 3 hold four consecutive units)
    float* td = const_cast<float*>(W.tile[wave]);
    float* th = const_cast<float*>(W.tile[wave]) + UDE_TILE;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int at = c * UDE_STRIDE + 8 * q + 4 * hf;
      *reinterpret_cast<float4*>(td + at) =
          make_float4(d2[4 * q], d2[4 * q + 1], d2[4 * q + 2], d2[4 * q + 3]);
      *reinterpret_cast<float4*>(th + at) =
          make_float4(h1[4 * q], h1[4 * q + 1], h1[4 * q + 2], h1[4 * q + 3]);
    }

    // delta h1 = W2^T delta2 on the matrix cores, delta1 = delta h1 (1 - h1^2)
    W.reload();
    v16f e1 = {0};
#pragma unroll
    for (int k = 0; k < 16; ++k) e1 = mfma32(W.a2b(k), d2[k], e1);
    W.reload();
    float p0 = 0.f, p1 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float d1 = e1[r] * fmaT(-h1[r], h1[r], 1.f);
      g.b1[r] = g.b1[r] + d1;
      g.w1[0][r] = fmaT(d1, y[0], g.w1[0][r]);
      g.w1[1][r] = fmaT(d1, y[1], g.w1[1][r]);
      p0 = fmaT(W.w1(0, r), d1, p0);
      p1 = fmaT(W.w1(1, r), d1, p1);
    }
    const float n0 = ude_join(p0), n1 = ude_join(p1);
    // Lotka-Volterra: J = [[a - b y1, -b y0], [d y1, d y0 - g]]
    gy[0] = n0 + fmaT(LV_D * y[1], w[1], (LV_A - LV_B * y[1]) * w[0]);
    gy[1] = n1 + fmaT(LV_D * y[0] - LV_G, w[1], -LV_B * y[0] * w[0]);

    // dW2 += sum over the wave's trajectories of delta2 h1^T: K = trajectories
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int row = (2 * k + hf) * UDE_STRIDE + c;
      g.w2 = mfma32(td[row], th[row], g.w2);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};

// ---------------------------------------------------------------- kernels --
constexpr int32_t LANE_IDLE = -1;  // a lane past the end of the ensemble

// Record / solve / frozen-mesh replay of the UDE (Tsit5, FP32): the explicit
// record with a wave-uniform loop -- lanes whose trajectory is done take
// zero-length steps until the whole wavefront is done.  Both lanes of a
// trajectory take its steps; what goes to memory, the lower one writes (a
// save state's and the final state's component hf each).
template <int MODE, bool CKPT>
__global__ void __launch_bounds__(256, 2) ude_forward_kernel(const FwdArgs a) {
  using Sys = LvUdeOn<UdeRegW>;
  using Tab = Tsit5;
  using T = float;
  constexpr int D = 2;
  constexpr int RB = TapeRec<T, D>::BYTES;
  constexpr int YB = StateBytes<T, D>::BYTES;
  constexpr int CH = RB / 16;
  const int K = CKPT ? a.rec.page_steps : PAGE_STEPS;
  const int64_t n = a.ivp.n;
  const int hf = (threadIdx.x >> 5) & 1, lane_c = threadIdx.x & 31;
  const int64_t tr = (int64_t)blockIdx.x * UDE_BLOCK_TRAJ + (threadIdx.x >> 6) * UDE_TRAJ + lane_c;
  const bool valid = tr < n;
  const bool writes = hf == 0;  // this lane writes for its trajectory
  __shared__ double s_times[65];
  __shared__ uint4 s_tape[(MODE == MODE_SOLVE || CKPT) ? 1 : TAPE_GROUP * CH * 256];
  __shared__ double s_h[CKPT ? H_GROUP * 256 : 1];
  UdeRegW wts;
  wts.load((const float*)a.ivp.params);
  if (threadIdx.x < 65)
    s_times[threadIdx.x] = (int)threadIdx.x < a.ivp.n_save ? save_time_at(a.ivp.st, threadIdx.x)
                                                          : INFINITY;
  __syncthreads();
  const float* p = reinterpret_cast<const float*>(&wts);
  const double t0 = a.ivp.t0, t1 = a.ivp.t1;
  const double rtol = a.ivp.rtol, atol = a.ivp.atol;
  const int ns = a.ivp.n_save;
  T* ysv = (T*)a.y_save;
  const RecView& R = a.rec;

  T y[D], k1[D];
#pragma unroll
  for (int c = 0; c < D; ++c) y[c] = valid ? ((const T*)a.ivp.y0)[c * n + tr] : T(1);
  Sys::rhs(y, p, k1);
  int32_t status = valid ? LANE_OK : LANE_IDLE;
  if (valid) {
#pragma unroll
    for (int c = 0; c < D; ++c)
      if (!isfinite(y[c]) || !isfinite(k1[c])) status = LANE_NONFINITE;
  }
  double t = t0, h = 0.0;
  int32_t S_mesh = 0;
  if constexpr (MODE == MODE_FROZEN) {
    if (valid) {
      S_mesh = a.mesh_S[tr];
      if (S_mesh < 0 || (int64_t)S_mesh > a.cap) {
        S_mesh = 0;
        status = LANE_MAX_STEPS;
      }
    }
  } else {
    const double h_init = initial_step<Sys, Tab, T>(y, p, k1, t0, t1, rtol, atol);
    h = a.ivp.h0 > 0.0 ? fmin(a.ivp.h0, t1 - t0) : h_init;
  }

  T yp[D], k1p[D];
#pragma unroll
  for (int c = 0; c < D; ++c) {
    yp[c] = y[c];
    k1p[c] = k1[c];
  }
  if constexpr (MODE != MODE_SOLVE) {
    if (valid && writes) R.first_page[tr] = -1;
  }
  double tp = t0;
  int next_save = 0;
  T* ys_out = ysv + hf * n + tr;  // component hf of the next save state
  int32_t* sidx_out = R.save_idx + tr;
  double* sdt_out = R.save_dt + tr;
  const int64_t ys_stride = (int64_t)D * n;
  double ts = s_times[0];
  bool side = false;
  int32_t S = 0, trials = 0;
  bool prev_rej = false;
  int32_t page = -1;
  char* pg = nullptr;

  while (true) {
    bool act = status == LANE_OK &&
               (side || (MODE == MODE_FROZEN ? (S < S_mesh) : (t < t1)));
    if (!__any(act)) break;
    double hh = 0.0;
    bool last = false;
    if (act) {
      if (!side) {
        if constexpr (MODE == MODE_FROZEN) {
          hh = a.mesh_h[(int64_t)S * n + tr];
          last = (S == S_mesh - 1);
          ++trials;
        } else {
          if (trials >= a.ivp.max_steps) {
            status = LANE_MAX_STEPS;
            act = false;
          } else if (h < 16.0 * EPS64 * fmax(fabs(t), 1.0)) {
            status = LANE_DT_UNDERFLOW;
            act = false;
          } else {
            ++trials;
            if (t + h >= t1) {
              h = t1 - t;
              last = true;
            }
            hh = h;
          }
        }
      } else {
        hh = ts - tp;
      }
    }

    // one evaluation of the step map by every lane (idle lanes: h = 0)
    T yb[D], kb[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      yb[c] = side ? yp[c] : y[c];
      kb[c] = side ? k1p[c] : k1[c];
    }
    T Yunused[Tab::S][D];
    T ylast[D], klast[D], ynew[D];
    double esum[D];
    step_push<Sys, Tab, T, Tab::S, false, false, MODE != MODE_FROZEN>(
        yb, kb, p, T(hh), Yunused, ylast, klast, ynew, esum);
#pragma unroll
    for (int c = 0; c < D; ++c) ynew[c] = ylast[c];
    double err = 0.0, fac0 = 0.0;
    if constexpr (MODE != MODE_FROZEN) {
      err = err_ms_sum<T, D>(yb, ynew, hh, esum, rtol, atol);  // RMS norm squared
      fac0 = err >= 0.0 ? step_factor<2 * (Tab::QEMB + 1)>(err) : 0.0;
    }
    if (!act) continue;

    if (side) {
      *ys_out = hf ? ynew[1] : ynew[0];
      ys_out += ys_stride;
      if constexpr (MODE != MODE_SOLVE) {
        if (writes) {
          *sidx_out = S - 1;
          *sdt_out = hh;
        }
        sidx_out += n;
        sdt_out += n;
      }
      ++next_save;
      ts = s_times[next_save];
      side = ts < t;
      continue;
    }

    if (MODE == MODE_FROZEN || err <= 1.0) {
      if constexpr (MODE != MODE_SOLVE) {
        const int slot = S % K;
        const int kpage = S / K;
        const bool need = (slot == 0);
        const bool over = need && (kpage >= R.static_pages);
        // one page for the trajectory's two lanes
        uint64_t got = wave_bump(&R.counters[CNT_PAGES], over && writes);
        if (need) {
          int32_t np_;
          if (!over) {
            np_ = (int32_t)(tr * R.static_pages + kpage);
          } else {
            got = __shfl((unsigned long long)got, lane_c);
            if (got >= (uint64_t)(R.n_pages - R.n_static)) {
              status = LANE_NOSPACE;
              continue;
            }
            np_ = (int32_t)(R.n_static + (int64_t)got);
            if (writes) {
              const int64_t li = (int64_t)np_ - R.n_static;
              R.links[2 * li] = page;
              R.links[2 * li + 1] = -1;
              if (page >= R.n_static)
                R.links[2 * ((int64_t)page - R.n_static) + 1] = np_;
              else
                R.first_page[tr] = np_;
            }
          }
          page = np_;
          pg = R.pages + (int64_t)page * R.page_bytes;
        }
        if (!writes) {
        } else if constexpr (CKPT) {
          if (need) store_state<T, D>(pg, yb);
          s_h[((slot & (H_GROUP - 1))) * 256 + threadIdx.x] = hh;
          if ((slot & (H_GROUP - 1)) == H_GROUP - 1)
            flush_h(s_h, H_GROUP, pg + YB + (slot - (H_GROUP - 1)) * 8);
        } else {
          stage_rec<T, D>(s_tape, ((slot & (TAPE_GROUP - 1))) * CH, hh, yb);
          if ((slot & (TAPE_GROUP - 1)) == TAPE_GROUP - 1)
            flush_recs<T, D>(s_tape, TAPE_GROUP, pg + (slot - (TAPE_GROUP - 1)) * RB);
        }
      }
      ++S;
      tp = t;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        yp[c] = y[c];
        k1p[c] = k1[c];
        y[c] = ynew[c];
        k1[c] = klast[c];
      }
      t = last ? t1 : t + hh;
      if constexpr (MODE != MODE_FROZEN) {
        h = hh * fmax(0.2, fmin(prev_rej ? 1.0 : 10.0, fac0));
        prev_rej = false;
      }
      side = ts < t;
    } else {
      h = hh * fmax(0.2, fac0);
      prev_rej = true;
    }
  }
  if (!valid) return;

  if constexpr (MODE != MODE_SOLVE) {
    if (!writes) {
    } else if constexpr (CKPT) {
      const int rem = S % H_GROUP;
      if (rem > 0 && pg != nullptr) flush_h(s_h, rem, pg + YB + ((S - rem) % K) * 8);
    } else {
      const int rem = S % TAPE_GROUP;
      if (rem > 0 && pg != nullptr) {
        const int slot0 = (S - rem) % K;
        flush_recs<T, D>(s_tape, rem, pg + slot0 * RB);
      }
    }
  }
  const bool ok = (status == LANE_OK);
  for (; next_save < ns; ++next_save) {
    *ys_out = !ok ? T(NAN) : hf ? y[1] : y[0];
    ys_out += ys_stride;
    if constexpr (MODE != MODE_SOLVE) {
      if (writes) {
        *sidx_out = ok ? S : -1;
        *sdt_out = ok ? s_times[next_save] - t : NAN;
      }
      sidx_out += n;
      sdt_out += n;
    }
  }
  if constexpr (MODE != MODE_SOLVE) {
    ((T*)R.y_final)[hf * n + tr] = hf ? y[1] : y[0];
    if (writes) {
      R.steps[tr] = S;
      R.n_trial[tr] = trials;
      R.last_page[tr] = page;
      R.status[tr] = status;
    }
  }
  if (writes && a.lane_status) a.lane_status[tr] = status;
}

// Fixed-order sum over the 32 lanes of this lane's half (result valid in
// the lane with c = 0).
__device__ __forceinline__ float half_sum(float v) {
  v = v + __shfl_xor(v, 16);
  v = v + __shfl_xor(v, 8);
  v = v + __shfl_xor(v, 4);
  v = v + __shfl_xor(v, 2);
  v = v + __shfl_xor(v, 1);
  return v;
}

// Reverse sweep of the UDE with the weight gradient summed over the
// ensemble: one partial [UDE_NP] per block (its wavefronts' sums added in
// order) in the workspace, summed by reduce_partials_kernel in a fixed order.
//
// CKPT: the wavefront goes through the segments by their index from the start
// of the mesh, the last first.  All its trajectories that have segment f
// replay it together (a replay trip evaluates the field only), then reverse
// it together; those with fewer segments idle until theirs comes.  The
// trips add up to the wavefront's longest trajectory, replayed and reversed.
template <bool CKPT>
__global__ void __launch_bounds__(64 * UDE_WAVES, 2) ude_adjoint_kernel(const AdjArgs a) {
  using Sys = LvUdeSweep;
  using Tab = Tsit5;
  using T = float;
  constexpr int D = 2, SU = Tab::SU;
  constexpr int RB = TapeRec<T, D>::BYTES;
  constexpr int YB = StateBytes<T, D>::BYTES;
  const int K = CKPT ? a.rec.page_steps : PAGE_STEPS;
  const int64_t n = a.ivp.n;
  const int wave = threadIdx.x >> 6;
  const int hf = (threadIdx.x >> 5) & 1;
  const int64_t tr = (int64_t)blockIdx.x * UDE_BLOCK_TRAJ + wave * UDE_TRAJ + (threadIdx.x & 31);
  const bool valid = tr < n;
  const RecView& R = a.rec;
  __shared__ UdeLds s_lds;
  // the stage states of the step and their cotangents, each lane its own
  // (indexed by the stage loop, which registers cannot be)
  __shared__ float s_Y[SU][D][64 * UDE_WAVES];
  __shared__ float s_Yb[SU][D][64 * UDE_WAVES];
  ude_load_weights(s_lds, (const float*)a.ivp.params);
  __syncthreads();
  const bool ok = valid && R.status[tr] == LANE_OK;
  UdeGrad g = {};
  T lam[D] = {0.f, 0.f};
  double loss = 0.0;
  const T two_scale = T(2.0 * a.scale);

  const int32_t S = ok ? R.steps[tr] : 0;
  int32_t page = ok ? R.last_page[tr] : -1;
  T ycur[D];
#pragma unroll
  for (int c = 0; c < D; ++c) ycur[c] = ok ? ((const T*)R.y_final)[c * n + tr] : T(1);
  int s = ok ? R.n_save - 1 : -1;
  const int32_t* sidx_p = R.save_idx + (int64_t)(s < 0 ? 0 : s) * n + (valid ? tr : 0);
  const double* sdt_p = R.save_dt + (int64_t)(s < 0 ? 0 : s) * n + (valid ? tr : 0);
  int32_t sidx = ok ? *sidx_p : -1;
  double sdt = ok ? *sdt_p : 0.0;
  auto next_save = [&]() {
    --s;
    sidx_p -= n;
    sdt_p -= n;
    if (s >= 0) {
      sidx = *sidx_p;
      sdt = *sdt_p;
    }
  };
  int32_t i = S;
  int slot = S > 0 ? (S - 1) % K : 0;
  char* scr = CKPT && valid ? (char*)a.scratch + (int64_t)tr * K * RB : nullptr;

  // the stages of the step of size hh from yb, by every lane
  T k0[D], Y[SU][D], ylast[D], klast[D], ys[D];
  float4 h2[SU][4];

  // Reverse every trajectory's steps down to mesh point lo (at lo = 0 with
  // the saves based there).
  auto reverse_to = [&](int32_t lo) {
    // What the lane does next: the saves on mesh point i itself at once, then
    // a side step (side) or a mesh step (rev alone); false: nothing down to lo.
    bool side = false, rev = false;
    auto next = [&]() {
      const bool mine = ok && (i > lo || lo == 0);
      while (mine && s >= 0 && sidx == i && sdt == 0.0) {
        T w[D];
        save_cotangent<T, D>(a, s, tr, ycur, two_scale, w, loss);
#pragma unroll
        for (int c = 0; c < D; ++c) lam[c] = lam[c] + w[c];
        next_save();
      }
      side = mine && (s >= 0 && sidx == i);
      rev = mine && (side || i > lo);
    };
    next();
    bool more = __any(rev);
    // (tested at the end of a trip only: with an exit in its middle the loop
    // holds the gradient accumulators twice, and spills)
    while (more) {
      T yb[D] = {T(1), T(1)};
      double hh = 0.0;
      if (rev) {
        if (side) {
          hh = sdt;
#pragma unroll
          for (int c = 0; c < D; ++c) yb[c] = ycur[c];
        } else {
          load_rec<T, D>((CKPT ? scr : R.pages + (int64_t)page * R.page_bytes) + slot * RB, hh,
                         yb);
        }
      }
      UdeKeep keep{&s_lds, h2, 0};
      const float* p = reinterpret_cast<const float*>(&keep);
      Sys::rhs(yb, p, k0);
      step_push<Sys, Tab, T, SU, true, true, false>(yb, k0, p, T(hh), Y, ylast, klast, ys,
                                                    nullptr);
      T w[D] = {T(0), T(0)};
      if (rev && side) {
        save_cotangent<T, D>(a, s, tr, ys, two_scale, w, loss);
      } else if (rev) {
#pragma unroll
        for (int c = 0; c < D; ++c) w[c] = lam[c];
      }

      // reverse through the stages (every lane, zero cotangent where idle).
      // One stage per trip of a loop that is not unrolled, so that one copy
      // of the VJP (and its registers) serves all stages.  Tsit5's b_j and
      // a_lj (l > j) are all nonzero, so the sum is
      // b_j w + a_{j+1,j} Ybar_{j+1} + ... in index order, as unrolled.
      static_assert(Tab::B[0] != 0.0 && Tab::B[5] != 0.0 && Tab::A[5][4] != 0.0 &&
                        Tab::A[5][0] != 0.0 && Tab::A[4][0] != 0.0,
                    "dense lower triangle expected");
      T lin[D];
#pragma unroll
      for (int c = 0; c < D; ++c) {
        lin[c] = w[c];
#pragma unroll
        for (int q = 0; q < SU; ++q) s_Y[q][c][threadIdx.x] = Y[q][c];
      }
#pragma unroll 1
      for (int j = SU - 1; j >= 0; --j) {
        T kb[D], Yj[D], Ybj[D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
          Yj[c] = s_Y[j][c][threadIdx.x];
          kb[c] = s_lds.coef[j][0] * w[c];
        }
#pragma unroll 1
        for (int l = j + 1; l < SU; ++l) {
#pragma unroll
          for (int c = 0; c < D; ++c)
            kb[c] = fmaT(s_lds.coef[j][l], s_Yb[l][c][threadIdx.x], kb[c]);
        }
#pragma unroll
        for (int c = 0; c < D; ++c) kb[c] = T(hh) * kb[c];
        Sys::vjp(Yj, s_lds, h2[j], kb, Ybj, g);
#pragma unroll
        for (int c = 0; c < D; ++c) {
          lin[c] = lin[c] + Ybj[c];
          s_Yb[j][c][threadIdx.x] = Ybj[c];
        }
      }
      if (rev && side) {
#pragma unroll
        for (int c = 0; c < D; ++c) lam[c] = lam[c] + lin[c];
        next_save();
      } else if (rev) {
#pragma unroll
        for (int c = 0; c < D; ++c) {
          lam[c] = lin[c];
          ycur[c] = yb[c];
        }
        --i;
        if (--slot < 0) {
          slot = K - 1;
          if (i > 0) page = prev_page(R, page);
        }
      }
      next();
      more = __any(rev);
    }
  };

  if constexpr (CKPT) {
    const int F = S > 0 ? (S - 1) / K : -1;  // this trajectory's last segment
    const int F_max = wave_max(F);
    // (f = 0 also where no trajectory has steps: the saves at the initial state)
    for (int f = F_max > 0 ? F_max : 0; f >= 0; --f) {
      // replay segment f: the record (h, state) of each of its steps into the
      // trajectory's scratch page (its two lanes write the same; each reads
      // what it wrote)
      const int len = f <= F ? slot + 1 : 0;
      const int len_max = wave_max(len);
      T y[D] = {T(1), T(1)};
      const double* hs = nullptr;
      double h_next = 0.0;
      if (len > 0) {
        const char* pgp = R.pages + (int64_t)page * R.page_bytes;
        load_state<T, D>(pgp, y);
        hs = (const double*)(pgp + YB);
        h_next = hs[0];
      }
      for (int j = 0; j < len_max; ++j) {
        const double hh = h_next;  // loaded a step ahead
        h_next = 0.0;
        if (j + 1 < len) h_next = hs[j + 1];
        if (j < len) store_rec<T, D>(scr + j * RB, hh, y);
        if (j + 1 < len_max) {  // the last step's end state is not needed
          using Fwd = LvUdeOn<UdeLds>;
          const float* p = reinterpret_cast<const float*>(&s_lds);
          Fwd::rhs(y, p, k0);
          step_push<Fwd, Tab, T, SU, false, true, false>(y, k0, p, T(hh), Y, ylast, klast, ys,
                                                         nullptr);
          if (j + 1 < len) {
#pragma unroll
            for (int c = 0; c < D; ++c) y[c] = ys[c];
          }
        }
      }
      reverse_to(f * K);
    }
  } else {
    reverse_to(0);
  }
  if (a.loss_kind != LOSS_COTANGENT) loss = a.scale * loss;

  if (valid) {
    T* gyo = (T*)a.grad_y0;
    if (gyo) gyo[hf * n + tr] = !ok ? T(NAN) : hf ? lam[1] : lam[0];
    if (hf == 0 && a.loss_out)
      a.loss_out[tr] = !ok ? NAN : (a.loss_kind == LOSS_COTANGENT ? 0.0 : loss);
  }

  // this wavefront's partial of the weight gradient, in parameter order (its
  // tiles are free now), then the block's: the wavefronts' added in order
  const int l = __lane_id(), c = l & 31;
  float* part = s_lds.tile[wave];
#pragma unroll
  for (int r = 0; r < 16; ++r) part[UDE_OW2 + 32 * ude_unit(r, hf) + c] = g.w2[r];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int u = ude_unit(r, hf);
    const float w30 = half_sum(g.w3[0][r]), w31 = half_sum(g.w3[1][r]);
    const float b2 = half_sum(g.b2[r]);
    const float w10 = half_sum(g.w1[0][r]), w11 = half_sum(g.w1[1][r]);
    const float b1 = half_sum(g.b1[r]);
    if (c == 0) {
      part[UDE_OW3 + u] = w30;
      part[UDE_OW3 + 32 + u] = w31;
      part[UDE_OB2 + u] = b2;
      part[UDE_OW1 + 2 * u] = w10;
      part[UDE_OW1 + 2 * u + 1] = w11;
      part[UDE_OB1 + u] = b1;
    }
  }
  const float b30 = half_sum(g.b3[0]), b31 = half_sum(g.b3[1]);
  if (l == 0) {
    part[UDE_OB3] = b30;
    part[UDE_OB3 + 1] = b31;
  }
  __syncthreads();
  float* out = (float*)a.workspace + (int64_t)blockIdx.x * UDE_NP;
  for (int q = threadIdx.x; q < UDE_NP; q += 64 * UDE_WAVES) {
    float v = s_lds.tile[0][q];
#pragma unroll
    for (int w = 1; w < UDE_WAVES; ++w) v = v + s_lds.tile[w][q];
    out[q] = v;
  }
}

}  // namespace ens
