// Rollout schedule "quad": four lanes per sample, sixteen samples per wavefront, the
// network on the matrix cores -- FP32 (v_mfma_f32_16x16x4_f32), or BF16 / FP16
// operands with FP32 accumulation (v_mfma_f32_16x16x32_{bf16,f16}) -- for the
// throughput regime (tens of thousands of samples, or many problems at once).
//
// Lane l = 16 g + j: sample j of the wave, lane group g (0..3).  The 16 samples are the
// 16 columns of every product out^T = W in^T, so a sample's values never mix with
// another's.  With the instruction's layouts (A[i][k] in lane i + 16 k, B[k][j] in lane
// j + 16 k, D[i][j] in lane j + 16 (i / 4), item i % 4):
//   layer 1: two k-steps; lane group g supplies input g (state component g) in the
//            first and (v_0, v_1, 1, 0)[g] in the second (the 1 carries b1);
//   layer 2: the accumulator of layer 1 holds neurons 16 m + 4 g + r in lane group g,
//            item r -- exactly the k-row lane group g supplies at k-step (m, r), so
//            the activations never leave their lane; b2 enters as the accumulator;
//   layer 3: output o is placed in row 4 o, so it lands in lane group o, item 0: each
//            lane receives derivative g of its own sample, and lane group g carries
//            state component g (summed in 64 bits beside the FP32 running sum that the network reads).
// Kinematics and cost run in chunks of 16 steps, lane-parallel: lane group g takes
// four consecutive steps of the chunk for its sample, with exclusive scans over the
// four lane groups (v_permlane16_swap / v_permlane32_swap).  The noise of a chunk is
// drawn before the chunk (four draws per lane) and kept in memory for the weighted
// perturbation sum at the end (drawn again where there is no such memory).
#include "kernels_common.hip.h"

namespace mppi {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float qf32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float qf32x2;

constexpr int kQuadBlock = 256;
constexpr int kQuadWaves = 4;
constexpr int kQuadSamples = 64;   // per block
constexpr int kQuadChunk = 16;     // steps per chunk
// A wave's LDS: rows 0..16 of kQuadRow floats, row s holding the network's inputs of its 16
// samples at step s of the chunk: [16][4] state components (row 16: the state after the
// chunk) and [16][4] of (v_0, v_1, 1, 0), the clamped control and the constants of lane
// groups 2 and 3.  One address serves both and the state's write to the next row.
constexpr int kQuadRow = 128;
constexpr double kFp32Range = 0x1.ffffffp127;   // the smallest value that rounds to infinity in FP32
constexpr int kQuadWaveLds = (kQuadChunk + 1) * kQuadRow;

__device__ __forceinline__ float q_as_f(uint32_t v) { return __builtin_bit_cast(float, v); }
__device__ __forceinline__ uint32_t q_as_u(float v) { return __builtin_bit_cast(uint32_t, v); }

// Every lane of a column (the four lanes of one sample) receives the values of all
// four lane groups: v[0..3] = value of lane group 0..3.
__device__ __forceinline__ void all4(float x, float v[4]) {
  auto p = __builtin_amdgcn_permlane16_swap(q_as_u(x), q_as_u(x), false, false);
  // p[0]: rows 0,1 -> row 0's value, rows 2,3 -> row 2's; p[1]: rows 1 and 3
  auto q0 = __builtin_amdgcn_permlane32_swap(p[0], p[0], false, false);   // [v0 | v0], [v2 | v2]
  auto q1 = __builtin_amdgcn_permlane32_swap(p[1], p[1], false, false);   // [v1 | v1], [v3 | v3]
  v[0] = q_as_f(q0[0]);
  v[2] = q_as_f(q0[1]);
  v[1] = q_as_f(q1[0]);
  v[3] = q_as_f(q1[1]);
}

// The same for a 64-bit value.
__device__ __forceinline__ void all4(double x, double v[4]) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  float lo[4], hi[4];
  all4(q_as_f((uint32_t)b), lo);
  all4(q_as_f((uint32_t)(b >> 32)), hi);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] = __builtin_bit_cast(double, ((uint64_t)q_as_u(hi[i]) << 32) | q_as_u(lo[i]));
}

// Exclusive prefix of the four lane groups' values for lane group g, and their sum, the
// same bits in the four lanes of a column.
__device__ __forceinline__ double scan4_excl(double v, int g, double& total) {
  double V[4];
  all4(v, V);
  double s = V[0], p = 0.0;
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    p = i == g ? s : p;
    s = s + V[i];
  }
  total = s;
  return p;
}

// v + v in the lanes 8, 4, 2 and 1 apart of each 16-lane row in turn: the row's sum in every
// lane (DPP moves; once the lanes 8 apart agree, rotating by 4 meets the lane 4 apart).
template <int CTRL>
__device__ __forceinline__ float q_dpp(float v) {
  return q_as_f((uint32_t)__builtin_amdgcn_mov_dpp((int)q_as_u(v), CTRL, 0xf, 0xf, true));
}
constexpr int kQRor8 = 0x128, kQRor4 = 0x124, kQXor2 = 0x4E, kQXor1 = 0xB1;
__device__ __forceinline__ float row_sum(float v) {
  v += q_dpp<kQRor8>(v);
  v += q_dpp<kQRor4>(v);
  v += q_dpp<kQXor2>(v);
  v += q_dpp<kQXor1>(v);
  return v;
}
__device__ __forceinline__ float row_min(float v) {
  v = fminf(v, q_dpp<kQRor8>(v));
  v = fminf(v, q_dpp<kQRor4>(v));
  v = fminf(v, q_dpp<kQXor2>(v));
  v = fminf(v, q_dpp<kQXor1>(v));
  return v;
}

// tanh of four values, PRE: of x from x * kTanhScale.  The empty asm statements keep the four
// in step: each stage's results are used only after all four have been issued, so the
// latency of one exp or rcp is covered by the others' (the compiler, short of
// registers, ran them one after the other: K = 65536, FP32, two waves per SIMD 745 -> 702
// us; K = 16384, FP32, h = 32, one wave 116 -> 107 us).  The values are tanh_f's and
// tanh_prescaled's.
template <bool PRE>
__device__ __forceinline__ void tanh4(const qf32x4 d, float h[4]) {
  float e[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_exp2f(PRE ? d[r] : d[r] * kTanhScale);
  asm("" : "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]));
#pragma unroll
  for (int r = 0; r < 4; ++r) e[r] = e[r] + 1.0f;
  asm("" : "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]));
#pragma unroll
  for (int r = 0; r < 4; ++r) e[r] = __builtin_amdgcn_rcpf(e[r]);
  asm("" : "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]));
#pragma unroll
  for (int r = 0; r < 4; ++r) h[r] = __builtin_fmaf(-2.0f, e[r], 1.0f);
}

constexpr int kQPrecFP32 = 0;
constexpr int kQPrecBF16 = 1;
constexpr int kQPrecFP16 = 2;

template <int PREC, int HID> struct QuadNet;

// FP32: v_mfma_f32_16x16x4_f32, one k-row per lane group, for layers 1 and 2; layer 3
// (4 outputs) on v_mfma_f32_4x4x1_16b_f32, whose 16 blocks of 4 lanes (one lane group,
// 4 samples) each take the 4 outputs x 4 samples of one hidden unit per call, so that
// no row of the product is idle: lane group g sums the hidden units 16m + 4g + r, and the
// four groups' partial sums are then added across the rows (two permlane swaps).
template <int HID>
struct QuadNet<kQPrecFP32, HID> {
  static constexpr int NM = HID / 16;
  float A1[NM][2];
  float A2[NM][NM][4];
  float A3[NM][4];
  qf32x4 C2[NM];
  qf32x4 C3;

  __device__ explicit QuadNet(const float* __restrict__ P, int g, int i) {
    const float* W1 = P;
    const float* b1 = W1 + HID * 6;
    const float* W2 = b1 + HID;
    const float* b2 = W2 + HID * HID;
    const float* W3 = b2 + HID;
    const float* b3 = W3 + 4 * HID;
    // layers 1 and 2 form tanh's argument already multiplied by 2 log2(e)
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int n = 16 * m + i;
      A1[m][0] = kTanhScale * W1[n * 6 + g];
      A1[m][1] = kTanhScale * (g == 0 ? W1[n * 6 + 4] : g == 1 ? W1[n * 6 + 5] : g == 2 ? b1[n] : 0.0f);
#pragma unroll
      for (int mi = 0; mi < NM; ++mi)
#pragma unroll
        for (int r = 0; r < 4; ++r) A2[m][mi][r] = kTanhScale * W2[n * HID + 16 * mi + 4 * g + r];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        C2[m][r] = kTanhScale * b2[16 * m + 4 * g + r];
        A3[m][r] = W3[(i & 3) * HID + 16 * m + 4 * g + r];   // output i & 3 of its block
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) C3[r] = g == 0 ? b3[r] : 0.0f;   // row r of a block: output r
  }

  // f = derivative (lane group g) of this lane's sample; b0 = state component g,
  // b1 = (v_0, v_1, 1, 0)[g].
  __device__ __forceinline__ float eval(float b0, float b1) const {
    float h1[NM][4];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      qf32x4 d = {0.0f, 0.0f, 0.0f, 0.0f};
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(A1[m][0], b0, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(A1[m][1], b1, d, 0, 0, 0);
      tanh4<true>(d, h1[m]);
    }
    float h2[NM][4];
    qf32x4 d2[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) d2[m] = C2[m];
#pragma unroll
    for (int mi = 0; mi < NM; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < NM; ++m)
          d2[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(A2[m][mi][r], h1[mi][r], d2[m], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < NM; ++m) tanh4<true>(d2[m], h2[m]);
    qf32x4 d3 = C3;   // lane (g, i): d3[o] = group g's part of output o of sample i
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) d3 = __builtin_amdgcn_mfma_f32_4x4x1f32(A3[m][r], h2[m][r], d3, 0, 0, 0);
    // lane groups 0, 1 keep outputs 0, 1 and groups 2, 3 outputs 2, 3 (sums of groups
    // g and g ^ 2), then each group keeps its own output (sum of the pair g, g ^ 1)
    const auto p0 = __builtin_amdgcn_permlane32_swap(q_as_u(d3[0]), q_as_u(d3[2]), false, false);
    const auto p1 = __builtin_amdgcn_permlane32_swap(q_as_u(d3[1]), q_as_u(d3[3]), false, false);
    const float a = q_as_f(p0[0]) + q_as_f(p0[1]);
    const float b = q_as_f(p1[0]) + q_as_f(p1[1]);
    const auto p2 = __builtin_amdgcn_permlane16_swap(q_as_u(a), q_as_u(b), false, false);
    return q_as_f(p2[0]) + q_as_f(p2[1]);
  }
};

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 qbf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 qf16x8;

template <int PREC> struct QuadOps;
template <> struct QuadOps<kQPrecBF16> {
  typedef qbf16x8 vec;
  static __device__ __forceinline__ qf32x4 mma(vec a, vec b, qf32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ vec pack(const float v[8]) {
    vec r;
#pragma unroll
    for (int c = 0; c < 8; ++c) r[c] = (__bf16)v[c];
    return r;
  }
};
template <> struct QuadOps<kQPrecFP16> {
  typedef qf16x8 vec;
  static __device__ __forceinline__ qf32x4 mma(vec a, vec b, qf32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ vec pack(const float v[8]) {
    vec r;
#pragma unroll
    for (int c = 0; c < 8; ++c) r[c] = (_Float16)v[c];
    return r;
  }
};

// BF16 / FP16 operands, FP32 accumulation: v_mfma_f32_16x16x32_{bf16,f16}, eight k
// slots per lane group (A[i][k] in lane i + 16 (k / 8), item k % 8; B likewise).
// Layer 1 uses slots 0 (state component g) and 1 ((v_0, v_1, 1, 0)[g]) of each
// group; k-block kb of layers 2 and 3 takes tiles 2 kb (items 0..3) and 2 kb + 1
// (items 4..7), i.e. neurons 16 (2 kb + c / 4) + 4 g + c % 4 -- again what lane group
// g holds of the previous layer's accumulators.
template <int PREC, int HID>
struct QuadNet {
  typedef QuadOps<PREC> Ops;
  typedef typename Ops::vec vec;
  static constexpr int NM = HID / 16;
  static constexpr int NKB = NM / 2;
  vec A1[NM];
  vec A2[NM][NKB];
  vec A3[NKB];
  qf32x4 C2[NM];
  qf32x4 C3;

  static constexpr float kPre = PREC == kQPrecBF16 ? kTanhScale : 1.0f;
  static __device__ __forceinline__ int neuron(int kb, int g, int c) {
    return 16 * (2 * kb + (c >> 2)) + 4 * g + (c & 3);
  }

  __device__ explicit QuadNet(const float* __restrict__ P, int g, int i) {
    const float* W1 = P;
    const float* b1 = W1 + HID * 6;
    const float* W2 = b1 + HID;
    const float* b2 = W2 + HID * HID;
    const float* W3 = b2 + HID;
    const float* b3 = W3 + 4 * HID;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int n = 16 * m + i;
      // BF16: layers 1 and 2 form tanh's argument already multiplied by 2 log2(e) (the
      // scaled weights are rounded to BF16; measured at K = 16384, the cost error drops
      // from 1.2-1.35e-2 to 1.0-1.1e-2).  FP16 keeps the unscaled weights: scaled, its
      // cost error rose from 8-9e-4 to 2.2-2.4e-3.
      float v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      v[0] = kPre * W1[n * 6 + g];
      v[1] = kPre * (g == 0 ? W1[n * 6 + 4] : g == 1 ? W1[n * 6 + 5] : g == 2 ? b1[n] : 0.0f);
      A1[m] = Ops::pack(v);
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = kPre * W2[n * HID + neuron(kb, g, c)];
        A2[m][kb] = Ops::pack(v);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) C2[m][r] = kPre * b2[16 * m + 4 * g + r];
    }
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      float v[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = (i & 3) == 0 ? W3[(i >> 2) * HID + neuron(kb, g, c)] : 0.0f;
      A3[kb] = Ops::pack(v);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) C3[r] = r == 0 ? b3[g] : 0.0f;
  }

  __device__ __forceinline__ float eval(float b0, float b1) const {
    float v[8] = {b0, b1, 0, 0, 0, 0, 0, 0};
    const vec B1 = Ops::pack(v);
    float h1[NM][4];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const qf32x4 d = Ops::mma(A1[m], B1, qf32x4{0.0f, 0.0f, 0.0f, 0.0f});
      tanh4<PREC == kQPrecBF16>(d, h1[m]);
    }
    vec B2[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = h1[2 * kb + (c >> 2)][c & 3];
      B2[kb] = Ops::pack(v);
    }
    float h2[NM][4];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      qf32x4 d = C2[m];
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) d = Ops::mma(A2[m][kb], B2[kb], d);
      tanh4<PREC == kQPrecBF16>(d, h2[m]);
    }
    qf32x4 d3 = C3;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = h2[2 * kb + (c >> 2)][c & 3];
      d3 = Ops::mma(A3[kb], Ops::pack(v), d3);
    }
    return d3[0];
  }
};

// One tile of 64 samples (tile * 64 ... + 63) of one problem.
//
// What bounds it: issue.  A matrix-core instruction and a vector instruction do not overlap
// on gfx950, also from different waves (microbenchmarks: 32 cycles per 16x16x4 FP32
// product plus 4.4 per vector instruction, 2.2 for an FP32 add, multiply or fma that two
// waves issue together, 8.2 per exp or rcp), so a step of 16 samples costs its 704 (h = 32)
// matrix cycles plus every vector instruction.  Hence everything that does not belong to
// the chain is done once per sample and step, in the lane that draws the step's noise (the
// clamped control and the control cost) or that evaluates its cost; the heading is checked
// for non-finite values once per chunk and x_d at the end: what is not finite there stays
// so, since every step adds to it.  242 -> ~170 vector instructions per wave-step beside the
// matrix products (a third of that from the 64-bit sums); with tanh4 above, before -> after:
// batched form (512 instances, 1.01e8 steps) 4.69 -> 4.07 ms; T = 100, h = 64: FP32 K = 65536 759 -> 678
// us, BF16 332 -> 264 us, FP16 365 -> 296 us, K = 16384 (one wave per SIMD) FP32 226 -> 188, BF16
// 124 -> 91, FP16 129 -> 99 us; h = 32, FP32, K = 16384 131 -> 93 us.
template <int PREC, int HID, bool RECEDE = true>
__device__ void quad_rollout_tile(const RolloutArgs& a, int tile, float* sU, float* sX, float* red) {
  const int T = __builtin_amdgcn_readfirstlane(a.T);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4;
  const int j = lane & 15;
  const int k = tile * kQuadSamples + wv * 16 + j;
  const bool valid = k < a.K;
  const bool zm = k >= a.K_imp;   // exploration sample: v = eps, delta = eps - u
  // v = eps + m_u u, delta = eps - m_z u, with one of the two 1 and the other 0 (exact)
  const float m_u = zm ? 0.0f : 1.0f, m_z = zm ? 1.0f : 0.0f;
  float* wX = sX + wv * kQuadWaveLds;
  // The stored noise of the wave's 16 samples ([T][16] pairs), or null.  Marked as global
  // memory: in the batched form the pointer is itself read from memory and would be taken
  // for a generic one, whose stores the next LDS read waits for.
  typedef __attribute__((address_space(1))) qf32x2 global_pair;
  global_pair* wS = a.eps_store ? (global_pair*)(a.eps_store + ((size_t)tile * kQuadWaves + wv) * (size_t)T * 32)
                                : nullptr;

  for (int i = threadIdx.x; i < 2 * T; i += kQuadBlock) sU[i] = a.U[i];
  __syncthreads();

  const QuadNet<PREC, HID> net(a.params, g, j);
  float x0v[kStateDim];
#pragma unroll
  for (int i = 0; i < kStateDim; ++i) x0v[i] = a.x0_dev ? a.x0_dev[i] : a.x0[i];
  // Sums over the steps are held in 64 bits: state component g (roll, v_x, v_y, theta_dot),
  // of which the network reads the FP32 running sum xh, the pose entering the chunk (the
  // same in the four lanes of a sample) and the cost.  A 64-bit add takes as long as one
  // FP32 instruction; the error-free FP32 sums it replaces took seven or eight.
  float xh = x0v[3 + g];
  double xd = xh, th_c = x0v[2], px_c = x0v[0], py_c = x0v[1], S64 = 0.0;
  bool ok = true;
  uint64_t in_range = ~0ull;         // the wave's lanes whose positions were inside FP32's range
  wX[j * 4 + g] = xh;                // row 0 = the state entering the chunk
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<float2*>(wX + (4 * q + g) * kQuadRow + 64 + j * 4 + 2) = make_float2(1.0f, 0.0f);
  // a horizon of less than a chunk leaves rows that no step writes: their sums are
  // multiplied by a zero step, so they must be finite
  if (T < kQuadChunk)
    for (int s = 1; s <= kQuadChunk; ++s) wX[s * kQuadRow + j * 4 + g] = 0.0f;

  for (int cs = 0; cs < T; cs += kQuadChunk) {
    const int n = __builtin_amdgcn_readfirstlane(min(kQuadChunk, T - cs));
    // the noise of the chunk: lane (g, j) draws steps cs + g + 4 q of its own sample
    // (past the horizon a clamped step, discarded), forms their clamped controls for the
    // chain and their control cost, and keeps the noise where it reads it back below
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int s = 4 * q + g;
      const int t = min(cs + s, T - 1);
      float e0, e1;
      draw_eps((uint32_t)t, (uint32_t)k, a.nk, e0, e1);
      const float2 u = *reinterpret_cast<const float2*>(sU + 2 * t);
      const float v0 = __builtin_amdgcn_fmed3f(__builtin_fmaf(u.x, m_u, e0), a.u_lo0, a.u_hi0);
      const float v1 = __builtin_amdgcn_fmed3f(__builtin_fmaf(u.y, m_u, e1), a.u_lo1, a.u_hi1);
      *reinterpret_cast<float2*>(wX + s * kQuadRow + 64 + j * 4) = make_float2(v0, v1);
      if (s < n) {
        if (wS) wS[(uint32_t)(t * 16 + j)] = qf32x2{e0, e1};
        S64 += (double)(a.gcs0 * (u.x * __builtin_fmaf(-u.x, m_z, e0)));
        S64 += (double)(a.gcs1 * (u.y * __builtin_fmaf(-u.y, m_z, e1)));
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // the serial chain over the chunk; the step's control (or constant) is read one step ahead
    // (row 16's place for controls is read and not used)
    {
      float* p = wX + j * 4 + g;
      float v = p[64];
      for (int s = 0; s < n; ++s) {
        const float vn = p[kQuadRow + 64];
        const float y = a.dt * net.eval(xh, v);
        xh = xh + y;
        xd = xd + (double)y;
        p += kQuadRow;
        p[0] = (float)xd;
        v = vn;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // kinematics and cost of the chunk: lane group g takes steps cs + 4 g .. cs + 4 g + 3; a
    // step past the horizon has a zero time step
    const float* row = wX + 4 * g * kQuadRow + j * 4;   // the state before the lane's first step
    bool live[4];
    float dq[4], dth[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      live[q] = 4 * g + q < n;
      dq[q] = live[q] ? a.dt : 0.0f;
      dth[q] = dq[q] * row[q * kQuadRow + 3];
    }
    // heading before each of the lane's steps
    double th[4], th_sum;
    {
      const double d1 = (double)dth[0] + (double)dth[1], d2 = d1 + (double)dth[2];
      th[0] = th_c + scan4_excl(d2 + (double)dth[3], g, th_sum);
      th[1] = th[0] + (double)dth[0];
      th[2] = th[0] + d1;
      th[3] = th[0] + d2;
    }
    // position after each of them
    double px[4], py[4], px_sum, py_sum;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float vx = row[q * kQuadRow + 1], vy = row[q * kQuadRow + 2];
      float sn, c_;
      sincosf((float)th[q], &sn, &c_);
      const double dx = (double)(dq[q] * (c_ * vx - sn * vy)), dy = (double)(dq[q] * (sn * vx + c_ * vy));
      px[q] = q == 0 ? dx : px[q - 1] + dx;
      py[q] = q == 0 ? dy : py[q - 1] + dy;
    }
    {
      const double bx = px_c + scan4_excl(px[3], g, px_sum), by = py_c + scan4_excl(py[3], g, py_sum);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        px[q] = bx + px[q];
        py[q] = by + py[q];
        // a position outside FP32's range at any step makes the sample non-finite, also where
        // a later step leads back
        in_range &= __ballot(fabs(px[q]) < kFp32Range) & __ballot(fabs(py[q]) < kFp32Range);
      }
    }
    // (held as the wave's masks, and before the loads: as a condition per lane, which the
    // compiler moves behind them, it spilled ten more registers at h = 32: batched form 4.24 ms
    // against 4.13, now 4.13)
    __builtin_amdgcn_sched_barrier(0);
    // every map and decay load at once
    float mv[4][4], fxv[4], fyv[4], dec[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t off[4];
      map_taps64(a.cost, px[q], py[q], off, fxv[q], fyv[q]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        mv[q][i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.map) + off[i]);
      dec[q] = a.decay[(uint32_t)(min(cs + 4 * g + q, T - 1) + 1)];
    }
    float zeta[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) zeta[q] =
          slip_angle(a.cost, row[(q + 1) * kQuadRow + 1], row[(q + 1) * kQuadRow + 2]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float c =
          state_cost_h(a.cost, bilerp(mv[q], fxv[q], fyv[q]), dec[q], row[(q + 1) * kQuadRow + 1], zeta[q]);
      S64 += (double)(live[q] ? c : 0.0f);
    }
    // the pose entering the next chunk
    th_c += th_sum;
    px_c += px_sum;
    py_c += py_sum;
    ok = ok && finite_f((float)th_c);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // the chunk's last state (as the cost reads it) enters the next chunk as its row 0
    wX[j * 4 + g] = (float)xd;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  ok = ok && ((in_range >> lane) & 1) && finite_f(xh) && finite_f((float)xd);

  // S_k: the four lanes' sums
  double S4[4];
  all4(S64, S4);
  float S = (float)(((S4[0] + S4[1]) + S4[2]) + S4[3]);
  float okv[4];
  all4(ok ? 1.0f : 0.0f, okv);
  const bool okc = okv[0] != 0.0f && okv[1] != 0.0f && okv[2] != 0.0f && okv[3] != 0.0f;
  if (!valid || !okc || !finite_f(S)) S = kInf;
  if (valid && g == 0) store_through(a.S + k, S);   // read by the host or Algorithm 3's update

  if (a.cem_zeta > 0) {
    // Algorithm 3: the sample's delta row (lane group g regenerates steps g, g + 4, ...)
    if (valid) {
      float* drow = a.D + (size_t)k * 2 * T;
      for (int t = g; t < T; t += 4) {
        float e0, e1;
        draw_eps((uint32_t)t, (uint32_t)k, a.nk, e0, e1);
        if (zm) {
          e0 -= sU[2 * t];
          e1 -= sU[2 * t + 1];
        }
        drow[2 * t] = e0;
        drow[2 * t + 1] = e1;
      }
    }
    return;   // the cross-entropy update runs in the launch that follows
  }

  // ---- the block's softmin partial ----------------------------------------------------
  float* scratch = red + kQuadWaves * 2 * kTMax;   // [8]
  const float wmin = row_min(S);
  if (lane == 0) scratch[wv] = wmin;
  __syncthreads();
  const float rho = fminf(fminf(scratch[0], scratch[1]), fminf(scratch[2], scratch[3]));
  const float e = rel_weight(S, rho, a.inv_lambda);
  const float esum = row_sum(e);
  if (lane == 0) scratch[4 + wv] = esum;
  // N[t] = sum_k e_k delta_{k,t}: lane group g takes steps t = g, g + 4, ... of its sample
  // (the stored noise, written by this lane in the chunk draws, or drawn again) and the 16
  // samples of a row are summed in DPP moves.  A sample past K has weight zero.
  const bool any_zm = a.K_imp < a.K;
  auto add_step = [&](int t, float e0, float e1) {
    if (any_zm) {
      const float2 u = *reinterpret_cast<const float2*>(sU + 2 * min(t, T - 1));
      e0 = __builtin_fmaf(-u.x, m_z, e0);
      e1 = __builtin_fmaf(-u.y, m_z, e1);
    }
    const float n0 = row_sum(e * e0), n1 = row_sum(e * e1);
    if (j == 0 && t < T) *reinterpret_cast<float2*>(red + wv * 2 * kTMax + 2 * t) = make_float2(n0, n1);
  };
  if (wS) {
    for (int t0 = 0; t0 < T; t0 += 16) {   // four loads in flight
      qf32x2 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = t0 + 4 * q + g;
        v[q] = t < T ? wS[(uint32_t)(t * 16 + j)] : qf32x2{0.0f, 0.0f};
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (t0 + 4 * q < T) add_step(t0 + 4 * q + g, v[q][0], v[q][1]);
    }
  } else {
    for (int t0 = 0; t0 < T; t0 += 4) {
      const int t = t0 + g;
      float e0, e1;
      draw_eps((uint32_t)min(t, T - 1), (uint32_t)k, a.nk, e0, e1);
      add_step(t, e0, e1);
    }
  }
  __syncthreads();
  float* N_lds = sX;   // the chunks are no longer read
  for (int o = threadIdx.x; o < 2 * T; o += kQuadBlock)
    N_lds[o] = ((red[o] + red[2 * kTMax + o]) + red[2 * 2 * kTMax + o]) + red[3 * 2 * kTMax + o];
  const float eta = ((scratch[4] + scratch[5]) + scratch[6]) + scratch[7];
  finish_iteration<kQuadBlock, kModelNet, RECEDE, HID>(a, tile, rho, eta, N_lds, red);
}

// Waves per SIMD: three at h = 32 (at most 168 registers), two at h = 64 (at most 256; with
// one, the FP32 form ran about a fifth slower at K = 65536).
template <int PREC, int HID>
__global__ __launch_bounds__(kQuadBlock, HID == 32 ? 3 : 2) void rollout_quad_kernel(RolloutArgs a) {
  if (a.iter_dev) a.nk.iter = *a.iter_dev;   // the device counter, advanced by the final merge
  __shared__ __attribute__((aligned(16))) float sU[2 * kTMax];
  __shared__ __attribute__((aligned(16))) float sX[kQuadWaves * kQuadWaveLds];
  __shared__ __attribute__((aligned(16))) float red[kQuadWaves * 2 * kTMax + 8];
  quad_rollout_tile<PREC, HID>(a, blockIdx.x, sU, sX, red);
}

// Batched form on quad tiles: each block takes items (instance, tile of 64 samples)
// from the launch's work queue in the order of the items list; the shared map, network
// and decay table come from kernel arguments.  A tile's arithmetic and an instance's
// merge order do not depend on the grid or the item order.  Three waves per SIMD (a few
// registers spill; about a tenth faster on the 512-instance workload than two).
__global__ __launch_bounds__(kQuadBlock, 3) void rollout_batch_quad_kernel(const RolloutArgs* __restrict__ inst,
                                                                      const int2* __restrict__ items, int n_items,
                                                                      const float* __restrict__ map,
                                                                      const float* __restrict__ params,
                                                                      const float* __restrict__ decay,
                                                                      unsigned* __restrict__ queue) {
  __shared__ __attribute__((aligned(16))) float sU[2 * kTMax];
  __shared__ __attribute__((aligned(16))) float sX[kQuadWaves * kQuadWaveLds];
  __shared__ __attribute__((aligned(16))) float red[kQuadWaves * 2 * kTMax + 8];
  for (;;) {
    const int b = next_work_item(queue, n_items);
    if (b < 0) break;
    const int2 it = items[b];
    RolloutArgs a = inst[it.x];
    a.map = map;
    a.params = params;
    a.decay = decay;
    a.nk.iter = *a.iter_dev;
    quad_rollout_tile<kQPrecFP32, 32, false>(a, it.y, sU, sX, red);
  }
}

template __global__ void rollout_quad_kernel<kQPrecFP32, 32>(RolloutArgs);
template __global__ void rollout_quad_kernel<kQPrecFP32, 64>(RolloutArgs);
template __global__ void rollout_quad_kernel<kQPrecBF16, 32>(RolloutArgs);
template __global__ void rollout_quad_kernel<kQPrecBF16, 64>(RolloutArgs);
template __global__ void rollout_quad_kernel<kQPrecFP16, 32>(RolloutArgs);
template __global__ void rollout_quad_kernel<kQPrecFP16, 64>(RolloutArgs);

}  // namespace mppi
