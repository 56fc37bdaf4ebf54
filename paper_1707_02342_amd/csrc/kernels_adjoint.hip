// Adjoint rollout: gradient of the free-energy objective
//   J = -lambda log((1/K) sum_k exp(-S_k/lambda)) = rho - lambda log(eta~/K)
// (the Monte-Carlo estimate of -lambda times the free energy, Eq. FreeEnergy) with
// respect to the nominal controls U and every parameter of the dynamics network.
//
// dJ/dS_k = w_k (the weights of Algorithm 2), so every sample's reverse sweep is
// seeded with w_k and the per-sample gradients add up directly.  The layout is the
// forward "wave" layout: 32 lanes per sample, lane (row r, column c) owning hidden
// unit j = 16 r + c, two samples per wavefront, eight per block.
//
// Memory: the forward pass stored the full state every `ckpt_every` steps.  The
// sweep walks the segments backwards.  As in the forward pass only the dynamic states
// x_d (the network never reads the pose) and their cotangents p_d form serial chains, so
// each segment is taken in three phases:
//   1. chain: the x_d recurrence from the checkpoint, 32 lanes per sample, keeping the
//      states and both layers' activations in LDS;
//   2. pose, lane-parallel over the segment's steps (at most 16, one 16-lane row, the two
//      rows of a sample alike): heading and position by scans, the gradient of the cost at
//      the post-step states, and -- since the cotangents of the pose depend on the network
//      through nothing but these -- their suffix sums p_x, p_y, p_theta, which reduces the
//      pose's part in the sweep to one known term per step ("drive"),
//        D_t = (0, dt (p_x cos + p_y sin), dt (p_y cos - p_x sin), dt p_theta);
//   3. reverse chain, one component of p_d per lane of each quad:
//        a2 = (W3^T dt p_d)(1 - h2^2);  a1 = (W2^T a2)(1 - h1^2);  g_in = W1^T a1;
//        dJ/du_t = g'(v_t) g_in[4:6];  p_d <- p_d + D_t + g_in[0:4] + dc/dx_d(x_t),
//      with dW3 += dt p_d h2^T, dW1 += a1 in^T on the vector ALU and dW2 += a2 h1^T, the two
//      samples of the wave together, as one v_mfma_f32_32x32x2_f32 per step: lane
//      32 half + j holds element j of sample `half`, which is the product's operand layout
//      as it stands (64 cycles against ~150 for the 32 DPP products it replaces).
// The control-cost term gamma eps_t / Sigma weighted by w_k sums to gamma Delta_t / Sigma
// and is added by the final reduction.
//
// What bounds it: the vector ALU and the latency of the two chains, ~160 instructions per
// step and wave.  Evaluating pose, cost gradient and their cotangents in all 32 lanes of
// every step, unrolled over 16 steps with the activations in registers (266 registers, one
// wave per SIMD, 86 KB of code), took 320-330 us at K = 4096, T = 100, C = 10; this
// form (188 registers, 11 KB) 102-104 us, 32 TFLOP/s of the 8064 flop per sample-step.
#include "wave_common.hip.h"

namespace mppi {

constexpr int kAdjMaxSeg = 16;   // steps of a segment (one 16-lane row)
constexpr int kNP32 = 1412;      // parameters of the 6-32-32-4 network

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

namespace {

constexpr int kRowMirror = 0x140;   // lane i of a row reads lane 15 - i

// Inclusive / exclusive sums over the 16 lanes of a row, and the sum over the lane itself
// and all later lanes of its row (suffix), in DPP moves.
__device__ __forceinline__ float row_incl(float v) {
  v = v + dpp_upd<kRowShr + 1>(0.0f, v);
  v = v + dpp_upd<kRowShr + 2>(0.0f, v);
  v = v + dpp_upd<kRowShr + 4>(0.0f, v);
  v = v + dpp_upd<kRowShr + 8>(0.0f, v);
  return v;
}
__device__ __forceinline__ float row_excl(float v) { return row_incl(dpp_upd<kRowShr + 1>(0.0f, v)); }
__device__ __forceinline__ float row_suffix(float v) { return dpp_f<kRowMirror>(row_incl(dpp_f<kRowMirror>(v))); }
__device__ __forceinline__ float row_suffix_excl(float v) { return dpp_f<kRowMirror>(row_excl(dpp_f<kRowMirror>(v))); }

// The value v holds in the first lane of the caller's 32-lane half.
__device__ __forceinline__ float first_of_half(float v) {
  const float lo = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  const float hi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  return (threadIdx.x & 32) ? hi : lo;
}

// acc + sum_o x_o w[o], x_o the value of x in lane o of each quad.
__device__ __forceinline__ float quad_dot(float acc, float x, float w0, float w1, float w2, float w3) {
  asm volatile(
      "s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %1, %2 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %1, %3 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %1, %4 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %1, %5 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf"
      : "+v"(acc) : "v"(x), "v"(w0), "v"(w1), "v"(w2), "v"(w3));
  return acc;
}

// g[o] += x_o y, x_o the value of x in lane o of each quad.
__device__ __forceinline__ void quad_axpy(float (&g)[4], float x, float y) {
  asm volatile(
      "s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %4, %5 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %5 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %5 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %5 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf"
      : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]), "+v"(g[3]) : "v"(x), "v"(y));
}

}  // namespace

// LDS: per sample the clamped controls (each step's entry later holds its dJ/du), then a
// region for the segment's states, drives and activations that the block's reduction of
// the parameter gradients reuses.
size_t adjoint_smem_bytes(int T, int ckpt_every) {
  const size_t C = (size_t)ckpt_every;
  const size_t seg = 2 * kWaveSlots * (C + 1) * 4 + 4 * C * 128;
  const size_t red = 4 * (size_t)kNP32;
  return sizeof(float) * (kWaveSlots * (size_t)((2 * T + 3) & ~3) + (seg > red ? seg : red));
}

__global__ __launch_bounds__(kWaveBlock, 2) void adjoint_wave_kernel(AdjointArgs a) {
  constexpr int HID = 32;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int T = a.T, C = a.ckpt_every;
  const int eStride = (2 * T + 3) & ~3;
  float* sV = smem;                                    // [8][2T] clamped controls, then dJ/du
  float* sX = sV + kWaveSlots * eStride;               // [8][C + 1][4] states x_d of the segment
  float* sD = sX + kWaveSlots * (C + 1) * 4;           // [8][C + 1][4] drives (row n: see below)
  float* sH = sD + kWaveSlots * (C + 1) * 4;           // [4 waves][C][2][64] activations h1, h2
  float* sRed = sX;                                    // [4][1412], after every segment

  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int half = lane >> 5;
  const int c32 = lane & 31;
  const int r = c32 >> 4;
  const int col = lane & 15;
  const int comp = lane & 3;
  const int slot = wv * 2 + half;
  const int k = blockIdx.x * kWaveSlots + slot;
  const bool valid = k < a.K;
  float* myV = sV + slot * eStride;
  float* myX = sX + slot * (C + 1) * 4;
  float* myD = sD + slot * (C + 1) * 4;
  float* myH = sH + wv * C * 128 + lane;

  // ---- network constants of this lane ----------------------------------------------
  const float* W1 = a.params;
  const float* b1 = W1 + HID * 6;
  const float* W2 = b1 + HID;
  const float* b2 = W2 + HID * HID;
  const float* W3 = b2 + HID;
  const float* b3 = W3 + 4 * HID;
  const int j = 16 * r + col;
  int src[16];
  src[0] = col;
  src[1] = ror_src<1>(col);   src[2] = ror_src<2>(col);   src[3] = ror_src<3>(col);
  src[4] = ror_src<4>(col);   src[5] = ror_src<5>(col);   src[6] = ror_src<6>(col);
  src[7] = ror_src<7>(col);   src[8] = ror_src<8>(col);   src[9] = ror_src<9>(col);
  src[10] = ror_src<10>(col); src[11] = ror_src<11>(col); src[12] = ror_src<12>(col);
  src[13] = ror_src<13>(col); src[14] = ror_src<14>(col); src[15] = ror_src<15>(col);
  // forward: layers 1 and 2 form tanh's argument already multiplied by 2 log2(e), layer 3
  // is a reduce-scatter over each quad times dt (see the wave kernel)
  float w1[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) w1[i] = kTanhScale * W1[j * 6 + i];
  const float bb1 = kTanhScale * b1[j];
  float wP[16], wQ[16], tP[16], tQ[16];   // rows of W2 (forward) and columns of it (reverse)
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    wP[s] = kTanhScale * W2[col * HID + 16 * r + src[s]];
    wQ[s] = kTanhScale * W2[(16 + col) * HID + 16 * r + src[s]];
    tP[s] = W2[(16 * r + src[s]) * HID + col];
    tQ[s] = W2[(16 * r + src[s]) * HID + 16 + col];
  }
  const float bP = (r == 0) ? kTanhScale * b2[col] : 0.0f;
  const float bQ = (r == 1) ? kTanhScale * b2[16 + col] : 0.0f;
  const float wKA = a.dt * W3[comp * HID + j];
  const float wKB = a.dt * W3[(comp ^ 2) * HID + j];
  const float wSA = a.dt * W3[(comp ^ 1) * HID + j];
  const float wSB = a.dt * W3[(comp ^ 3) * HID + j];
  const float bKA = (c32 < 4) ? a.dt * b3[comp] : 0.0f;
  // reverse: dt W3^T by output, W1^T as reduce-scatters (the state inputs over each quad, the
  // two controls over lane pairs)
  const float w30 = a.dt * W3[0 * HID + j], w31 = a.dt * W3[1 * HID + j];
  const float w32 = a.dt * W3[2 * HID + j], w33 = a.dt * W3[3 * HID + j];
  const float iKA = W1[j * 6 + comp], iKB = W1[j * 6 + (comp ^ 2)];
  const float iSA = W1[j * 6 + (comp ^ 1)], iSB = W1[j * 6 + (comp ^ 3)];
  const float uK = W1[j * 6 + 4 + (lane & 1)], uS = W1[j * 6 + 4 + ((lane & 1) ^ 1)];

  // ---- weight of this sample ---------------------------------------------------------
  const float rho = a.stats[0], eta = a.stats[1];
  const float Sk = valid ? a.S[k] : kInf;
  const float wk = (Sk < kInf && rho < kInf && eta > 0.0f) ? expf(-(Sk - rho) * a.inv_lambda) / eta : 0.0f;
  // a sample with zero weight contributes nothing; it re-runs from the zero state so
  // that no non-finite value of its own trajectory can reach the sums
  const bool live = wk > 0.0f;

  // ---- the controls of every step ----------------------------------------------------
  for (int t = c32; t < T; t += 32) {
    float e0, e1;
    draw_eps((uint32_t)t, (uint32_t)k, a.nk, e0, e1);
    myV[2 * t] = fminf(fmaxf(a.U[2 * t] + e0, a.u_lo0), a.u_hi0);
    myV[2 * t + 1] = fminf(fmaxf(a.U[2 * t + 1] + e1, a.u_lo1), a.u_hi1);
  }
  const float lo_i = (lane & 1) ? a.u_lo1 : a.u_lo0, hi_i = (lane & 1) ? a.u_hi1 : a.u_hi0;

  // ---- accumulators -----------------------------------------------------------------
  float gX[4] = {0, 0, 0, 0}, gV0 = 0.0f, gV1 = 0.0f, gb1 = 0.0f, gb2 = 0.0f;   // dW1 by input, db1, db2
  float gW3[4] = {0, 0, 0, 0}, gb3 = 0.0f;                                      // over dt
  f32x16 gW2 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  float pd = 0.0f;                            // cotangent of x_d, component comp
  float pc0 = 0.0f, pc1 = 0.0f, pc2 = 0.0f;   // cotangents of p_x, p_y, theta

  const int nseg = (T + C - 1) / C;
  const int n_ckpt = a.n_ckpt;
  // the checkpoint a segment starts from, loaded one segment ahead
  const float* cp = a.ckpt + (size_t)(valid ? k : 0) * n_ckpt * kCkptStride;
  float c_px, c_py, c_th, c_xd;
  auto load_ckpt = [&](int sgi) {
    const float* q = cp + (size_t)sgi * kCkptStride;
    c_px = q[0];
    c_py = q[1];
    c_th = q[2];
    c_xd = q[3 + comp];
  };
  load_ckpt(nseg - 1);
  for (int sgi = nseg - 1; sgi >= 0; --sgi) {
    const int t0 = sgi * C;
    const int n = min(C, T - t0);
    const float px0 = live ? c_px : 0.0f, py0 = live ? c_py : 0.0f, th0 = live ? c_th : 0.0f;
    float xh = live ? c_xd : 0.0f;
    if (sgi > 0) load_ckpt(sgi - 1);
    // ---- 1. the chain of the segment from its checkpoint ----
    myX[comp] = xh;   // every lane of a component holds and stores the same bits
    wave_lds_fence();
    float2 vc = *reinterpret_cast<const float2*>(myV + 2 * t0);
    for (int q = 0; q < n; ++q) {
      const float2 vn = *reinterpret_cast<const float2*>(myV + 2 * min(t0 + q + 1, T - 1));
      float acc = __builtin_fmaf(w1[4], vc.x, bb1);
      acc = __builtin_fmaf(w1[5], vc.y, acc);
      const float h1 = tanh_prescaled(quad_dot(acc, xh, w1[0], w1[1], w1[2], w1[3]));
      const float h2 = tanh_prescaled(mul32(bP, bQ, h1, wP, wQ));
      const float A = __builtin_fmaf(wKA, h2, bKA) + dpp_f<kQuadXor1>(wSA * h2);
      const float B = wKB * h2 + dpp_f<kQuadXor1>(wSB * h2);
      float g = A + dpp_f<kQuadXor2>(B);
      g = g + dpp_f<kRowRor + 8>(g);
      g = g + dpp_f<kRowRor + 4>(g);
      xh = xh + add_rows(g);
      myH[q * 128] = h1;
      myH[q * 128 + 64] = h2;
      myX[4 * (q + 1) + comp] = xh;
      vc = vn;
    }
    wave_lds_fence();
    // ---- 2. pose, cost gradient and drives: lane `col` takes step t0 + col ----
    {
      const bool lq = col < n;
      const int qc = min(col, n - 1);
      const float4 xs = *reinterpret_cast<const float4*>(myX + 4 * qc);
      const float4 xn = *reinterpret_cast<const float4*>(myX + 4 * qc + 4);
      const float th = th0 + row_excl(lq ? a.dt * xs.w : 0.0f);
      float sth, cth;
      sincosf(th, &sth, &cth);
      const float px = px0 + row_incl(lq ? a.dt * (cth * xs.y - sth * xs.z) : 0.0f);
      const float py = py0 + row_incl(lq ? a.dt * (sth * xs.y + cth * xs.z) : 0.0f);
      float gpx, gpy, gvx, gvy;
      state_cost_grad(a.cost, a.map, px, py, xn.y, xn.z, gpx, gpy, gvx, gvy);
      const bool lw = lq && live;
      gvx = lw ? wk * gvx : 0.0f;
      gvy = lw ? wk * gvy : 0.0f;
      const float p0 = pc0 + row_suffix(lw ? wk * gpx : 0.0f);
      const float p1 = pc1 + row_suffix(lw ? wk * gpy : 0.0f);
      const float e = lq ? a.dt * (p0 * (-sth * xs.y - cth * xs.z) + p1 * (cth * xs.y - sth * xs.z)) : 0.0f;
      const float p2 = pc2 + row_suffix_excl(e);   // before this step's own term
      // row q: D_q and the cost gradient at the state before step q (the post-step state of
      // step q - 1); row n: the cost gradient at the segment's last post-step state
      const float d1 = a.dt * (p0 * cth + p1 * sth) + dpp_upd<kRowShr + 1>(0.0f, gvx);
      const float d2 = a.dt * (p1 * cth - p0 * sth) + dpp_upd<kRowShr + 1>(0.0f, gvy);
      if (lq) {
        *reinterpret_cast<float4*>(myD + 4 * col) = make_float4(0.0f, d1, d2, a.dt * p2);
        if (col == n - 1) *reinterpret_cast<float4*>(myD + 4 * n) = make_float4(0.0f, gvx, gvy, 0.0f);
      }
      pc0 = first_of_half(p0);
      pc1 = first_of_half(p1);
      pc2 = first_of_half(p2 + e);
    }
    wave_lds_fence();
    // ---- 3. the reverse chain ----
    pd = pd + myD[4 * n + comp];
    float h1 = myH[(n - 1) * 128], h2 = myH[(n - 1) * 128 + 64];
    float xq = myX[4 * (n - 1) + comp], dr = myD[4 * (n - 1) + comp];
    vc = *reinterpret_cast<const float2*>(myV + 2 * (t0 + n - 1));
    for (int q = n - 1; q >= 0; --q) {
      // the next step's values are read one step ahead
      const int qn = max(q - 1, 0);
      const float h1n = myH[qn * 128], h2n = myH[qn * 128 + 64];
      const float xqn = myX[4 * qn + comp], drn = myD[4 * qn + comp];
      const float2 vn = *reinterpret_cast<const float2*>(myV + 2 * (t0 + qn));
      const float a2 = quad_dot(0.0f, pd, w30, w31, w32, w33) * __builtin_fmaf(-h2, h2, 1.0f);
      quad_axpy(gW3, pd, h2);
      gb3 += pd;
      gb2 += a2;
      gW2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a2, h1, gW2, 0, 0, 0);
      const float a1 = mul32(0.0f, 0.0f, a2, tP, tQ) * __builtin_fmaf(-h1, h1, 1.0f);
      const float A = iKA * a1 + dpp_f<kQuadXor1>(iSA * a1);
      const float B = iKB * a1 + dpp_f<kQuadXor1>(iSB * a1);
      float u = uK * a1 + dpp_f<kQuadXor1>(uS * a1);
      float g = A + dpp_f<kQuadXor2>(B);
      u = u + dpp_f<kQuadXor2>(u);
      g = g + dpp_f<kRowRor + 8>(g);
      u = u + dpp_f<kRowRor + 8>(u);
      g = g + dpp_f<kRowRor + 4>(g);
      u = u + dpp_f<kRowRor + 4>(u);
      pd = (pd + dr) + add_rows(g);
      u = add_rows(u);
      gb1 += a1;
      quad_axpy(gX, xq, a1);
      gV0 = __builtin_fmaf(vc.x, a1, gV0);
      gV1 = __builtin_fmaf(vc.y, a1, gV1);
      // g' = 1 strictly inside the bounds (where the clamped control is v itself), else 0
      const float vi = (lane & 1) ? vc.y : vc.x;
      myV[2 * (t0 + q) + (lane & 1)] = (vi > lo_i && vi < hi_i) ? u : 0.0f;
      h1 = h1n;
      h2 = h2n;
      xq = xqn;
      dr = drn;
      vc = vn;
    }
    wave_lds_fence();
  }

  // ---- block reduction of the parameter gradients -------------------------------------
  // Lane (r, c) of every sample holds the same parameter entries (dW2 already sums the two
  // samples of the wave), so the two samples are added across the halves and the four
  // waves through LDS.
  auto pair = [&](float v) { return v + other_half(v); };
  __syncthreads();   // the segments' LDS of every wave is no longer read
  float* red = sRed + wv * kNP32;
  const float v1[8] = {pair(gX[0]), pair(gX[1]), pair(gX[2]), pair(gX[3]), pair(gV0), pair(gV1), pair(gb1), pair(gb2)};
  const float v3[5] = {a.dt * pair(gW3[0]), a.dt * pair(gW3[1]), a.dt * pair(gW3[2]), a.dt * pair(gW3[3]),
                       a.dt * pair(gb3)};
  if (half == 0) {
#pragma unroll
    for (int i = 0; i < 6; ++i) red[j * 6 + i] = v1[i];
    red[192 + j] = v1[6];
    red[1248 + j] = v1[7];
#pragma unroll
    for (int o = 0; o < 4; ++o) red[1280 + o * HID + j] = v3[o];
    if (c32 < 4) red[1408 + c32] = v3[4];
  }
  // item v of the product's accumulator: row (a2) 8 (v / 4) + 4 half + v % 4, column (h1) c32
#pragma unroll
  for (int v = 0; v < 16; ++v) red[224 + (8 * (v >> 2) + 4 * half + (v & 3)) * HID + c32] = gW2[v];
  __syncthreads();
  const int stride = kNP32 + 2 * T;
  float* out = a.gpart + (size_t)blockIdx.x * stride;
  for (int i = threadIdx.x; i < kNP32; i += kWaveBlock)
    out[i] = ((sRed[i] + sRed[kNP32 + i]) + sRed[2 * kNP32 + i]) + sRed[3 * kNP32 + i];
  for (int o = threadIdx.x; o < 2 * T; o += kWaveBlock) {
    float acc = 0.0f;
#pragma unroll
    for (int sl = 0; sl < kWaveSlots; ++sl) acc += sV[sl * eStride + o];
    out[kNP32 + o] = acc;
  }
}

// Sum of the G per-block gradient partials [G][stride] in two passes with a fixed
// order.  Pass 1: row chunk y (rows [y G / R, (y+1) G / R)) of 64 columns per block;
// the four waves take every fourth row of the chunk and their sums are added in wave
// order.  Pass 2: the R chunk sums in chunk order, plus the control-cost term
// gamma * Delta_t / Sigma_ii of dJ/du_t.
__global__ __launch_bounds__(256) void adjoint_reduce_partial_kernel(const float* __restrict__ gpart, int G,
                                                                     int stride, int R,
                                                                     float* __restrict__ partial) {
  __shared__ float red[4][64];
  const int col = blockIdx.x * 64 + (threadIdx.x & 63);
  const int sub = threadIdx.x >> 6;
  const int y = blockIdx.y;
  const int g0 = (int)(((long long)y * G) / R), g1 = (int)(((long long)(y + 1) * G) / R);
  float acc = 0.0f;
  if (col < stride)
    for (int g = g0 + sub; g < g1; g += 4) acc += __builtin_nontemporal_load(gpart + (size_t)g * stride + col);
  red[sub][threadIdx.x & 63] = acc;
  __syncthreads();
  if (sub == 0 && col < stride) {
    const int c = threadIdx.x;
    partial[(size_t)y * stride + col] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
  }
}

__global__ __launch_bounds__(256) void adjoint_reduce_final_kernel(const float* __restrict__ partial, int R,
                                                                   int T, const float* __restrict__ stats,
                                                                   float gcs0, float gcs1, float* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int stride = kNP32 + 2 * T;
  if (i >= stride) return;
  float acc = 0.0f;
  for (int y = 0; y < R; ++y) acc += partial[(size_t)y * stride + i];
  if (i >= kNP32) {
    const int o = i - kNP32;
    acc += ((o & 1) ? gcs1 : gcs0) * stats[2 + o];
  }
  out[i] = acc;
}

}  // namespace mppi
