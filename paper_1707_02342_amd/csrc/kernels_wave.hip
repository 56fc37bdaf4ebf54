// Rollout schedule "wave": 32 lanes per sample, two samples per wavefront, for the
// latency-bound regime (a few thousand samples, e.g. K = 1920, T = 100), where one
// lane per sample would leave most of the chip idle while each lane walks a
// 100-step serial chain.
//
// Only the dynamic states x_d = (roll, v_x, v_y, theta_dot) form a serial chain: the
// network reads x_d and the control, never the pose (Section VI-B).  So the kernel
// splits each sample's work into four phases:
//
//  A. noise: each of the sample's 32 lanes draws eps for steps t = lane + 32 i
//     (Philox + Box-Muller), kept in registers and copied to LDS;
//  B. the serial x_d chain, one network evaluation per step with the 32 hidden
//     units spread one per lane:
//       layer 1: lane (row r, column c) owns neuron j = 16 r + c; the four state
//                components live in the lanes of each quad (component = lane & 3) and
//                reach every lane through quad_perm DPP operands of v_fmac_f32;
//       layer 2: each lane accumulates two outputs (c and 16 + c) over the 16 inputs
//                of its own row, reading them with row_ror DPP operands of
//                v_fmac_f32; v_permlane16_swap then exchanges the half sums between
//                the sample's two rows, so lane (r, c) ends with neuron 16 r + c;
//       layer 3: four products per lane, a reduce-scatter over each row (quad_perm
//                exchanges for bits 0 and 1 of the lane, row_ror 8 and 4 for bits 3
//                and 2) leaves output (lane & 3) in every lane, and a second
//                permlane16 swap adds the two rows;
//       update:  x_d += dt f, one component per lane, with the exact sum kept beside the FP32
//                running sum that the network reads (see kDefer below);
//     with the basis-function model (MODEL = kModelBasis) phase A also forms, for
//     each of the lane's steps, everything that depends on the control alone (sin and
//     tan of the steering and the four basis functions of the throttle and steering
//     only, times Theta) into LDS; in the chain the four state components reach every
//     lane of the quad through quad_perm DPP moves, every lane forms the 21 raw products
//     of the state (normalisers folded into its column of Theta) and lane (component c)
//     sums its own output: no cross-lane reduction and no transcendental on the chain;
//  C. kinematics and cost, lane-parallel over t: theta and the position are prefix
//     sums of their Euler increments (64-bit scans across the 32 lanes), then the cost at
//     every post-step state and the control-cost term, summed over t;
//  D. the block's softmin partial (rho_g, eta_g, N_g) for the merge kernel.
//
// The network arithmetic of phase B is exactly the FP32 network of the lane
// schedule with a different summation order.
#include "wave_common.hip.h"

namespace mppi {

// Waves per SIMD: with its 64-bit sums the compiler's own choice is one less than the bound
// here (137 and 210 registers), which costs more than the few registers that then spill:
// K = 6001, T = 150 124 -> 110 us (114 with error-free FP32 sums), K = 8192, T = 100 85 -> 82.
// With the weights staged through LDS (ChainStage) 105 and 78, K = 4096, T = 100 55 -> 51.5.
// (That is the network; for the basis-function model: up to 128 steps K = 8192, T = 64 53.7 us
// without and 44.0 with, the error-free sums took 45.8; beyond, where 34 registers would
// spill, 254 with and 250 without at K = 8192, T = 256 and 134 and 130 at K = 9000, T = 150.)
template <int HID, int NQ, int MODEL>
__global__ __launch_bounds__(kWaveBlock, NQ <= 4 ? 4 : MODEL == kModelNet ? 3 : 1) void rollout_wave_kernel(RolloutArgs a) {
  static_assert(HID == 32, "the wave schedule maps 32 hidden units onto 32 lanes");
  extern __shared__ float smem[];
  // Up to 128 steps (NQ = 4) the chain stores the uncompensated state hi_t and each
  // increment y_t, and phase C forms the compensated sums from them lane-parallel;
  // beyond (NQ = 8) the chain keeps the exact sum itself, in 64 bits (less LDS per block).
  constexpr bool kDefer = NQ <= 4;
  constexpr int kXW = kDefer ? 8 : 4;                // floats per step in sX
  constexpr bool kNetV = MODEL == kModelNet;         // the chain reads the clamped controls from sV
  const int T = a.T;
  const int T4 = (T + 4) & ~3;                       // padded row counts (16-byte aligned)
  const int eStride = (2 * T + 3) & ~3;
  float* sU = smem;                                  // [2T]
  float* sE = sU + eStride;                          // [8][2T] noise
  float* sV = sE + kWaveSlots * eStride;             // network model: [8][2T] clamped controls g(v)
  float* sX = sV + (kNetV ? kWaveSlots * eStride : 0);   // [8][T4][kXW]
  // [4][2T] wave partials of phase D (in the deferred layout they reuse sX, which phase C
  // has finished reading before the barrier that precedes them)
  float* red = kDefer ? sX : sX + kWaveSlots * T4 * kXW;
  float* scratch = kDefer ? sX + kWaveSlots * T4 * kXW : red + 4 * eStride;   // [16]
  float* sB = scratch + 16;                          // basis model: [8][T][8] control terms

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
  const bool zm = k >= a.K_imp;   // exploration sample: v = eps, delta = eps - u
  float* myE = sE + slot * eStride;
  float* myV = sV + slot * eStride;
  float4* myX = reinterpret_cast<float4*>(sX + slot * T4 * kXW);   // [T4] (NQ = 8) or [T4][2] (hi, y)

  // ---- the launch's inputs: every load is issued at once, the ones that the draws and the
  // controls need first.  (Absent inputs are read from the parameters' addresses, so that no
  // load is in a branch.  The basis-function model has no weights to wait for with it and reads
  // the counter as a scalar: K = 8500-10500, T <= 20, where a fifth block per compute unit
  // starts late, 31.8 -> 29.1 us at K = 9000, T = 10.)
  constexpr bool kNet = MODEL == kModelNet;
  constexpr int kURegs = (64 * NQ + kWaveBlock - 1) / kWaveBlock;   // 2T <= 64 NQ
  const int tid = threadIdx.x;
  const uint32_t* iter_p = a.iter_dev ? a.iter_dev : reinterpret_cast<const uint32_t*>(a.params);
  const uint32_t iter_in = kNet ? __hip_atomic_load(iter_p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *iter_p;
  float u_in[kURegs];
#pragma unroll
  for (int i = 0; i < kURegs; ++i) u_in[i] = a.U[min(tid + i * kWaveBlock, 2 * T - 1)];
  ChainStage<kWaveBlock> stage;
  if constexpr (kNet) stage.load(a.params);
  // the device counter is advanced by the final merge
  if (a.iter_dev) a.nk.iter = (uint32_t)__builtin_amdgcn_readfirstlane((int)iter_in);
#pragma unroll
  for (int i = 0; i < kURegs; ++i)
    if (tid + i * kWaveBlock < 2 * T) sU[tid + i * kWaveBlock] = u_in[i];
  __syncthreads();

  // basis-function model: this lane's column of Theta with each basis function's
  // normaliser folded in (the chain multiplies raw products such as sin(u_delta) tan(alpha_f))
  constexpr int kRaw = 21;
  constexpr int kRawIdx[kRaw] = {1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19, 20, 21, 22};
  constexpr float kRawScale[kRaw] = {0.1f, 1.0f / 1200.0f, 1.0f / (1200.0f * 1200.0f),
                                     1.0f / (1200.0f * 1200.0f * 1200.0f), 1.0f / 25.0f, 0.1f, 0.1f,
                                     1.0f / 40.0f, 1.0f / 1400.0f, 1.0f / (1400.0f * 1400.0f),
                                     1.0f / (1400.0f * 1400.0f * 1400.0f), 1.0f / 40.0f,
                                     1.0f / (40.0f * 40.0f), 1.0f / (40.0f * 40.0f * 40.0f), 1.0f / 50.0f,
                                     1.0f, 1.0f, 1.0f / 3.0f, 0.2f, 0.01f, 0.001f};
  float kc[kRaw];
#pragma unroll
  for (int i = 0; i < kRaw; ++i) kc[i] = kNet ? 0.0f : a.params[kRawIdx[i] * 4 + comp] * kRawScale[i];

  float x0v[kStateDim];
#pragma unroll
  for (int i = 0; i < kStateDim; ++i) x0v[i] = a.x0_dev ? a.x0_dev[i] : a.x0[i];

  // ---- A: noise ---------------------------------------------------------------------
  // (draws for steps past T use a clamped step index and are discarded; keeping the
  // chunks free of branches lets the independent draws interleave)
  float ea[NQ], eb[NQ];
  const int NT = (T + 31) >> 5;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    ea[i] = 0.0f;
    eb[i] = 0.0f;
    if (i < NT) {
      const int t = min(32 * i + c32, T - 1);
      draw_eps((uint32_t)t, (uint32_t)k, a.nk, ea[i], eb[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int t = 32 * i + c32;
    if (i < NT && t < T) {
      myE[2 * t] = ea[i];
      myE[2 * t + 1] = eb[i];
      if constexpr (kNetV) {
        // g(v) of the step (v = u + eps, or eps for an exploration sample), for the chain
        const float u0 = sU[2 * t], u1 = sU[2 * t + 1];
        myV[2 * t] = fminf(fmaxf(zm ? ea[i] : u0 + ea[i], a.u_lo0), a.u_hi0);
        myV[2 * t + 1] = fminf(fmaxf(zm ? eb[i] : u1 + eb[i], a.u_lo1), a.u_hi1);
      }
    }
  }
  if constexpr (MODEL == kModelBasis) {
    // the terms of each of the lane's steps that depend on the control alone:
    // {sin u_delta, -tan u_delta, u_delta, 0} and, per output o, Theta[1][o] u_F
    // + Theta[9][o] sin u_delta + Theta[24][o] u_F^2 + Theta[25][o] u_F^3
    float* myB = sB + slot * T * 8;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int t = 32 * i + c32;
      if (i < NT && t < T) {
        const float u0 = sU[2 * t], u1 = sU[2 * t + 1];
        const float vc0 = fminf(fmaxf(zm ? ea[i] : u0 + ea[i], a.u_lo0), a.u_hi0);
        const float vc1 = fminf(fmaxf(zm ? eb[i] : u1 + eb[i], a.u_lo1), a.u_hi1);
        const float sd = sinf(vc0);
        const float ntd = -tanf(vc0);
        const float u2 = vc1 * vc1, u3 = vc1 * u2;
        float c[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          float acc = a.params[0 * 4 + o] * vc1;
          acc = __builtin_fmaf(a.params[8 * 4 + o], sd, acc);
          acc = __builtin_fmaf(a.params[23 * 4 + o], u2, acc);
          c[o] = __builtin_fmaf(a.params[24 * 4 + o], u3, acc);
        }
        *reinterpret_cast<float4*>(myB + 8 * t) = make_float4(sd, ntd, vc0, 0.0f);
        *reinterpret_cast<float4*>(myB + 8 * t + 4) = make_float4(c[0], c[1], c[2], c[3]);
      }
    }
  }
  // the network's constants, staged where the states go
  ChainWeights cw;
  if constexpr (kNet) {
    stage.store(sX, a.dt);
    __syncthreads();
    cw.read(sX, c32);
    __syncthreads();
  }
  const auto& w1 = cw.w1;
  const auto& wP = cw.wP;
  const auto& wQ = cw.wQ;
  const float bb1 = cw.bb1, bP = cw.bP, bQ = cw.bQ;
  const float wKA = cw.wKA, wKB = cw.wKB, wSA = cw.wSA, wSB = cw.wSB, bKA = cw.bKA;
  float xh = x0v[3 + comp];           // the FP32 running sum hi_t that the network reads
  double xd = xh;                     // NQ = 8: the state's exact sum, kept by the chain
  if (c32 < 4) sX[slot * T4 * kXW + c32] = x0v[3 + c32];
  if (a.ckpt && valid && c32 < kStateDim)
    a.ckpt[(size_t)k * (T / a.ckpt_every + 1) * kCkptStride + c32] = x0v[c32];
  __syncthreads();

  // ---- B: serial chain of the dynamic states ---------------------------------------
  {
  float2 vc = make_float2(0.0f, 0.0f);
  if constexpr (kNetV) vc = *reinterpret_cast<const float2*>(myV);
  // the lane's store slot in sX: hi_{t+1} (lanes with bit 2 clear) or y_t (bit 2 set)
  const int xs_off = slot * T4 * kXW + ((lane & 4) ? 4 + comp : kXW + comp);
  // basis model: this step's control terms, also read one step ahead
  const float* myB = sB + slot * T * 8;
  float4 bq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float cq = 0.0f;
  if constexpr (MODEL == kModelBasis) {
    bq = *reinterpret_cast<const float4*>(myB);
    cq = myB[4 + comp];
  }
  for (int t = 0; t < T; ++t) {
    // next step's control is read one step ahead (LDS latency off the chain)
    const int tn = min(t + 1, T - 1);
    float2 vc_next = vc;
    if constexpr (kNetV) vc_next = *reinterpret_cast<const float2*>(myV + 2 * tn);
    float y;   // dt * f of the lane's component
    const float xcur = xh;
    if constexpr (MODEL == kModelBasis) {
      // bq = {sin u_delta, -tan u_delta, u_delta, 0}, cq = the control-only terms
      const float4 bq_next = *reinterpret_cast<const float4*>(myB + 8 * tn);
      const float cq_next = myB[8 * tn + 4 + comp];
      const float roll = dpp_f<0x00>(xcur), vx = dpp_f<0x55>(xcur);   // quad_perm:[i,i,i,i]
      const float vy = dpp_f<0xAA>(xcur), om = dpp_f<0xFF>(xcur);
      // tyre tangents: tan(arctan z) = z above v_x = 0.1, the steering alone below
      const bool mv = vx > 0.1f;
      const float rv = __builtin_amdgcn_rcpf(vx);
      const float q = vy * rv, w = om * rv;
      const float tf = mv ? __builtin_fmaf(0.45f, w, q) - bq.z : bq.y;
      const float tr = mv ? __builtin_fmaf(-0.35f, w, q) : 0.0f;
      const float qq = mv ? q : 0.0f;
      const float sf = bq.x * tf, tf2 = tf * tf, tr2 = tr * tr;
      const float atf = fabsf(tf), atr = fabsf(tr);
      const float rx = roll * vx, vx2 = vx * vx;
      const float raw[kRaw] = {vx, sf, sf * atf, sf * tf2, om * vy, om, vy, qq, tf, tf * atf, tf * tf2,
                               tr, tr * atr, tr * tr2, om * vx, roll, roll * om, rx, rx * om, vx2, vx * vx2};
      float p0 = cq, p1 = 0.0f, p2 = 0.0f, p3 = 0.0f;
#pragma unroll
      for (int i = 0; i < kRaw; i += 4) {
        p0 = __builtin_fmaf(kc[i], raw[i], p0);
        if (i + 1 < kRaw) p1 = __builtin_fmaf(kc[i + 1], raw[i + 1], p1);
        if (i + 2 < kRaw) p2 = __builtin_fmaf(kc[i + 2], raw[i + 2], p2);
        if (i + 3 < kRaw) p3 = __builtin_fmaf(kc[i + 3], raw[i + 3], p3);
      }
      y = a.dt * ((p0 + p1) + (p2 + p3));
      bq = bq_next;
      cq = cq_next;
    } else {
      // layer 1
      const float h1 = tanh_prescaled(chain_layer1(xcur, vc, bb1, w1));
      const float h2 = tanh_prescaled(mul32(bP, bQ, h1, wP, wQ));   // layer 2
      // layer 3 (times dt): reduce-scatter of the four outputs over each quad, then the
      // quads of the row and the two rows
      const float A = __builtin_fmaf(wKA, h2, bKA) + dpp_f<kQuadXor1>(wSA * h2);   // output oA, lanes L, L^1
      const float B = wKB * h2 + dpp_f<kQuadXor1>(wSB * h2);                         // output oB, lanes L, L^1
      float g = A + dpp_f<kQuadXor2>(B);                                             // output oA, the quad
      g = g + dpp_f<kRowRor + 8>(g);
      g = g + dpp_f<kRowRor + 4>(g);
      y = add_rows(g);
    }
    // every lane of a component holds the same bits (y and the update are formed alike
    // in all of them), so all lanes store: no branch in the step loop
    xh = xh + y;
    if constexpr (kDefer) {
      sX[xs_off + t * kXW] = (lane & 4) ? y : xh;   // y_t at entry t, hi_{t+1} at entry t + 1
    } else {
      xd = xd + (double)y;
      sX[slot * T4 * kXW + (t + 1) * kXW + comp] = (float)xd;
    }
    vc = vc_next;
  }
  }
  __syncthreads();

  // ---- C: kinematics and cost, parallel over t ---------------------------------------
  // Lane c owns the contiguous steps [c*npl, (c+1)*npl).  theta(t) = theta_0 + dt sum_{s<t}
  // theta_dot(s) and p(t+1) = p_0 + dt sum_{s<=t} R(theta(s)) v(s) are formed as
  // 64-bit lane sums plus 64-bit scans across the 32 lanes.  The positions of all the lane's steps are formed first, then every map and decay load
  // is issued before the first is used (one memory round trip), then the costs.
  const int npl = NT;
  const int tb = c32 * npl;
  // x_d at the lane's steps, xv[q] = x_d(tb + q) for q = 0..NQ (the state before step
  // tb + q and after step tb + q - 1).  Deferred layout: x_d(t) = hi_t + lo_t, where lo_t
  // sums the rounding errors err_s = (hi_s + y_s) - fl(hi_s + y_s), s < t (error-free
  // two-sum), in the lane and then by a scan across the lanes; the chain's own sums
  // hi_{s+1} = fl(hi_s + y_s) are recomputed here.
  float4 xv[NQ + 1];
  if constexpr (kDefer) {
    float4 hv[NQ], yv[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int t = tb + q;
      const bool live = q < npl && t < T;
      hv[q] = live ? myX[2 * t] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      yv[q] = live ? myX[2 * t + 1] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    float hs[NQ][4], lq[NQ][4];
    float lsum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float hq[4] = {hv[q].x, hv[q].y, hv[q].z, hv[q].w};
      const float yq[4] = {yv[q].x, yv[q].y, yv[q].z, yv[q].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float e_;
        two_sum(hq[c], yq[c], hs[q][c], e_);
        lsum[c] = lsum[c] + e_;
        lq[q][c] = lsum[c];
      }
    }
    float pre[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) pre[c] = scan32_excl(lsum[c], c32);
    xv[0] = make_float4(hv[0].x + pre[0], hv[0].y + pre[1], hv[0].z + pre[2], hv[0].w + pre[3]);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      xv[q + 1] = make_float4(hs[q][0] + (pre[0] + lq[q][0]), hs[q][1] + (pre[1] + lq[q][1]),
                              hs[q][2] + (pre[2] + lq[q][2]), hs[q][3] + (pre[3] + lq[q][3]));
  }
  auto xpre = [&](int q) -> float4 {   // x_d before step tb + q
    if constexpr (kDefer) return xv[q]; else return myX[tb + q];
  };
  auto xpost = [&](int q) -> float4 {  // x_d after step tb + q
    if constexpr (kDefer) return xv[q + 1]; else return myX[tb + q + 1];
  };
  // theta before each of the lane's steps and after the last: sums and scans in 64 bits
  // (dead slots add zero and keep the last live pose)
  double th[NQ + 1];
  th[0] = 0.0;
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    th[q + 1] = th[q] + (double)((q < npl && tb + q < T) ? a.dt * xpre(q).w : 0.0f);
  {
    const double base = x0v[2] + (scan32_incl64(th[NQ]) - th[NQ]);
#pragma unroll
    for (int q = 0; q <= NQ; ++q) th[q] = base + th[q];
  }
  double px[NQ], py[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double dx = 0.0, dy = 0.0;
    if (q < npl && tb + q < T) {
      const float4 xs = xpre(q);
      float sn, cs;
      sincosf((float)th[q], &sn, &cs);
      dx = (double)(a.dt * (cs * xs.y - sn * xs.z));
      dy = (double)(a.dt * (sn * xs.y + cs * xs.z));
    }
    px[q] = q == 0 ? dx : px[q - 1] + dx;
    py[q] = q == 0 ? dy : py[q - 1] + dy;
  }
  {
    const double bx = x0v[0] + (scan32_incl64(px[NQ - 1]) - px[NQ - 1]);
    const double by = x0v[1] + (scan32_incl64(py[NQ - 1]) - py[NQ - 1]);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      px[q] = bx + px[q];
      py[q] = by + py[q];
    }
  }
  // all gathers at once (indices are clamped to the map, steps to [1, T])
  float mv[NQ][4], fxv[NQ], fyv[NQ], dec[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    uint32_t off[4];
    map_taps64(a.cost, px[q], py[q], off, fxv[q], fyv[q]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      mv[q][i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.map) + off[i]);
    dec[q] = a.decay[min(tb + q, T - 1) + 1];
  }
  double S64 = 0.0;
  bool ok = true;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int t = tb + q;
    if (q < npl && t < T) {
      const float4 xn = xpost(q);
      const float px1 = (float)px[q], py1 = (float)py[q], th1 = (float)th[q + 1];
      if (a.ckpt && ((t + 1) % a.ckpt_every) == 0 && valid) {
        float* cp = a.ckpt + ((size_t)k * (T / a.ckpt_every + 1) + (t + 1) / a.ckpt_every) * kCkptStride;
        cp[0] = px1; cp[1] = py1; cp[2] = th1;
        cp[3] = xn.x; cp[4] = xn.y; cp[5] = xn.z; cp[6] = xn.w;
      }
      const float zeta = slip_angle(a.cost, xn.y, xn.z);
      S64 += (double)state_cost_h(a.cost, bilerp(mv[q], fxv[q], fyv[q]), dec[q], xn.y, zeta);
      const float u0 = sU[2 * t], u1 = sU[2 * t + 1];
      const float d0 = zm ? myE[2 * t] - u0 : myE[2 * t];
      const float d1 = zm ? myE[2 * t + 1] - u1 : myE[2 * t + 1];
      S64 += (double)(a.gcs0 * (u0 * d0) + a.gcs1 * (u1 * d1));
      ok = ok && finite_f(px1) && finite_f(py1) && finite_f(th1) && finite_f(xn.x) &&
           finite_f(xn.y) && finite_f(xn.z) && finite_f(xn.w);
    }
  }
  float S = (float)sum32_64(S64);
  const bool okc = all32(ok);
  if (!valid || !okc || !finite_f(S)) S = kInf;
  if (valid && c32 == 0) store_through(a.S + k, S);   // read by the host or Algorithm 3's update

  if (a.cem_zeta > 0) {
    // Algorithm 3: the sample's delta row, for the elite average
    if (valid) {
      float* drow = a.D + (size_t)k * 2 * T;
      for (int o = c32; o < 2 * T; o += 32) drow[o] = zm ? myE[o] - sU[o] : myE[o];
    }
    return;   // the cross-entropy update runs in the launch that follows
  }

  // ---- D: softmin partial of the block's samples ------------------------------------
  const float wmin = fminf(S, other_half(S));
  if (lane == 0) scratch[wv] = wmin;
  __syncthreads();
  const float rho = fminf(fminf(scratch[0], scratch[1]), fminf(scratch[2], scratch[3]));
  const float e = rel_weight(S, rho, a.inv_lambda);
  const float epair = e + other_half(e);
  if (lane == 0) scratch[4 + wv] = epair;
  const int eStrideRed = eStride;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    if (i < NT) {
      const int t = 32 * i + c32;
      const int tc = min(t, T - 1);
      const float d0 = zm ? ea[i] - sU[2 * tc] : ea[i];
      const float d1 = zm ? eb[i] - sU[2 * tc + 1] : eb[i];
      const float n0 = e * d0, n1 = e * d1;
      const float p0 = n0 + other_half(n0);
      const float p1 = n1 + other_half(n1);
      if (half == 0 && t < T) {
        red[wv * eStrideRed + 2 * t] = p0;
        red[wv * eStrideRed + 2 * t + 1] = p1;
      }
    }
  }
  __syncthreads();
  float* N_lds = sE;   // the noise rows are no longer read
  for (int o = threadIdx.x; o < 2 * T; o += kWaveBlock)
    N_lds[o] = ((red[o] + red[eStrideRed + o]) + red[2 * eStrideRed + o]) + red[3 * eStrideRed + o];
  const float eta = ((scratch[4] + scratch[5]) + scratch[6]) + scratch[7];
  finish_iteration<kWaveBlock, MODEL, true, HID>(a, blockIdx.x, rho, eta, N_lds, red);
}

template __global__ void rollout_wave_kernel<32, 4, kModelNet>(RolloutArgs);
template __global__ void rollout_wave_kernel<32, 8, kModelNet>(RolloutArgs);
template __global__ void rollout_wave_kernel<32, 4, kModelBasis>(RolloutArgs);
template __global__ void rollout_wave_kernel<32, 8, kModelBasis>(RolloutArgs);

// Dynamic LDS bytes the wave kernel needs for horizon T.
// (The layout of the kernel's LDS: the deferred-compensation layout up to T = 128,
// where launch_wave picks NQ = 4.)
size_t wave_smem_bytes(int T, int model) {
  const size_t e = (size_t)((2 * T + 3) & ~3);
  const size_t T4 = (size_t)((T + 4) & ~3);
  const bool defer = T <= 128;
  const size_t v = model == kModelNet ? (size_t)kWaveSlots * e : 0;
  const size_t x = (size_t)kWaveSlots * T4 * (defer ? 8 : 4);
  const size_t red = defer ? 0 : 4 * e;
  const size_t basis = model == kModelBasis ? (size_t)kWaveSlots * T * 8 : 0;
  const size_t behind = x + red + 16 + basis;   // the chain's constants pass through here
  return sizeof(float) * (e + kWaveSlots * e + v + (behind > kChainWords ? behind : (size_t)kChainWords));
}

}  // namespace mppi
