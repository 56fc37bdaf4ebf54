// Rollout schedule "wave", split form: the 32-lanes-per-sample layout of the wave
// kernel (two samples per wavefront, eight per block) with the block doubled to eight
// waves, so that every SIMD holds a chain wave and a cost wave of the same two samples.
// For the latency-bound regime where a launch fits the device in one block per CU
// (K up to 8 x CUs, e.g. K = 1920) and horizons up to 128 steps.
//
// Only the dynamic states x_d form a serial chain (the network never reads the pose,
// Section VI-B); the noise and the clamp of Algorithm 1 precede it and the kinematics
// and state cost of Section VI-C follow it.  So:
//
//  all waves: draw the noise of every sample and step of the block and form the
//    clamped controls g(v) (network) or the control-only terms (basis model) in LDS;
//  chain wave (waves 0..3, raised issue priority): runs the chain as the wave kernel's
//    deferred form does -- layer 1 from quad_perm DPP operands, layer 2 in row_ror DPP
//    operands of v_fmac_f32 and a v_permlane16_swap, layer 3 (times dt) as a
//    reduce-scatter, the uncompensated state hi_{t+1} = hi_t + y_t and its increment
//    y_t stored to LDS -- and publishes each finished chunk of steps with a
//    workgroup-scope release of a per-pair counter in LDS.  The chunks hold 32 steps
//    except the first, which holds the remainder of T: a chunk costs the cost wave
//    about the same time whatever its length, and with the short chunk first the cost
//    wave has finished every chunk but the last when the chain ends;
//  cost wave (waves 4..7): follows the chain one chunk behind: for chunk c it waits
//    (acquire) for the chain's counter, forms the compensated states x_d(t) = hi_t + lo_t
//    (the two-sum errors of the chain's sums, scanned across the lanes), the heading and
//    the position by 64-bit scans carried from chunk to chunk, and the state and
//    control costs of the chunk's steps (one step per lane).
//
// The cost wave waits only for the chain of its own block, which never waits, so every
// wait ends.  After both roles, all 512 threads form the block's softmin partial from the
// eight costs and the noise rows, and finish_iteration merges and updates as in every
// rollout kernel.  The costs equal the wave kernel's up to the summation order of the
// compensation terms and of the kinematic scans.
//
// Multi-step receding launch (the MULTI instances with n_steps > 1, launched
// cooperatively so that every block is resident): G rollout blocks and up to 16 merger
// blocks.  A rollout block loops over the steps, keeping the chain's network constants in
// registers and the model's parameters (for the plant step) in LDS.  At the end of step s
// each thread writes its column of the block's partial row through as a word that also
// holds the step's number (see kMergeCopies); the block draws step s + 1's noise (which
// does not depend on U) and then polls the merged row, each thread its own column, and
// runs the final stage itself -- normalisation, smoothing, update, shift, plant step -- so
// that step s + 1 starts from U and the plant state in its own LDS with no further memory
// round trip.  Every block computes the same values in the same order; block 0 alone
// writes U, the plant state, the statistics and the histories.  A merger block owns a
// sixteenth of the columns (several on a device with fewer free units): it reads these of
// all G rows (one 128-byte line each), merges them in the two levels of finish_iteration in
// the same order, and writes its part of the merged row.  A word is never overwritten while
// another block may still need it: a rollout block writes step s + 1's row after it has read step s's merged row, which
// every merger wrote after reading all of step s's rows.  Every wait is bounded: a block
// that gives up sets the status and leaves.  The results equal those of one launch per
// step bit for bit.
//
// What bounds a step (paper-shaped): the latency of the chain (~20 us), then of the
// exchange.  Replaced: a merger per group of 16 rows (each row written, waited for and
// flagged, the group row likewise, and all 15 group rows merged again by every rollout
// block): 32.0 -> 29.8 us per paper-shaped step (basis-function model 28.9 -> 26.2); with the
// cost waves' scans in 64 bits 29.4 (26.0), with the chain's loop where the compiler puts it
// 28.6 (25.8), with four steps per turn of that loop 28.0 (24.0), with layer 1 as one block
// 27.1.
#include "wave_common.hip.h"

namespace mppi {

constexpr int kSplitBlock = 512;   // 4 chain waves + 4 cost waves, 8 samples
constexpr int kSplitPairs = 4;     // sample pairs per block (one chain and one cost wave each)
// floats of the model's parameters a multi-step launch stages in LDS (the space is sized
// for the 6-32-32-4 network, 1412 floats; the basis model stages its Theta, 100)
constexpr int kSplitParams = 6 * 32 + 32 + 32 * 32 + 32 + 4 * 32 + 4;
constexpr int kSplitBasisParams = 25 * 4;

// the plant layout moves each of the network's parameters to a place of its own in the
// same space, and its 16-byte words (the W2 and W3 sections) start on 16-byte boundaries
constexpr bool plant_layout_fits() {
  bool seen[kSplitParams] = {};
  for (int i = 0; i < kSplitParams; ++i) {
    const int d = plant_layout_index(i, 32);
    if (d < 0 || d >= kSplitParams || seen[d]) return false;
    seen[d] = true;
  }
  return (7 * 32) % 4 == 0 && (8 * 32 + 32 * 32) % 4 == 0;
}
static_assert(plant_layout_fits(), "the plant layout must permute the 6-32-32-4 parameter vector");

namespace {

__device__ __forceinline__ void wait_count(unsigned* f, unsigned v) {
  while (__hip_atomic_load(f, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < v) __builtin_amdgcn_s_sleep(1);
}

__device__ __forceinline__ void publish_count(unsigned* f, unsigned v) {
  __hip_atomic_store(f, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The value v holds in the last lane of the caller's 32-lane half.
__device__ __forceinline__ float last_of_half(float v) {
  const float lo = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 31));
  const float hi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
  return (threadIdx.x & 32) ? hi : lo;
}

__device__ __forceinline__ double last_of_half(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = as_u(last_of_half(as_f((uint32_t)b))), hi = as_u(last_of_half(as_f((uint32_t)(b >> 32))));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The controls the chain reads for step t of a sample from its noise e: the clamped
// g(v) (network; v = u + eps, or eps for an exploration sample) into v2 = myV + 2t, or the
// basis model's control-only terms into b8 = myB + 8t.
template <int MODEL>
__device__ __forceinline__ void step_controls(const RolloutArgs& a, float u0, float u1, float e0, float e1, bool zm,
                                              float* v2, float* b8) {
  const float vc0 = fminf(fmaxf(zm ? e0 : u0 + e0, a.u_lo0), a.u_hi0);
  const float vc1 = fminf(fmaxf(zm ? e1 : u1 + e1, a.u_lo1), a.u_hi1);
  if constexpr (MODEL == kModelNet) {
    v2[0] = vc0;
    v2[1] = vc1;
  } else {
    // {sin u_delta, -tan u_delta, u_delta, 0} and, per output o, Theta[1][o] u_F
    // + Theta[9][o] sin u_delta + Theta[24][o] u_F^2 + Theta[25][o] u_F^3
    const float sd = sinf(vc0);
    const float ntd = -tanf(vc0);
    const float w2 = vc1 * vc1, w3 = vc1 * w2;
    float c[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      float acc = a.params[0 * 4 + o] * vc1;
      acc = __builtin_fmaf(a.params[8 * 4 + o], sd, acc);
      acc = __builtin_fmaf(a.params[23 * 4 + o], w2, acc);
      c[o] = __builtin_fmaf(a.params[24 * 4 + o], w3, acc);
    }
    *reinterpret_cast<float4*>(b8) = make_float4(sd, ntd, vc0, 0.0f);
    *reinterpret_cast<float4*>(b8 + 4) = make_float4(c[0], c[1], c[2], c[3]);
  }
}

// Every block draws the noise of all its samples and steps for iteration `iter` into sE
// (one (slot, t) pair per thread at a time, then passed to `then`).
template <class F>
__device__ __forceinline__ void draw_block_noise(const RolloutArgs& a, uint32_t iter, int kb, int T, int eStride,
                                                 float* sE, F&& then) {
  NoiseKey nk = a.nk;
  nk.iter = iter;
  for (int i = threadIdx.x; i < kWaveSlots * T; i += kSplitBlock) {
    const int slot = i / T, t = i - slot * T;
    float e0, e1;
    // the two-instruction products: two waves per SIMD wait for each draw (0.4-0.8 us of a
    // launch against the one-instruction form)
    draw_eps<false>((uint32_t)t, (uint32_t)(kb + slot), nk, e0, e1);
    sE[slot * eStride + 2 * t] = e0;
    sE[slot * eStride + 2 * t + 1] = e1;
    then(slot, t, e0, e1);
  }
}

// A word of a multi-step launch: a value and the number of its step, written through to
// the device's point of coherence / read from there.
__device__ __forceinline__ void store_word(uint64_t* p, float v, unsigned step) {
  __hip_atomic_store(p, ((uint64_t)step << 32) | as_u(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_word(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool word_ready(uint64_t w, unsigned step) { return (unsigned)(w >> 32) == step; }
__device__ __forceinline__ float word_value(uint64_t w) { return as_f((uint32_t)w); }

// The smallest value of each 16-lane row, in every lane.
__device__ __forceinline__ float row16_min(float v) {
  v = fminf(v, dpp_f<kRowRor + 8>(v));
  v = fminf(v, dpp_f<kRowRor + 4>(v));
  v = fminf(v, dpp_f<kQuadXor2>(v));
  return fminf(v, dpp_f<kQuadXor1>(v));
}

}  // namespace

// The launch's arguments, read again at each step of a multi-step launch from the kernel
// argument segment (the kernel's one explicit argument sits at its start) through a
// pointer the compiler cannot see through: otherwise every field would be held in
// scalar registers over all steps, and the surplus spilled to vector lanes and read back
// in every phase of every step.  Valid only in code inlined into the kernel: in a function
// the kernel calls, the kernel argument segment pointer reads as null.
__device__ __forceinline__ const RolloutArgs& reload_args() {
  uint64_t v = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(v));
  return *(const RolloutArgs*)(const __attribute__((address_space(4))) RolloutArgs*)v;
}

constexpr int kStatusTimeout = 6;   // a multi-step launch gave up waiting for another block

// Polls of one wait in a multi-step launch before the block gives up (0 in the arguments:
// 1 << 20: each poll waits for its load, so of the order of a second).
__device__ __forceinline__ unsigned spin_limit(const RolloutArgs& a) { return a.spin_limit ? a.spin_limit : (1u << 20); }

// Multi-step launch, one of the merger blocks (8 waves, G <= 256 rows): at every step takes the
// parts first, first + stride, ... (one where the device has a unit for each merger):
// reads the part's columns of every rollout block's row as they arrive, merges them as the
// blocks of one launch are merged -- per group of 16 rows relative to the group's minimum,
// then the group rows, every sum in row order, so that the merged row has the same bits --
// and writes the part of the merged row in kMergeCopies copies.  lds: (cw + 3) G +
// 18 * 32 floats.  Inlined into the kernel, since it reads the arguments with
// reload_args().
__device__ __forceinline__ void merge_columns_block(int n_steps, int first, int stride, float* lds) {
  constexpr int kPass = 8;   // rows per thread: 256 rows of at most 16 lanes over 512 threads
  __shared__ unsigned s_stop;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) s_stop = 0u;
  __syncthreads();
  for (int step = 0, m = first; step < n_steps;) {
    const RolloutArgs& as = reload_args();
    const int G = as.G, T2 = 2 * as.T, M = merge_parts(as.T), cw = merge_columns(as.T), LW = merge_line_words(cw);
    const int words = 2 + min(cw, T2 - m * cw);   // of the line that carry a value
    const unsigned target = as.step_base + (unsigned)step + 1u;
    const unsigned limit = spin_limit(as);
    const int vs = cw + 1;                        // columns of a row in LDS: eta, then the cw columns
    float* sRho = lds;                            // [G]
    float* sV = sRho + G;                         // [G][vs]
    float* sS = sV + G * vs;                      // [256] the rows' scales
    float* sN = sS + 256;                         // [16][18] per group: rho_g, then eta_g and the columns
    // ---- every row's line: LW / 2 lanes per row, two words a lane -------------------------
    const int sh = LW == 16 ? 3 : 4, l2 = 2 * (tid & ((1 << sh) - 1)), r0 = tid >> sh, dr = kSplitBlock >> sh;
    const uint64_t* src = as.sync + ((size_t)r0 * M + m) * LW + l2;
    const size_t ds = (size_t)dr * M * LW;
    const bool two = l2 + 1 < words;
    uint64_t w0[kPass], w1[kPass];
    bool ok = false;
    // until the wave's first rows are there, one word each; then everything at once
    for (unsigned i = 0; i < limit && !ok; ++i) {
      const bool act = r0 < G && l2 == 0;
      const uint64_t w = act ? load_word(src) : 0;
      ok = __all(!act || word_ready(w, target));
      if (!ok) __builtin_amdgcn_s_sleep(1);
    }
    if (ok) {
      ok = false;
      for (unsigned i = 0; i < limit && !ok; ++i) {
#pragma unroll
        for (int p = 0; p < kPass; ++p) {
          const bool act = r0 + p * dr < G && l2 < words;
          w0[p] = act ? load_word(src + p * ds) : 0;
          w1[p] = act && two ? load_word(src + p * ds + 1) : 0;
        }
        bool all = true;
#pragma unroll
        for (int p = 0; p < kPass; ++p) {
          const bool act = r0 + p * dr < G && l2 < words;
          all = all && (!act || (word_ready(w0[p], target) && (!two || word_ready(w1[p], target))));
        }
        ok = __all(all);
      }
    }
    if (!ok && lane == 0) {
      s_stop = 1u;
      __hip_atomic_store(as.status, kStatusTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (ok) {
#pragma unroll
      for (int p = 0; p < kPass; ++p) {
        const int row = r0 + p * dr;
        if (row < G && l2 < words) {
          if (l2 == 0) sRho[row] = word_value(w0[p]);
          else sV[row * vs + l2 - 1] = word_value(w0[p]);
          if (two) sV[row * vs + l2] = word_value(w1[p]);
        }
      }
    }
    __syncthreads();
    if (s_stop) return;
    const int ngrp = (G + 15) >> 4;               // merge_group_size(G) is 16 up to 256 rows
    // ---- group level: a 16-lane row per group, lane i its row i, then its columns i - 1, i + 15
    if (tid < 256) {
      const int g = tid >> 4, i = tid & 15;
      const int n_in = min(16, G - 16 * g);
      const bool in = i < n_in;
      const float rr = in ? sRho[16 * g + i] : kInf;
      const float ee = in ? sV[(16 * g + i) * vs] : 0.0f;
      const float rho = row16_min(rr);
      sS[tid] = ee > 0.0f ? expf(-(rr - rho) * as.inv_lambda) : 0.0f;
      wave_lds_fence();
      float acc0 = 0.0f, acc1 = 0.0f;
      const float* v = sV + 16 * g * vs;
      const bool c0 = i < words - 1, c1 = i + 16 < words - 1;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float s = sS[16 * g + q];
        acc0 = __builtin_fmaf(s, (q < n_in && c0) ? v[q * vs + i] : 0.0f, acc0);
        if (LW > 16) acc1 = __builtin_fmaf(s, (q < n_in && c1) ? v[q * vs + i + 16] : 0.0f, acc1);
      }
      float* n = sN + g * 18;
      if (i == 0) n[0] = rho;
      n[1 + i] = acc0;
      if (i == 0) n[17] = acc1;                   // column 16, there when cw = 16
    }
    __syncthreads();
    // ---- the group rows, in one wave: lane i of each row its group i, then word l of the line
    if (tid < 64) {
      const int i = lane & 15;
      const float rg = i < ngrp ? sN[i * 18] : kInf;
      const float eg = i < ngrp ? sN[i * 18 + 1] : 0.0f;
      const float rho = row16_min(rg);
      const float sg = eg > 0.0f ? expf(-(rg - rho) * as.inv_lambda) : 0.0f;
      const int l = lane & (LW - 1);              // word l: rho, eta, columns
      float acc = 0.0f;
      const float* n = sN + max(min(l, 17), 1);
#pragma unroll
      for (int g = 0; g < 16; ++g)
        acc = __builtin_fmaf(lane_value(sg, g), g < ngrp ? n[g * 18] : 0.0f, acc);
      const float out = l == 0 ? rho : acc;
      if (l < words) {
        uint64_t* dst = as.sync + ((size_t)G * M + m) * LW + l;
        for (int c = lane >> (sh + 1); c < kMergeCopies; c += 64 >> (sh + 1)) store_word(dst + (size_t)c * M * LW, out, target);
      }
    }
    m += stride;
    if (m >= M) {
      m = first;
      ++step;
    }
  }
}

template <int MODEL, bool MULTI>
__global__ __launch_bounds__(kSplitBlock) void rollout_wave_split_kernel(RolloutArgs a) {
  constexpr int HID = 32;
  constexpr bool kNet = MODEL == kModelNet;
  extern __shared__ float smem[];
  __shared__ unsigned s_abort;
  __shared__ float s_xn[kStateDim];                  // the step's plant state (multi-step: then the next step's)
  const int T = a.T;
  const int T4 = (T + 4) & ~3;
  const int eStride = (2 * T + 3) & ~3;
  const int nch = (T + 31) >> 5;                     // chunks of up to 32 steps (at most 4)
  const int r0 = T - 32 * (nch - 1);                 // steps in chunk 0 (1..32); every later chunk has 32
  const int n_steps = MULTI && a.n_steps > 1 ? a.n_steps : 1;
  float* sU = smem;                                  // [2T]
  float* sE = sU + eStride;                          // [8][2T] noise
  float* sV = sE + kWaveSlots * eStride;             // network: [8][2T] clamped controls
  float* sX = sV + (kNet ? kWaveSlots * eStride : 0);    // [8][T4][8]: hi_t, y_t
  unsigned* sFlag = reinterpret_cast<unsigned*>(sX + kWaveSlots * T4 * 8);   // [4] chain progress, [4] spare
  float* sS = reinterpret_cast<float*>(sFlag + 8);   // [8] costs
  float* sB = sS + 8;                                // basis model: [8][T][8] control terms
  float* sC = sB + (kNet ? 0 : kWaveSlots * T * 8);  // network: the chain's constants
  float* sP = sC + (kNet ? kChainWords : 0);         // basis model, multi-step: the parameters (the plant step)
  // after both roles: the block's N row (the clamped controls or the basis terms are no
  // longer read) and the merge's working row (the states are no longer read)
  float* N_lds = kNet ? sV : sB;
  float* lds = sX;
  if constexpr (MULTI) {
    if ((int)blockIdx.x >= a.G) {   // a merger block
      merge_columns_block(n_steps, (int)blockIdx.x - a.G, (int)gridDim.x - a.G, smem);
      return;
    }
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = tid >> 6;
  const bool chain = wv < kSplitPairs;
  const int pair = wv & (kSplitPairs - 1);
  const int half = lane >> 5;
  const int c32 = lane & 31;
  const int r = c32 >> 4;
  const int col = lane & 15;
  const int comp = lane & 3;
  const int slot = pair * 2 + half;
  const int kb = blockIdx.x * kWaveSlots;
  const int k = kb + slot;
  const bool valid = k < a.K;
  const bool zm = k >= a.K_imp;   // exploration sample: v = eps, delta = eps - u
  float* myE = sE + slot * eStride;
  float* myV = sV + slot * eStride;
  float* myB = sB + slot * T * 8;
  float* myX = sX + slot * T4 * 8;
  unsigned* chainCnt = sFlag + pair;

  // ---- the launch's inputs: every load is issued at once, the ones that the draws and the
  // controls need first.  The network's weights pass through LDS in the order in which a
  // chain lane holds them.  Read from global memory by the chain lanes, each load waited for
  // by itself before the draws, the chain began 4.9 us into the launch at T <= 64 and 5.4 at
  // T = 100; now 2.6 and 3.4.
  // (Absent inputs are read from the parameters' addresses, so that no load is in a branch.)
  const uint32_t* iter_p = a.iter_dev ? a.iter_dev : reinterpret_cast<const uint32_t*>(a.params);
  const uint32_t iter_in = __hip_atomic_load(iter_p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const float u_in = a.U[min(tid, 2 * T - 1)];   // 2T <= 256
  float x_in = load_through((a.x0_dev ? a.x0_dev : a.params) + min(tid, kStateDim - 1));
  ChainStage<kSplitBlock> stage;
  if constexpr (kNet) stage.load(a.params);
  if (!a.x0_dev) x_in = a.x0[min(tid, kStateDim - 1)];
  // the device counter is advanced by the final merge
  const uint32_t iter0 = a.iter_dev ? (uint32_t)__builtin_amdgcn_readfirstlane((int)iter_in) : a.nk.iter;
  if (tid < 2 * T) sU[tid] = u_in;
  if (tid < kStateDim) s_xn[tid] = x_in;
  if (tid < 2 * kSplitPairs) sFlag[tid] = 0u;
  if (tid == 0) s_abort = 0u;
  __syncthreads();
  // the noise of every sample and step, and (a single step) the controls with it
  draw_block_noise(a, iter0, kb, T, eStride, sE, [&](int sl, int t, float e0, float e1) {
    if constexpr (!MULTI)
      step_controls<MODEL>(a, sU[2 * t], sU[2 * t + 1], e0, e1, kb + sl >= a.K_imp, sV + sl * eStride + 2 * t,
                           sB + sl * T * 8 + 8 * t);
  });
  if constexpr (!MULTI)
    if (tid < kWaveSlots * 4) sX[(tid >> 2) * T4 * 8 + (tid & 3)] = s_xn[3 + (tid & 3)];
  if constexpr (kNet) stage.store(sC, a.dt);
  if constexpr (MULTI || !kNet)   // the plant step's copy of the parameters (a network in its plant layout)
    for (int i = tid; i < (kNet ? kSplitParams : kSplitBasisParams); i += kSplitBlock)
      sP[kNet ? plant_layout_index(i, HID) : i] = a.params[i];
  __syncthreads();

  // ---- the chain's constants, kept in registers over every step ----------------------
  ChainWeights cw;
  if (kNet && chain) cw.read(sC, c32);
  const auto& w1 = cw.w1;
  const auto& wP = cw.wP;
  const auto& wQ = cw.wQ;
  const float bb1 = cw.bb1, bP = cw.bP, bQ = cw.bQ;
  const float wKA = cw.wKA, wKB = cw.wKB, wSA = cw.wSA, wSB = cw.wSB, bKA = cw.bKA;
  // basis-function model: this lane's column of Theta with each normaliser folded in
  constexpr int kRaw = 21;
  constexpr int kRawIdx[kRaw] = {1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19, 20, 21, 22};
  constexpr float kRawScale[kRaw] = {0.1f, 1.0f / 1200.0f, 1.0f / (1200.0f * 1200.0f),
                                     1.0f / (1200.0f * 1200.0f * 1200.0f), 1.0f / 25.0f, 0.1f, 0.1f,
                                     1.0f / 40.0f, 1.0f / 1400.0f, 1.0f / (1400.0f * 1400.0f),
                                     1.0f / (1400.0f * 1400.0f * 1400.0f), 1.0f / 40.0f,
                                     1.0f / (40.0f * 40.0f), 1.0f / (40.0f * 40.0f * 40.0f), 1.0f / 50.0f,
                                     1.0f, 1.0f, 1.0f / 3.0f, 0.2f, 0.01f, 0.001f};
  float kc[kRaw] = {};
  if (!kNet && chain) {
#pragma unroll
    for (int i = 0; i < kRaw; ++i) kc[i] = sP[kRawIdx[i] * 4 + comp] * kRawScale[i];
  }
  if (chain) __builtin_amdgcn_s_setprio(2);

  for (int step = 0; step < n_steps; ++step) {
    const RolloutArgs& as = MULTI ? reload_args() : a;
    // this step's counter word and history entries
    const uint32_t iter = iter0 + (uint32_t)step;
    float* const u0_out = (as.u0_out && MULTI) ? as.u0_out + 2 * step : as.u0_out;
    float* const x_copy = (as.x_copy && MULTI) ? as.x_copy + kStateDim * step : as.x_copy;
    // this step's U (sU) and plant state: the launch's, then the block's own final stage's
    float x0v[kStateDim];
#pragma unroll
    for (int i = 0; i < kStateDim; ++i) x0v[i] = s_xn[i];
    if constexpr (MULTI) {
      // the controls of every sample and step; the state entry 0 of every sample
      for (int i = tid; i < kWaveSlots * T; i += kSplitBlock) {
        const int sl = i / T, t = i - sl * T;
        step_controls<MODEL>(as, sU[2 * t], sU[2 * t + 1], sE[sl * eStride + 2 * t], sE[sl * eStride + 2 * t + 1],
                             kb + sl >= as.K_imp, sV + sl * eStride + 2 * t, sB + sl * T * 8 + 8 * t);
      }
      if (tid < kWaveSlots * 4) sX[(tid >> 2) * T4 * 8 + (tid & 3)] = x0v[3 + (tid & 3)];
      __syncthreads();
    }

    if (chain) {
      // ---- chain wave ----------------------------------------------------------------
      float xh = x0v[3 + comp];   // hi_t of the lane's component
      float2 vc = make_float2(0.0f, 0.0f);
      float4 bq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      float cq = 0.0f;
      if constexpr (kNet) {
        vc = *reinterpret_cast<const float2*>(myV);
      } else {
        bq = *reinterpret_cast<const float4*>(myB);
        cq = myB[4 + comp];
      }
      // the lane's store slot: hi_{t+1} (lanes with bit 2 clear) or y_t (bit 2 set)
      float* xs = myX + ((lane & 4) ? 4 + comp : 8 + comp);
      for (int c = 0; c < nch; ++c) {
        const int t1 = r0 + 32 * c;
        // four steps per turn of the loop: between branches the compiler moves one step's loads,
        // stores and counters into the next step's chain (20 us of chain at T = 100 -> 19; with a
        // branch after each step, taken or not, 22).  Eight gain no more.
        const auto step_of = [&](int t) __attribute__((always_inline)) {
          const int tn = min(t + 1, T - 1);
          float y;   // dt * f of the lane's component
          if constexpr (MODEL == kModelBasis) {
            const float4 bq_next = *reinterpret_cast<const float4*>(myB + 8 * tn);
            const float cq_next = myB[8 * tn + 4 + comp];
            const float roll = dpp_f<0x00>(xh), vx = dpp_f<0x55>(xh);   // quad_perm:[i,i,i,i]
            const float vy = dpp_f<0xAA>(xh), om = dpp_f<0xFF>(xh);
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
            y = as.dt * ((p0 + p1) + (p2 + p3));
            bq = bq_next;
            cq = cq_next;
          } else {
            const float2 vc_next = *reinterpret_cast<const float2*>(myV + 2 * tn);
            // layer 1
            const float h1 = tanh_prescaled(chain_layer1(xh, vc, bb1, w1));
            const float h2 = tanh_prescaled(mul32(bP, bQ, h1, wP, wQ));   // layer 2
            // layer 3 (times dt)
            const float A = __builtin_fmaf(wKA, h2, bKA) + dpp_f<kQuadXor1>(wSA * h2);
            const float B = wKB * h2 + dpp_f<kQuadXor1>(wSB * h2);
            float g = A + dpp_f<kQuadXor2>(B);
            g = g + dpp_f<kRowRor + 8>(g);
            g = g + dpp_f<kRowRor + 4>(g);
            y = add_rows(g);
            vc = vc_next;
          }
          xh = xh + y;
          xs[8 * t] = (lane & 4) ? y : xh;   // y_t at entry t, hi_{t+1} at entry t + 1
        };
        int t = c > 0 ? t1 - 32 : 0;
        for (; t + 4 <= t1; t += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) step_of(t + u);
        }
        for (; t < t1; ++t) step_of(t);
        publish_count(chainCnt, (unsigned)(step * nch + c + 1));
      }
    } else {
      // ---- cost wave -----------------------------------------------------------------
      if (as.ckpt && valid && c32 < kStateDim)
        as.ckpt[(size_t)k * (T / as.ckpt_every + 1) * kCkptStride + c32] = x0v[c32];
      // carries from chunk to chunk: the compensation lo of each x_d component; the heading,
      // the position and the cost in 64 bits
      float lo[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      double th_c = x0v[2], px_c = x0v[0], py_c = x0v[1], S64 = 0.0;
      bool ok = true;
      for (int c = 0; c < nch; ++c) {
        wait_count(chainCnt, (unsigned)(step * nch + c + 1));
        const int t = (c > 0 ? r0 + 32 * (c - 1) : 0) + c32;
        const bool live = c > 0 || c32 < r0;
        const int tc = min(t, T - 1);
        const float4 hv = live ? *reinterpret_cast<const float4*>(myX + 8 * tc) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const float4 yv = live ? *reinterpret_cast<const float4*>(myX + 8 * tc + 4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        // compensated states before (xp) and after (xn) step t
        const float hq[4] = {hv.x, hv.y, hv.z, hv.w};
        const float yq[4] = {yv.x, yv.y, yv.z, yv.w};
        float xp[4], xn[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float s_, e_;
          two_sum(hq[i], yq[i], s_, e_);
          const float ex = scan32_excl(e_, c32);
          const float lt = lo[i] + ex;                 // lo_t
          xp[i] = hq[i] + lt;
          xn[i] = s_ + (lt + e_);
          lo[i] = lo[i] + last_of_half(ex + e_);       // the chunk's errors
        }
        // heading before the step: theta_0 + dt * (sum of the previous steps' theta_dot)
        const double dth = (double)(live ? as.dt * xp[3] : 0.0f);
        const double th1 = th_c + scan32_incl64(dth);   // after the step
        float sn, cs;
        sincosf((float)(th1 - dth), &sn, &cs);
        // position after the step: p_0 + dt * (sum over s <= t of R(theta_s) v_s)
        const double px = px_c + scan32_incl64((double)(live ? as.dt * (cs * xp[1] - sn * xp[2]) : 0.0f));
        const double py = py_c + scan32_incl64((double)(live ? as.dt * (sn * xp[1] + cs * xp[2]) : 0.0f));
        th_c = last_of_half(th1);
        px_c = last_of_half(px);
        py_c = last_of_half(py);
        // cost of the post-step state and the control cost of the step
        uint32_t off[4];
        float fx, fy;
        map_taps64(as.cost, px, py, off, fx, fy);
        const char* map = reinterpret_cast<const char*>(as.map);
        const float mv[4] = {*reinterpret_cast<const float*>(map + off[0]), *reinterpret_cast<const float*>(map + off[1]),
                             *reinterpret_cast<const float*>(map + off[2]), *reinterpret_cast<const float*>(map + off[3])};
        const float dec = as.decay[tc + 1];
        const float zeta = slip_angle(as.cost, xn[1], xn[2]);   // while the map values arrive
        if (live) {
          const float px1 = (float)px, py1 = (float)py;
          if (as.ckpt && ((t + 1) % as.ckpt_every) == 0 && valid) {
            float* cp = as.ckpt + ((size_t)k * (T / as.ckpt_every + 1) + (t + 1) / as.ckpt_every) * kCkptStride;
            cp[0] = px1; cp[1] = py1; cp[2] = (float)th1;
            cp[3] = xn[0]; cp[4] = xn[1]; cp[5] = xn[2]; cp[6] = xn[3];
          }
          S64 += (double)state_cost_h(as.cost, bilerp(mv, fx, fy), dec, xn[1], zeta);
          const float u0 = sU[2 * t], u1 = sU[2 * t + 1];
          const float d0 = zm ? myE[2 * t] - u0 : myE[2 * t];
          const float d1 = zm ? myE[2 * t + 1] - u1 : myE[2 * t + 1];
          S64 += (double)(as.gcs0 * (u0 * d0) + as.gcs1 * (u1 * d1));
          ok = ok && finite_f(px1) && finite_f(py1) && finite_f((float)th1) && finite_f(xn[0]) && finite_f(xn[1]) &&
               finite_f(xn[2]) && finite_f(xn[3]);
          if (as.cem_zeta > 0 && valid) {
            float* drow = as.D + (size_t)k * 2 * T;
            drow[2 * t] = d0;
            drow[2 * t + 1] = d1;
          }
        }
      }
      float S = (float)sum32_64(S64);
      if (!valid || !all32(ok) || !finite_f(S)) S = kInf;
      if (valid && c32 == 0) store_through(as.S + k, S);   // read by the host or Algorithm 3's update
      if (c32 == 0) sS[slot] = S;
    }
    __syncthreads();
    if (as.cem_zeta > 0) return;   // the cross-entropy update runs in the launch that follows

    // ---- the block's softmin partial (rho_g, eta_g, N_g) ------------------------------
    float Sk[kWaveSlots];
#pragma unroll
    for (int q = 0; q < kWaveSlots; ++q) Sk[q] = sS[q];
    float rho = Sk[0];
#pragma unroll
    for (int q = 1; q < kWaveSlots; ++q) rho = fminf(rho, Sk[q]);
    float wgt[kWaveSlots];
    float eta = 0.0f;
#pragma unroll
    for (int q = 0; q < kWaveSlots; ++q) {
      wgt[q] = rel_weight(Sk[q], rho, as.inv_lambda);
      eta += wgt[q];
    }
    const auto column = [&](int o) {   // N_g of column o
      const float u = sU[o];
      float n = 0.0f;
#pragma unroll
      for (int q = 0; q < kWaveSlots; ++q) {
        const float e = sE[q * eStride + o];
        n = __builtin_fmaf(wgt[q], (kb + q >= as.K_imp) ? e - u : e, n);
      }
      return n;
    };
    if constexpr (MULTI) {
      // ---- multi-step launch: the row goes to the merger blocks, the merged row comes back
      // and this block runs the final stage itself (2T <= 256: a column per thread) -------
      const int T2 = 2 * T, M = merge_parts(T), cw = merge_columns(T), LW = merge_line_words(cw);
      const unsigned target = as.step_base + (unsigned)step + 1u;
      uint64_t* const row = as.sync + (size_t)blockIdx.x * M * LW;
      const int m = tid / cw;
      const int word = m * LW + 2 + (tid - m * cw);
      if (tid < T2) {
        store_word(row + word, column(tid), target);
      } else if (tid >= 256 && tid < 256 + 2 * M) {
        const int h = tid - 256;
        store_word(row + (h >> 1) * LW + (h & 1), (h & 1) ? eta : rho, target);
      }
      FinalStage<kSplitBlock, MODEL, true, HID, kNet> fs;
      fs.prefetch_local(as, sU, x0v);
      __syncthreads();   // the block's noise and costs are no longer read
      // the next step's noise does not depend on its U: drawn while the merge completes
      if (step + 1 < n_steps) draw_block_noise(as, iter + 1u, kb, T, eStride, sE, [](int, int, float, float) {});
      float rho_m = 0.0f, eta_m = 0.0f;
      if (tid < 256) {   // whole waves: every thread of a column polls its own word and its line's head
        const uint64_t* src = as.sync + (size_t)(as.G + (int)(blockIdx.x % kMergeCopies)) * M * LW;
        const bool act = tid < T2;
        const unsigned limit = spin_limit(as);
        uint64_t w = 0, h0 = 0, h1 = 0;
        bool ok = false;
        for (unsigned i = 0; i < limit && !ok; ++i) {
          if (act) {
            w = load_word(src + word);
            h0 = load_word(src + m * LW);
            h1 = load_word(src + m * LW + 1);
          }
          ok = __all(!act || (word_ready(w, target) && word_ready(h0, target) && word_ready(h1, target)));
        }
        if (act) lds[tid] = word_value(w);
        rho_m = word_value(h0);
        eta_m = word_value(h1);
        if (!ok && lane == 0) {
          s_abort = 1u;
          __hip_atomic_store(as.status, kStatusTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      __syncthreads();
      if (s_abort) break;
      const bool fin = (rho_m < kInf) && (eta_m > 0.0f);
      fs.apply(as, lds, fin, fin ? 1.0f / eta_m : 0.0f, sP, rho_m, fin ? eta_m : 0.0f, iter, u0_out, x_copy,
               blockIdx.x == 0, sU, s_xn);
      __syncthreads();   // the next step's U (sU) and plant state (s_xn)
    } else {
      for (int o = tid; o < 2 * T; o += kSplitBlock) N_lds[o] = column(o);
      const StepTarget target{iter, u0_out, x_copy};
      finish_iteration<kSplitBlock, MODEL, true, HID>(as, blockIdx.x, rho, eta, N_lds, lds, as.params, &target);
    }
  }
}

template __global__ void rollout_wave_split_kernel<kModelNet, false>(RolloutArgs);
template __global__ void rollout_wave_split_kernel<kModelBasis, false>(RolloutArgs);
template __global__ void rollout_wave_split_kernel<kModelNet, true>(RolloutArgs);
template __global__ void rollout_wave_split_kernel<kModelBasis, true>(RolloutArgs);

// Dynamic LDS bytes of the split kernel for horizon T (T <= 128).
size_t wave_split_smem_bytes(int T, int model) {
  const size_t e = (size_t)((2 * T + 3) & ~3);
  const size_t T4 = (size_t)((T + 4) & ~3);
  const size_t v = model == kModelNet ? (size_t)kWaveSlots * e : 0;
  const size_t basis = model == kModelBasis ? (size_t)kWaveSlots * T * 8 : (size_t)kChainWords;
  return sizeof(float) * (e + kWaveSlots * e + v + (size_t)kWaveSlots * T4 * 8 + 8 + 8 + basis + kSplitParams);
}

}  // namespace mppi
