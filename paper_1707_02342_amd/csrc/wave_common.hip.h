// Cross-lane building blocks of the 32-lanes-per-sample layout (two samples per
// wavefront; lane = 32 * sample + 16 * row + column).  Shared by the forward
// ("wave") rollout and the adjoint rollout.
#pragma once

#include "kernels_common.hip.h"

namespace mppi {

constexpr int kWaveBlock = 256;
constexpr int kWaveSlots = 8;        // samples per block

__device__ __forceinline__ float as_f(uint32_t v) { return __builtin_bit_cast(float, v); }
__device__ __forceinline__ uint32_t as_u(float v) { return __builtin_bit_cast(uint32_t, v); }

// acc += src[dpp lane] * w, as one v_fmac_f32 with a DPP source operand.  The first
// use after src was written is preceded by two wait states (VALU write -> DPP read).
#define FMAC_DPP(acc, src, w, ctrl) \
  asm volatile("v_fmac_f32_dpp %0, %1, %2 " ctrl " row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(src), "v"(w))
#define FMAC_DPP_FIRST(acc, src, w, ctrl)                                                        \
  asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 " ctrl " row_mask:0xf bank_mask:0xf" : "+v"(acc) \
      : "v"(src), "v"(w))

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return as_f((uint32_t)__builtin_amdgcn_mov_dpp((int)as_u(v), CTRL, 0xf, 0xf, true));
}

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}

constexpr int kRowRor = 0x120;        // row_ror:s = 0x120 + s
constexpr int kQuadXor1 = 0xB1;       // quad_perm:[1,0,3,2]
constexpr int kQuadXor2 = 0x4E;       // quad_perm:[2,3,0,1]

// Column (0..15) whose value lane `col` reads through row_ror:S.
template <int S>
__device__ __forceinline__ int ror_src(int col) {
  return dpp_i<kRowRor + S>(col);
}

// Exchange between the two 16-lane rows of each 32-lane half: returns the pair
// (new first operand, new second operand) of v_permlane16_swap.
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  auto r = __builtin_amdgcn_permlane16_swap(as_u(a), as_u(b), false, false);
  a = as_f(r[0]);
  b = as_f(r[1]);
}

// Sum of v over the sample's two rows, the same bits in both rows.
__device__ __forceinline__ float add_rows(float v) {
  float x = v, y = v;
  swap_rows(x, y);
  return x + y;
}

constexpr int kRowShr = 0x110;        // row_shr:s = 0x110 + s
constexpr int kRowBcast15 = 0x142;    // lane 15 of each row to every lane of the next row

// DPP move with a row mask: lanes of the rows in ROWMASK whose source lane exists take
// v from it; every other lane keeps `old`.
template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ float dpp_upd(float old, float v) {
  return as_f((uint32_t)__builtin_amdgcn_update_dpp((int)as_u(old), (int)as_u(v), CTRL, ROWMASK, 0xF, false));
}

// The same for a 64-bit value, 0 in the lanes without a source.
template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ double dpp_zero64(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = as_u(dpp_upd<CTRL, ROWMASK>(0.0f, as_f((uint32_t)b)));
  const uint32_t hi = as_u(dpp_upd<CTRL, ROWMASK>(0.0f, as_f((uint32_t)(b >> 32))));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Inclusive sums of v over the 32 lanes of a half-wave in 64 bits: within each 16-lane row
// (shifts 1, 2, 4, 8), then the first row's total added to the second row.  An FP64 add
// takes as long as one FP32 instruction; the error-free FP32 pairs that these sums
// replace took eight per step.
__device__ __forceinline__ double scan32_incl64(double v) {
  v = v + dpp_zero64<kRowShr + 1>(v);
  v = v + dpp_zero64<kRowShr + 2>(v);
  v = v + dpp_zero64<kRowShr + 4>(v);
  v = v + dpp_zero64<kRowShr + 8>(v);
  return v + dpp_zero64<kRowBcast15, 0xA>(v);
}

// Exclusive scan of v over the 32 lanes of a half-wave (lane 0 of each half gets 0), in
// DPP moves: shift up one lane, scan within each 16-lane row, add the first row's total
// to the second row.
__device__ __forceinline__ float scan32_excl(float v, int c32) {
  const bool col0 = (c32 & 15) == 0;
  const float sh = dpp_upd<kRowShr + 1>(0.0f, v);
  const float bh = dpp_upd<kRowBcast15, 0xA>(0.0f, v);
  v = col0 ? bh : sh;
  v = v + dpp_upd<kRowShr + 1, 0xF>(0.0f, v);
  v = v + dpp_upd<kRowShr + 2, 0xF>(0.0f, v);
  v = v + dpp_upd<kRowShr + 4, 0xF>(0.0f, v);
  v = v + dpp_upd<kRowShr + 8, 0xF>(0.0f, v);
  v = v + dpp_upd<kRowBcast15, 0xA>(0.0f, v);
  return v;
}

// Sum of v over the 32 lanes, the same bits in every lane: butterflies within each row,
// then the two rows.
__device__ __forceinline__ double sum32_64(double v) {
  v = v + dpp_zero64<kRowRor + 8>(v);
  v = v + dpp_zero64<kRowRor + 4>(v);
  v = v + dpp_zero64<kQuadXor2>(v);
  v = v + dpp_zero64<kQuadXor1>(v);
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  float xl = as_f((uint32_t)b), yl = xl, xh = as_f((uint32_t)(b >> 32)), yh = xh;
  swap_rows(xl, yl);
  swap_rows(xh, yh);
  return __builtin_bit_cast(double, ((uint64_t)as_u(xh) << 32) | as_u(xl)) +
         __builtin_bit_cast(double, ((uint64_t)as_u(yh) << 32) | as_u(yl));
}

// The value of v in the lane 32 apart (the other half of the wave).
__device__ __forceinline__ float other_half(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(as_u(v), as_u(v), false, false);
  // r[0] holds the first half's values in both halves, r[1] the second half's
  return as_f((threadIdx.x & 32) ? r[0] : r[1]);
}

// Whether p holds in every lane of the calling lane's 32-lane half.
__device__ __forceinline__ bool all32(bool p) {
  const unsigned long long m = __ballot(p);
  const unsigned half = (threadIdx.x & 32) ? (unsigned)(m >> 32) : (unsigned)m;
  return half == 0xFFFFFFFFu;
}

// LDS that only one wave writes and reads: the order of its accesses for the compiler.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Layer 1 of the chain: b + W1 (x_d, g(v)) for the lane's hidden unit, x the lane's component
// of x_d.  One block, the controls' two products first: x is its input, so they stand between
// the instruction that wrote x and the first DPP read of it, which needs two wait states.
// (The compiler does not look for that inside a block, and products formed outside depend on
// the controls alone: it moved them above the write.  A paper-shaped multi-step step takes
// 27.1 us so, 28.0 with them outside; the wave kernel the same either way.)
__device__ __forceinline__ float chain_layer1(float x, float2 v, float b, const float (&w)[6]) {
  float acc;
  asm volatile(
      "v_fma_f32 %0, %6, %8, %10\n\t"
      "v_fmac_f32 %0, %7, %9\n\t"
      "v_fmac_f32_dpp %0, %1, %2 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %1, %3 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %1, %4 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %1, %5 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf"
      : "=&v"(acc)
      : "v"(x), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(v.x), "v"(v.y), "v"(b));
  return acc;
}

// One row's part of a 32 x 32 product: P += sum_s wP[s] h[ror s], Q likewise (the row's
// 16 values of h through row_ror), then the sums of the sample's two rows: lane (r, c)
// returns output 16 r + c.  Four interleaved accumulators, so that none is read by the
// instruction right after the one that wrote it, and rotations 2..15 in one block (no wait
// states inserted between them): the DPP source h was written before the four instructions
// forming P, Q, P2 and Q2, the block's inputs, more than the two wait states a DPP read needs.
__device__ __forceinline__ float mul32(float P, float Q, float h, const float (&wP)[16], const float (&wQ)[16]) {
  P = __builtin_fmaf(wP[0], h, P);
  Q = __builtin_fmaf(wQ[0], h, Q);
  float P2 = wP[1] * dpp_f<kRowRor + 1>(h);
  float Q2 = wQ[1] * dpp_f<kRowRor + 1>(h);
  asm volatile(
      "v_fmac_f32_dpp %0, %4, %5 row_ror:2 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %6 row_ror:2 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %7 row_ror:3 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %8 row_ror:3 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %9 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %10 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %11 row_ror:5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %12 row_ror:5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %13 row_ror:6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %14 row_ror:6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %15 row_ror:7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %16 row_ror:7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %17 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %18 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %19 row_ror:9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %20 row_ror:9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %21 row_ror:10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %22 row_ror:10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %23 row_ror:11 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %24 row_ror:11 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %25 row_ror:12 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %26 row_ror:12 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %27 row_ror:13 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %28 row_ror:13 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %0, %4, %29 row_ror:14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %1, %4, %30 row_ror:14 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %2, %4, %31 row_ror:15 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f32_dpp %3, %4, %32 row_ror:15 row_mask:0xf bank_mask:0xf"
      : "+v"(P), "+v"(Q), "+v"(P2), "+v"(Q2)
      : "v"(h), "v"(wP[2]), "v"(wQ[2]), "v"(wP[3]), "v"(wQ[3]), "v"(wP[4]), "v"(wQ[4]), "v"(wP[5]), "v"(wQ[5]),
        "v"(wP[6]), "v"(wQ[6]), "v"(wP[7]), "v"(wQ[7]), "v"(wP[8]), "v"(wQ[8]), "v"(wP[9]), "v"(wQ[9]),
        "v"(wP[10]), "v"(wQ[10]), "v"(wP[11]), "v"(wQ[11]), "v"(wP[12]), "v"(wQ[12]), "v"(wP[13]), "v"(wQ[13]),
        "v"(wP[14]), "v"(wQ[14]), "v"(wP[15]), "v"(wQ[15]));
  P = P + P2;
  Q = Q + Q2;
  swap_rows(P, Q);
  return P + Q;
}

// The network constants of the chain (the 6-32-32-4 network on 32 lanes per sample, see the
// wave kernel's phase B), staged through LDS in the order in which a chain lane holds them:
// lane 16 r + col, kChainRow words each (kChainRow / 4 is odd: the lanes' 16-byte reads fall
// on different banks), scaled: wP[16], wQ[16], w1[6], bb1, the layer-2 bias, wKA, wSA, wKB,
// wSB, bKA.  Each lane gathering its 45 weights from global memory took 3 us of a launch.
constexpr int kChainRow = 52;
constexpr int kChainW1 = 32, kChainB1 = 38, kChainB2 = 39, kChainW3 = 40, kChainB3 = 44;
constexpr int kChainWords = 32 * kChainRow;

// One block's part in it, NT threads: load() issues the loads, store() writes to LDS.
template <int NT>
struct ChainStage {
  static constexpr int H = 32, kW2 = H * H / NT;
  static constexpr int kRest = 6 * H + H + H + 4 * H + 4;   // W1, b1 and, behind W2, b2, W3, b3
  static constexpr int kRestRegs = (kRest + NT - 1) / NT;
  static_assert(NT % H == 0 && H * H % NT == 0, "");
  float w2[kW2], rest[kRestRegs];

  __device__ __forceinline__ void load(const float* params) {
#pragma unroll
    for (int i = 0; i < kW2; ++i) w2[i] = params[7 * H + threadIdx.x + i * NT];
#pragma unroll
    for (int i = 0; i < kRestRegs; ++i) {
      const int e = threadIdx.x + i * NT;
      rest[i] = params[e < 7 * H ? e : min(e, kRest - 1) + H * H];
    }
  }

  __device__ __forceinline__ void store(float* sC, float dt) const {
    const int tid = threadIdx.x;
    // W2[n][16 r + s] is lane 16 r + (n & 15)'s weight of the rotation by (n - s) & 15;
    // layers 1 and 2 form tanh's argument already multiplied by 2 log2(e)
#pragma unroll
    for (int i = 0; i < kW2; ++i) {
      const int n = (tid + i * NT) >> 5;
      sC[((tid & 16) + (n & 15)) * kChainRow + (n & 16) + ((n - tid) & 15)] = kTanhScale * w2[i];
    }
    constexpr int oB2 = 7 * H, oW3 = oB2 + H, oB3 = oW3 + 4 * H;
#pragma unroll
    for (int i = 0; i < kRestRegs; ++i) {
      const int e = tid + i * NT;
      if (e < oB2) {
        const int l = e < 6 * H ? e / 6 : e - 6 * H;
        sC[l * kChainRow + (e < 6 * H ? kChainW1 + e - 6 * l : kChainB1)] = kTanhScale * rest[i];
      } else if (e < oW3) {
        sC[(e - oB2) * kChainRow + kChainB2] = kTanhScale * rest[i];
      } else if (e < kRest) {   // layer 3 times dt: W3[o][l] is lane l's weight number o ^ (l & 3)
        const int q = e - oW3, l = e < oB3 ? q & 31 : q - 4 * H;
        sC[l * kChainRow + (e < oB3 ? kChainW3 + ((q >> 5) ^ (l & 3)) : kChainB3)] = dt * rest[i];
      }
    }
  }
};

struct ChainWeights {
  float w1[6] = {}, wP[16] = {}, wQ[16] = {};
  float bb1 = 0.0f, bP = 0.0f, bQ = 0.0f;
  // layer 3 times dt, as a reduce-scatter over each quad with the weights placed per lane:
  // lane L keeps output oA = L & 3 (its final one) and oB = oA ^ 2 (passed on in the second
  // exchange), and sends outputs oA ^ 1 and oA ^ 3 to its partner L ^ 1, whose oA and oB they
  // are; dt b3 enters once per output, in the lanes 0..3 of each sample
  float wKA = 0.0f, wKB = 0.0f, wSA = 0.0f, wSB = 0.0f, bKA = 0.0f;

  __device__ __forceinline__ void read(const float* sC, int c32) {
    const float* c = sC + c32 * kChainRow;
    const auto c4 = [&](int i) { return *reinterpret_cast<const float4*>(c + i); };
#pragma unroll
    for (int q = 0; q < 16; q += 4) {
      const float4 p = c4(q), v = c4(16 + q);
      wP[q] = p.x; wP[q + 1] = p.y; wP[q + 2] = p.z; wP[q + 3] = p.w;
      wQ[q] = v.x; wQ[q + 1] = v.y; wQ[q + 2] = v.z; wQ[q + 3] = v.w;
    }
    const float4 p = c4(kChainW1), v = c4(kChainW1 + 4), w = c4(kChainW3);
    w1[0] = p.x; w1[1] = p.y; w1[2] = p.z; w1[3] = p.w; w1[4] = v.x; w1[5] = v.y;
    bb1 = v.z;
    bP = c32 < 16 ? v.w : 0.0f;
    bQ = c32 < 16 ? 0.0f : v.w;
    wKA = w.x; wSA = w.y; wKB = w.z; wSB = w.w;
    bKA = c32 < 4 ? c[kChainB3] : 0.0f;
  }
};

}  // namespace mppi
