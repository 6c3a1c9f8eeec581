// Device-side evaluation of the RICS surrogate network on gfx950 MFMA.
//
// Network: 4 -> 128 -> 128 -> 128 -> 128 -> 3, SiLU after the hidden layers,
// linear output; 50,563 parameters, flat as [W1 (128x4 row-major), b1, W2, b2,
// W3, b3, W4, b4, W5 (3x128), b5].  Weights enter the matrix cores as bfloat16;
// every activation and back-propagated gradient enters as three bfloat16 terms
// hi + mid + lo (each the rounding of what the previous terms leave), so a
// product costs three v_mfma_f32_16x16x32_bf16 that share the weight operand
// and the network evaluates at float32 accuracy with float32 accumulation.
//
// One wavefront evaluates a group of 16 samples at a time as Z^T = W A^T: the
// 16 samples are the MFMA's N dimension, the neurons its M dimension.  With the
// 16x16x32 operand layout (lane l, g = l/16, r = l%16):
//   A (weights, 16 x 32):  lane holds A[r][8g + i], i = 0..7
//   B (activations, 32x16): lane holds B[8g + i][r]
//   D (16 x 16):           lane holds D[4g + j][r], j = 0..3
// the outputs of m-tiles 2K and 2K+1 already sit in the lanes that feed the
// B operand of k-step K, in the neuron order perm(K, g, i) = 32K + 4g + i
// (i < 4) and 32K + 16 + 4g + (i - 4) (i >= 4).  The weight tiles are stored
// pre-permuted in that order, so activations stay in registers between layers.
// Layers with 3 or 4 inputs (the input layer, and W5^T in the backward pass)
// pack the three split terms along K into one MFMA.
#pragma once

#include "pic1d_dev.h"

namespace pic1d {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int MLP_IN = 4, MLP_OUT = 3, MLP_W = 128;
constexpr int MLP_NPARAM = 50563;
constexpr int MLP_OFF_W1 = 0, MLP_OFF_B1 = 512;
constexpr int MLP_OFF_W2 = 640, MLP_OFF_B2 = 17024;
constexpr int MLP_OFF_W3 = 17152, MLP_OFF_B3 = 33536;
constexpr int MLP_OFF_W4 = 33664, MLP_OFF_B4 = 50048;
constexpr int MLP_OFF_W5 = 50176, MLP_OFF_B5 = 50560;

// Tiles of 64 lanes x 8 bfloat16.  Forward: W1 (8 m-tiles), W2..W4 (8 m x 4 k
// tiles each, index T*4+K), W5 (4 k-tiles).  Backward: W2^T..W4^T (T*4+K, T the
// input-neuron tile), W5^T (8 tiles).
constexpr int FT_L1 = 0, FT_H0 = 8, FT_OUT = 104, FT_TOTAL = 108;
constexpr int BT_H0 = 0, BT_OUT = 96, BT_TOTAL = 104;
constexpr int MLP_BIAS = 4 * MLP_W + 4;      // b1..b4, b5 (3) + pad: float offsets 0,128,256,384,512

// input box of the network (log10 gamma, s/L, log10 b, kT/keV), mapped to [-1, 1]
__host__ __device__ constexpr float mlp_in_lo(int k) { return k == 0 ? 0.0f : k == 1 ? 0.0f : k == 2 ? -2.0f : 0.3f; }
__host__ __device__ constexpr float mlp_in_hi(int k) { return k == 0 ? 8.0f : k == 1 ? 1.0f : k == 2 ? 3.0f : 1.0f; }

__host__ __device__ inline int mlp_perm(int K, int g, int i) {
    return 32 * K + (i < 4 ? 4 * g + i : 16 + 4 * g + (i - 4));
}

struct Split3 {
    bf16x8 hi, mid, lo;
};

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// Two values at a time: one packed conversion per term, and its halves widened back
// by a shift and a mask (converting value by value, the compiler makes a conversion
// and a permute of each).
__device__ __forceinline__ void split3(const float (&v)[8], Split3& s) {
    uint32_t* hi = reinterpret_cast<uint32_t*>(&s.hi);
    uint32_t* mid = reinterpret_cast<uint32_t*>(&s.mid);
    uint32_t* lo = reinterpret_cast<uint32_t*>(&s.lo);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        auto pack = [](float a, float b) {
            return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
        };
        auto low = [](uint32_t w) { return __builtin_bit_cast(float, w << 16); };
        auto high = [](uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); };
        const float a = v[2 * i], b = v[2 * i + 1];
        const uint32_t h = pack(a, b);
        const float a1 = a - low(h), b1 = b - high(h);
        const uint32_t m = pack(a1, b1);
        hi[i] = h;
        mid[i] = m;
        lo[i] = pack(a1 - low(m), b1 - high(m));
    }
}

__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

__device__ __forceinline__ float silu_grad_f(float z) {
    const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-z));
    return s * fmaf(z, 1.0f - s, 1.0f);
}

// B operand of the input layer for sample values x[0..3] (already normalised):
// positions 0..3 hi, 4..7 mid, 8..11 lo, zero beyond.  Lanes g = 0, 1 carry
// data; the caller provides each lane the inputs of sample r of its group.
__device__ __forceinline__ bf16x8 mlp_input_operand(const float (&x)[4], int g) {
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = (__bf16)0.0f;
    if (g < 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const __bf16 h = (__bf16)x[k];
            const float r1 = x[k] - (float)h;
            const __bf16 m = (__bf16)r1;
            const __bf16 l = (__bf16)(r1 - (float)m);
            if (g == 0) { b[k] = h; b[4 + k] = m; }
            else b[k] = l;
        }
    }
    return b;
}

// SiLU of m-tiles 2K, 2K+1 as the B operand of k-step K.
struct SiluOperand {
    __device__ __forceinline__ void operator()(const f32x4& t0, const f32x4& t1, Split3& s) const {
        float v[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = silu_f(t0[j]);
            v[4 + j] = silu_f(t1[j]);
        }
        split3(v, s);
    }
};

// The m-tiles 2K, 2K+1 themselves as the B operand of k-step K.
struct PlainOperand {
    __device__ __forceinline__ void operator()(const f32x4& t0, const f32x4& t1, Split3& s) const {
        const float v[8] = {t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]};
        split3(v, s);
    }
};

// One 128 -> 128 layer on a 16-sample group: out[T] = bias + sum_K W(T,K) B(K) over
// the three terms of B.  The loops run K, term, tile, so that consecutive MFMAs
// write eight different accumulators (independent chains); each tile sums in the
// order K0 hi, K0 mid, K0 lo, K1 hi, ...  An operand is formed right before its MFMAs, so
// that only one is live (12 registers instead of 48), and the scheduler is kept from
// hoisting the next one's: two wavefronts then fit a SIMD (the pusher spills four
// registers, outside of its loop over the layers).  They
// overlap one's vector with the other's matrix instructions (which leave the vector
// unit half of their 16 cycles; mixing the two within a wavefront, one MFMA to four
// vector instructions, was 6% slower).
template <class WPtr>
__device__ __forceinline__ void hidden_layer(WPtr w, int base, const float* __restrict__ bias, const f32x4 (&in)[8],
                                             f32x4 (&out)[8]) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
#pragma unroll
    for (int T = 0; T < 8; ++T) out[T] = *reinterpret_cast<const f32x4*>(bias + 16 * T + 4 * g);
#pragma unroll
    for (int K = 0; K < 4; ++K) {
        bf16x8 wt[8];
#pragma unroll
        for (int T = 0; T < 8; ++T) wt[T] = w[(base + T * 4 + K) * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);       // the weights' latency passes under the operand
        Split3 op;
        SiluOperand()(in[2 * K], in[2 * K + 1], op);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int T = 0; T < 8; ++T) out[T] = mfma(wt[T], op.hi, out[T]);
#pragma unroll
        for (int T = 0; T < 8; ++T) out[T] = mfma(wt[T], op.mid, out[T]);
#pragma unroll
        for (int T = 0; T < 8; ++T) out[T] = mfma(wt[T], op.lo, out[T]);
    }
}

// Forward pass of one 16-sample group.  `bin` is the input operand of this
// lane; returns D of the output layer (lanes g == 0: outputs 0..2 of sample r).
template <class WPtr>
__device__ __forceinline__ f32x4 mlp_group_forward(WPtr wf, const float* __restrict__ bias, const bf16x8& bin) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
    f32x4 acc[8];
#pragma unroll
    for (int T = 0; T < 8; ++T) {
        acc[T] = *reinterpret_cast<const f32x4*>(bias + 16 * T + 4 * g);
        acc[T] = mfma(wf[(FT_L1 + T) * 64 + lane], bin, acc[T]);
    }
#pragma unroll 1
    for (int h = 0; h < 3; ++h) {
        f32x4 next[8];
        hidden_layer(wf, FT_H0 + 32 * h, bias + MLP_W * (h + 1), acc, next);
#pragma unroll
        for (int T = 0; T < 8; ++T) acc[T] = next[T];
    }
    // one output tile: three partial sums (one per term) keep three MFMA chains in flight
    f32x4 o_hi, o_mid = {0.0f, 0.0f, 0.0f, 0.0f}, o_lo = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 4; ++j) o_hi[j] = (g == 0 && j < 3) ? bias[4 * MLP_W + j] : 0.0f;
#pragma unroll
    for (int K = 0; K < 4; ++K) {
        Split3 op;
        SiluOperand()(acc[2 * K], acc[2 * K + 1], op);
        const bf16x8 w = wf[(FT_OUT + K) * 64 + lane];
        o_hi = mfma(w, op.hi, o_hi);
        o_mid = mfma(w, op.mid, o_mid);
        o_lo = mfma(w, op.lo, o_lo);
    }
    f32x4 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) out[j] = o_hi[j] + (o_mid[j] + o_lo[j]);
    return out;
}

// B operand of W5^T in the backward pass for dL/d(out) d3[0..2] of sample r of the
// group: positions 0..2 hi, 3..5 mid, 6..8 lo.
__device__ __forceinline__ bf16x8 mlp_output_operand(const float (&d3)[3], int g) {
    __bf16 hi[3], mi[3], lo[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        hi[j] = (__bf16)d3[j];
        const float r1 = d3[j] - (float)hi[j];
        mi[j] = (__bf16)r1;
        lo[j] = (__bf16)(r1 - (float)mi[j]);
    }
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = (__bf16)0.0f;
    if (g == 0) {
        b[0] = hi[0]; b[1] = hi[1]; b[2] = hi[2];
        b[3] = mi[0]; b[4] = mi[1]; b[5] = mi[2];
        b[6] = lo[0]; b[7] = lo[1];
    } else if (g == 1) {
        b[0] = lo[2];
    }
    return b;
}

// The 16-sample group of a block of four wavefronts: wavefront w holds the m-tiles 2w
// and 2w+1 of every layer (32 neurons), forms the operand of k-step w from them and
// shares it through LDS, so that a layer costs a quarter of the time it takes one
// wavefront.  Each tile sums in the order of hidden_layer.
struct GroupOperands {
    bf16x8 t[2][4][3][64];      // double-buffered: [buffer][k-step][term][lane]
};

template <class Operand>
__device__ __forceinline__ void share_operand(GroupOperands& sh, int buf, int w, const f32x4 (&in)[2], Operand operand) {
    const int lane = threadIdx.x & 63;
    Split3 op;
    operand(in[0], in[1], op);
    sh.t[buf][w][0][lane] = op.hi;
    sh.t[buf][w][1][lane] = op.mid;
    sh.t[buf][w][2][lane] = op.lo;
    __syncthreads();        // (the other buffer's readers passed the barrier before)
}

// The weight tiles of wavefront w's two m-tiles of a 128 -> 128 layer.
template <class WPtr>
__device__ __forceinline__ void load_pair(WPtr wt, int base, int w, bf16x8 (&o)[2][4]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int K = 0; K < 4; ++K) o[t][K] = wt[(base + (2 * w + t) * 4 + K) * 64 + lane];
}

// out[t] += W(2w+t, .) B over the shared operands.
__device__ __forceinline__ void hidden_pair(const GroupOperands& sh, int buf, const bf16x8 (&wt)[2][4], f32x4 (&out)[2]) {
    const int lane = threadIdx.x & 63;
    bf16x8 b[4][3];
#pragma unroll
    for (int K = 0; K < 4; ++K)
#pragma unroll
        for (int term = 0; term < 3; ++term) b[K][term] = sh.t[buf][K][term][lane];
    __builtin_amdgcn_sched_barrier(0);       // all reads in flight before the first product
#pragma unroll
    for (int K = 0; K < 4; ++K)
#pragma unroll
        for (int term = 0; term < 3; ++term)
#pragma unroll
            for (int t = 0; t < 2; ++t) out[t] = mfma(wt[t][K], b[K][term], out[t]);
}

// The output layer over the shared operands (every wavefront the same): its tiles w and
// bias b.
__device__ __forceinline__ f32x4 output_layer(const GroupOperands& sh, int buf, const bf16x8 (&w)[4], const float (&b)[3]) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
    f32x4 o[3] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int j = 0; j < 3; ++j) o[0][j] = g == 0 ? b[j] : 0.0f;
    bf16x8 op[4][3];
#pragma unroll
    for (int K = 0; K < 4; ++K)
#pragma unroll
        for (int term = 0; term < 3; ++term) op[K][term] = sh.t[buf][K][term][lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int K = 0; K < 4; ++K)
#pragma unroll
        for (int term = 0; term < 3; ++term) o[term] = mfma(w[K], op[K][term], o[term]);
    f32x4 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) out[j] = o[0][j] + (o[1][j] + o[2][j]);
    return out;
}

}  // namespace pic1d
