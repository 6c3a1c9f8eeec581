// RICS surrogate network: training samples, bfloat16-MFMA forward, backward and
// weight-gradient kernels, Adam, and the C ABI of the pic1d_mlp_* calls.
//
// The network and its operand layout are described in mlp_dev.h.  What it
// learns, for momenta u >= 0 on the R_max = 4 dipole line (Appendix B.2):
//   o1 = log10(|F_hat| / |gamma mu - u|) = log10(A_F g(y) / x^2)   (Eq. contdrag)
//   o2 = log10(Ndot_hat)                                           (Eq. scatteringNdot)
//   o3 = log10(eps), eps = gamma (1 - (1 + 2b)^-1/2)               (Appendix A.3)
// as functions of (log10 gamma, s/L, log10 b, kT), with b an independent field
// strength.  The training samples are computed here in float64 from those
// closed forms; the loss is the mean squared error of the normalised targets.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/pic1d.h"
#include "mlp_dev.h"

namespace pic1d {

int set_global_error(int code, const std::string& msg);
inline int fail(void*, int code, const std::string& msg) { return set_global_error(code, msg); }

constexpr uint32_t STREAM_MLP_SAMPLE = 7, STREAM_MLP_INIT = 8, STREAM_MLP_BATCH = 9;
constexpr int MLP_MAX_ATTEMPTS = 64;
constexpr int MLP_CHUNK = 256;          // samples per weight-gradient block
constexpr int WGRAD_ROLES = 8;          // blocks per chunk: two per 128 x 128 layer, the input and the output layer
constexpr int MLP_TPB = 256;
constexpr int FWD_LDS_TPB = 768;
constexpr int ADAM_BLOCKS = (MLP_NPARAM + MLP_TPB - 1) / MLP_TPB;   // one parameter per thread

// float64 constants of the RICS prefactors (CODATA 2018; R* = 1e6 cm)
constexpr double kMlpRe = 2.8179403262e-13, kMlpLbar = 3.8615926796e-11, kMlpMeC2 = 510.99895, kMlpRstar = 1.0e6;

// ---------------------------------------------------------------------------
// training samples
// ---------------------------------------------------------------------------

// cos(theta) at arc-length fraction f of the line r = R sin^2(theta), s = 0 at the
// northern footpoint: P(v) = P(v0)(1 - 2f) with P(v) = v (1+3v^2)^1/2 + asinh(3^1/2 v)/3^1/2
// (Appendix B.2), by safeguarded Newton (P' = 2 (1 + 3 v^2)^1/2).
__device__ double mlp_cos_at(double R, double f) {
    const double v0 = sqrt(1.0 - 1.0 / R);
    auto P = [](double v) { return v * sqrt(1.0 + 3.0 * v * v) + asinh(1.7320508075688772 * v) / 1.7320508075688772; };
    const double target = P(v0) * (1.0 - 2.0 * f);
    double lo = -v0, hi = v0, v = v0 * (1.0 - 2.0 * f);
    for (int it = 0; it < 60; ++it) {
        const double e = P(v) - target;
        if (e > 0.0) hi = fmin(hi, v); else lo = fmax(lo, v);
        double vn = v - e / (2.0 * sqrt(1.0 + 3.0 * v * v));
        if (!(vn >= lo && vn <= hi)) vn = 0.5 * (lo + hi);
        if (fabs(vn - v) <= 1e-17 * (1.0 + fabs(v))) { v = vn; break; }
        v = vn;
    }
    return v;
}

// (o1, o2, o3, y) of one input point, float64
__device__ void mlp_targets(const float (&xin)[4], double R, double (&o)[3], double& y) {
    const double lg = xin[0], sl = xin[1], lb = xin[2], kT = xin[3];
    const double gam = exp10(lg);
    const double u = sqrt(fmax(gam * gam - 1.0, 0.0));
    const double b = exp10(lb);
    const double c = mlp_cos_at(R, sl);
    const double mu = 2.0 * c / sqrt(1.0 + 3.0 * c * c);
    const double x = R * (1.0 - c * c);
    const double th = kT / kMlpMeC2;
    y = b / (th * (gam - u * mu));
    const double base = kMlpRe * kMlpRstar / (4.0 * kMlpLbar * kMlpLbar);
    const double em1 = expm1(fmin(y, 700.0));
    o[0] = log10(base * th * th * th * y * y * y / em1 / (x * x));
    o[1] = log10(base * th * th * y * y / em1 / (x * x * gam));
    const double q = sqrt(1.0 + 2.0 * b);
    o[2] = log10(gam * (1.0 - 1.0 / q));
}

__global__ __launch_bounds__(MLP_TPB) void k_mlp_samples(uint32_t k0, uint32_t k1, int64_t first, int64_t n,
                                                         float R, float4* __restrict__ X, float4* __restrict__ O,
                                                         int* __restrict__ err) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t id = (uint64_t)(first + i);
        bool done = false;
        for (int a = 0; a < MLP_MAX_ATTEMPTS && !done; ++a) {
            const uint4 w = philox4x32_10(make_uint4((uint32_t)id, (uint32_t)(id >> 32), (uint32_t)a, STREAM_MLP_SAMPLE),
                                          k0, k1);
            const double u0 = (double)(w.x >> 8) * 0x1.0p-24, u1 = (double)(w.y >> 8) * 0x1.0p-24;
            const double u2 = (double)(w.z >> 8) * 0x1.0p-24, u3 = (double)(w.w >> 8) * 0x1.0p-24;
            const float xin[4] = {(float)(8.0 * u0), (float)u1, (float)(-2.0 + 5.0 * u2), (float)(0.3 + 0.7 * u3)};
            double o[3], y;
            mlp_targets(xin, (double)R, o, y);
            if (y <= (double)Y_CUT) {
                X[i] = make_float4(xin[0], xin[1], xin[2], xin[3]);
                O[i] = make_float4((float)o[0], (float)o[1], (float)o[2], 0.0f);
                done = true;
            }
        }
        if (!done) atomicExch(err, 1);
    }
}

// sums (pass 0) or sums of squared deviations from mean (pass 1) of the three
// target columns, one float64 partial per block and column
__global__ __launch_bounds__(MLP_TPB) void k_mlp_stats(const float4* __restrict__ O, int64_t n, int pass,
                                                       const double* __restrict__ mean, double* __restrict__ part) {
    __shared__ double sh[3][MLP_TPB];
    double acc[3] = {0.0, 0.0, 0.0};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 o = O[i];
        const double v[3] = {o.x, o.y, o.z};
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[k] += pass == 0 ? v[k] : (v[k] - mean[k]) * (v[k] - mean[k]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) sh[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int s = MLP_TPB / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
#pragma unroll
            for (int k = 0; k < 3; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x < 3) part[blockIdx.x * 3 + threadIdx.x] = sh[threadIdx.x][0];
}

// ---------------------------------------------------------------------------
// parameters -> bfloat16 MFMA tiles
// ---------------------------------------------------------------------------

__device__ __forceinline__ float mlp_w(const float* p, int layer, int o, int i) {
    switch (layer) {
        case 1: return p[MLP_OFF_W1 + o * 4 + i];
        case 2: return p[MLP_OFF_W2 + o * 128 + i];
        case 3: return p[MLP_OFF_W3 + o * 128 + i];
        case 4: return p[MLP_OFF_W4 + o * 128 + i];
        default: return p[MLP_OFF_W5 + o * 128 + i];
    }
}

__global__ __launch_bounds__(MLP_TPB) void k_mlp_pack(const float* __restrict__ p, bf16x8* __restrict__ ft,
                                                      bf16x8* __restrict__ bt, float* __restrict__ bias) {
    const int n_f = FT_TOTAL * 64, n_b = BT_TOTAL * 64;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n_f + n_b + MLP_BIAS; e += gridDim.x * blockDim.x) {
        if (e < n_f + n_b) {
            const bool fwd = e < n_f;
            const int t = fwd ? e / 64 : (e - n_f) / 64;
            const int lane = e & 63, g = lane >> 4, r = lane & 15;
            bf16x8 v;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float w = 0.0f;
                const int pp = 8 * g + i;
                if (fwd) {
                    if (t < FT_H0) {
                        w = pp < 12 ? mlp_w(p, 1, 16 * t + r, pp & 3) : 0.0f;
                    } else if (t < FT_OUT) {
                        const int h = (t - FT_H0) / 32, idx = (t - FT_H0) % 32, T = idx / 4, K = idx % 4;
                        w = mlp_w(p, h + 2, 16 * T + r, mlp_perm(K, g, i));
                    } else {
                        const int K = t - FT_OUT;
                        w = r < 3 ? mlp_w(p, 5, r, mlp_perm(K, g, i)) : 0.0f;
                    }
                } else {
                    if (t < BT_OUT) {
                        const int h = t / 32, idx = t % 32, T = idx / 4, K = idx % 4;
                        w = mlp_w(p, h + 2, mlp_perm(K, g, i), 16 * T + r);
                    } else {
                        const int T = t - BT_OUT;
                        w = pp < 9 ? mlp_w(p, 5, pp % 3, 16 * T + r) : 0.0f;
                    }
                }
                v[i] = (__bf16)w;
            }
            (fwd ? ft[e] : bt[e - n_f]) = v;
        } else {
            const int k = e - n_f - n_b;
            float b = 0.0f;
            if (k < 128) b = p[MLP_OFF_B1 + k];
            else if (k < 256) b = p[MLP_OFF_B2 + k - 128];
            else if (k < 384) b = p[MLP_OFF_B3 + k - 256];
            else if (k < 512) b = p[MLP_OFF_B4 + k - 384];
            else if (k < 515) b = p[MLP_OFF_B5 + k - 512];
            bias[k] = b;
        }
    }
}

// Glorot-uniform weights from Philox (counter (p, 0, 0, STREAM_MLP_INIT)), zero biases
__global__ __launch_bounds__(MLP_TPB) void k_mlp_init(uint32_t k0, uint32_t k1, float* __restrict__ p) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < MLP_NPARAM; e += gridDim.x * blockDim.x) {
        int fin = 0, fout = 0;
        bool weight = true;
        if (e < MLP_OFF_B1) { fin = 4; fout = 128; }
        else if (e < MLP_OFF_W2) weight = false;
        else if (e < MLP_OFF_B2) { fin = 128; fout = 128; }
        else if (e < MLP_OFF_W3) weight = false;
        else if (e < MLP_OFF_B3) { fin = 128; fout = 128; }
        else if (e < MLP_OFF_W4) weight = false;
        else if (e < MLP_OFF_B4) { fin = 128; fout = 128; }
        else if (e < MLP_OFF_W5) weight = false;
        else if (e < MLP_OFF_B5) { fin = 128; fout = 3; }
        else weight = false;
        float v = 0.0f;
        if (weight) {
            const uint4 w = philox4x32_10(make_uint4((uint32_t)e, 0u, 0u, STREAM_MLP_INIT), k0, k1);
            v = sqrtf(6.0f / (float)(fin + fout)) * (2.0f * uniform24(w.x) - 1.0f);
        }
        p[e] = v;
    }
}

// ---------------------------------------------------------------------------
// forward / backward over a batch
// ---------------------------------------------------------------------------

__device__ __forceinline__ void mlp_normalise(const float4& x, float (&xn)[4]) {
    const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) xn[k] = (v[k] - mlp_in_lo(k)) * (2.0f / (mlp_in_hi(k) - mlp_in_lo(k))) - 1.0f;
}

// Inference: raw inputs X (n x 4) -> network outputs out (n x 3, normalised targets), a
// 16-sample group per wavefront at a time.
template <class WPtr>
__device__ __forceinline__ void forward_groups(WPtr ft, const float* bias, const float4* __restrict__ X, int64_t n,
                                               float* __restrict__ out) {
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t q = wave; q * 16 < n; q += nwave) {
        const int64_t row = q * 16 + r;
        float xn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < n && g < 2) mlp_normalise(X[row], xn);
        const bf16x8 bin = mlp_input_operand(xn, g);
        const f32x4 o = mlp_group_forward(ft, bias, bin);
        if (g == 0 && row < n) {
            out[row * 3 + 0] = o[0];
            out[row * 3 + 1] = o[1];
            out[row * 3 + 2] = o[2];
        }
    }
}

__global__ __launch_bounds__(MLP_TPB) void k_mlp_forward(const bf16x8* __restrict__ ft, const float* __restrict__ bias,
                                                         const float4* __restrict__ X, int64_t n,
                                                         float* __restrict__ out) {
    forward_groups(ft, bias, X, n, out);
}

// ... with the weights in LDS, one block per CU and three wavefronts per SIMD: each
// group otherwise reads 108 KB of them through the L2, about half of what that can
// deliver.  Bound by vector issue (1,500 instructions and 308 MFMAs a group): 317 us a
// call at 1e6 samples, 345 without; from 262,144 samples on the groups make up for the
// staging (110 us either way there).  32-sample groups on 32x32x16 MFMAs give the same
// bits and half the weight reads, but two wavefronts per SIMD at best: 352 us.
__global__ __launch_bounds__(FWD_LDS_TPB) __attribute__((amdgpu_waves_per_eu(FWD_LDS_TPB / 256))) void k_mlp_forward_lds(
    const bf16x8* __restrict__ ft, const float* __restrict__ bias, const float4* __restrict__ X, int64_t n,
    float* __restrict__ out) {
    __shared__ bf16x8 sW[FT_TOTAL * 64];
    __shared__ __align__(16) float sB[MLP_BIAS];
    for (int e = threadIdx.x; e < FT_TOTAL * 64; e += FWD_LDS_TPB) sW[e] = ft[e];
    for (int e = threadIdx.x; e < MLP_BIAS; e += FWD_LDS_TPB) sB[e] = bias[e];
    __syncthreads();
    forward_groups((const bf16x8*)sW, (const float*)sB, X, n, out);
}

// Inference on a small batch, a block of four wavefronts per group (GroupOperands), from
// the parameters themselves: the rounding to bfloat16 and the order of k_mlp_pack's
// tiles are two 16-byte loads and four packed conversions per tile and lane, so no
// packing launch comes first.  Latency-bound; at 1,000 samples the call takes 28.6 us
// (34.7 with the packing and a group per wavefront).  Beyond FWD_SMALL samples the
// blocks' float32 weights (202 KB each from L2) cost more than the launch.
__global__ __launch_bounds__(MLP_TPB) __attribute__((amdgpu_waves_per_eu(2))) void k_mlp_forward_small(
    const float* __restrict__ p, const float4* __restrict__ X, int64_t n, float* __restrict__ out) {
    __shared__ GroupOperands sh;
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15, w = threadIdx.x >> 6;
    auto rounded = [](const float4& a, const float4& b) {
        bf16x8 t;
        t[0] = (__bf16)a.x; t[1] = (__bf16)a.y; t[2] = (__bf16)a.z; t[3] = (__bf16)a.w;
        t[4] = (__bf16)b.x; t[5] = (__bf16)b.y; t[6] = (__bf16)b.z; t[7] = (__bf16)b.w;
        return t;
    };
    const float4 none = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    // operand of k-step K from a row of 128 weights (mlp_perm's order)
    auto row_tile = [&](const float* row, int K) {
        const float4* q = reinterpret_cast<const float4*>(row + 32 * K + 4 * g);
        return rounded(q[0], q[4]);
    };
    constexpr int OFF_W[3] = {MLP_OFF_W2, MLP_OFF_W3, MLP_OFF_W4};
    int buf = 0;
    for (int64_t q = blockIdx.x; q * 16 < n; q += gridDim.x) {
        const int64_t row = q * 16 + r;
        float xn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (row < n && g < 2) mlp_normalise(X[row], xn);
        const bf16x8 bin = mlp_input_operand(xn, g);
        f32x4 z[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int o = 16 * (2 * w + k);
            const float4 w1 = *reinterpret_cast<const float4*>(p + MLP_OFF_W1 + 4 * (o + r));
            z[k] = *reinterpret_cast<const f32x4*>(p + MLP_OFF_B1 + o + 4 * g);
            z[k] = mfma(rounded(g < 2 ? w1 : none, g == 0 ? w1 : none), bin, z[k]);
        }
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            bf16x8 wt[2][4];
            f32x4 next[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int o = 16 * (2 * w + k);
#pragma unroll
                for (int K = 0; K < 4; ++K) wt[k][K] = row_tile(p + OFF_W[h] + MLP_W * (o + r), K);
                next[k] = *reinterpret_cast<const f32x4*>(p + OFF_W[h] + MLP_W * MLP_W + o + 4 * g);
            }
            share_operand(sh, buf, w, z, SiluOperand());
            hidden_pair(sh, buf, wt, next);
            z[0] = next[0];
            z[1] = next[1];
            buf ^= 1;
        }
        bf16x8 wo[4];
#pragma unroll
        for (int K = 0; K < 4; ++K) {
            const bf16x8 t = row_tile(p + MLP_OFF_W5 + MLP_W * min(r, 2), K);      // (rows 3 .. 15 are zero)
            wo[K] = r < 3 ? t : rounded(none, none);
        }
        float b5[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) b5[j] = p[MLP_OFF_B5 + j];
        share_operand(sh, buf, w, z, SiluOperand());
        const f32x4 o = output_layer(sh, buf, wo, b5);
        buf ^= 1;
        if (w == 0 && g == 0 && row < n) {
            out[row * 3 + 0] = o[0];
            out[row * 3 + 1] = o[1];
            out[row * 3 + 2] = o[2];
        }
    }
}

struct TrainArgs {
    const bf16x8* ft;
    const bf16x8* bt;
    const float* bias;
    const float4* X;          // inputs (raw)
    const float* T;           // explicit normalised targets (n x 3), or null
    const float4* O;          // sample targets (o1, o2, o3), used with norm when T is null
    const float* norm;        // mean[3], std[3]
    int64_t n_batch;          // samples in the batch
    int64_t n_pool;           // sample pool size; batch rows draw from it when > 0
    uint32_t step, k0, k1;
    float4* XN;               // normalised inputs of the batch rows
    float* Z;                 // pre-activations, 4 x rows x 128
    float* DS;                // dL/dz, 4 x rows x 128
    float4* DOUT;             // dL/d(out), rows x 4
    int64_t zlayer;
    double* loss_part;        // one partial sum of squared errors per block
};

// A product rounded to float32, whatever it is subtracted from next.
__device__ __forceinline__ float mul_rounded(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}

// Forward and backward over a batch: pre-activations Z, dL/d(out), dL/dz of the hidden
// layers DS and the loss.  A block of four wavefronts takes a group of 16 samples at a
// time (GroupOperands); the pre-activations stay in registers for the way back.
// Latency-bound at training batches, where a group or two are all a block gets: 18 us at
// 8,192 samples for both directions, 17 and 19 us with a group per wavefront and a
// kernel for each direction.  Larger batches gain too, as the pre-activations are not
// read back: 94 us at 65,536 samples for 50 and 65, 1.53 ms at 1,048,576 for 0.68 and 1.33.
__global__ __launch_bounds__(MLP_TPB) __attribute__((amdgpu_waves_per_eu(2))) void k_mlp_train(TrainArgs a) {
    __shared__ GroupOperands sh;
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15, w = threadIdx.x >> 6;
    const int64_t rows = a.zlayer / MLP_W;
    double lsum = 0.0;
    int buf = 0;
    for (int64_t q = blockIdx.x; q * 16 < rows; q += gridDim.x) {
        const int64_t row = q * 16 + r;
        const bool valid = row < a.n_batch;
        const int64_t at = row * MLP_W + 32 * w + 4 * g;      // this lane's neurons: at .. at+3 and at+16 .. at+19
        float xn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float t[3] = {0.0f, 0.0f, 0.0f};
        if (valid && g < 2) {
            int64_t src = row;
            if (a.n_pool > 0) {
                const uint4 p = philox4x32_10(make_uint4(a.step, (uint32_t)row, (uint32_t)(row >> 32), STREAM_MLP_BATCH),
                                              a.k0, a.k1);
                const uint64_t h = ((uint64_t)p.x << 32) | p.y;
                src = (int64_t)__umul64hi(h, (uint64_t)a.n_pool);
            }
            mlp_normalise(a.X[src], xn);
            if (g == 0) {
                if (a.T) {
                    t[0] = a.T[src * 3]; t[1] = a.T[src * 3 + 1]; t[2] = a.T[src * 3 + 2];
                } else {
                    const float4 o = a.O[src];
                    t[0] = (o.x - a.norm[0]) / a.norm[3];
                    t[1] = (o.y - a.norm[1]) / a.norm[4];
                    t[2] = (o.z - a.norm[2]) / a.norm[5];
                }
            }
        }
        const bf16x8 bin = mlp_input_operand(xn, g);
        f32x4 z[4][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int T = 2 * w + k;
            z[0][k] = *reinterpret_cast<const f32x4*>(a.bias + 16 * T + 4 * g);
            z[0][k] = mfma(a.ft[(FT_L1 + T) * 64 + lane], bin, z[0][k]);
        }
        bf16x8 wt[2][4];
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            load_pair(a.ft, FT_H0 + 32 * h, w, wt);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                *reinterpret_cast<f32x4*>(a.Z + h * a.zlayer + at + 16 * k) = z[h][k];
                z[h + 1][k] = *reinterpret_cast<const f32x4*>(a.bias + MLP_W * (h + 1) + 16 * (2 * w + k) + 4 * g);
            }
            share_operand(sh, buf, w, z[h], SiluOperand());
            hidden_pair(sh, buf, wt, z[h + 1]);
            buf ^= 1;
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) *reinterpret_cast<f32x4*>(a.Z + 3 * a.zlayer + at + 16 * k) = z[3][k];
        share_operand(sh, buf, w, z[3], SiluOperand());
        bf16x8 wo[4];
#pragma unroll
        for (int K = 0; K < 4; ++K) wo[K] = a.ft[(FT_OUT + K) * 64 + lane];
        const float b5[3] = {a.bias[4 * MLP_W], a.bias[4 * MLP_W + 1], a.bias[4 * MLP_W + 2]};
        const f32x4 o = output_layer(sh, buf, wo, b5);
        buf ^= 1;
        float d[3] = {0.0f, 0.0f, 0.0f};
        if (g == 0) {
            const float c = 2.0f / (3.0f * (float)a.n_batch);
            if (valid) {
                const float e0 = o[0] - t[0], e1 = o[1] - t[1], e2 = o[2] - t[2];
                d[0] = c * e0;
                d[1] = c * e1;
                d[2] = c * e2;
                if (w == 0) lsum += (double)e0 * e0 + (double)e1 * e1 + (double)e2 * e2;
            }
            if (w == 0) {
                a.DOUT[row] = make_float4(d[0], d[1], d[2], 0.0f);
                a.XN[row] = make_float4(xn[0], xn[1], xn[2], xn[3]);
            }
        }
        // back: dL/da of the last hidden layer, then through SiLU' and W^T layer by layer
#pragma unroll
        for (int j = 0; j < 3; ++j) d[j] = __shfl(d[j], r, 64);
        const bf16x8 bdo = mlp_output_operand(d, g);
        f32x4 acc[2];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            acc[k] = mfma(a.bt[(BT_OUT + 2 * w + k) * 64 + lane], bdo, f32x4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
        for (int h = 3; h >= 0; --h) {
            if (h > 0) load_pair(a.bt, BT_H0 + 32 * (h - 1), w, wt);      // W_{h+1}^T maps dL/dz_h to dL/da_{h-1}
#pragma unroll
            for (int k = 0; k < 2; ++k) {
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[k][j] = mul_rounded(acc[k][j], silu_grad_f(z[h][k][j]));
                *reinterpret_cast<f32x4*>(a.DS + h * a.zlayer + at + 16 * k) = acc[k];
            }
            if (h == 0) break;
            share_operand(sh, buf, w, acc, PlainOperand());
            acc[0] = acc[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            hidden_pair(sh, buf, wt, acc);
            buf ^= 1;
        }
    }
    if (w == 0) {
        for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
        if (lane == 0) a.loss_part[blockIdx.x] = lsum;
    }
}

// The activation rounded to float32 before it is split (mlp_dev.h's operands take the
// product into the first subtraction unrounded).
__device__ __forceinline__ float silu_rounded(float z) {
    return mul_rounded(z, __builtin_amdgcn_rcpf(1.0f + __expf(-z)));
}

// c += A B over the six products of the operands' terms above 2^-24 relative.
__device__ __forceinline__ f32x4 mfma6(const Split3& A, const Split3& B, f32x4 c) {
    c = mfma(A.hi, B.hi, c);
    c = mfma(A.hi, B.mid, c);
    c = mfma(A.mid, B.hi, c);
    c = mfma(A.hi, B.lo, c);
    c = mfma(A.lo, B.hi, c);
    return mfma(A.mid, B.mid, c);
}

// Weight and bias gradients of one layer over one chunk of MLP_CHUNK rows:
// dW[o][i] = sum_s delta[s][o] a[s][i], db[o] = sum_s delta[s][o]; both operands
// enter as three bfloat16 terms.  A lane's operand is eight samples of one neuron: it
// reads them straight from the row-major arrays (16 lanes share a 64-byte piece of a
// row), so nothing is transposed.  In the 128 x 128 layers a block of four wavefronts
// takes half the output neurons, 16 per wavefront; each wavefront forms a quarter of
// the activations' operands, once per block, and shares them through LDS.
// grid = (chunks, WGRAD_ROLES);
// partial[chunk][param] in the flat packing.  Bound by latency and the operands'
// formation: 15.5 us at 8,192 rows, where staging float32 through LDS and splitting it
// again for every tile took 84 us.
__global__ __launch_bounds__(MLP_TPB) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_mlp_wgrad(
    const float4* __restrict__ XN, const float* __restrict__ Z, const float* __restrict__ DS,
    const float4* __restrict__ DOUT, int64_t zlayer, float* __restrict__ partial) {
    constexpr int KSTEPS = MLP_CHUNK / 32;
    __shared__ bf16x8 sA[2][8][3][64];           // activation operands of a k-step, double-buffered
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15, w = threadIdx.x >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * MLP_CHUNK;
    float* out = partial + (int64_t)blockIdx.x * MLP_NPARAM;
    const int role = blockIdx.y;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    // eight samples (rows 8g .. 8g+7 of a k-step) of neuron column c
    auto column = [&](const float* base, int ks, int c, float (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = base[(row0 + 32 * ks + 8 * g + i) * MLP_W + c];
    };
    auto silu8 = [](const float (&z)[8], Split3& s) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = silu_rounded(z[i]);
        split3(v, s);
    };
    // the sum over a k-step's 32 samples in their order, from the four lanes that hold a
    // neuron's samples to its lane g = 3
    auto ordered_sum = [&](const float (&d)[8]) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q > 0) s = __shfl(s, 16 * (q - 1) + r, 64);
#pragma unroll
            for (int i = 0; i < 8; ++i) s += d[i];
        }
        return s;
    };
    if (role < WGRAD_ROLES - 2) {
        const int layer = 2 + (role >> 1);       // 2, 3, 4
        const int To = 4 * (role & 1) + w;
        const float* D = DS + (layer - 1) * zlayer;
        const float* Zp = Z + (layer - 2) * zlayer;
        f32x4 acc[8];
        float db = 0.0f;
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = zero;
        float dv[8], z0[8], z1[8];
        auto load = [&](int ks) {
            column(D, ks, 16 * To + r, dv);
            column(Zp, ks, 32 * w + r, z0);
            column(Zp, ks, 32 * w + 16 + r, z1);
        };
        load(0);
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const int buf = ks & 1;
            Split3 A, B;
            split3(dv, A);
            db += ordered_sum(dv);
            silu8(z0, B);
            sA[buf][2 * w][0][lane] = B.hi;
            sA[buf][2 * w][1][lane] = B.mid;
            sA[buf][2 * w][2][lane] = B.lo;
            silu8(z1, B);
            sA[buf][2 * w + 1][0][lane] = B.hi;
            sA[buf][2 * w + 1][1][lane] = B.mid;
            sA[buf][2 * w + 1][2][lane] = B.lo;
            __syncthreads();                     // (the buffer's readers of two k-steps ago passed the last one)
            if (ks + 1 < KSTEPS) load(ks + 1);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                Split3 Bt[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    Bt[t].hi = sA[buf][4 * h + t][0][lane];
                    Bt[t].mid = sA[buf][4 * h + t][1][lane];
                    Bt[t].lo = sA[buf][4 * h + t][2][lane];
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[4 * h + t] = mfma6(A, Bt[t], acc[4 * h + t]);
            }
        }
        const int offW = layer == 2 ? MLP_OFF_W2 : layer == 3 ? MLP_OFF_W3 : MLP_OFF_W4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int o = 16 * To + 4 * g + j;
#pragma unroll
            for (int t = 0; t < 8; ++t) out[offW + o * MLP_W + 16 * t + r] = acc[t][j];
        }
        if (g == 3) out[offW + MLP_W * MLP_W + 16 * To + r] = db;
    } else if (role == WGRAD_ROLES - 2) {
        // the input layer
        f32x4 acc[2] = {zero, zero};
        float db[2] = {0.0f, 0.0f};
        for (int ks = 0; ks < KSTEPS; ++ks) {
            float x[8], d[8];
            Split3 A, B;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[i] = r < 4 ? reinterpret_cast<const float*>(XN + row0 + 32 * ks + 8 * g + i)[r] : 0.0f;
            split3(x, B);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                column(DS, ks, 32 * w + 16 * t + r, d);
                split3(d, A);
                db[t] += ordered_sum(d);
                acc[t] = mfma6(A, B, acc[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (r < 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) out[MLP_OFF_W1 + (32 * w + 16 * t + 4 * g + j) * 4 + r] = acc[t][j];
            if (g == 3) out[MLP_OFF_B1 + 32 * w + 16 * t + r] = db[t];
        }
    } else {
        // the output layer: three rows
        f32x4 acc[2] = {zero, zero};
        float db = 0.0f;
        const float* Zp = Z + 3 * zlayer;
        for (int ks = 0; ks < KSTEPS; ++ks) {
            float d[8], z[8];
            Split3 A, B;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                d[i] = r < 3 ? reinterpret_cast<const float*>(DOUT + row0 + 32 * ks + 8 * g + i)[r] : 0.0f;
            split3(d, A);
            db += ordered_sum(d);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                column(Zp, ks, 32 * w + 16 * t + r, z);
                silu8(z, B);
                acc[t] = mfma6(A, B, acc[t]);
            }
        }
        if (g == 0) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
#pragma unroll
                for (int t = 0; t < 2; ++t) out[MLP_OFF_W5 + j * MLP_W + 32 * w + 16 * t + r] = acc[t][j];
            }
        }
        if (g == 3 && w == 0 && r < 3) out[MLP_OFF_B5 + r] = db;
    }
}

// Sum of the chunk partials (fixed order) and, if apply, one Adam step
// (Kingma & Ba 2015, Algorithm 1) with bias corrections bc1 = 1 - beta1^t, bc2 = 1 - beta2^t.
struct AdamArgs {
    float lr, beta1, omb1, beta2, omb2, eps, bc1, bc2;   // omb = 1 - beta, bc = 1 - beta^t (formed in float64)
};

// Writes parameter e's bfloat16 value to its places in the MFMA tiles (the inverse of
// k_mlp_pack's reading; the tiles' zeros stay as k_mlp_pack left them).
struct PackedNet {
    __bf16* ft;
    __bf16* bt;
    float* bias;
};

__device__ __forceinline__ void mlp_repack(const PackedNet& n, int e, float v) {
    const __bf16 b = (__bf16)v;
    auto put = [](__bf16* tiles, int tile, int g, int r, int i, __bf16 x) { tiles[(tile * 64 + 16 * g + r) * 8 + i] = x; };
    // position (K, g, i) of an input neuron in mlp_perm's order
    auto place = [](int neuron, int& K, int& g, int& i) {
        const int m = neuron & 31;
        K = neuron >> 5;
        g = (m & 15) >> 2;
        i = (m & 3) + (m < 16 ? 0 : 4);
    };
    int K, g, i;
    if (e < MLP_OFF_B1) {
        const int o = e >> 2, k = e & 3;
        put(n.ft, FT_L1 + (o >> 4), 0, o & 15, k, b);
        put(n.ft, FT_L1 + (o >> 4), 0, o & 15, 4 + k, b);
        put(n.ft, FT_L1 + (o >> 4), 1, o & 15, k, b);
    } else if (e < MLP_OFF_W2) {
        n.bias[e - MLP_OFF_B1] = v;
    } else if (e < MLP_OFF_W5) {
        constexpr int LAYER = MLP_W * MLP_W + MLP_W;
        const int h = (e - MLP_OFF_W2) / LAYER, k = (e - MLP_OFF_W2) - h * LAYER;
        if (k < MLP_W * MLP_W) {
            const int o = k >> 7, in = k & 127;
            place(in, K, g, i);
            put(n.ft, FT_H0 + 32 * h + (o >> 4) * 4 + K, g, o & 15, i, b);
            place(o, K, g, i);
            put(n.bt, BT_H0 + 32 * h + (in >> 4) * 4 + K, g, in & 15, i, b);
        } else {
            n.bias[MLP_W * (h + 1) + k - MLP_W * MLP_W] = v;
        }
    } else if (e < MLP_OFF_B5) {
        const int o = (e - MLP_OFF_W5) >> 7, in = (e - MLP_OFF_W5) & 127;
        place(in, K, g, i);
        put(n.ft, FT_OUT + K, g, o, i, b);
        for (int pp = o; pp < 9; pp += 3) put(n.bt, BT_OUT + (in >> 4), pp >> 3, in & 15, pp & 7, b);
    } else {
        n.bias[4 * MLP_W + e - MLP_OFF_B5] = v;
    }
}

// With n.ft set, the updated parameters also replace theirs in the packed tiles: the
// next training step needs no launch of k_mlp_pack.
__global__ __launch_bounds__(MLP_TPB) void k_mlp_adam(const float* __restrict__ partial, int nchunk,
                                                      float* __restrict__ p, float* __restrict__ m,
                                                      float* __restrict__ v, float* __restrict__ grad_out, int apply,
                                                      AdamArgs h, PackedNet n) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < MLP_NPARAM; e += gridDim.x * blockDim.x) {
        float gsum = 0.0f;
#pragma unroll 8
        for (int c = 0; c < nchunk; ++c) gsum += partial[(int64_t)c * MLP_NPARAM + e];
        if (grad_out) grad_out[e] = gsum;
        if (apply) {
            const float mm = h.beta1 * m[e] + h.omb1 * gsum;
            const float vv = h.beta2 * v[e] + h.omb2 * gsum * gsum;
            m[e] = mm;
            v[e] = vv;
            const float pn = p[e] - h.lr * (mm / h.bc1) / (sqrtf(vv / h.bc2) + h.eps);
            p[e] = pn;
            if (n.ft) mlp_repack(n, e, pn);
        }
    }
}

}  // namespace pic1d

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
using namespace pic1d;

namespace {

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

AdamArgs adam_args(double lr, double beta1, double beta2, double eps, int64_t t) {
    AdamArgs h;
    h.lr = (float)lr;
    h.beta1 = (float)beta1;
    h.omb1 = (float)(1.0 - beta1);
    h.beta2 = (float)beta2;
    h.omb2 = (float)(1.0 - beta2);
    h.eps = (float)eps;
    h.bc1 = (float)(1.0 - std::pow(beta1, (double)t));
    h.bc2 = (float)(1.0 - std::pow(beta2, (double)t));
    return h;
}

struct MlpWork {
    bf16x8* ft = nullptr;
    bf16x8* bt = nullptr;
    float* bias = nullptr;
    float* master = nullptr;
    float* m = nullptr;
    float* v = nullptr;
    float* grad = nullptr;
    float* norm = nullptr;
    float4* X = nullptr;
    float4* O = nullptr;
    float4* XN = nullptr;
    float4* DOUT = nullptr;
    float* Z = nullptr;
    float* DS = nullptr;
    float* partial = nullptr;
    double* loss_part = nullptr;
    double* stat_part = nullptr;
    double* mean_dev = nullptr;
    int* err = nullptr;
    int64_t rows = 0;            // batch rows rounded up to MLP_CHUNK
    int nchunk = 0;
    size_t bytes = 0;
};

constexpr int FWD_BLOCKS = 1024;
constexpr int64_t FWD_SMALL = 4096;
constexpr int64_t FWD_LARGE = 262144;

// blocks of k_mlp_train: a 16-sample group each, at most two rounds of the chip
int train_blocks(int64_t rows) { return (int)std::min<int64_t>(FWD_BLOCKS, rows / 16); }
constexpr int STAT_BLOCKS = 512;

// Carve the training workspace: tiles, parameters and Adam moments, the sample
// pool (n_pool rows of inputs and targets), the per-batch activations and the
// weight-gradient partials.  With base == nullptr only the size is computed.
MlpWork mlp_layout(char* base, int64_t batch, int64_t n_pool) {
    MlpWork w;
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        char* p = base ? base + off : nullptr;
        off = align256(off + bytes);
        return p;
    };
    w.rows = ((batch + MLP_CHUNK - 1) / MLP_CHUNK) * MLP_CHUNK;
    w.nchunk = (int)(w.rows / MLP_CHUNK);
    w.ft = reinterpret_cast<bf16x8*>(take(sizeof(bf16x8) * FT_TOTAL * 64));
    w.bt = reinterpret_cast<bf16x8*>(take(sizeof(bf16x8) * BT_TOTAL * 64));
    w.bias = reinterpret_cast<float*>(take(sizeof(float) * MLP_BIAS));
    w.master = reinterpret_cast<float*>(take(sizeof(float) * MLP_NPARAM));
    w.m = reinterpret_cast<float*>(take(sizeof(float) * MLP_NPARAM));
    w.v = reinterpret_cast<float*>(take(sizeof(float) * MLP_NPARAM));
    w.grad = reinterpret_cast<float*>(take(sizeof(float) * MLP_NPARAM));
    w.norm = reinterpret_cast<float*>(take(sizeof(float) * 8));
    w.X = reinterpret_cast<float4*>(take(sizeof(float4) * std::max<int64_t>(n_pool, 1)));
    w.O = reinterpret_cast<float4*>(take(sizeof(float4) * std::max<int64_t>(n_pool, 1)));
    w.XN = reinterpret_cast<float4*>(take(sizeof(float4) * w.rows));
    w.DOUT = reinterpret_cast<float4*>(take(sizeof(float4) * w.rows));
    w.Z = reinterpret_cast<float*>(take(sizeof(float) * 4 * w.rows * MLP_W));
    w.DS = reinterpret_cast<float*>(take(sizeof(float) * 4 * w.rows * MLP_W));
    w.partial = reinterpret_cast<float*>(take(sizeof(float) * (size_t)w.nchunk * MLP_NPARAM));
    w.loss_part = reinterpret_cast<double*>(take(sizeof(double) * FWD_BLOCKS));
    w.stat_part = reinterpret_cast<double*>(take(sizeof(double) * 3 * STAT_BLOCKS));
    w.mean_dev = reinterpret_cast<double*>(take(sizeof(double) * 4));
    w.err = reinterpret_cast<int*>(take(sizeof(int) * 4));
    w.bytes = off;
    return w;
}

#define MLP_TRY(expr)                                                                               \
    do {                                                                                            \
        hipError_t e_ = (expr);                                                                     \
        if (e_ != hipSuccess) return fail(nullptr, PIC1D_EDEVICE, std::string(#expr ": ") + hipGetErrorString(e_)); \
    } while (0)

int check_workspace(void* ws, size_t have, size_t need) {
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) != 0 || have < need)
        return fail(nullptr, PIC1D_ENOMEM, "workspace missing, misaligned (256 B) or smaller than pic1d_mlp_workspace_size");
    return PIC1D_OK;
}

void split_seed(uint64_t seed, uint32_t& k0, uint32_t& k1) {
    k0 = (uint32_t)seed;
    k1 = (uint32_t)(seed >> 32);
}

// one forward + backward + weight-gradient pass over the batch rows already
// addressed by `fa`; leaves the chunk partials in w.partial
int run_grad(const MlpWork& w, TrainArgs fa, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_train, dim3(train_blocks(w.rows)), dim3(MLP_TPB), 0, s, fa);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(w.nchunk, WGRAD_ROLES), dim3(MLP_TPB), 0, s, w.XN, w.Z, w.DS, w.DOUT,
                       (int64_t)(w.rows * MLP_W), w.partial);
    MLP_TRY(hipGetLastError());
    return PIC1D_OK;
}

double sum_loss(const MlpWork& w, int nblocks, hipStream_t s) {
    double h[FWD_BLOCKS];          // on the stack: the allocation-free entry point uses this too
    nblocks = std::min(nblocks, FWD_BLOCKS);
    if (hipMemcpyAsync(h, w.loss_part, sizeof(double) * nblocks, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return NAN;
    double t = 0.0;
    for (int b = 0; b < nblocks; ++b) t += h[b];
    return t;
}

// The loss and gradient of n samples on a carved workspace w (pic1d_mlp_loss_grad
// and its allocation-free variant).
int loss_grad_on(const MlpWork& w, const float* params, int64_t n, const float* x, const float* t, float* grad,
                 double* loss, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_pack, dim3(64), dim3(MLP_TPB), 0, s, params, w.ft, w.bt, w.bias);
    TrainArgs fa{};
    fa.ft = w.ft; fa.bias = w.bias; fa.X = reinterpret_cast<const float4*>(x); fa.T = t;
    fa.n_batch = n; fa.n_pool = 0; fa.XN = w.XN; fa.Z = w.Z; fa.DS = w.DS; fa.DOUT = w.DOUT; fa.bt = w.bt;
    fa.zlayer = w.rows * MLP_W; fa.loss_part = w.loss_part;
    if (int rc = run_grad(w, fa, s)) return rc;
    hipLaunchKernelGGL(k_mlp_adam, dim3(ADAM_BLOCKS), dim3(MLP_TPB), 0, s, w.partial, w.nchunk, nullptr, nullptr, nullptr, grad,
                       0, adam_args(0.0, 0.0, 0.0, 1.0, 1), PackedNet{});
    MLP_TRY(hipGetLastError());
    const double l = sum_loss(w, train_blocks(w.rows), s);
    if (loss) *loss = l / (3.0 * (double)n);
    return PIC1D_OK;
}

// ---------------------------------------------------------------------------
// Scratch of pic1d_mlp_loss_grad_static: the workspace of a batch of up to
// MLP_STATIC_MAX_ROWS samples as a file-scope device array, held by each GPU the
// library runs on until the process ends.  In host code `scratch` names a host
// stand-in, never the device memory: the device address comes from
// hipGetSymbolAddress, taken once per device with that device current.
// ---------------------------------------------------------------------------
constexpr int64_t MLP_STATIC_MAX_ROWS = 2048;
constexpr size_t MLP_STATIC_BYTES = (size_t)12 << 20;
constexpr int MLP_STATIC_MAX_DEVICES = 64;

}  // namespace

static __device__ __align__(256) unsigned char scratch[MLP_STATIC_BYTES];

namespace {

std::mutex g_scratch_mutex;
void* g_scratch_ptr[MLP_STATIC_MAX_DEVICES] = {};

int static_scratch(void** out) {
    int dev = -1;
    MLP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MLP_STATIC_MAX_DEVICES)
        return fail(nullptr, PIC1D_EDEVICE, "device index beyond the static scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(nullptr, PIC1D_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PIC1D_OK;
}

}  // namespace

extern "C" {

int pic1d_mlp_param_count(void) { return MLP_NPARAM; }

int pic1d_mlp_workspace_size(int64_t batch, int64_t n_pool, size_t* bytes) {
    if (!bytes || batch <= 0 || n_pool < 0) return fail(nullptr, PIC1D_EINVAL, "bad arguments");
    *bytes = mlp_layout(nullptr, batch, n_pool).bytes;
    return PIC1D_OK;
}

int pic1d_mlp_samples(uint64_t seed, int64_t first, int64_t n, float* x, float* o, void* workspace,
                      size_t workspace_bytes, void* stream) {
    if (n < 0 || first < 0 || (n > 0 && (!x || !o)) || (reinterpret_cast<uintptr_t>(x) & 15) ||
        (reinterpret_cast<uintptr_t>(o) & 15))
        return fail(nullptr, PIC1D_EINVAL, "bad arguments (x, o: device, 16-byte aligned, n x 4 floats)");
    if (int rc = check_workspace(workspace, workspace_bytes, PIC1D_MLP_SAMPLES_WORKSPACE)) return rc;
    if (n == 0) return PIC1D_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int* err = static_cast<int*>(workspace);
    MLP_TRY(hipMemsetAsync(err, 0, sizeof(int), s));
    uint32_t k0, k1;
    split_seed(seed, k0, k1);
    const int blocks = (int)std::min<int64_t>((n + MLP_TPB - 1) / MLP_TPB, 65536);
    hipLaunchKernelGGL(k_mlp_samples, dim3(blocks), dim3(MLP_TPB), 0, s, k0, k1, first, n, 4.0f,
                       reinterpret_cast<float4*>(x), reinterpret_cast<float4*>(o), err);
    MLP_TRY(hipGetLastError());
    int h = 0;
    MLP_TRY(hipMemcpyAsync(&h, err, sizeof(int), hipMemcpyDeviceToHost, s));
    MLP_TRY(hipStreamSynchronize(s));
    if (h) return fail(nullptr, PIC1D_ENONFINITE, "sample stream exhausted its attempts");
    return PIC1D_OK;
}

int pic1d_mlp_forward(const float* params, int64_t n, const float* x, float* out, void* workspace,
                      size_t workspace_bytes, void* stream) {
    if (!params || n < 0 || (n > 0 && (!x || !out)) || (reinterpret_cast<uintptr_t>(x) & 15))
        return fail(nullptr, PIC1D_EINVAL, "bad arguments");
    const MlpWork need = mlp_layout(nullptr, 1, 0);
    if (int rc = check_workspace(workspace, workspace_bytes, need.bytes)) return rc;
    const MlpWork w = mlp_layout(static_cast<char*>(workspace), 1, 0);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // (the small kernel reads the parameters 16 bytes at a time)
    if (n > 0 && n <= FWD_SMALL && (reinterpret_cast<uintptr_t>(params) & 15) == 0) {
        hipLaunchKernelGGL(k_mlp_forward_small, dim3((unsigned)((n + 15) / 16)), dim3(MLP_TPB), 0, s, params,
                           reinterpret_cast<const float4*>(x), n, out);
    } else if (n > 0) {
        hipLaunchKernelGGL(k_mlp_pack, dim3(64), dim3(MLP_TPB), 0, s, params, w.ft, w.bt, w.bias);
        const float4* X = reinterpret_cast<const float4*>(x);
        if (n >= FWD_LARGE) {
            int dev = 0, n_cu = 0;
            MLP_TRY(hipGetDevice(&dev));
            MLP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
            hipLaunchKernelGGL(k_mlp_forward_lds, dim3(n_cu), dim3(FWD_LDS_TPB), 0, s, w.ft, w.bias, X, n, out);
        } else {
            const int blocks = (int)std::min<int64_t>(FWD_BLOCKS, (n + 63) / 64);
            hipLaunchKernelGGL(k_mlp_forward, dim3(blocks), dim3(MLP_TPB), 0, s, w.ft, w.bias, X, n, out);
        }
    }
    MLP_TRY(hipGetLastError());
    MLP_TRY(hipStreamSynchronize(s));
    return PIC1D_OK;
}

int pic1d_mlp_loss_grad(const float* params, int64_t n, const float* x, const float* t, float* grad, double* loss,
                        void* workspace, size_t workspace_bytes, void* stream) {
    if (!params || n <= 0 || !x || !t || !grad || (reinterpret_cast<uintptr_t>(x) & 15))
        return fail(nullptr, PIC1D_EINVAL, "bad arguments");
    const MlpWork need = mlp_layout(nullptr, n, 0);
    if (int rc = check_workspace(workspace, workspace_bytes, need.bytes)) return rc;
    const MlpWork w = mlp_layout(static_cast<char*>(workspace), n, 0);
    return loss_grad_on(w, params, n, x, t, grad, loss, static_cast<hipStream_t>(stream));
}

int pic1d_mlp_loss_grad_static(const float* params, int64_t n, const float* x, const float* t, float* grad,
                               double* loss, void* stream) {
    if (!params || n <= 0 || !x || !t || !grad || (reinterpret_cast<uintptr_t>(x) & 15))
        return fail(nullptr, PIC1D_EINVAL, "bad arguments");
    if (n > MLP_STATIC_MAX_ROWS)
        return fail(nullptr, PIC1D_EINVAL,
                    "n exceeds the static scratch of pic1d_mlp_loss_grad_static (at most 2048 samples per call)");
    // every layout up to the maximum batch fits the array (checked, not assumed)
    if (mlp_layout(nullptr, MLP_STATIC_MAX_ROWS, 0).bytes > MLP_STATIC_BYTES)
        return fail(nullptr, PIC1D_ENOMEM, "static scratch smaller than the layout of its maximum batch");
    void* base = nullptr;
    if (int rc = static_scratch(&base)) return rc;
    const MlpWork w = mlp_layout(static_cast<char*>(base), n, 0);
    return loss_grad_on(w, params, n, x, t, grad, loss, static_cast<hipStream_t>(stream));
}

int pic1d_mlp_adam(float* params, float* m, float* v, const float* grad, int64_t t, double lr, double beta1,
                   double beta2, double eps, void* stream) {
    if (!params || !m || !v || !grad || t < 1 || !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0))
        return fail(nullptr, PIC1D_EINVAL, "bad arguments");
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_mlp_adam, dim3(ADAM_BLOCKS), dim3(MLP_TPB), 0, s, grad, 1, params, m, v, nullptr, 1,
                       adam_args(lr, beta1, beta2, eps, t), PackedNet{});
    MLP_TRY(hipGetLastError());
    MLP_TRY(hipStreamSynchronize(s));
    return PIC1D_OK;
}

int pic1d_mlp_train(const pic1d_mlp_train_config* c, pic1d_mlp_train_result* res) {
    if (!c || !res || c->n_samples <= 0 || c->batch <= 0 || c->steps < 0 || !(c->lr > 0.0f) ||
        !(c->lr_final >= 0.0f) || !res->params || !res->norm)
        return fail(nullptr, PIC1D_EINVAL, "bad arguments");
    const MlpWork need = mlp_layout(nullptr, c->batch, c->n_samples);
    if (int rc = check_workspace(c->workspace, c->workspace_bytes, need.bytes)) return rc;
    const MlpWork w = mlp_layout(static_cast<char*>(c->workspace), c->batch, c->n_samples);
    hipStream_t s = static_cast<hipStream_t>(c->stream);
    const auto t0 = std::chrono::steady_clock::now();
    uint32_t k0, k1;
    split_seed(c->seed, k0, k1);

    // samples and their normalisation
    MLP_TRY(hipMemsetAsync(w.err, 0, sizeof(int), s));
    hipLaunchKernelGGL(k_mlp_samples, dim3((int)std::min<int64_t>((c->n_samples + MLP_TPB - 1) / MLP_TPB, 65536)),
                       dim3(MLP_TPB), 0, s, k0, k1, (int64_t)0, c->n_samples, 4.0f, w.X, w.O, w.err);
    hipLaunchKernelGGL(k_mlp_stats, dim3(STAT_BLOCKS), dim3(MLP_TPB), 0, s, w.O, c->n_samples, 0, nullptr, w.stat_part);
    std::vector<double> part(3 * STAT_BLOCKS);
    MLP_TRY(hipMemcpyAsync(part.data(), w.stat_part, sizeof(double) * part.size(), hipMemcpyDeviceToHost, s));
    int herr = 0;
    MLP_TRY(hipMemcpyAsync(&herr, w.err, sizeof(int), hipMemcpyDeviceToHost, s));
    MLP_TRY(hipStreamSynchronize(s));
    if (herr) return fail(nullptr, PIC1D_ENONFINITE, "sample stream exhausted its attempts");
    double mean[4] = {0, 0, 0, 0}, var[3] = {0, 0, 0};
    for (int b = 0; b < STAT_BLOCKS; ++b)
        for (int k = 0; k < 3; ++k) mean[k] += part[b * 3 + k];
    for (int k = 0; k < 3; ++k) mean[k] /= (double)c->n_samples;
    MLP_TRY(hipMemcpyAsync(w.mean_dev, mean, sizeof(double) * 4, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_mlp_stats, dim3(STAT_BLOCKS), dim3(MLP_TPB), 0, s, w.O, c->n_samples, 1, w.mean_dev,
                       w.stat_part);
    MLP_TRY(hipMemcpyAsync(part.data(), w.stat_part, sizeof(double) * part.size(), hipMemcpyDeviceToHost, s));
    MLP_TRY(hipStreamSynchronize(s));
    for (int b = 0; b < STAT_BLOCKS; ++b)
        for (int k = 0; k < 3; ++k) var[k] += part[b * 3 + k];
    float norm[8] = {0};
    for (int k = 0; k < 3; ++k) {
        norm[k] = (float)mean[k];
        norm[3 + k] = (float)std::sqrt(var[k] / (double)c->n_samples);
        if (!(norm[3 + k] > 0.0f)) norm[3 + k] = 1.0f;
    }
    MLP_TRY(hipMemcpyAsync(w.norm, norm, sizeof(norm), hipMemcpyHostToDevice, s));

    // initial weights, zero moments
    if (c->init_params) {
        MLP_TRY(hipMemcpyAsync(w.master, c->init_params, sizeof(float) * MLP_NPARAM, hipMemcpyHostToDevice, s));
    } else {
        hipLaunchKernelGGL(k_mlp_init, dim3(64), dim3(MLP_TPB), 0, s, k0, k1, w.master);
    }
    MLP_TRY(hipMemsetAsync(w.m, 0, sizeof(float) * MLP_NPARAM, s));
    MLP_TRY(hipMemsetAsync(w.v, 0, sizeof(float) * MLP_NPARAM, s));
    MLP_TRY(hipMemsetAsync(w.XN, 0, sizeof(float4) * w.rows, s));

    TrainArgs fa{};
    fa.ft = w.ft; fa.bias = w.bias; fa.X = w.X; fa.T = nullptr; fa.O = w.O; fa.norm = w.norm;
    fa.n_batch = c->batch; fa.n_pool = c->n_samples; fa.k0 = k0; fa.k1 = k1;
    fa.XN = w.XN; fa.Z = w.Z; fa.DS = w.DS; fa.DOUT = w.DOUT; fa.bt = w.bt; fa.zlayer = w.rows * MLP_W; fa.loss_part = w.loss_part;
    const double b1 = c->beta1 > 0.0 ? c->beta1 : 0.9, b2 = c->beta2 > 0.0 ? c->beta2 : 0.999;
    const double eps = c->eps > 0.0 ? c->eps : 1e-8;
    const int nlog = std::max(0, std::min(res->n_loss, c->steps));
    int logged = 0;
    res->loss_first = NAN;
    hipLaunchKernelGGL(k_mlp_pack, dim3(64), dim3(MLP_TPB), 0, s, w.master, w.ft, w.bt, w.bias);
    const PackedNet net{reinterpret_cast<__bf16*>(w.ft), reinterpret_cast<__bf16*>(w.bt), w.bias};
    for (int t = 1; t <= c->steps; ++t) {
        fa.step = (uint32_t)t;
        if (int rc = run_grad(w, fa, s)) return rc;
        const double lr = c->lr_final + 0.5 * (c->lr - c->lr_final) *
                                            (1.0 + std::cos(3.141592653589793 * (double)(t - 1) / (double)c->steps));
        hipLaunchKernelGGL(k_mlp_adam, dim3(ADAM_BLOCKS), dim3(MLP_TPB), 0, s, w.partial, w.nchunk, w.master, w.m, w.v,
                           nullptr, 1, adam_args(lr, b1, b2, eps, t), net);
        MLP_TRY(hipGetLastError());
        const bool first = t == 1;
        const bool log_now = nlog > 0 && res->loss && logged < nlog &&
                             (int64_t)(t - 1) * nlog / c->steps >= logged;
        if (first || log_now || t == c->steps) {
            const double l = sum_loss(w, train_blocks(w.rows), s) / (3.0 * (double)c->batch);
            if (first) res->loss_first = l;
            if (log_now) res->loss[logged++] = l;
            if (t == c->steps) res->loss_last = l;
        }
    }
    MLP_TRY(hipMemcpyAsync(res->params, w.master, sizeof(float) * MLP_NPARAM, hipMemcpyDeviceToHost, s));
    MLP_TRY(hipStreamSynchronize(s));
    for (int k = 0; k < 6; ++k) res->norm[k] = norm[k];
    res->n_loss = logged;
    res->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return PIC1D_OK;
}

}  // extern "C"
