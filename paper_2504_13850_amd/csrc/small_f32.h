// Pieces shared by the fused steps of the small fp32 convolution networks
// (MobileNetV3-Large's and VGG-5's server parts): products over a few dozen
// samples and weight gradients on fp32 MFMA.  Operands are stored feature by
// feature, [C][ld], rows (sample, pixel) contiguous and padded with zeros to a
// multiple of 16.
#pragma once

#include "kernels.h"

namespace fo {
namespace {

__device__ __forceinline__ float hswish(float x) { return x * fminf(fmaxf(x + 3.f, 0.f), 6.f) * (1.f / 6.f); }
__device__ __forceinline__ float hswish_d(float x) { return x < -3.f ? 0.f : (x > 3.f ? 1.f : (2.f * x + 3.f) / 6.f); }
__device__ __forceinline__ float hsig(float x) { return fminf(fmaxf(x + 3.f, 0.f), 6.f) * (1.f / 6.f); }
__device__ __forceinline__ float hsig_d(float x) { return x > -3.f && x < 3.f ? 1.f / 6.f : 0.f; }

__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ void st4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }

// Element (channel c, row r) of an activation: p + (r / 16) sb + c sc + r % 16.
// sb = 16 is the channel-major layout; the batch as sent ([B][80][4][4], p NULL)
// has sb = 80 * 16, sc = 16.
struct Act2 {
    const float* p;
    int64_t sb, sc;
};
__device__ __forceinline__ const float* act_ptr(const Act2& a, const StepIn* in) {
    return a.p ? a.p : static_cast<const float*>(in->x);
}
__device__ __forceinline__ int64_t act_row(const Act2& a, int r) { return (int64_t)(r >> 4) * a.sb + (r & 15); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
// ------------------------------------------------------------------ layers over the samples (SE and classifier)
// Y[n][b] = epi(sum_k W(n, k) X[k][b]) on v_mfma_f32_16x16x4_f32: a workgroup
// takes 16 outputs of 32 samples, its eight waves an eighth of k each (the
// products are a few hundred long and at most 80 workgroups wide, so their time
// is the length of the k walk), added in order.  A wave keeps two running sums
// (the rounding error grows with their length).  TR: W(n, k) = W[k][n].
enum Epi : int { E_RELU, E_SCALE, E_HSWISH, E_LOGITS, E_DHSWISH, E_PLAIN, E_DRELU };
constexpr int LIN_T = 512;  // threads: eight waves, an eighth of k each
struct Lin {
    const float* W;
    const float* X;    // [K][ldb]
    const float* bias;
    float* out;        // [N][ldb]
    const float* aux;  // E_DHSWISH: the pre-activation, E_DRELU: the activation, [N][ldb]
    float* out2;       // E_HSWISH: the activation (out: before it); E_LOGITS: [B][N]
    const float* a2;   // E_SCALE: the maps [N][ld2] and their scaled copy
    float* h;
    int N, K, B, ldb, hw, ld2;
};

template <bool TR, int EPI>
__global__ void __launch_bounds__(LIN_T) linear_small(const Lin p) {
    __shared__ float red[8][2][256];
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * 16, b0 = blockIdx.y * 32;
    const int kper = (p.K + 127) / 128 * 16;
    const int k0 = min(w * kper, p.K), k1 = min(k0 + kper, p.K);
    const int n = min(n0 + tok, p.N - 1);
    const int c1 = min(b0 + 16 + tok, p.ldb - 1);
    const float *x0 = p.X + b0 + tok, *x1 = p.X + c1;
    f32x4 a0[2], a1[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) a0[h] = a1[h] = f32x4{0.f, 0.f, 0.f, 0.f};
    // 32 of k per turn, every load of a turn in flight before its first product.
    // K is a multiple of 8: a group of four is inside or outside as a whole.
    for (int k = k0; k < k1; k += 32) {
        float a[2][4], u[2][4], v[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kk = k + 16 * h + 4 * g, kc = min(kk, k1 - 4);
            if constexpr (TR) {
#pragma unroll
                for (int j = 0; j < 4; ++j) a[h][j] = p.W[(int64_t)(kc + j) * p.N + n];
            } else {
                const f32x4 t = ld4(p.W + (int64_t)n * p.K + kc);
#pragma unroll
                for (int j = 0; j < 4; ++j) a[h][j] = t[j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                u[h][j] = x0[(int64_t)(kc + j) * p.ldb];
                v[h][j] = x1[(int64_t)(kc + j) * p.ldb];
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool on = k + 16 * h + 4 * g < k1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float w = on ? a[h][j] : 0.f;
                a0[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, u[h][j], a0[h], 0, 0, 0);
                a1[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, v[h][j], a1[h], 0, 0, 0);
            }
        }
    }
    const f32x4 s0 = a0[0] + a0[1], s1 = a1[0] + a1[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        red[w][0][(4 * g + i) * 16 + tok] = s0[i];
        red[w][1][(4 * g + i) * 16 + tok] = s1[i];
    }
    __syncthreads();
    const int half = threadIdx.x >> 8, e = threadIdx.x & 255;
    const int on = n0 + (e >> 4), b = b0 + 16 * half + (e & 15);
    if (on >= p.N || b >= p.ldb) return;
    float v = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) v += red[s][half][e];
    const int64_t o = (int64_t)on * p.ldb + b;
    const bool in = b < p.B;  // padding samples hold zeros
    if constexpr (EPI == E_RELU) p.out[o] = in ? fmaxf(v + p.bias[on], 0.f) : 0.f;
    if constexpr (EPI == E_PLAIN) p.out[o] = in ? v : 0.f;
    if constexpr (EPI == E_DRELU) p.out[o] = in && p.aux[o] > 0.f ? v : 0.f;
    if constexpr (EPI == E_DHSWISH) p.out[o] = in ? v * hswish_d(p.aux[o]) : 0.f;
    if constexpr (EPI == E_HSWISH) {
        const float z = v + p.bias[on];
        p.out[o] = in ? z : 0.f;
        p.out2[o] = in ? hswish(z) : 0.f;
    }
    if constexpr (EPI == E_LOGITS) {
        if (in) p.out2[(int64_t)b * p.N + on] = v + p.bias[on];
    }
    if constexpr (EPI == E_SCALE) {
        const float z = in ? v + p.bias[on] : 0.f, s = hsig(z);
        p.out[o] = z;
        // the maps' padding rows too (a is zero there): the projection's weight gradient
        // multiplies them by zeros, and a shorter batch finds an earlier one's values there
        if (b * p.hw >= p.ld2) return;
        const float* a = p.a2 + (int64_t)on * p.ld2 + b * p.hw;
        float* h = p.h + (int64_t)on * p.ld2 + b * p.hw;
        for (int q = 0; q < p.hw; q += 4) st4(h + q, ld4(a + q) * s);
    }
}

// ------------------------------------------------------------------ classifier of ten classes
// Between the last hidden layer f [F][ldb] and its gradient, one workgroup:
// logits [B][10], mean cross-entropy (labels clamped and counted), dz, df = dz W
// (where f > 0 if RELU), the classifier's gradients and update (prm / grd: its
// weights [10][F], then its biases).  128 samples at a time in LDS.
template <int F, bool RELU>
__global__ void __launch_bounds__(1024) small_head(const float* __restrict__ f1, int ldb,
                                                   const StepIn* __restrict__ in, float* __restrict__ prm,
                                                   float* __restrict__ grd, float lr, int B,
                                                   float* __restrict__ logits, float* __restrict__ loss,
                                                   float* __restrict__ df1) {
    constexpr int C = 10, NB = 128, NG = (C * F + C + 1023) / 1024;
    __shared__ float f[F][NB + 1], dz[C][NB + 1], w[C * F], part[2];
    __shared__ int badw[2];
    const int t = threadIdx.x;
    for (int e = t; e < C * F; e += 1024) w[e] = prm[e];
    float grad[NG] = {}, mine = 0.f;
    int bad = 0;
    for (int b0 = 0; b0 < ldb; b0 += NB) {
        const int nb = min(NB, ldb - b0), nv = min(NB, B - b0);  // samples with padding, samples
        __syncthreads();
        for (int e = t; e < F * nb; e += 1024) {  // (f1's padding may hold anything)
            const int k = e / nb, b = e % nb;
            f[k][b] = b < nv ? f1[(int64_t)k * ldb + b0 + b] : 0.f;
        }
        __syncthreads();
        for (int e = t; e < nv * C; e += 1024) {
            const int n = e / nv, b = e % nv;
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            for (int k = 0; k < F; k += 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] = fmaf(f[k + j][b], w[n * F + k + j], s[j]);
            const float v = ((s[0] + s[1]) + (s[2] + s[3])) + prm[C * F + n];
            dz[n][b] = v;
            logits[(int64_t)(b0 + b) * C + n] = v;
        }
        __syncthreads();
        if (t < nv) {  // a thread per sample
            float m = -INFINITY, s = 0.f;
#pragma unroll
            for (int n = 0; n < C; ++n) m = fmaxf(m, dz[n][t]);
#pragma unroll
            for (int n = 0; n < C; ++n) s += expf(dz[n][t] - m);
            const float lse = m + logf(s);
            int y = in->labels[b0 + t];
            if (y < 0 || y >= C) {
                ++bad;
                y = y < 0 ? 0 : C - 1;
            }
            mine += lse - dz[y][t];
#pragma unroll
            for (int n = 0; n < C; ++n) dz[n][t] = (expf(dz[n][t] - lse) - (n == y ? 1.f : 0.f)) / (float)B;
        } else if (t < nb) {
#pragma unroll
            for (int n = 0; n < C; ++n) dz[n][t] = 0.f;
        }
        __syncthreads();
        for (int e = t; e < F * nb; e += 1024) {
            const int k = e / nb, b = e % nb;
            float s = 0.f;
#pragma unroll
            for (int n = 0; n < C; ++n) s = fmaf(dz[n][b], w[n * F + k], s);
            df1[(int64_t)k * ldb + b0 + b] = !RELU || f[k][b] > 0.f ? s : 0.f;  // (padding samples: dz = 0)
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int e = t + 1024 * i;
            float s = 0.f, u = 0.f;
            if (e < C * F) {
                for (int b = 0; b < nv; b += 2) {  // (an odd last sample is followed by zeros in both)
                    s = fmaf(dz[e / F][b], f[e % F][b], s);
                    u = fmaf(dz[e / F][b + 1], f[e % F][b + 1], u);
                }
            } else if (e < C * F + C) {
                for (int b = 0; b < nv; ++b) s += dz[e - C * F][b];
            }
            grad[i] += s + u;
        }
    }
    if (t < NB) {
        mine = wave_sum(mine);
        for (int o = 32; o > 0; o >>= 1) bad += __shfl_xor(bad, o);
        if ((t & 63) == 0) {
            part[t >> 6] = mine;
            badw[t >> 6] = bad;
        }
    }
    __syncthreads();  // (also: every read of the biases is done)
    if (t == 0) {
        loss[0] = (part[0] + part[1]) / (float)B;
        loss[1] = (float)(badw[0] + badw[1]);
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const int e = t + 1024 * i;
        if (e >= C * F + C) break;
        const float old = prm[e];
        grd[e] = grad[i];
        prm[e] = __builtin_fmaf(-lr, grad[i], old);
    }
}

// ------------------------------------------------------------------ weight gradients and their update
// dW[n][k] = sum_r dY[n][r] X[k][r] of a product, 32 x 32 per wave (four
// MFMA tiles fed by four 16-byte loads per 16 rows, both operands contiguous in
// r), the gradient stored and the weight updated (theta <- theta - lr g); the
// waves of a product's first column of tiles also add up its bias gradient.
struct WUnit {
    const float* dy;  // [N][ld]
    Act2 x;           // [K] rows
    int64_t w, bias;  // parameter offsets (bias: -1 without one)
    int N, K, ld, task0;  // ld: rows, a multiple of 16; task0: the product's first task
};
// id: the wave's tile of the product (wave-uniform).
__device__ __forceinline__ void wgrad_32x32(const WUnit& u, int id, const StepIn* __restrict__ in,
                                            float* __restrict__ prm, float* __restrict__ grd, float lr) {
    const int kt = (u.K + 31) / 32, n0 = id / kt * 32, k0 = id % kt * 32;
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4;
    const float* x = act_ptr(u.x, in);
    const float *yr[2], *xr[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        yr[i] = u.dy + (int64_t)min(n0 + 16 * i + tok, u.N - 1) * u.ld + 4 * g;
        xr[i] = x + (int64_t)min(k0 + 16 * i + tok, u.K - 1) * u.x.sc + 4 * g;
    }
    f32x4 acc[2][2];
    float bs[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ld = u.ld;
    const int64_t sb = u.x.sb;
    f32x4 y[2], v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        y[i] = ld4(yr[i]);
        v[i] = ld4(xr[i]);
    }
    for (int r = 0; r < ld; r += 16) {
        const int rn = min(r + 16, ld - 16);  // the next rows in flight during these products
        f32x4 yn[2], vn[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            yn[i] = ld4(yr[i] + rn);
            vn[i] = ld4(xr[i] + (rn >> 4) * sb);
            bs[i] += (y[i][0] + y[i][1]) + (y[i][2] + y[i][3]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)  // column n = lane % 16, rows k = 4 g ..: four weights per lane
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j][q], y[i][q], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            y[i] = yn[i];
            v[i] = vn[i];
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = n0 + 16 * i + tok;
        if (u.bias >= 0 && k0 == 0) {
            float s = bs[i];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (g == 0 && n < u.N) {
                grd[u.bias + n] = s;
                prm[u.bias + n] = __builtin_fmaf(-lr, s, prm[u.bias + n]);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = k0 + 16 * j + 4 * g;
            if (n >= u.N || k >= u.K) continue;
            const int64_t o = u.w + (int64_t)n * u.K + k;
            f32x4 w = ld4(prm + o);
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = __builtin_fmaf(-lr, acc[i][j][q], w[q]);
            st4(grd + o, acc[i][j]);
            st4(prm + o, w);
        }
    }
}

inline int pad16(int n) { return (n + 15) / 16 * 16; }

}  // namespace
}  // namespace fo
