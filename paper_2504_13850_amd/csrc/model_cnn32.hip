// Config 1: the tiny fp32 CNN server network, one training iteration of the
// activation branch of Alg. 4:
//   conv3x3 32->64 + bias + ReLU, maxpool 2x2, conv3x3 64->64 + bias + ReLU,
//   global average pool, linear 64->10, mean cross-entropy, backward, SGD.
// Everything is fp32; the activation gradient of the first conv is never
// formed.
//
// The network is 0.5 GFLOP at batch 16, so launches (4.5 us each) and the
// latency inside them are the step.  Convolutions run as implicit GEMMs on
// v_mfma_f32_16x16x4_f32 with one image and its border of zeros in LDS: in the
// forward and the input gradient 16 output channels by 16 pixels per wave (the
// weights' k = (tap, channel) is contiguous), in the weight gradients 16 input
// channels by nine taps per wave over the image's pixels.  Pooling, ReLU, the
// global average and their backward sit in the neighbouring convolution, and
// the second convolution's weight gradient shares a launch with its input
// gradient: 7 launches instead of 14, 176 -> 59 us at batch 16.
#include "model.h"
#include "small_f32.h"

namespace fo {

namespace {

constexpr int C0 = 32, C1 = 64, C2 = 64, H0 = 16, H1 = 8, P0 = H0 * H0, P1 = H1 * H1, NCLS = 10;
constexpr int64_t kW1 = (int64_t)C1 * 9 * C0, kW2 = (int64_t)C2 * 9 * C1, kFc = (int64_t)NCLS * C2;
constexpr int64_t oW1 = 0, oB1 = oW1 + kW1, oW2 = oB1 + C1, oB2 = oW2 + kW2, oWf = oB2 + C2;
constexpr int64_t kParams = oWf + kFc + NCLS;
constexpr int kShares = 64;  // shares of the images in a weight gradient (one image each at batch 16)
constexpr int T = 256;       // threads of a convolution kernel: four waves

struct Plan {
    float* p1;      // conv1 + ReLU, pooled [B][64][8][8]
    uint8_t* arg1;  // window position of its maximum (the first in row-major order)
    float* y2;      // conv2 + ReLU [B][64][8][8]
    float* h;       // global average [64][ldb], samples only (its padding is not written)
    float* dh;      // its gradient
    float* dp1;     // gradient of p1 where p1 > 0
    float *part1, *part2;  // the weight gradients' shares [shares][64][9 Ci + 1], the bias last
};
constexpr int kRow1 = 9 * C0 + 4, kRow2 = 9 * C1 + 4;  // a partial row: weights, bias, padding to 16 bytes

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// A product is kept as several running sums, added pairwise: the error of a sum
// grows with the length of its chain of additions.  Four in the first
// convolution and NP in the second and its input gradient (72 products each),
// NPW per image in the weight gradients (32 and 64 pixels each; three taps at a
// time, as two running sums of all nine leave no registers for a third wave per
// SIMD).  Median error of the gradient over 24 batches of 16: 6.6e-8, with half
// as many sums and one over all images 7.9e-8; the step takes 58.5 against 57.6 us.
constexpr int NP = 8, NPW = 2;
template <int N>
__device__ __forceinline__ f32x4 pairwise(const f32x4* a) {
    if constexpr (N == 1)
        return a[0];
    else
        return pairwise<N / 2>(a) + pairwise<N / 2>(a + N / 2);
}

// Rows y0 - 1 .. y0 + NR of an image [C][H][H] into xs[C][NR + 2][H + 2] (LDS), zeros outside.
template <int C, int H, int NR>
__device__ __forceinline__ void stage(const float* __restrict__ x, int y0, float* xs) {
    constexpr int W = H + 2, S = (NR + 2) * W;
    for (int e = threadIdx.x; e < C * (NR + 2) * (H / 4); e += T) {
        const int c = e / ((NR + 2) * (H / 4)), r = e / (H / 4) % (NR + 2), q = e % (H / 4), y = y0 + r - 1;
        const bool in = y >= 0 && y < H;
        const f32x4 v = ld4(x + c * H * H + (in ? y : 0) * H + 4 * q);
        float* o = xs + c * S + r * W + 1 + 4 * q;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = in ? v[i] : 0.f;
    }
    for (int e = threadIdx.x; e < C * (NR + 2); e += T) xs[e * W] = xs[e * W + W - 1] = 0.f;
}

// conv1 + ReLU + 2x2 max pool: block = (image, 16 channels, half the rows); a
// tile is 2 x 8 pixels, so a window's four values are lanes l, l ^ 1, l ^ 8, l ^ 9.
__global__ void __launch_bounds__(T) c1_fwd(const StepIn* __restrict__ in, const float* __restrict__ w,
                                            const float* __restrict__ bias, float* __restrict__ p1,
                                            uint8_t* __restrict__ arg1) {
    constexpr int NR = H0 / 2, W = H0 + 2, S = (NR + 2) * W;
    __shared__ float xs[C0 * S];
    const int b = blockIdx.x, co = blockIdx.y * 16, y0 = blockIdx.z * NR;
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    const f32x4 bv = ld4(bias + co + 4 * g);
    stage<C0, H0, NR>(static_cast<const float*>(in->x) + (int64_t)b * C0 * P0, y0, xs);
    __syncthreads();
    // the wave's two tiles: rows 2 wave, 2 wave + 1, columns 0-7 and 8-15
    const float* xr = xs + (2 * wave + (tok >> 3)) * W + (tok & 7);
    const float* wr = w + (int64_t)(co + tok) * 9 * C0 + 4 * g;
    f32x4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int s = 0; s < C0 / 16; ++s) {
            const f32x4 a = ld4(wr + t * C0 + 16 * s);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i][j] = mfma(a[j], xr[(16 * s + 4 * g + j) * S + t / 3 * W + t % 3 + 8 * i], acc[i][j]);
        }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const f32x4 z = pairwise<4>(acc[i]) + bv;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float v0 = fmaxf(z[k], 0.f), v1 = __shfl_xor(v0, 1), v2 = __shfl_xor(v0, 8), v3 = __shfl_xor(v1, 8);
            float best = v0;
            int at = 0;
            if (v1 > best) { best = v1; at = 1; }
            if (v2 > best) { best = v2; at = 2; }
            if (v3 > best) { best = v3; at = 3; }
            if ((tok & 9) == 0) {
                const int64_t o = ((int64_t)b * C1 + co + 4 * g + k) * P1 + (y0 / 2 + wave) * H1 + 4 * i + (tok & 7) / 2;
                p1[o] = best;
                arg1[o] = (uint8_t)at;
            }
        }
    }
}

// conv2 + ReLU and the global average: block = (image, 16 channels), 16 pixels per wave.
__global__ void __launch_bounds__(T) c2_fwd(const float* __restrict__ p1, const float* __restrict__ w,
                                            const float* __restrict__ bias, float* __restrict__ y2,
                                            float* __restrict__ h, int ldb) {
    constexpr int W = H1 + 2, S = W * W;
    __shared__ float xs[C1 * S], red[4][16];
    const int b = blockIdx.x, co = blockIdx.y * 16;
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    const f32x4 bv = ld4(bias + co + 4 * g);
    // the weights of a tap are loaded during the products of the one before
    const float* wr = w + (int64_t)(co + tok) * 9 * C1 + 4 * g;
    f32x4 a[2][C1 / 16];
#pragma unroll
    for (int s = 0; s < C1 / 16; ++s) a[0][s] = ld4(wr + 16 * s);
    stage<C1, H1, H1>(p1 + (int64_t)b * C1 * P1, 0, xs);
    __syncthreads();
    const int px = 16 * wave + tok;
    const float* xr = xs + px / H1 * W + px % H1;
    f32x4 acc[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        if (t + 1 < 9)
#pragma unroll
            for (int s = 0; s < C1 / 16; ++s) a[(t + 1) & 1][s] = ld4(wr + (t + 1) * C1 + 16 * s);
#pragma unroll
        for (int s = 0; s < C1 / 16; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4& c = acc[(4 * s + j) % NP];
                c = mfma(a[t & 1][s][j], xr[(16 * s + 4 * g + j) * S + t / 3 * W + t % 3], c);
            }
    }
    const f32x4 z = pairwise<NP>(acc) + bv;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float v = fmaxf(z[k], 0.f);
        y2[((int64_t)b * C2 + co + 4 * g + k) * P1 + px] = v;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (tok == 0) red[wave][4 * g + k] = v;
    }
    __syncthreads();
    if (threadIdx.x < 16)
        h[(int64_t)(co + threadIdx.x) * ldb + b] =
            ((red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x])) / (float)P1;
}

// The lane's bias gradient (its sum over the rows it held) over the four lane groups.
__device__ __forceinline__ float groups_sum(float v) {
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// conv2 backward.  Blocks below 4 * shares (first: they are the longest): conv2's
// weight and bias gradient of (share of the images, 16 output channels).  The
// rest: the input gradient of (image, 16 input channels) through the pool's
// ReLU; the gradient of conv2's output is [y2 > 0] dh / 64, formed while it is staged.
__global__ void __launch_bounds__(T) c2_bwd(const float* __restrict__ p1, const float* __restrict__ y2,
                                            const float* __restrict__ dh, int ldb, const float* __restrict__ w,
                                            float* __restrict__ dp1, float* __restrict__ part, int B, int shares) {
    constexpr int W = H1 + 2, S = W * W;
    __shared__ float xs[C1 * S];
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    if ((int)blockIdx.x >= 4 * shares) {
        const int b = blockIdx.x / 4 - shares, ci = blockIdx.x % 4 * 16;
        const float* wr = w + ci + tok;
        float a[2][16];  // a tap's weights, loaded during the products of the one before
        auto load = [&](int t) {
#pragma unroll
            for (int q = 0; q < 16; ++q) a[t & 1][q] = wr[((16 * (q / 4) + 4 * g + q % 4) * 9 + t) * C1];
        };
        load(0);
        for (int e = threadIdx.x; e < C2 * P1 / 4; e += T) {
            const int c = e / (P1 / 4), q = e % (P1 / 4) * 4;
            const f32x4 v = ld4(y2 + (int64_t)b * C2 * P1 + 4 * e);
            const float d = dh[(int64_t)c * ldb + b] / (float)P1;
            float* o = xs + c * S + (q / H1 + 1) * W + q % H1 + 1;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = v[i] > 0.f ? d : 0.f;
        }
        for (int e = threadIdx.x; e < C2 * 4 * (W - 1); e += T) {  // the border
            const int c = e / (4 * (W - 1)), k = e % (4 * (W - 1)), i = k % (W - 1);
            const int at = k / (W - 1) == 0   ? i
                           : k / (W - 1) == 1 ? (W - 1) * W + i + 1
                           : k / (W - 1) == 2 ? (i + 1) * W
                                              : i * W + W - 1;
            xs[c * S + at] = 0.f;
        }
        __syncthreads();
        const int px = 16 * wave + tok;
        const float* xr = xs + px / H1 * W + px % H1;
        f32x4 acc[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            if (t + 1 < 9) load(t + 1);
#pragma unroll
            for (int q = 0; q < 16; ++q)
                acc[q % NP] = mfma(a[t & 1][q], xr[(16 * (q / 4) + 4 * g + q % 4) * S + (2 - t / 3) * W + 2 - t % 3],
                                   acc[q % NP]);
        }
        const f32x4 v = pairwise<NP>(acc);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t o = ((int64_t)b * C1 + ci + 4 * g + k) * P1 + px;
            dp1[o] = p1[o] > 0.f ? v[k] : 0.f;
        }
        return;
    }
    const int share = blockIdx.x / 4, co = blockIdx.x % 4 * 16;
    f32x4 acc[9];
    float bs[4] = {};
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* xr = xs + (16 * wave + tok) * S;
    for (int b = share; b < B; b += shares) {
        if (b != share) __syncthreads();
        stage<C1, H1, H1>(p1 + (int64_t)b * C1 * P1, 0, xs);
        const float d1 = dh[(int64_t)(co + tok) * ldb + b] / (float)P1;
        f32x4 d[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            d[s] = ld4(y2 + ((int64_t)b * C2 + co + tok) * P1 + 16 * s + 4 * g);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                d[s][j] = d[s][j] > 0.f ? d1 : 0.f;
                bs[s] += d[s][j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            f32x4 c[3][NPW];
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int s = 0; s < NPW; ++s) c[kx][s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int px = 16 * s + 4 * g + j;
                    const float* x = xr + (px / H1 + ky) * W + px % H1;
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) c[kx][s % NPW] = mfma(x[kx], d[s][j], c[kx][s % NPW]);
                }
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) acc[3 * ky + kx] += pairwise<NPW>(c[kx]);
        }
    }
    float* o = part + ((int64_t)share * C2 + co + tok) * kRow2;
#pragma unroll
    for (int t = 0; t < 9; ++t) st4(o + t * C1 + 16 * wave + 4 * g, acc[t]);
    const float b4 = groups_sum((bs[0] + bs[1]) + (bs[2] + bs[3]));
    if (wave == 0 && g == 0) o[9 * C1] = b4;
}

// conv1's weight and bias gradient: block = (share of the images, 16 output
// channels); waves are the two blocks of 16 input channels by the image's two
// halves (added through LDS at the end).  The gradient of conv1's output is dp1
// at its window's maximum, formed in registers.
__global__ void __launch_bounds__(T) c1_wgrad(const StepIn* __restrict__ in, const float* __restrict__ dp1,
                                              const uint8_t* __restrict__ arg1, float* __restrict__ part, int B,
                                              int shares) {
    constexpr int W = H0 + 2, S = W * W;
    __shared__ __attribute__((aligned(16))) float xs[C0 * S];
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    const int share = blockIdx.x / 4, co = blockIdx.x % 4 * 16, cb = wave & 1, half = wave >> 1;
    f32x4 acc[9];
    float bs[4] = {};
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* xr = xs + (16 * cb + tok) * S;
    for (int b = share; b < B; b += shares) {
        if (b != share) __syncthreads();
        stage<C0, H0, H0>(static_cast<const float*>(in->x) + (int64_t)b * C0 * P0, 0, xs);
        // the lane's channel: pooled columns 2 g, 2 g + 1 of the half's four pooled rows
        const int64_t q = ((int64_t)b * C1 + co + tok) * P1 + 4 * half * H1 + 2 * g;
        float d[4][2];
        int at[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                d[r][c] = dp1[q + r * H1 + c];
                at[r][c] = arg1[q + r * H1 + c];
                bs[r] += d[r][c];
            }
        __syncthreads();
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            f32x4 c[3][NPW];
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int s = 0; s < NPW; ++s) c[kx][s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = at[r / 2][j / 2] == (r & 1) * 2 + (j & 1) ? d[r / 2][j / 2] : 0.f;
                    const float* x = xr + (8 * half + r + ky) * W + 4 * g + j;
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) c[kx][r % NPW] = mfma(x[kx], v, c[kx][r % NPW]);
                }
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) acc[3 * ky + kx] += pairwise<NPW>(c[kx]);
        }
    }
    const float b4 = groups_sum((bs[0] + bs[1]) + (bs[2] + bs[3]));
    __syncthreads();
    float* o = part + ((int64_t)share * C1 + co + tok) * kRow1;
    f32x4* red = reinterpret_cast<f32x4*>(xs) + cb * 64 * 10 + lane;
    if (half) {
#pragma unroll
        for (int t = 0; t < 9; ++t) red[64 * t] = acc[t];
        red[64 * 9] = f32x4{b4, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    if (half) return;
#pragma unroll
    for (int t = 0; t < 9; ++t) st4(o + t * C0 + 16 * cb + 4 * g, acc[t] + red[64 * t]);
    if (cb == 0 && g == 0) o[9 * C0] = b4 + red[64 * 9][0];
}
static_assert(2 * 64 * 10 * 4 <= C0 * (H0 + 2) * (H0 + 2), "partial sums of two waves in the image's LDS");

// Shares added in order, gradients stored, parameters updated: a thread per
// four weights of a row, or its bias.
__global__ void __launch_bounds__(T) c_update(const float* __restrict__ part1, const float* __restrict__ part2,
                                              int shares, float* __restrict__ prm, float* __restrict__ grd, float lr) {
    constexpr int Q1 = kRow1 / 4, Q2 = kRow2 / 4;
    int i = blockIdx.x * T + threadIdx.x;
    const bool first = i < C1 * Q1;
    if (!first) i -= C1 * Q1;
    if (!first && i >= C2 * Q2) return;
    const int nq = first ? Q1 : Q2, co = i / nq, q = i % nq;
    const int64_t stride = (int64_t)64 * nq * 4;
    const float* p = (first ? part1 : part2) + 4 * (int64_t)i;
    f32x4 s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 3 < shares; k += 4)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += ld4(p + (k + j) * stride);
    for (; k < shares; ++k) s[0] += ld4(p + k * stride);
    const f32x4 v = (s[0] + s[1]) + (s[2] + s[3]);
    if (q == nq - 1) {  // the bias
        const int64_t o = (first ? oB1 : oB2) + co;
        grd[o] = v[0];
        prm[o] = __builtin_fmaf(-lr, v[0], prm[o]);
        return;
    }
    const int64_t o = (first ? oW1 : oW2) + (int64_t)co * (nq - 1) * 4 + 4 * q;
    f32x4 w = ld4(prm + o);
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = __builtin_fmaf(-lr, v[j], w[j]);
    st4(grd + o, v);
    st4(prm + o, w);
}
static_assert(oB1 % 4 == 0 && oW2 % 4 == 0 && oB2 % 4 == 0, "16-byte parameter accesses");

size_t carve(Plan* P, int max_batch, Arena* ar) {
    const size_t B = max_batch, ldb = pad16(max_batch), sh = std::min(max_batch, kShares);
    size_t s = 0;
    auto take = [&](auto*& p, size_t n) {
        using U = std::remove_reference_t<decltype(*p)>;
        s += (n * sizeof(U) + 255) & ~size_t(255);
        if (ar) p = ar->template take<U>(n);
    };
    take(P->h, C2 * ldb);
    take(P->dh, C2 * ldb);
    take(P->p1, B * C1 * P1);
    take(P->y2, B * C2 * P1);
    take(P->dp1, B * C1 * P1);
    take(P->arg1, B * C1 * P1);
    take(P->part1, sh * C1 * kRow1);
    take(P->part2, sh * C2 * kRow2);
    return s;
}

size_t ws_bytes(const fo_model* m) {
    Plan P;
    return carve(&P, m->max_batch, nullptr);
}

fo_status init(fo_model* m) {
    Plan* P = new (std::nothrow) Plan();
    if (!P) return FO_ENOMEM;
    m->plan = P;
    carve(P, m->max_batch, &m->arena);
    if (!P->part2) {
        set_error("cnn32: workspace arena too small");
        return FO_ENOMEM;
    }
    return FO_OK;
}

fo_status step(fo_model* m, const fo_acts* acts, const int32_t* labels) {
    (void)labels;  // (the batch's data is read through m->dev_in)
    const Plan* P = (const Plan*)m->plan;
    hipStream_t s = m->stream;
    const int B = acts->batch, ldb = pad16(B), shares = std::min(B, kShares);
    float *prm = m->params, *grd = m->grads;
    // forward (Alg. 4: forward pass of M_s)
    hipLaunchKernelGGL(c1_fwd, dim3(B, C1 / 16, 2), dim3(T), 0, s, m->dev_in, prm + oW1, prm + oB1, P->p1, P->arg1);
    hipLaunchKernelGGL(c2_fwd, dim3(B, C2 / 16), dim3(T), 0, s, P->p1, prm + oW2, prm + oB2, P->y2, P->h, ldb);
    // loss f_s and backward (Alg. 4: backward pass of M_s)
    hipLaunchKernelGGL((small_head<C2, false>), dim3(1), dim3(1024), 0, s, P->h, ldb, m->dev_in, prm + oWf, grd + oWf,
                       m->lr, B, m->logits, m->loss, P->dh);
    hipLaunchKernelGGL(c2_bwd, dim3(4 * (B + shares)), dim3(T), 0, s, P->p1, P->y2, P->dh, ldb, prm + oW2, P->dp1,
                       P->part2, B, shares);
    hipLaunchKernelGGL(c1_wgrad, dim3(4 * shares), dim3(T), 0, s, m->dev_in, P->dp1, P->arg1, P->part1, B, shares);
    // SGD (Alg. 4: theta_s <- theta_s - gamma_s grad)
    hipLaunchKernelGGL(c_update, dim3((unsigned)cdiv(16 * (kRow1 + kRow2), T)), dim3(T), 0, s, P->part1, P->part2,
                       shares, prm, grd, m->lr);
    FO_LAUNCHED();
    return FO_OK;
}

void destroy(fo_model* m) {
    delete (Plan*)m->plan;
    m->plan = nullptr;
}

}  // namespace

int64_t cnn32_param_count() { return kParams; }

const Family* family_cnn32() {
    static const Family f = {(int64_t)C0 * P0 * 4, ws_bytes, init, step, destroy};
    return &f;
}

}  // namespace fo
