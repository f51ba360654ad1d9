// Config 9: the server part of the paper's VGG-5 (Table 4) split after its
// second pool, one training iteration of the activation branch of Alg. 4 in
// fp32 on [64, 8, 8] inputs (NCHW at the boundary):
//   conv3x3 64->64 (no bias) -> batch norm (batch statistics) -> ReLU ->
//   maxpool 2x2 -> flatten (C, H, W) -> fc 1024->128 + ReLU -> fc 128->10,
//   mean cross-entropy, backward, SGD.
// Batches of up to 128 samples take the fused step below.  In larger ones the
// convolution runs as an explicit im2col matrix [B*64][576] (k = (ky, kx, ci),
// the weight layout's order) times the weights on the fp32 product kernel, its
// output NHWC; batch norm is one workgroup per channel; the pool writes its
// output in (C, H, W) order so the flatten is the identity.  The input gradient
// of the convolution is never formed (nothing goes back to the devices).
#include "model.h"
#include "small_f32.h"

namespace fo {

namespace {

constexpr int CI = 64, CO = 64, HW = 8, HP = 4, KC = 9 * CI, F1 = 128, NCLS = 10, NF = CO * HP * HP;
constexpr float BN_EPS = 1e-5f;
constexpr int64_t kParams = (int64_t)CO * KC + 2 * CO + (int64_t)F1 * NF + F1 + (int64_t)NCLS * F1 + NCLS;
constexpr int kMaxSlices = 16;

inline int nblk(int64_t n) { return (int)cdiv(n, 256); }

// col[r][(ky*3 + kx)*CI + ci] = x[b][ci][y+ky-1][x+kx-1] (0 outside), r = (b*8 + y)*8 + x
__global__ void __launch_bounds__(256) im2col_kernel(const StepIn* __restrict__ in, float* __restrict__ col, int B) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)B * HW * HW * KC) return;
    const int k = (int)(i % KC);
    const int64_t r = i / KC;
    const int tap = k / CI, ci = k % CI, ky = tap / 3, kx = tap % 3;
    const int b = (int)(r / (HW * HW)), y = (int)(r / HW % HW), x = (int)(r % HW);
    const int yy = y + ky - 1, xx = x + kx - 1;
    const float* X = (const float*)in->x;
    col[i] = yy >= 0 && yy < HW && xx >= 0 && xx < HW ? X[(((int64_t)b * CI + ci) * HW + yy) * HW + xx] : 0.f;
}

// Block c: batch statistics of channel c over the R rows of z (NHWC), then
// xhat, y = ReLU(gamma xhat + beta); mean and variance in two passes.
__device__ __forceinline__ float block_sum(float v, float* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}
__global__ void __launch_bounds__(256) bn5_fwd(const float* __restrict__ z, const float* __restrict__ gam,
                                               const float* __restrict__ bet, float* __restrict__ xhat,
                                               float* __restrict__ y, float* __restrict__ rstd_out, int R) {
    __shared__ float red[4];
    const int c = blockIdx.x;
    float s = 0.f;
    for (int r = threadIdx.x; r < R; r += 256) s += z[(int64_t)r * CO + c];
    const float mu = block_sum(s, red) / R;
    float v = 0.f;
    for (int r = threadIdx.x; r < R; r += 256) {
        const float d = z[(int64_t)r * CO + c] - mu;
        v = fmaf(d, d, v);
    }
    const float rs = 1.f / sqrtf(block_sum(v, red) / R + BN_EPS);
    for (int r = threadIdx.x; r < R; r += 256) {
        const int64_t o = (int64_t)r * CO + c;
        const float xh = (z[o] - mu) * rs;
        xhat[o] = xh;
        y[o] = fmaxf(fmaf(gam[c], xh, bet[c]), 0.f);
    }
    if (threadIdx.x == 0) rstd_out[c] = rs;
}

// 2x2 max pool of y (NHWC [B][8][8][64]) into p ((C, H, W) order, [B][1024]),
// with the window position of the maximum (the first one in row-major order)
__global__ void __launch_bounds__(256) pool5_fwd(const float* __restrict__ y, float* __restrict__ p,
                                                 uint8_t* __restrict__ arg, int B) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= B * NF) return;
    const int b = i / NF, c = i / (HP * HP) % CO, oy = i / HP % HP, ox = i % HP;
    float best = -INFINITY;
    int at = 0;
    for (int w = 0; w < 4; ++w) {
        const int yy = 2 * oy + (w >> 1), xx = 2 * ox + (w & 1);
        const float v = y[(((int64_t)b * HW + yy) * HW + xx) * CO + c];
        if (v > best) {
            best = v;
            at = w;
        }
    }
    p[i] = best;
    arg[i] = (uint8_t)at;
}

// d(batch-norm output) at every pre-pool position: the pooled gradient where
// the position is its window's maximum, times the ReLU mask (y > 0)
__global__ void __launch_bounds__(256) pool5_relu_bwd(const float* __restrict__ dp, const uint8_t* __restrict__ arg,
                                                      const float* __restrict__ y, float* __restrict__ dbn, int B) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)B * HW * HW * CO) return;
    const int c = (int)(i % CO);
    const int64_t r = i / CO;
    const int b = (int)(r / (HW * HW)), yy = (int)(r / HW % HW), xx = (int)(r % HW);
    const int j = ((b * CO + c) * HP + yy / 2) * HP + xx / 2;
    const int w = (yy & 1) * 2 + (xx & 1);
    dbn[i] = arg[j] == w && y[i] > 0.f ? dp[j] : 0.f;
}

// Block c: dgamma = sum dy xhat, dbeta = sum dy, dz = gamma rstd (dy - dbeta/R - xhat dgamma/R)
__global__ void __launch_bounds__(256) bn5_bwd(const float* __restrict__ dy, const float* __restrict__ xhat,
                                               const float* __restrict__ gam, const float* __restrict__ rstd,
                                               float* __restrict__ dz, float* __restrict__ dgam,
                                               float* __restrict__ dbet, int R) {
    __shared__ float red[4];
    const int c = blockIdx.x;
    float sg = 0.f, sb = 0.f;
    for (int r = threadIdx.x; r < R; r += 256) {
        const int64_t o = (int64_t)r * CO + c;
        sg = fmaf(dy[o], xhat[o], sg);
        sb += dy[o];
    }
    const float dg = block_sum(sg, red), db = block_sum(sb, red);
    const float k = gam[c] * rstd[c];
    for (int r = threadIdx.x; r < R; r += 256) {
        const int64_t o = (int64_t)r * CO + c;
        dz[o] = k * (dy[o] - db / R - xhat[o] * dg / R);
    }
    if (threadIdx.x == 0) {
        dgam[c] = dg;
        dbet[c] = db;
    }
}

// ------------------------------------------------------------------ the fused step, batches of up to 128
// With a launch per product, norm and pool the step is 23 dependent launches of
// 4.5 us or little more (120.6 us at batch 32).  Here it is 8 (64.5 us): the convolution as an implicit GEMM of
// one image in LDS; batch norm, ReLU and pool by the workgroup that owns a
// channel over the whole batch; fc1; one workgroup for everything between the
// hidden layer and its gradient; the pooled gradient of a channel (a 16-column
// product) with the pool's, ReLU's and batch norm's backward; the weight
// gradients; their sums and the update.  Activations are stored feature by
// feature ([C][rows] and [features][ldb], samples padded with zeros to 16).
// At most 128 samples: a channel's rows (8,192) and the hidden layer of the
// whole batch have to fit in LDS.
constexpr int kFusedMax = 128;
constexpr int XP = 10, XS = XP * XP;  // an image with its border of zeros
constexpr int kWgShares = 32;         // samples' shares of the convolution's weight gradient
// offsets in the flat parameter vector
constexpr int64_t oWc = 0, oG = oWc + (int64_t)CO * KC, oBb = oG + CO, oW1 = oBb + CO, oB1 = oW1 + (int64_t)F1 * NF,
                  oW2 = oB1 + F1;

// One image of the batch into xs[ci][10][10] (LDS; the border is zeroed by the caller once).
__device__ __forceinline__ void stage_image(const StepIn* in, int b, float* xs) {
    const float* x = static_cast<const float*>(in->x) + (int64_t)b * CI * HW * HW;
    for (int e = threadIdx.x; e < CI * HW * HW / 4; e += 256) {
        const f32x4 v = ld4(x + 4 * e);
        const int ci = e / (HW * HW / 4), q = e % (HW * HW / 4) * 4;
        float* o = xs + ci * XS + (q / HW + 1) * XP + q % HW + 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = v[i];
    }
}
__device__ __forceinline__ void zero_image(float* xs) {
    for (int e = threadIdx.x; e < CI * XS; e += 256) xs[e] = 0.f;
    __syncthreads();
}

// z[co][b 64 + pixel] of 16 channels of one image: a wave takes 16 pixels,
// v_mfma_f32_16x16x4_f32 with the weights' rows as A (k = (tap, ci) contiguous,
// one 16-byte load per 16 k) and the pixels from LDS as B.  128 workgroups at
// batch 32, each 144 MFMAs long per wave (1.9 us).
__global__ void __launch_bounds__(256) v5_conv(const StepIn* __restrict__ in, const float* __restrict__ w,
                                               float* __restrict__ z, int64_t ld) {
    __shared__ float xs[CI * XS];
    const int b = blockIdx.x, lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    const int co = blockIdx.y * 16;
    // the weights of a tap are loaded during the products of the one before
    const float* wr = w + (int64_t)(co + tok) * KC + 4 * g;
    f32x4 a[2][CI / 16];
#pragma unroll
    for (int s = 0; s < CI / 16; ++s) a[0][s] = ld4(wr + 16 * s);
    zero_image(xs);
    stage_image(in, b, xs);
    __syncthreads();
    const int px = 16 * wave + tok, at = px / HW * XP + px % HW;
    // sixteen running sums of 36 products each, added pairwise (the rounding error grows with their length)
    f32x4 acc[CI / 16][4];
#pragma unroll
    for (int s = 0; s < CI / 16; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[s][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        if (t + 1 < 9)
#pragma unroll
            for (int s = 0; s < CI / 16; ++s) a[(t + 1) & 1][s] = ld4(wr + (t + 1) * CI + 16 * s);
#pragma unroll
        for (int s = 0; s < CI / 16; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[s][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    a[t & 1][s][j], xs[(16 * s + 4 * g + j) * XS + at + t / 3 * XP + t % 3], acc[s][j], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < CI / 16; ++s) acc[s][0] = (acc[s][0] + acc[s][1]) + (acc[s][2] + acc[s][3]);
    const f32x4 v = (acc[0][0] + acc[1][0]) + (acc[2][0] + acc[3][0]);
#pragma unroll
    for (int i = 0; i < 4; ++i) z[(co + 4 * g + i) * ld + b * HW * HW + px] = v[i];
}

// Channel c = block: batch norm over its R rows (in LDS), ReLU, 2x2 max pool
// into p[(c, 4, 4)][ldb] with the window position of the maximum (the first in
// row-major order).
__global__ void __launch_bounds__(512) v5_bn_pool(const float* __restrict__ z, int64_t ld,
                                                  const float* __restrict__ gam, const float* __restrict__ bet,
                                                  float* __restrict__ xhat, float* __restrict__ rstd_out,
                                                  float* __restrict__ p, uint8_t* __restrict__ arg, int B, int ldb) {
    __shared__ float y[kFusedMax * HW * HW], red[8];
    const int c = blockIdx.x, R = B * HW * HW, w = threadIdx.x >> 6;
    auto total = [&](float v) {
        v = wave_sum(v);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[w] = v;
        __syncthreads();
        return ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
    };
    float s = 0.f;
    for (int r = 4 * threadIdx.x; r < R; r += 4 * 512) {
        const f32x4 v = ld4(z + c * ld + r);
        st4(y + r, v);
        s += (v[0] + v[1]) + (v[2] + v[3]);
    }
    const float mu = total(s) / R;
    float q = 0.f;
    for (int r = threadIdx.x; r < R; r += 512) {
        const float d = y[r] - mu;
        q = fmaf(d, d, q);
    }
    const float rs = 1.f / sqrtf(total(q) / R + BN_EPS), ga = gam[c], be = bet[c];
    if (threadIdx.x == 0) rstd_out[c] = rs;
    for (int r = threadIdx.x; r < R; r += 512) {
        const float xh = (y[r] - mu) * rs;
        xhat[c * ld + r] = xh;
        y[r] = fmaxf(fmaf(ga, xh, be), 0.f);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HP * HP * ldb; i += 512) {  // samples adjacent
        const int o = i / ldb, b = i % ldb;
        float best = 0.f;
        int at = 0;
        if (b < B) {
            best = -INFINITY;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float v = y[b * HW * HW + (2 * (o / HP) + (k >> 1)) * HW + 2 * (o % HP) + (k & 1)];
                if (v > best) {
                    best = v;
                    at = k;
                }
            }
        }
        const int64_t e = (int64_t)(c * HP * HP + o) * ldb + b;
        p[e] = best;
        arg[e] = (uint8_t)at;
    }
}

// Channel c = block: dp of its 16 pooled positions (16 rows of a product over
// the hidden units), through the pool and the ReLU to the batch norm's output,
// the norm's backward and update, dz of the convolution [c][row].
__global__ void __launch_bounds__(512) v5_dp_bn(const float* __restrict__ df1, int ldb, const float* __restrict__ w1,
                                                const float* __restrict__ xhat, int64_t ld,
                                                const float* __restrict__ rstd, const uint8_t* __restrict__ arg,
                                                float* __restrict__ prm, float* __restrict__ grd, float lr,
                                                float* __restrict__ dzc, int B) {
    __shared__ float dp[HP * HP][kFusedMax], red[2][8];
    const int c = blockIdx.x, R = B * HW * HW, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, tok = lane & 15,
              g = lane >> 4;
    if (16 * wave < ldb) {  // a wave per 16 samples
        f32x4 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < F1 / 16; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = 16 * s + 4 * g + j;
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[(int64_t)n * NF + c * HP * HP + tok],
                                                              df1[n * ldb + 16 * wave + tok], acc[j], 0, 0, 0);
            }
        const f32x4 v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) dp[4 * g + i][16 * wave + tok] = v[i];
    }
    __syncthreads();
    // thread = (sample, pooled position): the gradient reaches the window's maximum if it is positive
    const float ga = prm[oG + c], be = prm[oBb + c], rs = rstd[c];
    float sg = 0.f, sb = 0.f;
    for (int i = threadIdx.x; i < B * HP * HP; i += 512) {
        const int b = i / (HP * HP), o = i % (HP * HP), k = arg[(int64_t)(c * HP * HP + o) * ldb + b];
        const int r = b * HW * HW + (2 * (o / HP) + (k >> 1)) * HW + 2 * (o % HP) + (k & 1);
        const float xh = xhat[c * ld + r];
        const float d = fmaf(ga, xh, be) > 0.f ? dp[o][b] : 0.f;
        dp[o][b] = d;
        sg = fmaf(d, xh, sg);
        sb += d;
    }
    sg = wave_sum(sg);
    sb = wave_sum(sb);
    if (lane == 0) {
        red[0][wave] = sg;
        red[1][wave] = sb;
    }
    __syncthreads();
    float dg = 0.f, db = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        dg += red[0][k];
        db += red[1][k];
    }
    const float kk = ga * rs, mg = dg / R, mb = db / R;
    for (int r = threadIdx.x; r < R; r += 512) {
        const int b = r / (HW * HW), yy = r / HW % HW, xx = r % HW, o = yy / 2 * HP + xx / 2;
        const float d = arg[(int64_t)(c * HP * HP + o) * ldb + b] == (yy & 1) * 2 + (xx & 1) ? dp[o][b] : 0.f;
        dzc[c * ld + r] = kk * (d - mb - xhat[c * ld + r] * mg);
    }
    if (threadIdx.x == 0) {
        grd[oG + c] = dg;
        grd[oBb + c] = db;
        prm[oG + c] = __builtin_fmaf(-lr, dg, ga);
        prm[oBb + c] = __builtin_fmaf(-lr, db, be);
    }
}

// Weight gradients.  The convolution's (blocks below `conv`): block = (share of
// the samples, 16 output channels), a wave holds 16 input channels by nine taps
// and walks the images staged in LDS; the shares go to part and are added by
// v5_update.  The rest: fc1's, 32 x 32 per wave, with its update.
__global__ void __launch_bounds__(256) v5_wgrad(const StepIn* __restrict__ in, const float* __restrict__ dzc,
                                                int64_t ld, int B, int shares, float* __restrict__ part, WUnit fc1,
                                                float* __restrict__ prm, float* __restrict__ grd, float lr) {
    __shared__ float xs[CI * XS];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int)blockIdx.x >= 4 * shares) {
        wgrad_32x32(fc1, (blockIdx.x - 4 * shares) * 4 + wave, in, prm, grd, lr);
        return;
    }
    const int lane = threadIdx.x & 63, tok = lane & 15, g = lane >> 4, share = blockIdx.x / 4, co = blockIdx.x % 4 * 16;
    zero_image(xs);
    f32x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* xr = xs + (16 * wave + tok) * XS;
    for (int b = share; b < B; b += shares) {
        if (b != share) __syncthreads();
        stage_image(in, b, xs);
        f32x4 d[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) d[s] = ld4(dzc + (co + tok) * ld + b * HW * HW + 16 * s + 4 * g);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int px = 16 * s + 4 * g + j;
                const float* x = xr + px / HW * XP + px % HW;
#pragma unroll
                for (int t = 0; t < 9; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t / 3 * XP + t % 3], d[s][j], acc[t], 0, 0, 0);
            }
    }
    float* o = part + ((int64_t)share * CO + co + tok) * KC + 16 * wave + 4 * g;
#pragma unroll
    for (int t = 0; t < 9; ++t) st4(o + t * CI, acc[t]);
}

// The convolution's weights: shares added in order, gradient stored, weight updated.
__global__ void __launch_bounds__(256) v5_update(const float* __restrict__ part, int shares, float* __restrict__ prm,
                                                 float* __restrict__ grd, float lr) {
    const int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    f32x4 s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 3 < shares; k += 4)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += ld4(part + (int64_t)(k + j) * CO * KC + i);
    for (; k < shares; ++k) s[0] += ld4(part + (int64_t)k * CO * KC + i);
    const f32x4 v = (s[0] + s[1]) + (s[2] + s[3]);
    f32x4 w = ld4(prm + oWc + i);
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = __builtin_fmaf(-lr, v[j], w[j]);
    st4(grd + oWc + i, v);
    st4(prm + oWc + i, w);
}
static_assert(CO * KC % 1024 == 0 && oW1 % 4 == 0 && F1 % 32 == 0 && NF % 128 == 0, "whole blocks");

struct Plan {
    // the fused step
    float *zc, *xhc, *dzc, *rsc, *pf, *f1f, *df1f, *wpart;
    uint8_t* argf;
    // larger batches
    const float *wc, *g, *bb, *w1, *b1, *w2, *b2;
    float *gwc, *gg, *gbb, *gw1, *gb1, *gw2, *gb2;
    float *col, *z, *xhat, *y, *rstd, *p, *f1, *dz, *df1, *dp, *dbn, *dconv, *part, *colws;
    uint8_t* arg;
    size_t part_floats;
};

size_t ws_bytes(const fo_model* m) {
    const size_t B = (size_t)m->max_batch, R = B * HW * HW;
    size_t s = 0;
    auto add = [&](size_t b) { s += (b + 255) & ~size_t(255); };
    add(sizeof(Plan));
    const size_t Bf = std::min<size_t>(B, kFusedMax), Rf = Bf * HW * HW, lf = pad16((int)Bf);
    for (int i = 0; i < 3; ++i) add(4 * CO * Rf);  // zc, xhc, dzc
    add(4 * CO);                           // rsc
    add(4 * NF * lf);                      // pf
    for (int i = 0; i < 2; ++i) add(4 * F1 * lf);  // f1f, df1f
    add(4 * (size_t)kWgShares * CO * KC);  // wpart
    add(NF * lf);                          // argf
    if (B <= kFusedMax) return s;
    add(4 * R * KC);                       // col
    for (int i = 0; i < 3; ++i) add(4 * R * CO);  // z, xhat, y
    add(4 * CO);                           // rstd
    add(4 * B * NF);                       // p
    add(B * NF);                           // arg
    add(4 * B * F1);                       // f1
    add(4 * B * NCLS);                     // dz
    add(4 * B * F1);                       // df1
    add(4 * B * NF);                       // dp
    add(4 * R * CO);                       // dbn
    add(4 * R * CO);                       // dconv
    add(4 * (size_t)kMaxSlices * CO * KC); // part
    add(4 * colsum_ws_floats((int)B, F1)); // colws
    return s;
}

fo_status init(fo_model* m) {
    Plan* P = new (std::nothrow) Plan();
    if (!P) return FO_ENOMEM;
    m->plan = P;
    const size_t B = (size_t)m->max_batch, R = B * HW * HW;
    const float* p = m->params;
    float* g = m->grads;
    auto take = [&](const float*& w, float*& gw, size_t n) {
        w = p;
        gw = g;
        p += n;
        g += n;
    };
    take(P->wc, P->gwc, (size_t)CO * KC);
    take(P->g, P->gg, CO);
    take(P->bb, P->gbb, CO);
    take(P->w1, P->gw1, (size_t)F1 * NF);
    take(P->b1, P->gb1, F1);
    take(P->w2, P->gw2, (size_t)NCLS * F1);
    take(P->b2, P->gb2, NCLS);
    Arena& a = m->arena;
    a.take<char>(sizeof(Plan));
    const size_t Bf = std::min<size_t>(B, kFusedMax), Rf = Bf * HW * HW, lf = pad16((int)Bf);
    for (float** q : {&P->zc, &P->xhc, &P->dzc}) *q = a.take<float>(CO * Rf);
    P->rsc = a.take<float>(CO);
    P->pf = a.take<float>(NF * lf);
    for (float** q : {&P->f1f, &P->df1f}) *q = a.take<float>(F1 * lf);
    P->wpart = a.take<float>((size_t)kWgShares * CO * KC);
    P->argf = a.take<uint8_t>(NF * lf);
    if (!P->argf) {
        set_error("vgg5: workspace arena too small");
        return FO_ENOMEM;
    }
    if (B <= kFusedMax) return FO_OK;
    P->col = a.take<float>(R * KC);
    P->z = a.take<float>(R * CO);
    P->xhat = a.take<float>(R * CO);
    P->y = a.take<float>(R * CO);
    P->rstd = a.take<float>(CO);
    P->p = a.take<float>(B * NF);
    P->arg = a.take<uint8_t>(B * NF);
    P->f1 = a.take<float>(B * F1);
    P->dz = a.take<float>(B * NCLS);
    P->df1 = a.take<float>(B * F1);
    P->dp = a.take<float>(B * NF);
    P->dbn = a.take<float>(R * CO);
    P->dconv = a.take<float>(R * CO);
    P->part_floats = (size_t)kMaxSlices * CO * KC;
    P->part = a.take<float>(P->part_floats);
    P->colws = a.take<float>(colsum_ws_floats((int)B, F1));
    if (!P->colws) {
        set_error("vgg5: workspace arena too small");
        return FO_ENOMEM;
    }
    return FO_OK;
}

GemmF32 prod(const float* A, int64_t am, int64_t ak, const float* B, int64_t bn, int64_t bk, float* C, int64_t ldc,
             int M, int N, int K) {
    GemmF32 g{};
    g.A = A;
    g.am = am;
    g.ak = ak;
    g.B = B;
    g.bn = bn;
    g.bk = bk;
    g.C = C;
    g.ldc = ldc;
    g.M = M;
    g.N = N;
    g.K = K;
    g.S = 1;
    g.auto_split = 1;
    return g;
}

fo_status fused_step(fo_model* m, const Plan* P, int B) {
    hipStream_t s = m->stream;
    const int ldb = pad16(B), shares = std::min(B, kWgShares);
    const int64_t ld = (int64_t)B * HW * HW;
    float *prm = m->params, *grd = m->grads;
    // forward (Alg. 4: forward pass of M_s)
    hipLaunchKernelGGL(v5_conv, dim3(B, CO / 16), dim3(256), 0, s, m->dev_in, prm + oWc, P->zc, ld);
    hipLaunchKernelGGL(v5_bn_pool, dim3(CO), dim3(512), 0, s, P->zc, ld, prm + oG, prm + oBb, P->xhc, P->rsc, P->pf,
                       P->argf, B, ldb);
    Lin l{};
    l.W = prm + oW1;
    l.X = P->pf;
    l.bias = prm + oB1;
    l.out = P->f1f;
    l.N = F1;
    l.K = NF;
    l.B = B;
    l.ldb = ldb;
    hipLaunchKernelGGL((linear_small<false, E_RELU>), dim3(F1 / 16, (unsigned)cdiv(ldb, 32)), dim3(LIN_T), 0, s, l);
    // loss and backward (Alg. 4: backward pass of M_s)
    hipLaunchKernelGGL((small_head<F1, true>), dim3(1), dim3(1024), 0, s, P->f1f, ldb, m->dev_in, prm + oW2, grd + oW2,
                       m->lr, B, m->logits, m->loss, P->df1f);
    hipLaunchKernelGGL(v5_dp_bn, dim3(CO), dim3(512), 0, s, P->df1f, ldb, prm + oW1, P->xhc, ld, P->rsc, P->argf, prm,
                       grd, m->lr, P->dzc, B);
    const WUnit fc1{P->df1f, Act2{P->pf, 16, ldb}, oW1, oB1, F1, NF, ldb, 0};
    hipLaunchKernelGGL(v5_wgrad, dim3(4 * shares + F1 / 32 * (NF / 32) / 4), dim3(256), 0, s, m->dev_in, P->dzc, ld, B,
                       shares, P->wpart, fc1, prm, grd, m->lr);
    hipLaunchKernelGGL(v5_update, dim3(CO * KC / 1024), dim3(256), 0, s, P->wpart, shares, prm, grd, m->lr);
    FO_LAUNCHED();
    return FO_OK;
}

fo_status step(fo_model* m, const fo_acts* acts, const int32_t* labels) {
    (void)labels;  // read through m->dev_in
    Plan* P = (Plan*)m->plan;
    hipStream_t s = m->stream;
    const int B = acts->batch, R = B * HW * HW;
    if (B <= kFusedMax) return fused_step(m, P, B);
    fo_status st = FO_OK;
    auto gemm = [&](const GemmF32& g) { return launch_gemm_f32(g, P->part, P->part_floats, s); };
#define TRY(x)                      \
    do {                            \
        st = (x);                   \
        if (st != FO_OK) return st; \
    } while (0)
    // forward (Alg. 4: forward pass of M_s)
    hipLaunchKernelGGL(im2col_kernel, dim3(nblk((int64_t)R * KC)), dim3(256), 0, s, m->dev_in, P->col, B);
    FO_LAUNCHED();
    TRY(gemm(prod(P->col, KC, 1, P->wc, KC, 1, P->z, CO, R, CO, KC)));
    hipLaunchKernelGGL(bn5_fwd, dim3(CO), dim3(256), 0, s, P->z, P->g, P->bb, P->xhat, P->y, P->rstd, R);
    hipLaunchKernelGGL(pool5_fwd, dim3(nblk((int64_t)B * NF)), dim3(256), 0, s, P->y, P->p, P->arg, B);
    FO_LAUNCHED();
    GemmF32 g1 = prod(P->p, NF, 1, P->w1, NF, 1, P->f1, F1, B, F1, NF);
    g1.bias = P->b1;
    g1.relu = 1;
    TRY(gemm(g1));
    GemmF32 g2 = prod(P->f1, F1, 1, P->w2, F1, 1, m->logits, NCLS, B, NCLS, F1);
    g2.bias = P->b2;
    TRY(gemm(g2));
    TRY(launch_xent(m->logits, m->dev_in, P->dz, m->loss, B, NCLS, s));
    // backward (Alg. 4: backward pass of M_s)
    TRY(gemm(prod(P->dz, 1, NCLS, P->f1, 1, F1, P->gw2, F1, NCLS, F1, B)));       // dW2 = dz^T f1
    TRY(launch_colsum(P->dz, NCLS, B, nullptr, NCLS, P->gb2, P->colws, s));
    GemmF32 gd = prod(P->dz, NCLS, 1, P->w2, 1, F1, P->df1, F1, B, F1, NCLS);     // df1 = dz W2 * (f1 > 0)
    gd.mask = P->f1;
    gd.ldmask = F1;
    TRY(gemm(gd));
    GemmF32 gw = prod(P->df1, 1, F1, P->p, 1, NF, P->gw1, NF, F1, NF, B);         // dW1 = df1^T p
    TRY(gemm(gw));
    TRY(launch_colsum(P->df1, F1, B, nullptr, F1, P->gb1, P->colws, s));
    TRY(gemm(prod(P->df1, F1, 1, P->w1, 1, NF, P->dp, NF, B, NF, F1)));          // dp = df1 W1
    hipLaunchKernelGGL(pool5_relu_bwd, dim3(nblk((int64_t)R * CO)), dim3(256), 0, s, P->dp, P->arg, P->y, P->dbn, B);
    hipLaunchKernelGGL(bn5_bwd, dim3(CO), dim3(256), 0, s, P->dbn, P->xhat, P->g, P->rstd, P->dconv, P->gg, P->gbb,
                       R);
    FO_LAUNCHED();
    GemmF32 gc = prod(P->dconv, 1, CO, P->col, 1, KC, P->gwc, KC, CO, KC, R);   // dWc = dconv^T col
    gc.S = std::min(kMaxSlices, std::max(1, R / 256));
    TRY(gemm(gc));
#undef TRY
    // SGD (Alg. 4)
    return launch_sgd(m->params, m->grads, nullptr, nullptr, nullptr, m->n_params, m->lr, 0.f, s);
}

void destroy(fo_model* m) {
    delete (Plan*)m->plan;
    m->plan = nullptr;
}

}  // namespace

int64_t vgg5_param_count() { return kParams; }

const Family* family_vgg5() {
    static const Family f = {(int64_t)CI * HW * HW * 4, ws_bytes, init, step, destroy};
    return &f;
}

}  // namespace fo
