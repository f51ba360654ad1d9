// The MobileNetV3-Large server step (config 10) in few launches, for batches
// of up to 128 samples.
//
// Its maps are small (4x4 and 2x2 pixels: 512 and 128 rows at batch 32) and
// every layer is followed by a training-mode batch norm, a reduction over all
// rows of a channel.  One launch per product, norm and convolution makes 245
// dependent launches of which nearly all take the 4.5 us that a launch costs
// here whatever it does.  But a channel of an expansion passes through its
// batch norm, hard-swish, depthwise convolution and second batch norm on its
// own, so a workgroup that owns four channels over all rows takes them from
// the 1x1 product to the squeeze in one launch, holding the rows in LDS; the
// backward does the same in reverse.  Four channels, because the product
// (thread = row, four channels per MFMA) is bound by reading the
// input once per workgroup through the CU's L2 port (64 B per cycle: 160 KB,
// 1 us at 80 channels), so fewer channels per workgroup only add work, and
// more leave CUs idle (46 to 240 workgroups as it is).
//   per block, forward:  expand + BN + dw + BN [-> SE fc1 -> SE fc2 + scale] -> project + BN (+ residual)
//   backward: input gradient of the block above + BN3 -> dh (+ dt) [-> dq -> dm] -> chain down to dz1
// Every weight gradient runs in one launch at the end, with its SGD update (all
// readers of the weights are done by then); norm and depthwise parameters are
// updated by the workgroup that owns their channel.  66 launches; at batch 32 the
// step takes 642 us against 1,325 with a launch per product, norm and convolution.
//
// Activations are stored channel by channel, [C][ld], rows (sample, pixel)
// contiguous and padded with zeros to a multiple of 16: a batch norm, a
// convolution and a weight gradient (a product over rows) all read them
// contiguously.  A step writes the padding that it reads (its place depends on
// the batch size, so what is there is another step's data).
#include "mbv3.h"
#include "small_f32.h"

namespace fo {
namespace mbv3 {
namespace {

constexpr int T = 1024;  // threads of a channel kernel: 16 waves, four per channel
constexpr int CG = 4;    // channels of a workgroup
constexpr int RMAX = kFusedMax * HIN * HIN;  // rows of a channel in LDS

// Sum over a channel's four waves (every wave of the workgroup calls it).
__device__ __forceinline__ float chan_sum(float v, float* red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, w0 = w & ~3;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    return (red[w0] + red[w0 + 1]) + (red[w0 + 2] + red[w0 + 3]);
}

// z[c][r] = sum_k x[k][r] w(c, k) for the workgroup's channels c0 .. c0 + 3 into
// sm[c R + r] (LDS).  TR: w(c, k) = W[k][c] (ldw columns), else W[c][k].
// A lane takes V adjacent rows (one load), a wave 64 V, and the k range is cut
// into as many shares as fill 16 waves, added in order through LDS.
// v_mfma_f32_4x4x1 (16 blocks of a 4 x 1 by 1 x 4 product): the 64 lanes of B are
// 64 rows, A the four channels' weights, broadcast from block k % 8 (cbsz 4,
// abid), so one register, lane l holding w(c0 + l % 4, k0 + l / 4), feeds eight k
// and a lane ends up with its rows' four channels.
// What bounds it: the inputs were written on other XCDs, so they arrive from
// beyond L2 at about 2 us; the time is how many bytes are in flight (up to
// 16 waves x 16 loads x 1 KB here).  K = 672 over 512 rows: 24.6 us, against 33
// with 4-byte loads and two shares; with the weights in scalar registers instead, each k
// waiting for its own cache line of W, the widest input gradient took 63 us.
// Sums of eight products are formed first and then added, which keeps the
// rounding error of the long reductions down.
constexpr int SMEM = 4 * CG * T;  // floats of LDS: 1,024 threads' partial sums of up to four rows
constexpr int S1 = SMEM / 2;      // the second array of the later phases starts here

template <bool TR, int V>
__device__ __forceinline__ void product4_v(const Act2& x, const float* xp, int K, const float* __restrict__ W, int ldw,
                                           int c0, int R, int lg, float* sm) {
    constexpr int KC = 8;
    typedef float vec __attribute__((ext_vector_type(V)));
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> lg), nks = T >> lg, rows = V << lg;
    const int kper = (K / KC + nks - 1) / nks * KC;
    const int k0 = min(ks * kper, K), k1 = min(k0 + kper, K);
    const int r0 = V * (threadIdx.x & ((1 << lg) - 1));
    const int wc = c0 + (threadIdx.x & 3), wk = (threadIdx.x & 31) >> 2;
    const float* xr = xp + act_row(x, min(r0, R - V));
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = zero;
    vec cur[KC], nxt[KC];
    float wv = 0.f, wn;
    auto load = [&](int k, vec (&v)[KC], float& w) {
        w = TR ? W[(int64_t)(k + wk) * ldw + wc] : W[(int64_t)wc * ldw + k + wk];
#pragma unroll
        for (int u = 0; u < KC; ++u) v[u] = *reinterpret_cast<const vec*>(xr + (k + u) * x.sc);
    };
    if (k0 < k1) load(k0, cur, wv);
    for (int k = k0; k < k1; k += KC) {
        load(min(k + KC, k1 - KC), nxt, wn);
        f32x4 p[V];
#pragma unroll
        for (int i = 0; i < V; ++i) p[i] = zero;
#define FO_K1(u)                                                                          \
    _Pragma("unroll") for (int i = 0; i < V; ++i)                                         \
        p[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(wv, cur[u][i], p[i], 4, u, 0);
        FO_K1(0) FO_K1(1) FO_K1(2) FO_K1(3) FO_K1(4) FO_K1(5) FO_K1(6) FO_K1(7)
#undef FO_K1
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] += p[i];
        wv = wn;
#pragma unroll
        for (int u = 0; u < KC; ++u) cur[u] = nxt[u];
    }
#pragma unroll
    for (int c = 0; c < CG; ++c) {
        vec o;
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] = acc[i][c];
        *reinterpret_cast<vec*>(sm + (ks * CG + c) * rows + r0) = o;
    }
    __syncthreads();
    float out[8];  // 4 rows / 1,024 of the sums, at most 8,192 / 1,024
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = threadIdx.x + T * q;
        out[q] = 0.f;
        if (e < CG * rows)
            for (int s = 0; s < nks; ++s) out[q] += sm[s * CG * rows + e];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = threadIdx.x + T * q;
        if (e < CG * rows && e % rows < R) sm[e / rows * R + e % rows] = out[q];
    }
    __syncthreads();
}
// Rows are a multiple of 4 (whole maps), K of 8.
template <bool TR>
__device__ __forceinline__ void product4(const Act2& x, const float* xp, int K, const float* __restrict__ W, int ldw,
                                         int c0, int R, float* sm) {
    if (R > 128)
        product4_v<TR, 4>(x, xp, K, W, ldw, c0, R, R > 1024 ? 9 : R > 512 ? 8 : R > 256 ? 7 : 6, sm);
    else if (R > 64)
        product4_v<TR, 2>(x, xp, K, W, ldw, c0, R, 6, sm);
    else
        product4_v<TR, 1>(x, xp, K, W, ldw, c0, R, 6, sm);
}

// The wave's share of its channel's rows: r = 64 (wave % 4) + lane + 256 i.
#define FO_ROWS(r, n) for (int r = (threadIdx.x & 255); r < (n); r += 256)

// Batch statistics of the channel's row zs[0..R): zs becomes xhat, which also
// goes to xh (global); returns 1 / sigma.
__device__ __forceinline__ float bn_stats(float* zs, float* xh, int R, float* red) {
    float s = 0.f;
    FO_ROWS(r, R) s += zs[r];
    const float mu = chan_sum(s, red) / R;
    float v = 0.f;
    FO_ROWS(r, R) {
        const float d = zs[r] - mu;
        v = fmaf(d, d, v);
    }
    const float rs = 1.f / sqrtf(chan_sum(v, red) / R + BN_EPS);
    FO_ROWS(r, R) {
        const float h = (zs[r] - mu) * rs;
        zs[r] = h;
        xh[r] = h;
    }
    return rs;
}

// One channel's norm backward: du (LDS) times act'(gamma xhat + beta) if act,
// its sums to the gradients (and the update), dz = gamma rstd (du - dbeta / R -
// xhat dgamma / R) back into du.  gi / bi: the parameters' offsets.
__device__ __forceinline__ void bn_grad(float* du, const float* xh, float rstd, int R, bool act, float* prm, float* grd,
                                        int64_t gi, int64_t bi, float lr, float* red) {
    const float g = prm[gi], b = prm[bi];
    float sg = 0.f, sb = 0.f;
    FO_ROWS(r, R) {
        const float x = xh[r];
        float d = du[r];
        if (act) {
            d *= hswish_d(fmaf(g, x, b));
            du[r] = d;
        }
        sg = fmaf(d, x, sg);
        sb += d;
    }
    const float dg = chan_sum(sg, red), db = chan_sum(sb, red);
    const float k = g * rstd, mg = dg / R, mb = db / R;
    FO_ROWS(r, R) du[r] = k * (du[r] - mb - xh[r] * mg);
    if ((threadIdx.x & 255) == 0) {
        grd[gi] = dg;
        grd[bi] = db;
        prm[gi] = __builtin_fmaf(-lr, dg, g);
        prm[bi] = __builtin_fmaf(-lr, db, b);
    }
}

// ------------------------------------------------------------------ forward
struct Expand {
    const StepIn* in;
    Act2 x;
    const float *wex, *g1, *b1, *wdw, *g2, *b2;
    float *xh1, *rs1, *xh2, *rs2, *a2, *m;  // m: [e][ldb] channel means, or NULL
    int cin, e, B, ld1, ld2, ldb;
};

// Four channels of a bottleneck from the expansion to the second hard-swish.
template <int KD, int H, int S>
__global__ void __launch_bounds__(T) mb_expand(const Expand p) {
    constexpr int HW = H * H, HO = (H + 2 * (KD / 2) - KD) / S + 1, HWO = HO * HO;
    __shared__ __attribute__((aligned(16))) float sm[SMEM];
    __shared__ float red[16];
    const int R = p.B * HW, Ro = p.B * HWO, c0 = blockIdx.x * CG;
    product4<false>(p.x, act_ptr(p.x, p.in), p.cin, p.wex, p.cin, c0, R, sm);
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = c0 + ch;
    float* z = sm + ch * R;
    float rs = bn_stats(z, p.xh1 + (int64_t)c * p.ld1, R, red);
    if ((threadIdx.x & 255) == 0) p.rs1[c] = rs;
    const float g1 = p.g1[c], b1 = p.b1[c];
    FO_ROWS(r, R) z[r] = hswish(fmaf(g1, z[r], b1));
    float w[KD * KD];
#pragma unroll
    for (int q = 0; q < KD * KD; ++q) w[q] = p.wdw[c * KD * KD + q];
    __syncthreads();
    float* z2 = sm + S1 + ch * Ro;
    FO_ROWS(r, Ro) {
        const int b = r / HWO, oy = r / HO % HO, ox = r % HO;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < KD * KD; ++q) {
            const int y = oy * S + q / KD - KD / 2, x = ox * S + q % KD - KD / 2;
            const bool in = y >= 0 && y < H && x >= 0 && x < H;
            const float t = z[b * HW + (in ? y * H + x : 0)];
            v = in ? fmaf(t, w[q], v) : v;
        }
        z2[r] = v;
    }
    __syncthreads();
    rs = bn_stats(z2, p.xh2 + (int64_t)c * p.ld2, Ro, red);
    if ((threadIdx.x & 255) == 0) p.rs2[c] = rs;
    const float g2 = p.g2[c], b2 = p.b2[c];
    FO_ROWS(r, p.ld2) {
        const float a = r < Ro ? hswish(fmaf(g2, z2[r], b2)) : 0.f;
        if (r < Ro) z2[r] = a;
        p.a2[(int64_t)c * p.ld2 + r] = a;
    }
    if (!p.m) return;
    __syncthreads();
    FO_ROWS(b, p.ldb) {
        float s = 0.f;
        if (b < p.B)
#pragma unroll
            for (int q = 0; q < HWO; ++q) s += z2[b * HWO + q];
        p.m[(int64_t)c * p.ldb + b] = s / HWO;
    }
}

struct Project {
    const StepIn* in;
    Act2 h;
    const float *w, *g, *b;
    Act2 res;  // the block's input when it is added to the output
    float *xh, *rs, *y;
    float* mean;  // the last 1x1 convolution: hard-swish and the channel means [C][ldb] instead of y
    int K, R, B, ld, ldb, has_res;
};

// Four output channels of a projection (or of the last 1x1 convolution) with
// their batch norm and the residual.
__global__ void __launch_bounds__(T) mb_project(const Project p) {
    __shared__ __attribute__((aligned(16))) float sm[SMEM];
    __shared__ float red[16];
    const int c0 = blockIdx.x * CG, R = p.R;
    product4<false>(p.h, p.h.p, p.K, p.w, p.K, c0, R, sm);
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = c0 + ch;
    float* z = sm + ch * R;
    const float rs = bn_stats(z, p.xh + (int64_t)c * p.ld, R, red);
    if ((threadIdx.x & 255) == 0) p.rs[c] = rs;
    const float g = p.g[c], b = p.b[c];
    if (p.mean) {
        FO_ROWS(r, R) z[r] = hswish(fmaf(g, z[r], b));
        __syncthreads();
        const int hw = R / p.B;
        FO_ROWS(i, p.ldb) {
            float s = 0.f;
            if (i < p.B)
                for (int q = 0; q < hw; ++q) s += z[i * hw + q];
            p.mean[(int64_t)c * p.ldb + i] = s / hw;
        }
        return;
    }
    const float* xr = p.has_res ? act_ptr(p.res, p.in) + c * p.res.sc : nullptr;
    FO_ROWS(r, p.ld) {
        float v = 0.f;
        if (r < R) v = fmaf(g, z[r], b) + (xr ? xr[act_row(p.res, r)] : 0.f);
        p.y[(int64_t)c * p.ld + r] = v;
    }
}

// ------------------------------------------------------------------ loss
// Mean cross-entropy of logits [B][200] (a wave per sample) and its gradient,
// transposed and padded: dz [200][ldb].  Labels are clamped and counted.
__global__ void __launch_bounds__(1024) mb_xent(const float* __restrict__ z, const StepIn* __restrict__ in,
                                                float* __restrict__ dz, float* __restrict__ loss, int B, int ldb) {
    constexpr int NW = 16, J = (NCLS + 63) / 64;
    __shared__ float part[NW];
    __shared__ int badw[NW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float mine = 0.f;
    int bad = 0;
    for (int b = w; b < ldb; b += NW) {
        if (b >= B) {
            for (int c = lane; c < NCLS; c += 64) dz[(int64_t)c * ldb + b] = 0.f;
            continue;
        }
        float v[J], m = -INFINITY, s = 0.f;
        int y = in->labels[b];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            v[j] = lane + 64 * j < NCLS ? z[(int64_t)b * NCLS + min(lane + 64 * j, NCLS - 1)] : -INFINITY;
            m = fmaxf(m, v[j]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
#pragma unroll
        for (int j = 0; j < J; ++j) s += lane + 64 * j < NCLS ? expf(v[j] - m) : 0.f;
        const float lse = m + logf(wave_sum(s));
        if (y < 0 || y >= NCLS) {
            bad++;
            y = y < 0 ? 0 : NCLS - 1;
        }
        mine += lse - z[(int64_t)b * NCLS + y];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = lane + 64 * j;
            if (c < NCLS) dz[(int64_t)c * ldb + b] = (expf(v[j] - lse) - (c == y ? 1.f : 0.f)) / (float)B;
        }
    }
    if (lane == 0) {
        part[w] = mine;
        badw[w] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        int nb = 0;
        for (int k = 0; k < NW; ++k) {
            t += part[k];
            nb += badw[k];
        }
        loss[0] = t / (float)B;
        loss[1] = (float)nb;
    }
}

// ------------------------------------------------------------------ backward
struct LastBwd {
    const float *dg, *xh, *rs;
    float *prm, *grd, *dz;
    int64_t gi, bi;
    float lr;
    int B, R, ld, ldb;
};
// Four channels of the last 1x1 convolution: the mean's gradient through
// hard-swish and the batch norm.
__global__ void __launch_bounds__(T) mb_last_bwd(const LastBwd p) {
    __shared__ float s0[CG * kFusedMax * 4], red[16];  // 2x2 maps
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = blockIdx.x * CG + ch, hw = p.R / p.B;
    float* d = s0 + ch * p.R;
    FO_ROWS(r, p.R) d[r] = p.dg[(int64_t)c * p.ldb + r / hw] / hw;
    bn_grad(d, p.xh + (int64_t)c * p.ld, p.rs[c], p.R, true, p.prm, p.grd, p.gi + c, p.bi + c, p.lr, red);
    FO_ROWS(r, p.ld) p.dz[(int64_t)c * p.ld + r] = r < p.R ? d[r] : 0.f;
}

struct BlkDx {
    Act2 dzu;            // dz1 of the block above (or of the last convolution), [K][ld]
    const float* wu;     // its expansion [K][co]
    const float* dyu;    // the gradient of its output when it has a residual, else NULL
    const float *xh, *rs;
    float *prm, *grd, *dy, *dz;
    int64_t gi, bi;
    float lr;
    int K, co, R, ld;
};
// Four channels of a block's output gradient (the input gradient of the block
// above, plus its residual) and their way through the projection's batch norm.
__global__ void __launch_bounds__(T) mb_dx(const BlkDx p) {
    __shared__ __attribute__((aligned(16))) float sm[SMEM];
    __shared__ float red[16];
    const int c0 = blockIdx.x * CG, R = p.R;
    product4<true>(p.dzu, p.dzu.p, p.K, p.wu, p.co, c0, R, sm);
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = c0 + ch;
    float* d = sm + ch * R;
    FO_ROWS(r, R) {
        const float v = d[r] + (p.dyu ? p.dyu[(int64_t)c * p.ld + r] : 0.f);
        d[r] = v;
        p.dy[(int64_t)c * p.ld + r] = v;
    }
    bn_grad(d, p.xh + (int64_t)c * p.ld, p.rs[c], R, false, p.prm, p.grd, p.gi + c, p.bi + c, p.lr, red);
    FO_ROWS(r, p.ld) p.dz[(int64_t)c * p.ld + r] = r < R ? d[r] : 0.f;
}

struct Chain {
    Act2 dz3;         // the projection's output gradient [co][ld2]
    const float* wpr;  // [co][e]
    const float *xh1, *rs1, *xh2, *rs2;
    const float *a2, *t, *dm;  // squeeze-excitation blocks
    float *dh, *dt;
    float *prm, *grd, *dz1;
    BlkOff o;
    float lr;
    int co, e, B, ld1, ld2, ldb;
};

// From da2 (LDS, d2, four channels of Ro rows) down to dz1: second batch norm,
// depthwise convolution (weight and input gradient), first batch norm.
template <int KD, int H, int S>
__device__ __forceinline__ void chain_down(const Chain& p, float* d2, float* s1, float* red, float* wred, int c0) {
    constexpr int HW = H * H, HO = (H + 2 * (KD / 2) - KD) / S + 1, HWO = HO * HO, KK = KD * KD;
    constexpr int SEG = 256 / KK;  // shares of the samples per tap
    const int R = p.B * HW, Ro = p.B * HWO;
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = c0 + ch, t = threadIdx.x & 255;
    float *d = d2 + ch * Ro, *a = s1 + ch * R;
    const float* xh1 = p.xh1 + (int64_t)c * p.ld1;
    const float g1 = p.prm[p.o.g1 + c], b1 = p.prm[p.o.b1 + c];
    float w[KK];
#pragma unroll
    for (int q = 0; q < KK; ++q) w[q] = p.prm[p.o.wdw + (int64_t)c * KK + q];
    FO_ROWS(r, R) a[r] = hswish(fmaf(g1, xh1[r], b1));
    bn_grad(d, p.xh2 + (int64_t)c * p.ld2, p.rs2[c], Ro, true, p.prm, p.grd, p.o.g2 + c, p.o.b2 + c, p.lr, red);
    __syncthreads();
    // the depthwise weight gradient: thread = (tap, share of the samples)
    if (t < KK * SEG) {
        const int q = t % KK, dy = q / KD - KD / 2, dx = q % KD - KD / 2;
        float s = 0.f;
        for (int b = t / KK; b < p.B; b += SEG) {
            float u = 0.f;
#pragma unroll
            for (int o = 0; o < HWO; ++o) {
                const int y = o / HO * S + dy, x = o % HO * S + dx;
                const bool in = y >= 0 && y < H && x >= 0 && x < H;
                const float v = a[b * HW + (in ? y * H + x : 0)];
                u = in ? fmaf(d[b * HWO + o], v, u) : u;
            }
            s += u;
        }
        wred[ch * 256 + t] = s;
    }
    __syncthreads();
    if (t < KK) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < SEG; ++k) s += wred[ch * 256 + k * KK + t];
        const int64_t i = p.o.wdw + (int64_t)c * KK + t;
        p.grd[i] = s;
        p.prm[i] = __builtin_fmaf(-p.lr, s, p.prm[i]);
    }
    // the input gradient, over a (read for the last time above)
    FO_ROWS(r, R) {
        const int b = r / HW, yy = r / H % H, xx = r % H;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < KK; ++q) {
            const int ty = yy + KD / 2 - q / KD, tx = xx + KD / 2 - q % KD;  // = oy S, ox S
            const bool in = ty >= 0 && tx >= 0 && ty % S == 0 && tx % S == 0 && ty / S < HO && tx / S < HO;
            const float u = d[b * HWO + (in ? ty / S * HO + tx / S : 0)];
            v = in ? fmaf(u, w[q], v) : v;
        }
        a[r] = v;
    }
    bn_grad(a, xh1, p.rs1[c], R, true, p.prm, p.grd, p.o.g1 + c, p.o.b1 + c, p.lr, red);
    FO_ROWS(r, p.ld1) p.dz1[(int64_t)c * p.ld1 + r] = r < R ? a[r] : 0.f;
}

// dh = dz3 Wpr for four channels; a block without squeeze-excitation goes on
// down to dz1, one with it leaves dh and the squeeze's gradient dt.
template <int KD, int H, int S, bool SE>
__global__ void __launch_bounds__(T) mb_dh(const Chain p) {
    constexpr int HO = (H + 2 * (KD / 2) - KD) / S + 1, HWO = HO * HO;
    __shared__ __attribute__((aligned(16))) float sm[SMEM];
    __shared__ float red[16], wred[CG * 256];
    const int c0 = blockIdx.x * CG, Ro = p.B * HWO;
    product4<true>(p.dz3, p.dz3.p, p.co, p.wpr, p.e, c0, Ro, sm);
    if constexpr (SE) {
        const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = c0 + ch;
        const float *d = sm + ch * Ro, *a = p.a2 + (int64_t)c * p.ld2;
        FO_ROWS(r, Ro) p.dh[(int64_t)c * p.ld2 + r] = d[r];
        FO_ROWS(b, p.ldb) {
            float v = 0.f;
            if (b < p.B) {
#pragma unroll
                for (int q = 0; q < HWO; ++q) v = fmaf(d[b * HWO + q], a[b * HWO + q], v);
                v *= hsig_d(p.t[(int64_t)c * p.ldb + b]);
            }
            p.dt[(int64_t)c * p.ldb + b] = v;
        }
    } else {
        chain_down<KD, H, S>(p, sm, sm + S1, red, wred, c0);
    }
}

// The rest of a squeeze-excitation block: da2 = dh hard-sigmoid(t) + dm / HW, down to dz1.
template <int KD, int H, int S>
__global__ void __launch_bounds__(T) mb_chain(const Chain p) {
    constexpr int HO = (H + 2 * (KD / 2) - KD) / S + 1, HWO = HO * HO;
    __shared__ float sm[SMEM], red[16], wred[CG * 256];
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), c = blockIdx.x * CG + ch, Ro = p.B * HWO;
    FO_ROWS(r, Ro) {
        const int64_t tb = (int64_t)c * p.ldb + r / HWO;
        sm[ch * Ro + r] = fmaf(p.dh[(int64_t)c * p.ld2 + r], hsig(p.t[tb]), p.dm[tb] / HWO);
    }
    chain_down<KD, H, S>(p, sm, sm + S1, red, wred, blockIdx.x * CG);
}

// ------------------------------------------------------------------ weight gradients and their update
constexpr int kUnits = 2 * NBLK + 1 + 2 * 5 + 2;
struct Units {
    WUnit u[kUnits];
    int n, tasks;
};

__global__ void __launch_bounds__(256) mb_wgrad(const Units p, const StepIn* __restrict__ in, float* __restrict__ prm,
                                                float* __restrict__ grd, float lr) {
    const int task = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (task >= p.tasks) return;
    int ui = 0;
    while (ui + 1 < p.n && p.u[ui + 1].task0 <= task) ++ui;
    wgrad_32x32(p.u[ui], task - p.u[ui].task0, in, prm, grd, lr);
}

constexpr bool all_by_four() {
    for (int j = 0; j < NBLK; ++j) {
        const BlkOff& o = kOffs.bk[j];
        for (int64_t v : {o.wex, o.g1, o.wdw, o.g2, o.wpr, o.g3})
            if (v % 4) return false;
        if (kBlk[j].se && (o.wse1 % 4 || o.wse2 % 4 || se_width(kBlk[j].e) % 8)) return false;
        if (kBlk[j].e % 8 || kBlk[j].co % 8) return false;
    }
    return kOffs.wl % 4 == 0 && kOffs.wf1 % 4 == 0 && kOffs.wf2 % 4 == 0;
}
static_assert(all_by_four(), "16-byte weight accesses, products over multiples of 8");

}  // namespace

// ------------------------------------------------------------------ plan
struct FBlk {
    float *xh1, *rs1, *xh2, *rs2, *a2, *m, *q, *t, *h, *xh3, *rs3, *y;
    float *dy, *dz3, *dh, *dt, *dq, *dm, *dz1;
};
struct Fused {
    FBlk b[NBLK];
    float *xhl, *rsl, *gp, *fpre, *f, *dz, *df, *dg, *dzl;
};

namespace {

int side(int j) { return j <= 5 ? 4 : 2; }  // of block j's input

size_t carve(Fused* F, int Bm, Arena* ar) {
    size_t s = 0;
    auto take = [&](float*& p, size_t n) {
        s += (n * sizeof(float) + 255) & ~size_t(255);
        if (ar) p = ar->take<float>(n);
    };
    const size_t ldb = pad16(Bm);
    for (int j = 0; j < NBLK; ++j) {
        const Shape& k = kBlk[j];
        FBlk& b = F->b[j];
        const size_t l1 = pad16(Bm * side(j) * side(j)), l2 = pad16(Bm * side(j + 1) * side(j + 1));
        for (float** p : {&b.xh1, &b.dz1}) take(*p, k.e * l1);
        for (float** p : {&b.xh2, &b.a2, &b.h, &b.dh}) take(*p, k.e * l2);
        for (float** p : {&b.m, &b.t, &b.dt, &b.dm, &b.q, &b.dq}) take(*p, k.e * ldb);
        for (float** p : {&b.xh3, &b.y, &b.dy, &b.dz3}) take(*p, k.co * l2);
        for (float** p : {&b.rs1, &b.rs2, &b.rs3}) take(*p, k.e);
    }
    const size_t ll = pad16(Bm * 4);
    for (float** p : {&F->xhl, &F->dzl}) take(*p, CLAST * ll);
    take(F->rsl, CLAST);
    for (float** p : {&F->gp, &F->dg}) take(*p, CLAST * ldb);
    for (float** p : {&F->fpre, &F->f, &F->df}) take(*p, F1 * ldb);
    take(F->dz, NCLS * ldb);
    return s;
}

}  // namespace

size_t fused_bytes(int max_batch) {
    Fused F;
    return carve(&F, std::min(max_batch, kFusedMax), nullptr);
}

fo_status fused_init(fo_model* m, int max_batch, Fused** out) {
    Fused* F = new (std::nothrow) Fused();
    if (!F) return FO_ENOMEM;
    *out = F;
    carve(F, std::min(max_batch, kFusedMax), &m->arena);
    if (!F->dz) {
        set_error("mbv3: workspace arena too small");
        return FO_ENOMEM;
    }
    return FO_OK;
}

void fused_destroy(Fused* f) { delete f; }

fo_status fused_step(fo_model* m, const Fused* F, int B) {
    static_assert(RMAX <= 2 * T && CG * RMAX <= S1, "rows of four channels in LDS");
    hipStream_t s = m->stream;
    float *prm = m->params, *grd = m->grads;
    const StepIn* in = m->dev_in;
    const int ldb = pad16(B);
    const float lr = m->lr;
    auto maps = [](const float* p, int ld) { return Act2{p, 16, ld}; };
    const Act2 batch = {nullptr, (int64_t)CIN * 16, 16};
    // linear layers over the samples
    auto lin = [&](const float* W, const float* X, int N, int K) {
        Lin l{};
        l.W = W;
        l.X = X;
        l.N = N;
        l.K = K;
        l.B = B;
        l.ldb = ldb;
        return l;
    };
    auto grid = [&](int N) { return dim3((unsigned)cdiv(N, 16), (unsigned)cdiv(ldb, 32)); };

    // ---------------- forward (Alg. 4: forward pass of M_s)
    for (int j = 0; j < NBLK; ++j) {
        const Shape& k = kBlk[j];
        const BlkOff& o = kOffs.bk[j];
        const FBlk& b = F->b[j];
        const int H = side(j), HO = side(j + 1), R = B * H * H, Ro = B * HO * HO, cin = j ? kBlk[j - 1].co : CIN;
        const int ld1 = pad16(R), ld2 = pad16(Ro);
        Expand e{};
        e.in = in;
        e.x = j ? maps(F->b[j - 1].y, ld1) : batch;
        e.wex = prm + o.wex; e.g1 = prm + o.g1; e.b1 = prm + o.b1;
        e.wdw = prm + o.wdw; e.g2 = prm + o.g2; e.b2 = prm + o.b2;
        e.xh1 = b.xh1; e.rs1 = b.rs1; e.xh2 = b.xh2; e.rs2 = b.rs2; e.a2 = b.a2;
        e.m = k.se ? b.m : nullptr;
        e.cin = cin; e.e = k.e; e.B = B; e.ld1 = ld1; e.ld2 = ld2; e.ldb = ldb;
        const dim3 ge(k.e / CG);
        if (k.k == 3) hipLaunchKernelGGL((mb_expand<3, 4, 1>), ge, dim3(T), 0, s, e);
        else if (H == 4) hipLaunchKernelGGL((mb_expand<5, 4, 2>), ge, dim3(T), 0, s, e);
        else hipLaunchKernelGGL((mb_expand<5, 2, 1>), ge, dim3(T), 0, s, e);
        const float* h = b.a2;
        if (k.se) {
            const int S = se_width(k.e);
            Lin l = lin(prm + o.wse1, b.m, S, k.e);
            l.bias = prm + o.bse1;
            l.out = b.q;
            hipLaunchKernelGGL((linear_small<false, E_RELU>), grid(S), dim3(LIN_T), 0, s, l);
            l = lin(prm + o.wse2, b.q, k.e, S);
            l.bias = prm + o.bse2;
            l.out = b.t;
            l.a2 = b.a2; l.h = b.h; l.hw = HO * HO; l.ld2 = ld2;
            hipLaunchKernelGGL((linear_small<false, E_SCALE>), grid(k.e), dim3(LIN_T), 0, s, l);
            h = b.h;
        }
        Project q{};
        q.in = in;
        q.h = maps(h, ld2);
        q.w = prm + o.wpr; q.g = prm + o.g3; q.b = prm + o.b3;
        q.has_res = k.stride == 1 && cin == k.co;
        q.res = e.x;
        q.xh = b.xh3; q.rs = b.rs3; q.y = b.y;
        q.K = k.e; q.R = Ro; q.B = B; q.ld = ld2; q.ldb = ldb;
        hipLaunchKernelGGL(mb_project, dim3(k.co / CG), dim3(T), 0, s, q);
    }
    const int Rl = B * 4, ldl = pad16(Rl), clast = kBlk[NBLK - 1].co;
    {
        Project q{};
        q.h = maps(F->b[NBLK - 1].y, ldl);
        q.w = prm + kOffs.wl; q.g = prm + kOffs.gl; q.b = prm + kOffs.bl;
        q.xh = F->xhl; q.rs = F->rsl; q.mean = F->gp;
        q.K = clast; q.R = Rl; q.B = B; q.ld = ldl; q.ldb = ldb;
        hipLaunchKernelGGL(mb_project, dim3(CLAST / CG), dim3(T), 0, s, q);
        Lin l = lin(prm + kOffs.wf1, F->gp, F1, CLAST);
        l.bias = prm + kOffs.bf1;
        l.out = F->fpre;
        l.out2 = F->f;
        hipLaunchKernelGGL((linear_small<false, E_HSWISH>), grid(F1), dim3(LIN_T), 0, s, l);
        l = lin(prm + kOffs.wf2, F->f, NCLS, F1);
        l.bias = prm + kOffs.bf2;
        l.out2 = m->logits;
        hipLaunchKernelGGL((linear_small<false, E_LOGITS>), grid(NCLS), dim3(LIN_T), 0, s, l);
    }
    hipLaunchKernelGGL(mb_xent, dim3(1), dim3(1024), 0, s, m->logits, in, F->dz, m->loss, B, ldb);
    FO_LAUNCHED();

    // ---------------- backward (Alg. 4: backward pass of M_s)
    Units un{};
    auto unit = [&](const float* dy, Act2 x, int64_t w, int64_t bias, int N, int K, int ld) {
        un.u[un.n++] = WUnit{dy, x, w, bias, N, K, ld, un.tasks};
        un.tasks += (int)(cdiv(N, 32) * cdiv(K, 32));
    };
    {
        Lin l = lin(prm + kOffs.wf2, F->dz, F1, NCLS);
        l.aux = F->fpre;
        l.out = F->df;
        hipLaunchKernelGGL((linear_small<true, E_DHSWISH>), grid(F1), dim3(LIN_T), 0, s, l);
        l = lin(prm + kOffs.wf1, F->df, CLAST, F1);
        l.out = F->dg;
        hipLaunchKernelGGL((linear_small<true, E_PLAIN>), grid(CLAST), dim3(LIN_T), 0, s, l);
        const LastBwd p{F->dg, F->xhl, F->rsl, prm, grd, F->dzl, kOffs.gl, kOffs.bl, lr, B, Rl, ldl, ldb};
        hipLaunchKernelGGL(mb_last_bwd, dim3(CLAST / CG), dim3(T), 0, s, p);
        unit(F->df, maps(F->gp, ldb), kOffs.wf1, kOffs.bf1, F1, CLAST, ldb);
        unit(F->dz, maps(F->f, ldb), kOffs.wf2, kOffs.bf2, NCLS, F1, ldb);
        unit(F->dzl, maps(F->b[NBLK - 1].y, ldl), kOffs.wl, -1, CLAST, clast, ldl);
    }
    for (int j = NBLK - 1; j >= 0; --j) {
        const Shape& k = kBlk[j];
        const BlkOff& o = kOffs.bk[j];
        const FBlk& b = F->b[j];
        const int H = side(j), HO = side(j + 1), R = B * H * H, Ro = B * HO * HO, cin = j ? kBlk[j - 1].co : CIN;
        const int ld1 = pad16(R), ld2 = pad16(Ro);
        const bool last = j == NBLK - 1;
        BlkDx d{};
        d.dzu = last ? maps(F->dzl, ldl) : maps(F->b[j + 1].dz1, ld2);
        d.wu = prm + (last ? kOffs.wl : kOffs.bk[j + 1].wex);
        d.K = last ? CLAST : kBlk[j + 1].e;
        d.dyu = !last && kBlk[j + 1].stride == 1 && k.co == kBlk[j + 1].co ? F->b[j + 1].dy : nullptr;
        d.xh = b.xh3; d.rs = b.rs3;
        d.prm = prm; d.grd = grd; d.dy = b.dy; d.dz = b.dz3;
        d.gi = o.g3; d.bi = o.b3; d.lr = lr;
        d.co = k.co; d.R = Ro; d.ld = ld2;
        hipLaunchKernelGGL(mb_dx, dim3(k.co / CG), dim3(T), 0, s, d);
        Chain c{};
        c.dz3 = maps(b.dz3, ld2);
        c.wpr = prm + o.wpr;
        c.xh1 = b.xh1; c.rs1 = b.rs1; c.xh2 = b.xh2; c.rs2 = b.rs2;
        c.a2 = b.a2; c.t = b.t; c.dm = b.dm; c.dh = b.dh; c.dt = b.dt;
        c.prm = prm; c.grd = grd; c.dz1 = b.dz1;
        c.o = o; c.lr = lr;
        c.co = k.co; c.e = k.e; c.B = B; c.ld1 = ld1; c.ld2 = ld2; c.ldb = ldb;
        const dim3 ge(k.e / CG);
        if (!k.se) {
            hipLaunchKernelGGL((mb_dh<3, 4, 1, false>), ge, dim3(T), 0, s, c);
        } else {
            const int S = se_width(k.e);
            if (k.k == 3) hipLaunchKernelGGL((mb_dh<3, 4, 1, true>), ge, dim3(T), 0, s, c);
            else if (H == 4) hipLaunchKernelGGL((mb_dh<5, 4, 2, true>), ge, dim3(T), 0, s, c);
            else hipLaunchKernelGGL((mb_dh<5, 2, 1, true>), ge, dim3(T), 0, s, c);
            Lin l = lin(prm + o.wse2, b.dt, S, k.e);
            l.aux = b.q;
            l.out = b.dq;
            hipLaunchKernelGGL((linear_small<true, E_DRELU>), grid(S), dim3(LIN_T), 0, s, l);
            l = lin(prm + o.wse1, b.dq, k.e, S);
            l.out = b.dm;
            hipLaunchKernelGGL((linear_small<true, E_PLAIN>), grid(k.e), dim3(LIN_T), 0, s, l);
            if (k.k == 3) hipLaunchKernelGGL((mb_chain<3, 4, 1>), ge, dim3(T), 0, s, c);
            else if (H == 4) hipLaunchKernelGGL((mb_chain<5, 4, 2>), ge, dim3(T), 0, s, c);
            else hipLaunchKernelGGL((mb_chain<5, 2, 1>), ge, dim3(T), 0, s, c);
            unit(b.dt, maps(b.q, ldb), o.wse2, o.bse2, k.e, S, ldb);
            unit(b.dq, maps(b.m, ldb), o.wse1, o.bse1, S, k.e, ldb);
        }
        unit(b.dz3, maps(k.se ? b.h : b.a2, ld2), o.wpr, -1, k.co, k.e, ld2);
        unit(b.dz1, j ? maps(F->b[j - 1].y, ld1) : batch, o.wex, -1, k.e, cin, ld1);
    }
    // ---------------- weight gradients and SGD (Alg. 4)
    hipLaunchKernelGGL(mb_wgrad, dim3((unsigned)cdiv(un.tasks, 4)), dim3(256), 0, s, un, in, prm, grd, lr);
    FO_LAUNCHED();
    return FO_OK;
}

}  // namespace mbv3
}  // namespace fo
