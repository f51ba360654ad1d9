// The server part of MobileNetV3-Large (config 10): its shapes, its activation
// functions and the interface of its fused step.
#pragma once

#include "kernels.h"
#include "model.h"

namespace fo {
namespace mbv3 {

constexpr int CIN = 80, HIN = 4, CLAST = 960, F1 = 1280, NCLS = 200, NBLK = 8;
constexpr float BN_EPS = 1e-5f;

struct Shape {
    int k, e, co, se, stride;
};
constexpr Shape kBlk[NBLK] = {{3, 200, 80, 0, 1}, {3, 184, 80, 0, 1}, {3, 184, 80, 0, 1}, {3, 480, 112, 1, 1},
                              {3, 672, 112, 1, 1}, {5, 672, 160, 1, 2}, {5, 960, 160, 1, 1}, {5, 960, 160, 1, 1}};
// squeeze width: e / 4 to a multiple of 8, at least 8, not below 90% of e / 4
constexpr int se_width(int e) {
    return (e / 4 + 4) / 8 * 8 < 8 ? 8
           : ((e / 4 + 4) / 8 * 8 < 0.9 * (e / 4) ? (e / 4 + 4) / 8 * 8 + 8 : (e / 4 + 4) / 8 * 8);
}

// Offsets of a block's parameters in the flat vector (se*: -1 without squeeze-excitation).
struct BlkOff {
    int64_t wex, g1, b1, wdw, g2, b2, wse1, bse1, wse2, bse2, wpr, g3, b3;
};
struct Offs {
    BlkOff bk[NBLK];
    int64_t wl, gl, bl, wf1, bf1, wf2, bf2, total;
};
constexpr Offs make_offs() {
    Offs o{};
    int64_t p = 0;
    int ci = CIN;
    for (int j = 0; j < NBLK; ++j) {
        const Shape& b = kBlk[j];
        BlkOff& k = o.bk[j];
        k.wex = p; p += (int64_t)b.e * ci;
        k.g1 = p; p += b.e;
        k.b1 = p; p += b.e;
        k.wdw = p; p += (int64_t)b.e * b.k * b.k;
        k.g2 = p; p += b.e;
        k.b2 = p; p += b.e;
        k.wse1 = k.bse1 = k.wse2 = k.bse2 = -1;
        if (b.se) {
            const int s = se_width(b.e);
            k.wse1 = p; p += (int64_t)s * b.e;
            k.bse1 = p; p += s;
            k.wse2 = p; p += (int64_t)b.e * s;
            k.bse2 = p; p += b.e;
        }
        k.wpr = p; p += (int64_t)b.co * b.e;
        k.g3 = p; p += b.co;
        k.b3 = p; p += b.co;
        ci = b.co;
    }
    o.wl = p; p += (int64_t)CLAST * ci;
    o.gl = p; p += CLAST;
    o.bl = p; p += CLAST;
    o.wf1 = p; p += (int64_t)F1 * CLAST;
    o.bf1 = p; p += F1;
    o.wf2 = p; p += (int64_t)NCLS * F1;
    o.bf2 = p; p += NCLS;
    o.total = p;
    return o;
}
constexpr Offs kOffs = make_offs();

// The fused step (k_mbv3.hip) for batches of at most kFusedMax samples: a
// channel's rows (16 per sample) have to fit in LDS four channels at a time.
constexpr int kFusedMax = 128;
struct Fused;
size_t fused_bytes(int max_batch);
fo_status fused_init(fo_model* m, int max_batch, Fused** out);  // carves m->arena
void fused_destroy(Fused* f);
fo_status fused_step(fo_model* m, const Fused* f, int B);

}  // namespace mbv3
}  // namespace fo
