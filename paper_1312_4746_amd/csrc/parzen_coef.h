// The pair exponent and the per (label, pixel) coefficients of the Parzen sum,
// shared by the exact kernel's files and the matrix-core path's preparation.
#pragma once

#include "cs_internal.h"

namespace cs {

constexpr double kLog2e = 1.4426950408889634;
constexpr double kLn2 = 0.6931471805599453;
constexpr int kRefSubset = 4;
constexpr float kRefMargin = 48.0f;

template <int NW>
__device__ __forceinline__ float pair_e(float px, float py, float pr, float pg, float pb,
                                        const uint32_t (&mx)[NW], const uint32_t *rw, float nA,
                                        float nB, float nC) {
    const float dx = px - __uint_as_float(rw[0]);
    const float dy = py - __uint_as_float(rw[1]);
    const float d2 = fmaf(dy, dy, dx * dx);
    const float dr = pr - __uint_as_float(rw[2]);
    const float dg = pg - __uint_as_float(rw[3]);
    const float db = pb - __uint_as_float(rw[4]);
    const float c2 = fmaf(db, db, fmaf(dg, dg, dr * dr));
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t = __popc(mx[w] ^ rw[8 + w]) + t;
    float e = (float)t * nB;
    e = fmaf(nC, c2, e);
    e = fmaf(nA, d2, e);
    return e;
}

// Per (label, pixel) coefficients of the pair exponent in log2 units, from
// the exact nearest-sample distance d (FP32):
//   nA = -log2(e) / (2 rho^2), nB = -log2(e) / beta, rho = alpha_rho max(d, r_f),
//   (nB = 0 when the texture factor is applied outside the sum, eq:joined),
//   K  = -log m_i - log(2 pi) - 1.5 log(2 pi sigma_c^2) - log(rho^2),
//   nR = -R with the log-sum-exp reference R = min(U, e^ + kRefMargin):
//   U = nA d^2 bounds every exponent from above, e^ is the largest exponent
//   over the nearest sample and kRefSubset strided samples of the label (an
//   achieved value, so the sum is at least 2^-kRefMargin).
// coef[l * npix + i] = {nA, nB, nR, K}; pixel i is subset[i] or i.
// Tiled layout (matrix-core path): slot i = tile * kTilePix + q, the pixel of
// fast_slot_row (the tile grid, or entry i of the subset); empty slots get
// {0, 0, -200, 0} (their terms vanish).
template <int NW>
__device__ __forceinline__ void coef_of(const ParzenArgs &a, float4 *__restrict__ coef, int64_t i, int l0, int l1) {
    const int64_t nslots = a.coef_tiled ? (int64_t)a.ntiles_pad * kTilePix : a.npix;
    if (i >= nslots) return;
    const int64_t N = (int64_t)a.H * a.W;
    const int W64 = (a.k + 63) / 64;
    int64_t pix;
    if (a.coef_tiled) {
        const int t = (int)(i / kTilePix), q = (int)(i - (int64_t)t * kTilePix);
        const int64_t row = fast_slot_row(a.subset, a.npix, a.H, a.W, a.tiles_x, a.ntiles_real, t, q);
        if (row < 0) {
            for (int l = l0; l < l1; ++l) coef[(int64_t)l * nslots + i] = make_float4(0.0f, 0.0f, -200.0f, 0.0f);
            return;
        }
        pix = fast_row_pixel(a.subset, row);
    } else {
        pix = a.subset ? (int64_t)a.subset[i] : i;
    }
    const uint32_t *mask32 = reinterpret_cast<const uint32_t *>(a.masks);
    const float nC = (float)(-kLog2e / (2.0 * a.sigma_c * a.sigma_c));
    const uint32_t w32 = (uint32_t)a.W, y = (uint32_t)pix / w32;  // (32-bit divisions: an image has fewer than 2^31 pixels)
    const float px = (float)((uint32_t)pix - y * w32), py = (float)y;
    const float pr = a.rgb[pix], pg = a.rgb[N + pix], pb = a.rgb[2 * N + pix];
    uint32_t mx[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) mx[w] = mask32[pix * 2 * W64 + w];
#pragma unroll 1
    for (int l = l0; l < l1; ++l) {
        const int d2min = a.d2[(int64_t)l * N + pix];
        const int64_t nearp = a.nearest[(int64_t)l * N + pix];
        // FP32 from here (the results are FP32; a few ulps against one rounding)
        const float fl2 = (float)(a.rho_floor * a.rho_floor);
        const float dm = fmaxf((float)d2min, fl2);
        const float rho2 = (float)(a.alpha_rho * a.alpha_rho) * dm;
        const float rho = sqrtf(rho2);
        const float nA = -(float)kLog2e / (2.0f * rho2);
        const float nB = a.texture_in_sum ? -(float)kLog2e / ((float)a.beta_scale * rho) : 0.0f;
        const float K = (float)a.kconst[l] - logf(rho2);
        uint32_t nrec[kRecWords];
#pragma unroll
        for (int w = 0; w < NW; ++w) nrec[8 + w] = mask32[nearp * 2 * W64 + w];
        const uint32_t ny = (uint32_t)nearp / w32;
        nrec[0] = __float_as_uint((float)((uint32_t)nearp - ny * w32));
        nrec[1] = __float_as_uint((float)ny);
        nrec[2] = __float_as_uint(a.rgb[nearp]);
        nrec[3] = __float_as_uint(a.rgb[N + nearp]);
        nrec[4] = __float_as_uint(a.rgb[2 * N + nearp]);
        float est = pair_e<NW>(px, py, pr, pg, pb, mx, nrec, nA, nB, nC);
        // Largest exponent over the nearest sample and an evenly strided subset of
        // the label's samples: an achieved value close to the maximum.
        const int s0 = a.seg_off[l], m = a.seg_off[l + 1] - s0;
        const int nsub = m < kRefSubset ? m : kRefSubset;
        const uint32_t *recw = reinterpret_cast<const uint32_t *>(a.recs);
        for (int j = 0; j < nsub; ++j) {
            const int64_t sidx = s0 + (int64_t)j * m / nsub;
            est = fmaxf(est, pair_e<NW>(px, py, pr, pg, pb, mx, recw + sidx * kRecWords, nA, nB, nC));
        }
        const float U = nA * (float)d2min;
        coef[(int64_t)l * nslots + i] = make_float4(nA, nB, -fminf(U, est + kRefMargin), K);
    }
}

}  // namespace cs
