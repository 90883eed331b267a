// Patch analysis for patches up to 11 x 11 on gfx950 (instantiated per patch
// size by the k_patch*.hip files; larger patches: k_analyze.hip): normalised
// Gaussian-masked gray patches (Sec. 3.1), the contraction a = O s on MFMA
// (Sec. 2) and its output: FP32 vectors, co-support masks, or (kPatchSelect)
// vectors and, of the FP32 products, the masks and lists of a median's bracket.
//
// Bound by the FP32 matrix units at large k (11 x 11, k = 242: two thirds of a
// tile's time; the halo, the statistics and the patches take the rest) and by
// the stores of a at small k.  1024 x 1024, 11 x 11, k = 242: 946 -> 700 us
// (BF16 products: 634 -> 340 us); 2048 x 2048, 7 x 7, k = 98: 964 -> 823 us
// (BF16 628 -> 538 us, 3.1 TB/s of stores); 481 x 321, 11 x 11, k = 242: 180 ->
// 136 us (before: one workgroup per tile, the operator read by each).
// kPatchSelect is bound by its vector instructions (some 20 per 64 entries for the
// tests and lists): 2048 x 2048, 7 x 7, k = 98, FP32 and BF16 products 1173 us,
// where the two analyses and a pass over the FP32 vectors took 1870 us; without
// listing anything 1090 us.
//
// Persistent workgroups of four waves walk tiles of TP pixels of one image
// row.  Wave w keeps the operator rows of the 16-row blocks w, w + 4, ... in
// registers as MFMA B fragments for all its tiles, so the operator is read
// once per workgroup (read per tile, its scattered rows kept the address unit
// of the L1 busier than the matrix cores: 0.46 of the time for those at
// 1024 x 1024, 11 x 11, k = 242).  Per tile:
// 1. the FP64 gray halo in LDS (requested and put there during the tile
//    before, ahead of most of its stores: a wait for loads also waits for
//    every older store);
// 2. mean and squared norm of every masked patch q_t = w_t g_t from column
//    sums (the Gaussian mask is a product of its row and its column factor):
//    nu2 = sum q^2 - n mu^2 in FP64.  Where that cancels (nu2 <= 1e-6 sum q^2,
//    a flat patch under a wide mask; a constant patch has nu2 = 0 exactly), and
//    where sum q^2 is so small that its terms may have lost bits below the
//    normal range (a narrow mask over black pixels), the sums run entry by
//    entry in the order of the definition;
// 3. s_t = (q_t - mu) (1 / nu) in FP64, rounded once to FP32, into LDS as four
//    runs of KF entries per pixel: lane group g of an MFMA operand takes run
//    g, so its A values are 16-byte aligned pieces of one row;
// 4. 16 pixels x 16 rows per MFMA chain, chains of at most 32 products whose
//    sums are added at the end (shorter chains: a smaller rounding bound).
//
// Output layout of the 16x16 MFMA tile: lane l, accumulator r holds pixel
// 4*(l/16) + r of the block and operator row l%16 of the row block.
#pragma once
#pragma clang fp contract(off)

#include <type_traits>

#include "cs_internal.h"
#include "cs_device.h"
#include "../../include/cosparse.h"

namespace cs {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int P>
struct PatchTile {
    static constexpr int h = (P - 1) / 2, n = P * P;
    static constexpr int KF = (n + 3) / 4;                // entries of a run (FP32 K steps)
    static constexpr int RS = (KF + 3) / 4 * 4;           // its place, 16-byte aligned
    static constexpr int ss = 4 * RS + 4;                 // row stride; ss / 4 odd: distinct banks
    static constexpr int CQ = patch_chain_quads(P);       // 16-product pieces per chain
    static constexpr int TP = 64;                         // pixels per tile
    static constexpr int hw = TP + 2 * h, halo = P * hw, halo_it = (halo + 255) / 256;
};

enum { kPatchAlpha = 0, kPatchMasks = 1, kPatchSelect = 2 };

// LDS of the mask output: the tile's co-support pieces (pixel major), its
// entries in between (one word of pixels per operator row), and the hand-offs
// of their exact evaluation.
constexpr int kNearList = 1024;
struct PatchNear {
    uint64_t mk[64 * 4];
    uint64_t rows[256];
    uint64_t part[4];
    int sums[4];
    uint16_t list[kNearList];
    uint8_t px[64];
};

template <class V>
using lds_ptr = __attribute__((address_space(3))) V *;

// Decides the tile's entries in between exactly: every sum sequential in t in
// FP64 (the order of the definition), mu = sum q / n, nu2 = sum (q - mu)^2,
// s_t = (q_t - mu) / sqrt(nu2) (0 when nu2 = 0), a_j = sum O_jt s_t.  Only the
// pixels that have such entries are formed, 32 at a time, in the place of the
// FP32 patches; the entries are listed row by row, so a wave reads few operator
// rows, and every thread takes one.  (One lane per entry inside the epilogue,
// the rest of its wave waiting, took 30.6 ms of masks at 1024 x 1024, 11 x 11,
// k = 242 in BF16, where a fifth of all entries lie in between; 4.3 ms here,
// and in FP32, where one in a few thousand does, 2.09 -> 1.76 ms.)
// mus, nus: places for 32 means and norms.
template <int P>
__device__ __noinline__ void resolve_near(const float *omega, const double *wmask, double tau, int W64,
                                          lds_ptr<const double> gh, lds_ptr<double> sd, lds_ptr<double> mus,
                                          lds_ptr<double> nus, lds_ptr<PatchNear> nr) {
#pragma clang fp contract(off)
    using T = PatchTile<P>;
    constexpr int n = T::n, hw = T::hw;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t mine = nr->rows[tid];
    uint32_t lo = (uint32_t)mine, hi = (uint32_t)(mine >> 32);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        lo |= (uint32_t)__shfl_xor((int)lo, d);
        hi |= (uint32_t)__shfl_xor((int)hi, d);
    }
    if (lane == 0) nr->part[wave] = (uint64_t)hi << 32 | lo;
    __syncthreads();
    const uint64_t px = nr->part[0] | nr->part[1] | nr->part[2] | nr->part[3];
    const int npx = __popcll(px);
    if (tid < 64 && (px >> tid & 1ull)) nr->px[__popcll(px & ((1ull << tid) - 1ull))] = (uint8_t)tid;
    __syncthreads();
    for (int b = 0; b < npx; b += 32) {
        const int cnt = min(32, npx - b);
        for (int e = tid; e < cnt * n; e += 256) {
            const int slot = e / n, t = e - slot * n;
            sd[e] = wmask[t] * gh[t / P * hw + nr->px[b + slot] + t % P];
        }
        __syncthreads();
        if (tid < cnt) {
            const lds_ptr<const double> q = sd + tid * n;
            double sum = 0.0;
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int v = 0; v < P; ++v) sum = sum + q[u * P + v];
            const double mu = sum / (double)n;
            double nu2 = 0.0;
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int v = 0; v < P; ++v) {
                    const double z = q[u * P + v] - mu;
                    nu2 = nu2 + z * z;
                }
            mus[tid] = mu;
            nus[tid] = nu2 == 0.0 ? 0.0 : sqrt(nu2);
        }
        __syncthreads();
        for (int e = tid; e < cnt * n; e += 256) {
            const int slot = e / n;
            const double nu = nus[slot];
            sd[e] = nu == 0.0 ? 0.0 : (sd[e] - mus[slot]) / nu;
        }
        // this thread's row's entries of these pixels, and their list places
        const uint64_t bits = mine & (~0ull << nr->px[b]) & (~0ull >> (63 - nr->px[b + cnt - 1]));
        const int c = __popcll(bits);
        int incl = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(incl, d);
            if (lane >= d) incl += v;
        }
        if (lane == 63) nr->sums[wave] = incl;
        __syncthreads();
        int off = incl - c, total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) off += nr->sums[w];
            total += nr->sums[w];
        }
        for (int w0 = 0; w0 < total; w0 += kNearList) {
            if (w0) __syncthreads();  // the list of the window before is done with
            int at = off - w0;
            for (uint64_t rest = bits; rest; rest &= rest - 1ull, ++at)
                if (at >= 0 && at < kNearList) nr->list[at] = (uint16_t)(tid << 6 | __builtin_ctzll(rest));
            __syncthreads();
            for (int e = tid; e < min(kNearList, total - w0); e += 256) {
                const int j = nr->list[e] >> 6, il = nr->list[e] & 63;
                const float *om = omega + (int64_t)j * n;
                const int s0 = (__popcll(px & ((1ull << il) - 1ull)) - b) * n;
                double acc = 0.0;
#pragma unroll 1
                for (int t0 = 0; t0 < n; t0 += 8) {
                    double sv[8];
                    float ov[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int t = t0 + u < n ? t0 + u : n - 1;
                        sv[u] = sd[s0 + t];
                        ov[u] = om[t];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (t0 + u < n) acc = acc + (double)ov[u] * sv[u];
                }
                if (fabs(acc) <= tau)
                    atomicOr(reinterpret_cast<unsigned int *>((PatchNear *)nr) + il * 2 * W64 + (j >> 5),
                             1u << (j & 31));
            }
        }
        __syncthreads();  // the patches and sums are formed anew
    }
}

// Workgroups per compute unit (waves per SIMD) that the operator fragments
// leave registers for.
constexpr int patch_waves(int p, int jb) { return jb * ((p * p + 3) / 4) <= 32 ? 4 : jb * ((p * p + 3) / 4) <= 64 ? 3 : 2; }
// The same for kPatchSelect, from an estimate of its registers (at 7 x 7, k = 98,
// BF16, four waves with 15 registers spilled: 1173 us, three without: 1227 us).
constexpr int patch_sel_regs(int p, int jb, bool bf16) {
    const int rs = ((p * p + 3) / 4 + 3) / 4 * 4;
    return 40 + 4 * ((p * (64 + p - 1) + 255) / 256) + jb * (rs + 14) + 18 + (bf16 ? jb * rs / 2 : 0);
}
constexpr int patch_waves_of(int p, int jb, int prec, int out) {
    if (out != kPatchSelect) return patch_waves(p, jb);
    const int r = patch_sel_regs(p, jb, prec == CS_BF16);
    return r <= 150 ? 4 : r <= 200 ? 3 : 2;
}

template <int P, int JB, int PREC, int OUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(patch_waves_of(P, JB, PREC, OUT))))
void k_patch(AnalyzeArgs a, int tiles_x, int ntiles) {
    using T = PatchTile<P>;
    constexpr int h = T::h, n = T::n, KF = T::KF, RS = T::RS, ss = T::ss, TP = T::TP, hw = T::hw;
    constexpr bool kSel = OUT == kPatchSelect;
    constexpr bool kB16 = PREC == CS_BF16, kF32 = !kB16 || kSel;  // the selection runs on the FP32 vectors
    if (a.skip && a.skip->br_ok) return;
    __shared__ double gh2[2][T::halo];  // this tile's gray halo and the next one's
    // sequential statistics a row of the patch at a time, the mask in LDS (the
    // other outputs have no registers for it)
    constexpr bool kSeqRow = OUT == kPatchAlpha;
    __shared__ double s_c1[hw], s_c2[hw], s_w[kSeqRow ? n : 1];
    __shared__ double s_mu[TP], s_ri[TP];  // mu and 1 / nu (0 for a zero patch)
    __shared__ __align__(16) float s[TP * ss];
    __shared__ char near_lds[OUT == kPatchMasks ? sizeof(PatchNear) : 1] __attribute__((aligned(16)));
    PatchNear *const nr = reinterpret_cast<PatchNear *>(near_lds);
    const int W64 = (a.k + 63) / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, jl = lane & 15;
    const int64_t N = (int64_t)a.H * a.W;
    const int nblk = (a.k + 15) / 16;
    // waves across operator blocks (4, or 2 or 1 where there are no more: the
    // waves then share out the pixels)
    const int js = nblk <= 2 ? nblk : 4, jw = wave & (js - 1), rb0 = wave / js, rbs = 4 / js;
    // mask weights, one per lane, read out by lane number (a scalar load per
    // weight waited for the scalar cache, 9.5k of 50k cycles per tile):
    // wrun lane i: entry KF wave + i; wrow lane i: the row factor of column i
    const int trun = KF * wave + lane;
    const double wrun = lane < KF && trun < n ? a.wmask[trun] : 0.0;
    const double wrow = a.wmask[h * P + (lane < P ? lane : 0)];
    auto of_lane = [](double v, int l) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, l), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), l);
        return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };

    // operator fragments: row 16 (jw + 4 u) + jl, run g (rows past k repeat
    // the last, their outputs are not used; entries past n are 0)
    float bf[kF32 ? JB : 1][kF32 ? RS : 1];
    s16x4 bb[kB16 ? JB : 1][kB16 ? RS / 4 : 1];
#pragma unroll
    for (int u = 0; u < JB; ++u) {
        const int j = 16 * (jw + 4 * u) + jl;
        const float *o = a.omega + (int64_t)(j < a.k ? j : a.k - 1) * n;
#pragma unroll
        for (int q = 0; q < RS / 4; ++q) {
            const int t0 = KF * g + 4 * q;
            float v[4];
            if (t0 + 4 <= n) {
                __builtin_memcpy(v, o + t0, 16);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = t0 + i < n ? o[t0 + i] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = 4 * q + i < KF ? v[i] : 0.0f;
                if constexpr (kF32) bf[u][4 * q + i] = x;
                if constexpr (kB16) bb[u][q][i] = bf16_rne(x);
            }
        }
    }
    float tin[OUT == kPatchMasks ? JB : 1], tout[OUT == kPatchMasks ? JB : 1];
    if constexpr (OUT == kPatchMasks) {
#pragma unroll
        for (int u = 0; u < JB; ++u) {
            const int j = 16 * (jw + 4 * u) + jl;
            tin[u] = j < a.k ? a.t_in[j] : 0.0f;
            tout[u] = j < a.k ? a.t_out[j] : 0.0f;
        }
    }
    unsigned long long nrecomp = 0;
    // kPatchSelect: the bracket, the rows' undecided intervals, the masks of
    // this tile and the last, this wave's list regions
    __shared__ float s_tin[kSel ? 256 : 1], s_tout[kSel ? 256 : 1];
    __shared__ uint64_t s_mk[2][kSel ? TP * 4 : 1];
    uint32_t blo = 0xFFFFFFFFu, bspan = 0, dbase = 0;
    uint64_t *breg = nullptr, *dreg = nullptr;
    uint32_t nb_w = 0, nd_w = 0, below = 0, region = 0, over = 0;  // wave-uniform
    uint64_t jvm[kSel ? JB : 1];  // the lanes that have a row
    if constexpr (kSel) {
        float ti = INFINITY, to = INFINITY;  // no bracket: nothing is listed
        if (a.sel_st->br_valid) {
            const double mm = *a.tau_max_margin;
            double tlo, thi;
            blo = a.sel_st->br_lo;
            bspan = a.sel_st->br_hi - blo;
            tau_interval((double)__uint_as_float(blo), (double)__uint_as_float(blo + bspan), mm, a.sel_frac, tlo, thi);
            dbase = tau_defer_base(tlo, mm);
            tau_row_interval(tlo, thi, tid < a.k ? a.tau_margins[tid] : 0.0, ti, to);
        }
        s_tin[tid] = ti;
        s_tout[tid] = to;
        s_mk[0][tid] = s_mk[1][tid] = 0;
        // what may be listed before a block that may list all its entries
        region = (uint32_t)a.sel_region > 256u * JB ? (uint32_t)a.sel_region - 256u * JB : 0u;
#pragma unroll
        for (int u = 0; u < JB; ++u) jvm[u] = __ballot(16 * (jw + 4 * u) + jl < a.k);
        const int64_t at = ((int64_t)blockIdx.x * 4 + wave) * a.sel_region;
        breg = a.sel_blist + at;
        dreg = a.sel_dlist + at;
    }
    // entry base + place (base wave-uniform) at `at` of a region, d above it
    auto put = [](uint64_t *reg, uint32_t at, uint64_t base, uint32_t place, uint32_t d) {
        const uint64_t e = base + place;
        uint32_t *o = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(reg) + 8u * at);
        const uint2 v = make_uint2((uint32_t)e, d << (kPackShift - 32) | (uint32_t)(e >> 32));
        *reinterpret_cast<uint2 *>(o) = v;
    };

    // places of this thread's halo entries, (row << 16) | column (32-bit
    // offsets from wave-uniform bases throughout: the operator fragments leave
    // few registers for addresses, and a spilled value waits for every store)
    uint32_t place[T::halo_it];
#pragma unroll
    for (int it = 0; it < T::halo_it; ++it) {
        const uint32_t idx = tid + 256 * it;
        place[it] = idx / hw << 16 | idx % hw;
    }
    float hr[T::halo_it], hg[T::halo_it], hb[T::halo_it];
    const float *const pr = a.rgb, *const pg = a.rgb + N, *const pb = a.rgb + 2 * N;
    auto request = [&](int tile) {  // the colours of a tile's halo (pixel 0 where there is none)
        const int row = tile / tiles_x, c0 = (tile - row * tiles_x) * TP;
        const int ncols = min(TP, a.W - c0) + 2 * h;
#pragma unroll
        for (int it = 0; it < T::halo_it; ++it) {
            const int rr = (int)(place[it] >> 16), cc = (int)(place[it] & 0xffffu);
            uint32_t src = 0;
            if (rr < P && cc < ncols)
                src = (uint32_t)reflect_idx(row - h + rr, a.H) * (uint32_t)a.W + (uint32_t)reflect_idx(c0 - h + cc, a.W);
            hr[it] = pr[src];
            hg[it] = pg[src];
            hb[it] = pb[src];
        }
    };
    auto arrive = [&](int tile, double *to) {  // the requested colours as gray values (0 past the row end)
        const int ncols = min(TP, a.W - (tile % tiles_x) * TP) + 2 * h;
#pragma unroll
        for (int it = 0; it < T::halo_it; ++it) {
            const int cc = (int)(place[it] & 0xffffu);
            if (tid + 256 * it < T::halo) to[tid + 256 * it] = cc < ncols ? gray64_of(hr[it], hg[it], hb[it]) : 0.0;
        }
    };
    const uint32_t lane_off = (uint32_t)(4 * g * a.k + jl);
    if (kSeqRow && tid < n) s_w[tid] = a.wmask[tid];
    int tile = blockIdx.x, par = 0;
    if (tile < ntiles) {
        request(tile);
        arrive(tile, gh2[0]);
    }
    int64_t last_pix = 0;  // kPatchSelect: the last tile's masks, still in LDS
    int last_words = 0;
    for (; tile < ntiles; tile += gridDim.x, par ^= 1) {
        const double *gh = gh2[par];
        const int row = tile / tiles_x, c0 = (tile - row * tiles_x) * TP;
        const int valid_px = min(TP, a.W - c0);
        if constexpr (OUT == kPatchMasks) {
            nr->mk[tid] = 0;
            nr->rows[tid] = 0;
        }
        __syncthreads();
        // 2. statistics: column sums, then each pixel's P columns
        static_assert(hw <= 128, "columns of two waves");
        if (wave < 2) {  // whole waves: a lane's weight is read from lanes past the last column too
            const int c = tid < hw ? tid : hw - 1;
            double c1 = 0.0, c2 = 0.0;
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const double w = of_lane(wrow, u), x = w * gh[u * hw + c];
                c1 += x;
                c2 += x * x;
            }
            if (tid < hw) {
                s_c1[c] = c1;
                s_c2[c] = c2;
            }
        } else if constexpr (kSel) {
            for (int idx = tid - 128; idx < last_words; idx += 128) a.masks[last_pix * W64 + idx] = s_mk[par ^ 1][idx];
        }
        __syncthreads();
        if (tid < TP) {
            double m = 0.0, q = 0.0;
#pragma unroll
            for (int v = 0; v < P; ++v) {
                const double w = of_lane(wrow, v);
                m += w * s_c1[tid + v];
                q += w * w * s_c2[tid + v];
            }
            double mu = m / (double)n, nu2 = q - m * mu;
            // (a term below the normal range is off by 2^-1074, nothing to a q above 2^-900)
            if (tid < valid_px && !(nu2 > 1e-6 * q && q > 0x1p-900)) {
                uint32_t any = 1;  // 0: a zero patch, told without its sums (black areas)
                if (q == 0.0) {
                    any = 0;
#pragma unroll 4
                    for (int t = 0; t < n; ++t) {
                        const uint64_t b = __builtin_bit_cast(uint64_t, gh[(t / P) * hw + tid + t % P]);
                        any |= (uint32_t)b | (uint32_t)(b >> 32);
                    }
                }
                if (any == 0) {
                    mu = nu2 = 0.0;
                } else if constexpr (kSeqRow) {
                    double sum = 0.0;
#pragma unroll 1
                    for (int u = 0; u < P; ++u)
#pragma unroll
                        for (int v = 0; v < P; ++v) sum = sum + s_w[u * P + v] * gh[u * hw + tid + v];
                    mu = sum / (double)n;
                    nu2 = 0.0;
#pragma unroll 1
                    for (int u = 0; u < P; ++u)
#pragma unroll
                        for (int v = 0; v < P; ++v) {
                            const double z = s_w[u * P + v] * gh[u * hw + tid + v] - mu;
                            nu2 = nu2 + z * z;
                        }
                } else {
                    double sum = 0.0;
                    for (int t = 0; t < n; ++t) sum = sum + a.wmask[t] * gh[(t / P) * hw + tid + t % P];
                    mu = sum / (double)n;
                    nu2 = 0.0;
                    for (int t = 0; t < n; ++t) {
                        const double z = a.wmask[t] * gh[(t / P) * hw + tid + t % P] - mu;
                        nu2 = nu2 + z * z;
                    }
                }
            }
            const double ri = nu2 == 0.0 || tid >= valid_px ? 0.0 : 1.0 / sqrt(nu2);
            s_ri[tid] = ri;
            s_mu[tid] = ri == 0.0 ? 0.0 : mu;
        }
        __syncthreads();
        // 3. FP32 patches: wave w writes run w of every pixel
#pragma unroll
        for (int i0 = 0; i0 < TP; i0 += 64) {
            const int i = i0 + lane;
            const double ri = s_ri[i], mu = s_mu[i];
#pragma unroll
            for (int q = 0; q < RS / 4; ++q) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int t = KF * wave + 4 * q + e;
                    const bool live = 4 * q + e < KF && t < n;
                    const int tt = live ? t : 0;
                    const double x = gh[(tt / P) * hw + i + tt % P];
                    v[e] = live ? (float)((of_lane(wrun, 4 * q + e) * x - mu) * ri) : 0.0f;
                }
                *reinterpret_cast<f32x4 *>(s + i * ss + wave * RS + 4 * q) = v;
                if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // the reads of later entries do not pile up in registers
            }
        }
        __syncthreads();
        const bool more = tile + (int)gridDim.x < ntiles;
        if (more) request(tile + gridDim.x);
        // 4. a = O s
        const int64_t pix0 = (int64_t)row * a.W + c0;
        const int nrb = (valid_px + 15) / 16;
        const int left = valid_px - 4 * g;
        auto block = [&](int rb, auto first) __attribute__((always_inline)) {
            const f32x4 *sr = reinterpret_cast<const f32x4 *>(s + (rb * 16 + jl) * ss + g * RS);
            f32x4 tot[kF32 ? JB : 1];
            if constexpr (kF32) {
#pragma unroll
                for (int q0 = 0; q0 < RS / 4; q0 += T::CQ) {
                    f32x4 acc[JB];
#pragma unroll
                    for (int u = 0; u < JB; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = q0; q < q0 + T::CQ && q < RS / 4; ++q) {
                        const f32x4 av = sr[q];
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (4 * q + i < KF)
#pragma unroll
                                for (int u = 0; u < JB; ++u)
                                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bf[u][4 * q + i], acc[u], 0,
                                                                                  0, 0);
                    }
#pragma unroll
                    for (int u = 0; u < JB; ++u) tot[u] = q0 == 0 ? acc[u] : tot[u] + acc[u];
                    __builtin_amdgcn_sched_barrier(0);  // one chain's accumulators at a time
                }
            }
            f32x4 hot[kB16 ? JB : 1];  // the BF16 products
            if constexpr (kB16) {
#pragma unroll
                for (int u = 0; u < JB; ++u) hot[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < RS / 4; ++q) {
                    const f32x4 av = sr[q];
                    const s16x4 ab = __builtin_bit_cast(
                        s16x4, make_uint2(bf16_pair(av[0], av[1]), bf16_pair(av[2], av[3])));
#pragma unroll
                    for (int u = 0; u < JB; ++u)
                        hot[u] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ab, bb[u][q], hot[u], 0, 0, 0);
                }
            }
            // the next tile's halo arrives ahead of this one's stores
            if (first.value && more) arrive(tile + gridDim.x, gh2[par ^ 1]);
            if constexpr (kSel) {
                // a list that is nearly full starts again: its call ends in the
                // general selection
                if (nb_w > region || nd_w > region) {
                    over = 1;
                    nb_w = nd_w = 0;
                }
                float ti[JB], to[JB];
#pragma unroll
                for (int u = 0; u < JB; ++u) {
                    ti[u] = s_tin[16 * (jw + 4 * u) + jl];
                    to[u] = s_tout[16 * (jw + 4 * u) + jl];
                }
                int col = 0;  // lane 8 u + 2 r + h: the mask pieces of pixels 8 h + r and 8 h + 4 + r
                uint64_t first_e = (uint64_t)(pix0 + rb * 16) * (uint64_t)a.k + 16 * jw;  // wave-uniform
#pragma unroll
                for (int r = 0; r < 4; ++r, first_e += a.k) {
                    const uint64_t pvm = __builtin_amdgcn_sicmp(left, rb * 16 + r, kSgt);
#pragma unroll
                    for (int u = 0; u < JB; ++u) {
                        if (jw + 4 * u >= nblk) break;
                        const uint64_t live = pvm & jvm[u];
                        const uint64_t e0 = first_e + 64 * u;
                        if (__builtin_amdgcn_inverse_ballot_w64(live)) {
                            float *out = a.alpha + e0 + lane_off;
                            if constexpr (kB16)
                                *out = hot[u][r];
                            else
                                *out = tot[u][r];
                        }
                        // rows past k and pixels past the row end get the key of
                        // +inf, which every test rejects (a bracket's intervals
                        // lie within FP32)
                        const float f = __builtin_amdgcn_inverse_ballot_w64(live) ? fabsf(tot[u][r]) : INFINITY;
                        const uint32_t x = __float_as_uint(f), d = x - blo;
                        below += (uint32_t)__popcll(__builtin_amdgcn_uicmp(x, blo, kUlt));
                        const uint64_t cm = __builtin_amdgcn_uicmp(d, bspan, kUle);
                        if (__builtin_amdgcn_inverse_ballot_w64(cm)) put(breg, nb_w + lane_prefix(cm), e0, lane_off, d);
                        nb_w += (uint32_t)__popcll(cm);
                        const uint64_t inb = __builtin_amdgcn_fcmpf(f, ti[u], kOle);
                        col = write_lane((int)(uint32_t)inb, u * 8 + r * 2, col);
                        col = write_lane((int)(uint32_t)(inb >> 32), u * 8 + r * 2 + 1, col);
                        const uint64_t dm = ~(inb | __builtin_amdgcn_fcmpf(f, to[u], kOgt));  // NaN: undecided
                        if (__builtin_amdgcn_inverse_ballot_w64(dm))
                            put(dreg, nd_w + lane_prefix(dm), e0, lane_off, min(x - dbase, kPackMax));
                        nd_w += (uint32_t)__popcll(dm);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                const int jb = jw + 4 * (lane >> 3);
                if (lane < 8 * JB && jb < nblk) {
                    uint16_t *mk = reinterpret_cast<uint16_t *>(s_mk[par]) + jb;
                    const int il = rb * 16 + 8 * (lane & 1) + (lane >> 1 & 3);
                    mk[il * 4 * W64] = (uint16_t)col;
                    mk[(il + 4) * 4 * W64] = (uint16_t)((uint32_t)col >> 16);
                }
                return;
            }
#pragma unroll
            for (int u = 0; u < JB; ++u) {
                const int jb = jw + 4 * u;
                if (jb >= nblk) break;
                const int j = 16 * jb + jl;
                const bool jv = j < a.k;
                uint32_t in_between = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool pv = rb * 16 + 4 * g + r < valid_px;
                    if constexpr (OUT == kPatchAlpha) {
                        float *out = a.alpha + ((pix0 + rb * 16 + r) * a.k + 16 * jb);  // wave-uniform
                        if (pv && jv) {
                            if constexpr (kB16)
                                out[lane_off] = hot[u][r];
                            else
                                out[lane_off] = tot[u][r];
                        }
                    }
                    if constexpr (OUT == kPatchMasks) {
                        float av;
                        if constexpr (kB16)
                            av = fabsf(hot[u][r]);
                        else
                            av = fabsf(tot[u][r]);
                        const bool in = av <= tin[u] && pv && jv;
                        if (!(av <= tin[u]) && !(av > tout[u]) && pv && jv) in_between |= 1u << r;
                        const unsigned long long bits = __ballot(in);
                        if (lane < 4)
                            reinterpret_cast<uint16_t *>(nr->mk)[(rb * 16 + 4 * lane + r) * 4 * W64 + jb] =
                                (uint16_t)(bits >> (16 * lane));
                    }
                }
                if constexpr (OUT == kPatchMasks) {
                    if (__ballot(in_between != 0)) {
                        uint32_t v = in_between << (4 * g);
                        v |= (uint32_t)__shfl_xor((int)v, 16);
                        v |= (uint32_t)__shfl_xor((int)v, 32);
                        if (g == 0 && v) reinterpret_cast<uint16_t *>(nr->rows)[j * 4 + rb] = (uint16_t)v;
                    }
                }
            }
        };
        if (rb0 < nrb)
            block(rb0, std::true_type{});
        else if (more)
            arrive(tile + gridDim.x, gh2[par ^ 1]);
#pragma unroll 1
        for (int rb = rb0 + rbs; rb < nrb; rb += rbs) block(rb, std::false_type{});
        if constexpr (OUT == kPatchMasks) {
            __syncthreads();
            const uint64_t mine = nr->rows[tid];
            nrecomp += (unsigned long long)__popcll(mine);
            if (__syncthreads_or(mine != 0))
                resolve_near<P>(a.omega, a.wmask, a.tau, W64, (lds_ptr<const double>)gh,
                                (lds_ptr<double>)reinterpret_cast<double *>(s), (lds_ptr<double>)s_mu,
                                (lds_ptr<double>)s_ri, (lds_ptr<PatchNear>)nr);
            for (int idx = tid; idx < valid_px * W64; idx += 256) a.masks[pix0 * W64 + idx] = nr->mk[idx];
        }
        if constexpr (kSel) {
            last_pix = pix0;
            last_words = valid_px * W64;
        }
        __syncthreads();
    }
    if constexpr (kSel) {
        for (int idx = tid; idx < last_words; idx += 256) a.masks[last_pix * W64 + idx] = s_mk[par ^ 1][idx];
        __shared__ uint32_t s_below[4];
        if (lane == 0) {
            const int w = blockIdx.x * 4 + wave;
            a.sel_bcnt[w] = nb_w;
            a.sel_dcnt[w] = nd_w;
            if (over) a.sel_st->br_over = 1;
            s_below[wave] = below;
        }
        __syncthreads();
        if (tid == 0) {
            a.sel_parts[blockIdx.x] = (unsigned long long)s_below[0] + s_below[1] + s_below[2] + s_below[3];
            if (blockIdx.x == 0) {
                a.sel_st->rg_waves = 4 * gridDim.x;
                a.sel_st->rg_size = (long long)a.sel_region;
                a.sel_st->br_dbase = dbase;
            }
        }
    }
    if constexpr (OUT == kPatchMasks) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) nrecomp += __shfl_xor(nrecomp, d);
        if (a.recomputed && lane == 0 && nrecomp) atomicAdd(a.recomputed, nrecomp);
    }
    // the set-up of the median selection that follows this kernel
    if (a.tau_st && blockIdx.x == 0) {
        tau_setup_state(a.tau_st, a.tau_hist3, a.tau_hist_words, a.tau_rank0, 256);
        tau_setup_margins(a.omega, a.k, n, a.tau_coef, a.tau_margins, a.tau_max_margin, 256);
    }
}

template <int P, int JB, int PREC, int OUT>
hipError_t launch_patch_k(const LaunchCtx &lc, const AnalyzeArgs &a) {
    using T = PatchTile<P>;
    const int tiles_x = (a.W + T::TP - 1) / T::TP;
    const int64_t ntiles = (int64_t)tiles_x * a.H;
    // as many workgroups as run at once: one wave per SIMD each
    const int64_t cap = (int64_t)lc.num_cu * patch_waves_of(P, JB, PREC, OUT);
    int64_t blocks = ntiles < cap ? ntiles : cap;
    if constexpr (OUT == kPatchSelect) {
        if (blocks > kGatherBlocks) blocks = kGatherBlocks;
        // the waves' regions share the lists, which have a place per entry
        AnalyzeArgs b = a;
        b.sel_region = (int64_t)a.H * a.W * a.k / (4 * blocks);
        hipLaunchKernelGGL((k_patch<P, JB, PREC, OUT>), dim3((unsigned)blocks), dim3(256), 0, lc.stream, b, tiles_x,
                           (int)ntiles);
    } else {
        hipLaunchKernelGGL((k_patch<P, JB, PREC, OUT>), dim3((unsigned)blocks), dim3(256), 0, lc.stream, a, tiles_x,
                           (int)ntiles);
    }
    return hipGetLastError();
}

template <int P, int PREC, int OUT>
hipError_t launch_patch_j(const LaunchCtx &lc, const AnalyzeArgs &a) {
    switch ((a.k + 63) / 64) {
        case 1: return launch_patch_k<P, 1, PREC, OUT>(lc, a);
        case 2: return launch_patch_k<P, 2, PREC, OUT>(lc, a);
        case 3: return launch_patch_k<P, 3, PREC, OUT>(lc, a);
        default: return launch_patch_k<P, 4, PREC, OUT>(lc, a);
    }
}

template <int P>
hipError_t launch_patch_p(const LaunchCtx &lc, const AnalyzeArgs &a, int precision) {
    if (a.sel_st) {
        if constexpr (P <= kPatchSelMax)
            return precision == CS_BF16 ? launch_patch_j<P, CS_BF16, kPatchSelect>(lc, a)
                                        : launch_patch_j<P, CS_FP32, kPatchSelect>(lc, a);
        return hipErrorInvalidValue;
    }
    if (a.masks)
        return precision == CS_BF16 ? launch_patch_j<P, CS_BF16, kPatchMasks>(lc, a)
                                    : launch_patch_j<P, CS_FP32, kPatchMasks>(lc, a);
    return precision == CS_BF16 ? launch_patch_j<P, CS_BF16, kPatchAlpha>(lc, a)
                                : launch_patch_j<P, CS_FP32, kPatchAlpha>(lc, a);
}

}  // namespace cs
