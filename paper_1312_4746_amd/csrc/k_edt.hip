// Exact squared Euclidean distance from every pixel to the nearest scribble
// sample of each label, with the identity of that sample, on gfx950.  This is
// the |x - x_{v_i}| that sets the spatial bandwidth rho_i(x) in Sec. 3.1.
//
// Separable transform on integer distances (exact):
//  1. columns: the rows of every column are cut into short segments; a first
//     kernel records the first and last seed row of each segment, a second one
//     carries the nearest seed rows from the other segments in and scans its
//     own segment both ways (lanes own adjacent columns, so loads coalesce);
//  2. rows: one workgroup per (label, row) stages f(q) = squared column
//     distance of every column q in LDS, and the smallest f over blocks of 16
//     columns and over runs of kWalk blocks; each thread owns columns c and
//     walks outward block by block, keeping the best (c - q)^2 + f(q).  A block
//     is scanned only when its nearest column and its smallest f could still
//     beat the best, a run is passed over when none of its blocks could, and
//     the walk stops once the nearest column of the next blocks is at least
//     that far.
//
// The row pass is bound by its vector instructions.  1024 x 1024, 16 labels: 495 ->
// 298 us with the runs (most of a walk passes far blocks of other labels' samples)
// and a multiply-add per column scanned; 481 x 321: 33 -> 28 us.  Whole runs cost
// short walks: with 50000 random samples the transform at 1024 x 1024 takes 172 us
// block by block, 231 by runs; decided lane by lane, 191.  The listed form
// waits for its loads: 2048 x 2048, 1171 -> 594 us with kWalkAhead minima and whole
// blocks requested together (runs, or an upper bound from the minima before the
// first scan, measured 624 and 657 us).  The column pass likewise: 220 -> 80 us
// with kSegAhead segments at a time.
#include "cs_internal.h"

namespace cs {

constexpr int kSegRows = 16;
constexpr int kSegAhead = 8;  // segments of a column read together in the search for the nearest seed row
constexpr int kWalk = 8;       // blocks of a row, on each side, that the row pass passes over together
constexpr int kShort = 8 * 16;  // columns to each side up to which the row pass looks at every block
constexpr int kWalkAhead = 4;  // ... and whose minima the listed pass reads together
constexpr int kNoSeed = -1;
constexpr int kRowBlk = 16;  // columns per block of the row pass
constexpr int32_t kInf = 0x3FFFFFFF;

// Per (label, segment, column): first and last seed row inside the segment.
__global__ __launch_bounds__(64) void k_edt_col_summary(const uint8_t *seeds, int H, int W,
                                                         int nseg, int32_t *first, int32_t *last) {
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int seg = blockIdx.y, l = blockIdx.z;
    if (c >= W) return;
    const int64_t N = (int64_t)H * W;
    const uint8_t *sd = seeds + (int64_t)l * N + c;
    const int r0 = seg * kSegRows, r1 = min(H, r0 + kSegRows);
    int f = kNoSeed, la = kNoSeed;
#pragma unroll 4
    for (int r = r0; r < r1; ++r) {
        if (sd[(int64_t)r * W]) {
            if (f < 0) f = r;
            la = r;
        }
    }
    const int64_t o = ((int64_t)l * nseg + seg) * W + c;
    first[o] = f;
    last[o] = la;
}

// Smallest value of each aligned group of 16 lanes (rotations within it).
__device__ __forceinline__ int min16(int v) {
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x128, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x124, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x122, 0xF, 0xF, false));
    return min(v, __builtin_amdgcn_update_dpp(v, v, 0x121, 0xF, 0xF, false));
}

// Nearest seed row in the column for every pixel of a segment, given the last
// seed row in the segments above it and the first in those below; MIN: also
// the smallest f over each block of kRowBlk columns, which an aligned group of as
// many lanes holds (every lane of the wave takes part, live: it has a column; a
// pass of its own over the rows took 80 us at 2048 x 2048, 10 labels, 26 more here).
template <bool MIN>
__device__ __forceinline__ void fill_segment(const uint8_t *seeds, int H, int W, int c, int seg, int l, int above,
                                             int below, int32_t *colrow, int32_t *bmin, bool live) {
    static_assert(kRowBlk == 16, "a block is a group of 16 lanes");
    const int64_t N = (int64_t)H * W;
    const int cc = live ? c : W - 1;
    const uint8_t *sd = seeds + (int64_t)l * N + cc;
    int32_t *cr = colrow + (int64_t)l * N + cc;
    const int nb = (W + kRowBlk - 1) / kRowBlk;
    const int r0 = seg * kSegRows, r1 = min(H, r0 + kSegRows);
    // the segment's seed bytes, loaded unconditionally (rows clamped) so that
    // the loads are in flight together
    bool sv[kSegRows];
#pragma unroll
    for (int i = 0; i < kSegRows; ++i) sv[i] = sd[(int64_t)min(r0 + i, H - 1) * W] != 0;
    int up[kSegRows];
    int lastr = above;
#pragma unroll
    for (int i = 0; i < kSegRows; ++i) {
        const int r = r0 + i;
        if (r < r1 && sv[i]) lastr = r;
        up[i] = lastr;
    }
    int nextr = below;
#pragma unroll
    for (int i = kSegRows - 1; i >= 0; --i) {
        const int r = r0 + i;
        if (r < r1 && sv[i]) nextr = r;
        const int a = up[i];
        int best = a;
        if (nextr >= 0 && (a < 0 || nextr - r < r - a)) best = nextr;
        if (live && r < r1) cr[(int64_t)r * W] = best;
        if constexpr (MIN) {
            const int m = min16(live && best >= 0 ? (r - best) * (r - best) : kInf);
            if (live && r < r1 && c % kRowBlk == 0) bmin[((int64_t)l * H + r) * nb + c / kRowBlk] = m;
        }
    }
}

template <bool MIN>
__global__ __launch_bounds__(64) void k_edt_col_fill(const uint8_t *seeds, int H, int W, int nseg,
                                                      const int32_t *first, const int32_t *last,
                                                      int32_t *colrow, int32_t *bmin) {
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int seg = blockIdx.y, l = blockIdx.z;
    if (!MIN && c >= W) return;
    const int64_t sbase = (int64_t)l * nseg * W + min(c, W - 1);
    int above = kNoSeed;  // last seed row in the segments above
    for (int s0 = seg - 1; s0 >= 0 && above < 0; s0 -= kSegAhead) {
        int v[kSegAhead];
#pragma unroll
        for (int i = 0; i < kSegAhead; ++i) v[i] = last[sbase + (int64_t)max(s0 - i, 0) * W];
#pragma unroll
        for (int i = kSegAhead - 1; i >= 0; --i) above = v[i] >= 0 ? v[i] : above;
    }
    int below = kNoSeed;  // first seed row in the segments below
    for (int s0 = seg + 1; s0 < nseg && below < 0; s0 += kSegAhead) {
        int v[kSegAhead];
#pragma unroll
        for (int i = 0; i < kSegAhead; ++i) v[i] = first[sbase + (int64_t)min(s0 + i, nseg - 1) * W];
#pragma unroll
        for (int i = kSegAhead - 1; i >= 0; --i) below = v[i] >= 0 ? v[i] : below;
    }
    fill_segment<MIN>(seeds, H, W, c, seg, l, above, below, colrow, bmin, c < W);
}

// Both steps in one launch for up to kColSegs segments: a workgroup has all
// segments of kColWidth columns, a thread one of them, and hands the summaries
// over in LDS (64 x 64: 7.9 -> 4.5 us, 481 x 321: 11.2 -> 9.6 us).
constexpr int kColWidth = 32, kColSegs = 1024 / kColWidth;
template <bool MIN>
__global__ __launch_bounds__(1024) void k_edt_cols(const uint8_t *seeds, int H, int W, int nseg, int32_t *colrow,
                                                   int32_t *bmin) {
    __shared__ int16_t s_first[kColSegs][kColWidth], s_last[kColSegs][kColWidth];
    const int x = threadIdx.x % kColWidth, seg = threadIdx.x / kColWidth, l = blockIdx.y;
    const int c = blockIdx.x * kColWidth + x;
    const bool live = c < W;
    const int r0 = seg * kSegRows, r1 = min(H, r0 + kSegRows);
    int f = kNoSeed, la = kNoSeed;
    if (live) {
        const uint8_t *sd = seeds + (int64_t)l * H * W + c;
        bool sv[kSegRows];
#pragma unroll
        for (int i = 0; i < kSegRows; ++i) sv[i] = sd[(int64_t)min(r0 + i, H - 1) * W] != 0;
#pragma unroll
        for (int i = 0; i < kSegRows; ++i)
            if (r0 + i < r1 && sv[i]) {
                if (f < 0) f = r0 + i;
                la = r0 + i;
            }
    }
    s_first[seg][x] = (int16_t)f;
    s_last[seg][x] = (int16_t)la;
    __syncthreads();
    if (!MIN && !live) return;
    int above = kNoSeed, below = kNoSeed;
    for (int s = 0; s < nseg; ++s) {
        if (s < seg && s_last[s][x] >= 0) above = s_last[s][x];
        if (s > seg && below < 0) below = s_first[s][x];
    }
    fill_segment<MIN>(seeds, H, W, c, seg, l, above, below, colrow, bmin, live);
}

// Smallest (c - q)^2 + f(q) over the columns q = q0 + i of a block from g_i = f(q0
// + i) + i^2: with e = c - q0 it is e^2 + min (g_i - 2 e i), one multiply-add per
// column and half a three-way minimum.
__device__ __forceinline__ int block_best(const int (&g)[kRowBlk], int e) {
    const int e2 = -2 * e;
    int m = g[0];
#pragma unroll
    for (int i = 1; i < kRowBlk; ++i) m = min(m, __mul24(e2, i) + g[i]);
    return __mul24(e, e) + m;
}

__global__ __launch_bounds__(1024) void k_edt_rows(const int32_t *colrow, int H, int W,
                                                    int32_t *d2, int32_t *nearest) {
    extern __shared__ int32_t lds[];
    const int nb = (W + kRowBlk - 1) / kRowBlk;
    // f: squared column distance plus the square of the column's place in its
    // block, kInf instead of the distance where the column has no seed, padded to
    // whole blocks with kInf (16-byte aligned: blocks are read as int4)
    int32_t *f = lds;
    int32_t *rowof = lds + nb * kRowBlk;      // nearest seed row of each column
    int32_t *fmin = lds + 2 * nb * kRowBlk;   // smallest f over each block
    int32_t *wmin = fmin + nb;                // smallest f over it and the kWalk - 1 blocks after it
    const int r = blockIdx.x, l = blockIdx.y;
    const int64_t N = (int64_t)H * W;
    const int32_t *cr = colrow + (int64_t)l * N + (int64_t)r * W;
    for (int c = threadIdx.x; c < nb * kRowBlk; c += blockDim.x) {
        const int q = c < W ? cr[c] : -1;
        rowof[c] = q;
        f[c] = (q < 0 ? kInf : (r - q) * (r - q)) + (c % kRowBlk) * (c % kRowBlk);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        int m = kInf;
        for (int i = 0; i < kRowBlk; ++i) m = min(m, f[b * kRowBlk + i] - i * i);
        fmin[b] = m;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        int m = kInf;
        for (int u = 0; u < kWalk; ++u) m = min(m, fmin[min(b + u, nb - 1)]);
        wmin[b] = m;
    }
    __syncthreads();
    int32_t *dd = d2 + (int64_t)l * N + (int64_t)r * W;
    int32_t *nn = nearest + (int64_t)l * N + (int64_t)r * W;
    for (int c = threadIdx.x; c < W; c += blockDim.x) {
        // The walk keeps only the smallest value and the block that first
        // reached it (strict improvement); the column is found afterwards in
        // that block, the first in ascending order with the smallest value.
        // Ties go as in a one-by-one scan: the own column first, then the
        // blocks in walk order, then ascending columns.
        const int cb = c / kRowBlk, ci = c - cb * kRowBlk;
        int best = f[c] - ci * ci, bb = -1;
        auto scan = [&](int b) {
            const int4 *f4 = reinterpret_cast<const int4 *>(f + b * kRowBlk);
            const int4 v0 = f4[0], v1 = f4[1], v2 = f4[2], v3 = f4[3];
            const int g[kRowBlk] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w,
                                    v2.x, v2.y, v2.z, v2.w, v3.x, v3.y, v3.z, v3.w};
            const int m = block_best(g, c - b * kRowBlk);
            if (m < best) {
                best = m;
                bb = b;
            }
        };
        scan(cb);  // own block, every column
        // blocks outward on both sides; a block is scanned only if its
        // nearest column and smallest f could beat the best so far, and the
        // walk stops once the nearest column of the next blocks is too far.
        // Where the best so far leaves every lane of the wave a run at most, as
        // among many samples, it goes block by block, else run by run.
        const bool more = !__all(best < kShort * kShort);
        for (int d = 1; !more; ++d) {
            const int bl = cb - d, br = cb + d;
            const int gl = c - (bl * kRowBlk + kRowBlk - 1);  // distance to the left block's last column
            const int gr = br * kRowBlk - c;                     // distance to the right block's first column
            const bool lok = bl >= 0 && gl * gl < best, rok = br < nb && gr * gr < best;
            if (!lok && !rok) break;
            if (lok && gl * gl + fmin[bl] < best) scan(bl);
            if (rok && gr * gr + fmin[br] < best) scan(br);
        }
        for (int d0 = 1; more; d0 += kWalk) {
            const int g0l = c - (cb - d0) * kRowBlk - (kRowBlk - 1), g0r = (cb + d0) * kRowBlk - c;
            const bool lok0 = cb - d0 >= 0 && g0l * g0l < best, rok0 = cb + d0 < nb && g0r * g0r < best;
            if (!lok0 && !rok0) break;
            // nothing within the next kWalk blocks on either side
            const bool lt = lok0 && g0l * g0l + wmin[max(cb - d0 - (kWalk - 1), 0)] < best;
            const bool rt = rok0 && g0r * g0r + wmin[cb + d0] < best;
            if (!lt && !rt) continue;
            for (int u = 0; u < kWalk; ++u) {
                const int bl = cb - d0 - u, br = cb + d0 + u;
                const int gl = c - (bl * kRowBlk + kRowBlk - 1), gr = br * kRowBlk - c;
                if (lt && bl >= 0 && gl * gl + fmin[bl] < best) scan(bl);
                if (rt && br < nb && gr * gr + fmin[br] < best) scan(br);
            }
        }
        int bq = c;
        if (bb >= 0) {
            const int e = c - bb * kRowBlk, rest = best - __mul24(e, e);
#pragma unroll
            for (int i = kRowBlk - 1; i >= 0; --i)
                if (__mul24(-2 * e, i) + f[bb * kRowBlk + i] == rest) bq = bb * kRowBlk + i;
        }
        if (best >= kInf) {  // no seed of this label anywhere (rejected before launch)
            dd[c] = -1;
            nn[c] = -1;
        } else {
            dd[c] = best;
            nn[c] = rowof[bq] * W + bq;
        }
    }
}

// The row pass for listed pixels only, one thread per (entry, label): the
// walk of k_edt_rows for the entry's column, reading f and the block minima
// from global memory instead of LDS (the same blocks are scanned in the same
// order, so the result and its ties are those of k_edt_rows).  Entries
// outside the image are skipped (the host rejects them after the launch).
__global__ __launch_bounds__(256) void k_edt_rows_list(const int32_t *colrow, const int32_t *bmin, int H,
                                                       int W, const int32_t *list, int64_t npix, int32_t *d2,
                                                       int32_t *nearest) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int l = blockIdx.y;
    if (e >= npix) return;
    const int64_t N = (int64_t)H * W;
    const int64_t pix = list[e];
    if (pix < 0 || pix >= N) return;
    const int r = (int)(pix / W), c = (int)(pix - (int64_t)r * W);
    const int nb = (W + kRowBlk - 1) / kRowBlk;
    const int32_t *cr = colrow + (int64_t)l * N + (int64_t)r * W;
    const int32_t *fm = bmin + ((int64_t)l * H + r) * nb;
    // f(q) + i^2 of a block's columns q = q0 + i (16-byte loads, which need no
    // alignment beyond the element's; past the row end, as in the full pass, kInf)
    auto block = [&](int b, int (&g)[kRowBlk]) {
        int rows[kRowBlk];
        if (b * kRowBlk + kRowBlk <= W) {
            __builtin_memcpy(rows, cr + b * kRowBlk, sizeof(rows));
        } else {
#pragma unroll
            for (int i = 0; i < kRowBlk; ++i) {
                const int q = b * kRowBlk + i;
                rows[i] = cr[min(q, W - 1)];
                if (q >= W) rows[i] = kNoSeed;
            }
        }
#pragma unroll
        for (int i = 0; i < kRowBlk; ++i) g[i] = (rows[i] < 0 ? kInf : __mul24(r - rows[i], r - rows[i])) + i * i;
    };
    const int cb = c / kRowBlk;
    const int own = cr[c];
    int best = own < 0 ? kInf : (r - own) * (r - own), bb = -1;
    auto scan = [&](int b) {
        int g[kRowBlk];
        block(b, g);
        const int m = block_best(g, c - b * kRowBlk);
        if (m < best) {
            best = m;
            bb = b;
        }
    };
    scan(cb);
    bool more = true;
    for (int d0 = 1; more; d0 += kWalkAhead) {
        int ml[kWalkAhead], mr[kWalkAhead];
#pragma unroll
        for (int u = 0; u < kWalkAhead; ++u) {
            ml[u] = fm[max(cb - d0 - u, 0)];
            mr[u] = fm[min(cb + d0 + u, nb - 1)];
        }
#pragma unroll
        for (int u = 0; u < kWalkAhead; ++u) {
            const int bl = cb - d0 - u, br = cb + d0 + u;
            const int gl = c - (bl * kRowBlk + kRowBlk - 1);
            const int gr = br * kRowBlk - c;
            const bool lok = bl >= 0 && gl * gl < best;
            const bool rok = br < nb && gr * gr < best;
            if (!lok && !rok) {
                more = false;
                break;
            }
            if (lok && gl * gl + ml[u] < best) scan(bl);
            if (rok && gr * gr + mr[u] < best) scan(br);
        }
    }
    int bq = c;
    if (bb >= 0) {
        int g[kRowBlk];
        block(bb, g);
        const int e = c - bb * kRowBlk;
#pragma unroll
        for (int i = kRowBlk - 1; i >= 0; --i)
            if (__mul24(e, e) + __mul24(-2 * e, i) + g[i] == best) bq = bb * kRowBlk + i;
    }
    const int64_t o = (int64_t)l * N + pix;
    if (best >= kInf) {
        d2[o] = -1;
        nearest[o] = -1;
    } else {
        d2[o] = best;
        nearest[o] = cr[bq] * W + bq;
    }
}

// Scratch: first/last summaries, 2 * L * ceil(H/16) * W int32, and (listed
// form) the block minima, L * H * ceil(W/16) int32.
size_t edt_scratch_bytes(int H, int W, int L) {
    const int nseg = (H + kSegRows - 1) / kSegRows;
    const size_t nb = (size_t)(W + kRowBlk - 1) / kRowBlk;
    return sizeof(int32_t) * (2 * (size_t)L * nseg * W + (size_t)L * H * nb);
}

hipError_t launch_edt(const LaunchCtx &lc, const uint8_t *seeds, int H, int W, int L,
                      int32_t *colrow, int32_t *d2, int32_t *nearest, int32_t *scratch,
                      const int32_t *list, int64_t npix) {
    const int nseg = (H + kSegRows - 1) / kSegRows;
    int32_t *first = scratch, *last = scratch + (size_t)L * nseg * W;
    // a short list (at most an eighth of the pixels) takes the per-entry row
    // pass; longer ones the full pass, whose rows share their staging
    const bool listed = list && npix * 8 <= (int64_t)H * W;
    int32_t *bmin = listed ? scratch + 2 * (size_t)L * nseg * W : nullptr;
    if (nseg <= kColSegs) {
        const dim3 grid((W + kColWidth - 1) / kColWidth, L), block(kColWidth * nseg);
        if (listed)
            hipLaunchKernelGGL(k_edt_cols<true>, grid, block, 0, lc.stream, seeds, H, W, nseg, colrow, bmin);
        else
            hipLaunchKernelGGL(k_edt_cols<false>, grid, block, 0, lc.stream, seeds, H, W, nseg, colrow, bmin);
    } else {
        const dim3 grid((W + 63) / 64, nseg, L);
        hipLaunchKernelGGL(k_edt_col_summary, grid, dim3(64), 0, lc.stream, seeds, H, W, nseg, first, last);
        if (listed)
            hipLaunchKernelGGL(k_edt_col_fill<true>, grid, dim3(64), 0, lc.stream, seeds, H, W, nseg, first, last, colrow, bmin);
        else
            hipLaunchKernelGGL(k_edt_col_fill<false>, grid, dim3(64), 0, lc.stream, seeds, H, W, nseg, first, last, colrow, bmin);
    }
    if (listed) {
        if (npix == 0) return hipGetLastError();
        hipLaunchKernelGGL(k_edt_rows_list, dim3((unsigned)((npix + 255) / 256), L), dim3(256), 0, lc.stream,
                           colrow, bmin, H, W, list, npix, d2, nearest);
        return hipGetLastError();
    }
    const size_t nbk = (size_t)(W + kRowBlk - 1) / kRowBlk;
    const size_t lds = sizeof(int32_t) * (2 * nbk * kRowBlk + 2 * nbk);
    hipError_t e = hipFuncSetAttribute((const void *)k_edt_rows,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int threads = (W + 63) / 64 * 64;
    if (threads > 1024) threads = 1024;
    hipLaunchKernelGGL(k_edt_rows, dim3(H, L), dim3(threads), lds, lc.stream, colrow, H, W, d2, nearest);
    return hipGetLastError();
}

}  // namespace cs
