// Co-support masks at tau = frac * median|a| with the mask decision fused
// into the candidate gather of the exact median (Sec. 2 co-support of a
// thresholded analysed vector; the threshold is a fixed fraction of the
// median magnitude).
//
// The separate path reads the N*k analysed vectors five times: three radix
// digits, the candidate gather and then the masks at the exact tau.  Here the
// gather pass decides the masks as well, and takes the place of the third
// digit: after two digits (the top 22 bits) the float median of the rounded
// |a| is known to lie in a bin [v_lo, v_hi] of 2^10 floats (at the medians
// and FP32 bounds of the 7 x 7 and 11 x 11 workloads, 0.6 and 0.25 of the
// candidate window's half-width 2m, so the window grows little), and the exact
// median lies in [v_lo - m, v_hi + m] (m the largest proven rounding bound),
// so tau lies in a short interval.  Every entry whose rounded |a| is clear of that interval by more
// than its row's margin is decided in the gather pass; the few others are
// listed and decided against the exact tau once it is selected, in FP64 where
// the rounded value is within the margin.  Masks and tau equal those of the
// separate path bit for bit.  The lists have room for every entry, so nothing
// depends on a host round trip.
#pragma clang fp contract(off)

#include "cs_internal.h"
#include "cs_device.h"

namespace cs {

namespace {
constexpr int kPx = 8;  // pixels per wave and round in the pixel-major pass
// rounds per wave before the number of workgroups is reached (64 x 64: four 11.2 us,
// one 7.3 us)
constexpr int kRoundsPerWave = 1;
// Candidate window [v_lo - 2m, v_hi + 2m] as float bit patterns (non-negative
// floats order like their bit patterns): an entry below it is exactly below
// the exact median, one above it exactly above.
__device__ __forceinline__ void candidate_window(double vlo, double vhi, double mm, TauState *st, bool record,
                                                 uint32_t &blo, uint32_t &bhi) {
    const double wlo = vlo - 2.0 * mm, whi = vhi + 2.0 * mm;
    if (record) {
        st->lo = wlo;
        st->hi = whi;
    }
    float flo = (float)wlo, fhi = (float)whi;
    if ((double)flo < wlo) flo = nextafterf(flo, INFINITY);
    if ((double)fhi > whi) fhi = nextafterf(fhi, -INFINITY);
    blo = wlo <= 0.0 ? 0u : __float_as_uint(flo);
    bhi = __float_as_uint(fhi);
}
}  // namespace

// ---- selection from a sampled bracket ----
// For long vectors the two digit passes are left out: the median's place is
// bracketed from a sample (2^17 entries spread over the vectors by the golden
// ratio, ranks 0.5 +- 1/128, 5.6 deviations of independent samples), the gather
// pass counts the entries below the bracket and lists those inside (some 1.6 %),
// and the median's bin is picked from the list.  Where the bracket turns out
// not to hold the median or its window (entries that the sample does not
// represent, as rows of very different norm at a k that the spread favours), the digit passes and their gather run after all.
// 1024 x 1024, 11 x 11, k = 242 (254 M entries): 730 us for the digit passes and
// the gather, 336 us for sample, pass, pick and window.

// Bins of the sample: 32 octaves below 2 of 256 each.
constexpr int kSampleBlocks = 32, kSample = kSampleBlocks * 4096;
constexpr uint32_t kBinBase = (127u - 31u) << 8;
__global__ __launch_bounds__(1024) void k_bracket_sample(const float *alpha, int64_t count, unsigned int *hist) {
    __shared__ unsigned int h[kBracketBins];
    for (int i = threadIdx.x; i < kBracketBins; i += 1024) h[i] = 0u;
    __syncthreads();
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint64_t i = (uint64_t)blockIdx.x * 4096 + u * 1024 + threadIdx.x;
        const uint64_t f = i * 0x9E3779B97F4A7C15ull;  // i times the golden ratio, mod 1
        v[u] = alpha[(int64_t)__umul64hi(f, (uint64_t)count)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t b = (__float_as_uint(v[u]) & 0x7FFFFFFFu) >> 15;
        const uint32_t c = b < kBinBase ? 0u : b - kBinBase;
        atomicAdd(&h[c < kBracketBins ? c : kBracketBins - 1], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBracketBins; i += 1024)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

// The same before any vector is there: kSample / 8 pixels spread by the golden
// ratio, eight rows of each chosen by a hash, in FP32 (a wave per pixel: its
// lanes form the patch, then eight take a row each).  On textured images with
// noise its median's rank was off by 0.11 % (one deviation, 12 images).
// One workgroup more computes the rows' margins.
constexpr int kPatchSampleBlocks = 256;
__global__ __launch_bounds__(1024) void k_patch_sample(AnalyzeArgs a, unsigned int *hist) {
    __shared__ unsigned int h[kBracketBins];
    __shared__ float s_p[16][128];
    if (blockIdx.x == kPatchSampleBlocks) {
        tau_setup_margins(a.omega, a.k, a.n, a.tau_coef, a.tau_margins, a.tau_max_margin, 1024);
        return;
    }
    const float *const rgb = a.rgb, *const omega = a.omega;
    const double *const wmask = a.wmask;
    const int H = a.H, W = a.W, p = a.p, k = a.k;
    for (int i = threadIdx.x; i < kBracketBins; i += 1024) h[i] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = p * p, hp = (p - 1) / 2;
    const int64_t N = (int64_t)H * W;
    constexpr int per = kSample / 8 / (kPatchSampleBlocks * 16);
    float *const sp = s_p[wave];
    const int t1 = lane + 64;
    const double w0 = lane < n ? wmask[lane] : 0.0, w1 = t1 < n ? wmask[t1] : 0.0;
    const int u0 = lane / p, v0 = lane - u0 * p, u1 = t1 / p, v1 = t1 - u1 * p;
    auto place = [&](int row, int col, int u, int v) {
        return (int64_t)reflect_idx(row + u - hp, H) * W + reflect_idx(col + v - hp, W);
    };
#pragma unroll
    for (int it = 0; it < per; ++it) {
        const uint64_t i = ((uint64_t)blockIdx.x * 16 + wave) * per + it;
        const int64_t pix = (int64_t)__umul64hi(i * 0x9E3779B97F4A7C15ull, (uint64_t)N);
        const int row = (int)(pix / W), col = (int)(pix - (int64_t)row * W);
        const double q0 = lane < n ? w0 * gray64(rgb, N, place(row, col, u0, v0)) : 0.0;
        const double q1 = t1 < n ? w1 * gray64(rgb, N, place(row, col, u1, v1)) : 0.0;
        double sum = q0 + q1;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
        const double mu = sum / n;
        const float z0 = lane < n ? (float)(q0 - mu) : 0.0f, z1 = t1 < n ? (float)(q1 - mu) : 0.0f;
        float nu2 = z0 * z0 + z1 * z1;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) nu2 += __shfl_xor(nu2, d);
        const float ri = nu2 > 0.0f ? 1.0f / sqrtf(nu2) : 0.0f;
        __builtin_amdgcn_wave_barrier();
        sp[lane] = z0 * ri;
        sp[t1] = z1 * ri;
        __builtin_amdgcn_wave_barrier();  // a wave's LDS accesses complete in order
        // row of this group of eight lanes
        uint64_t x = (i * 8 + (lane >> 3) + 1) * 0xD1B54A32D192ED03ull;
        x ^= x >> 32;
        const int j = (int)__umul64hi(x * 0x9E3779B97F4A7C15ull, (uint64_t)k);
        const float *om = omega + (int64_t)j * n;
        float acc = 0.0f;
        for (int t = lane & 7; t < n; t += 8) acc += om[t] * sp[t];
        acc += __shfl_xor(acc, 1);
        acc += __shfl_xor(acc, 2);
        acc += __shfl_xor(acc, 4);
        const uint32_t b = (__float_as_uint(acc) & 0x7FFFFFFFu) >> 15;
        const uint32_t c = b < kBinBase ? 0u : b - kBinBase;
        if ((lane & 7) == 0) atomicAdd(&h[c < kBracketBins ? c : kBracketBins - 1], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBracketBins; i += 1024)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

__global__ __launch_bounds__(1024) void k_select_setup(AnalyzeArgs a) {
    tau_setup_state(a.tau_st, a.tau_hist3, a.tau_hist_words, a.tau_rank0, 1024);
}

// The bracket: the bins of the sample's ranks 0.5 -+ 1/128, widened by three
// margins.  None where a row's undecided interval would reach past FP32 (a huge
// frac), whose end the passes over the entries give to places without an entry.
__global__ __launch_bounds__(1024) void k_bracket_pick(const unsigned int *hist, const double *max_margin, double frac,
                                                       TauState *st) {
    constexpr int per = kBracketBins / 1024;
    __shared__ unsigned int s_w[16], s_bin[2];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    unsigned int loc[per], sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        loc[i] = hist[t * per + i];
        sum += loc[i];
    }
    unsigned int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned int a = __shfl_up(incl, off);
        if (lane >= off) incl += a;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    unsigned int before = incl - sum;
    for (int w = 0; w < wave; ++w) before += s_w[w];
    constexpr unsigned int r[2] = {kSample / 2 - kSample / 128, kSample / 2 + kSample / 128};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        unsigned int acc = before;
#pragma unroll
        for (int i = 0; i < per; ++i) {
            if (r[e] >= acc && r[e] < acc + loc[i]) s_bin[e] = t * per + i;
            acc += loc[i];
        }
    }
    __syncthreads();
    if (t == 0) {
        const unsigned int b0 = s_bin[0], b1 = s_bin[1];
        // the outer bins hold what lies past them too
        const double m3 = 3.0 * *max_margin;
        const double lo = (double)__uint_as_float((b0 + kBinBase) << 15) - m3;
        const double hi = (double)__uint_as_float((b1 + 1 + kBinBase) << 15) + m3;
        const uint32_t blo = __float_as_uint((float)lo), bhi = __float_as_uint((float)hi);
        double tlo, thi;
        tau_interval((double)(float)lo, (double)(float)hi, *max_margin, frac, tlo, thi);
        const bool ok = b0 > 0 && b1 < kBracketBins - 1 && lo > 0.0 && hi < 4.0 && bhi - blo < kPackMax &&
                        thi + *max_margin < (double)__FLT_MAX__;
        st->br_valid = ok ? 1 : 0;
        if (ok) {
            int shift = 0;
            while (((bhi - blo) >> shift) >= (uint32_t)kBracketFine) ++shift;
            st->br_lo = blo;
            st->br_hi = bhi;
            st->br_shift = shift;
        }
    }
}

// Histogram of the listed entries' keys within the bracket.
__global__ __launch_bounds__(1024) void k_bracket_hist(const uint64_t *blist, const unsigned int *bcnt,
                                                       const TauState *st, unsigned int *fine) {
    __shared__ unsigned int h[kBracketFine];
    if (!st->br_valid) return;
    for (int i = threadIdx.x; i < kBracketFine; i += 1024) h[i] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63, nw = (int)st->rg_waves, shift = kPackShift + (int)st->br_shift;
    for (int r = blockIdx.x * 16 + (threadIdx.x >> 6); r < nw; r += gridDim.x * 16) {
        const uint64_t *src = blist + r * (int64_t)st->rg_size;
        const int n = (int)bcnt[r];
        for (int q0 = lane; q0 < n; q0 += 4 * 64) {
            uint64_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = src[q0 + 64 * u < n ? q0 + 64 * u : q0];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (q0 + 64 * u < n) atomicAdd(&h[v[u] >> shift], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBracketFine; i += 1024)
        if (h[i]) atomicAdd(&fine[i], h[i]);
}

// The median's bin, the candidate window around it and its entries from the
// list (regions as the list's); st->br_ok when the bracket holds the window.
__global__ __launch_bounds__(256) void k_bracket_window(const uint64_t *blist, const unsigned int *bcnt,
                                                        const unsigned int *fine, const double *max_margin,
                                                        TauState *st, unsigned long long *parts, int64_t *cand,
                                                        unsigned int *ccnt) {
    __shared__ unsigned long long s_w[2][4];
    __shared__ int s_bin;
    if (!st->br_valid || st->br_over) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int nb = (int)(st->rg_waves / 4);  // workgroups of the pass before
    // entries below the bracket, and the rank left inside it
    unsigned long long below = 0, sum = 0;
    for (int i = t; i < nb; i += 256) below += parts[i];
    unsigned int loc[kBracketFine / 256];
#pragma unroll
    for (int i = 0; i < kBracketFine / 256; ++i) {
        loc[i] = fine[t * (kBracketFine / 256) + i];
        sum += loc[i];
    }
    unsigned long long incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long a = __shfl_up(incl, off);
        if (lane >= off) incl += a;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) below += __shfl_xor(below, off);
    if (lane == 63) {
        s_w[0][wave] = incl;
        s_w[1][wave] = below;
    }
    if (t == 0) s_bin = -1;
    __syncthreads();
    below = s_w[1][0] + s_w[1][1] + s_w[1][2] + s_w[1][3];
    unsigned long long before = incl - sum;
    for (int w = 0; w < wave; ++w) before += s_w[0][w];
    const unsigned long long r0 = st->rank0;
    if (r0 >= below) {
        const unsigned long long r = r0 - below;
        unsigned long long acc = before;
#pragma unroll
        for (int i = 0; i < kBracketFine / 256; ++i) {
            if (r >= acc && r < acc + loc[i]) s_bin = t * (kBracketFine / 256) + i;
            acc += loc[i];
        }
    }
    __syncthreads();
    const int bin = s_bin;
    if (bin < 0) return;  // outside the bracket
    const uint32_t blo = st->br_lo, bhi = st->br_hi, shift = st->br_shift;
    const uint32_t klo = blo + ((uint32_t)bin << shift), khi = min(klo + (1u << shift) - 1u, bhi);
    uint32_t wlo, whi;
    const bool first = blockIdx.x == 0 && t == 0;
    candidate_window((double)__uint_as_float(klo), (double)__uint_as_float(khi), *max_margin, st, first, wlo, whi);
    if (wlo < blo || whi > bhi) return;
    if (first) {
        st->br_ok = 1;
        st->nparts = nb + gridDim.x;
    }
    const uint32_t clo = wlo - blo, chi = whi - blo;
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int nw = (int)st->rg_waves;
    unsigned int low = 0;
    for (int r = blockIdx.x * 4 + wave; r < nw; r += gridDim.x * 4) {
        const int64_t at = r * (int64_t)st->rg_size;
        const int n = (int)bcnt[r];
        unsigned int nc = 0;
        for (int q0 = 0; q0 < n; q0 += 4 * 64) {
            uint64_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = blist[at + min(q0 + 64 * u + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool live = q0 + 64 * u + lane < n;
                const uint32_t d = (uint32_t)(v[u] >> kPackShift);
                low += live && d < clo ? 1u : 0u;
                const bool in = live && d >= clo && d <= chi;
                const unsigned long long m = __ballot(in);
                if (in) cand[at + nc + __popcll(m & lt)] = (int64_t)(v[u] & ((1ull << kPackShift) - 1ull));
                nc += (unsigned int)__popcll(m);
            }
        }
        if (lane == 0) ccnt[r] = nc;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) low += __shfl_xor(low, off);
    __syncthreads();  // s_w is read above
    if (lane == 0) s_w[0][wave] = low;
    __syncthreads();
    if (t == 0) parts[nb + blockIdx.x] = s_w[0][0] + s_w[0][1] + s_w[0][2] + s_w[0][3];
}

// The gather pass.  Each wave takes a contiguous run of rounds of kPx
// consecutive pixels (kRoundsPerWave of them or more, the loads of the next in
// flight while one is decided), lane = row within a 64-bit mask word.  Its
// candidates and undecided entries go to its own region of cand and didx,
// which starts at its first entry (so it can never overflow), counted in
// ccnt and dcnt: no global atomics.  Per workgroup the count of entries below
// the candidate window goes to parts[blockIdx.x].
//
// Bound by the one reading of the vectors: 254 M entries (k = 242) in 266 us, 3.8
// TB/s; 411 M of k = 98, a quarter of whose lanes have no row, in 522 us.  The
// comparisons are wave masks in scalar registers, counted there, and the mask
// words are written into their lanes: with a ballot per test and a lane compare
// per word, vector instructions and spilled masks bound it (380 and 642 us).
//
// BR: the window is the whole sampled bracket [br_lo, br_hi] instead, the
// median's bin within it being picked afterwards from the listed entries; they
// and the undecided ones are listed with their keys (kPackShift).
template <int W64, bool BR>
__global__ __launch_bounds__(256) void k_median_mask_gather(const float *alpha, int64_t N, int k,
                                                            const double *max_margin, const double *margins,
                                                            double frac, TauState *st, int64_t *cand,
                                                            unsigned int *ccnt, unsigned long long *parts,
                                                            int64_t *didx, unsigned int *dcnt, uint64_t *masks,
                                                            const unsigned int *hist3) {
    if (BR ? !st->br_valid : st->br_ok) return;
    static_assert(kPx * W64 <= 64, "one mask word per lane");
    __shared__ unsigned long long red[4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double mm = *max_margin;
    uint32_t blo, bhi, dbase = 0;
    double vlo, vhi;
    if constexpr (BR) {
        blo = st->br_lo;
        bhi = st->br_hi;
        vlo = (double)__uint_as_float(blo);
        vhi = (double)__uint_as_float(bhi);
    } else {
        // the second digit, from its complete histogram: the target rank's
        // rounded |a| has the top 22 bits prefix, so it lies in [v_lo, v_hi]
        // (workgroup 0 records the digit)
        unsigned int prefix;
        unsigned long long rank;
        tau_pick_digit(hist3 + kHistBins, 10, st->pfx[1], st->rk[1], prefix, rank);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->pfx[2] = st->prefix = prefix;
            st->rk[2] = st->rank = rank;
        }
        vlo = (double)__uint_as_float(prefix);
        vhi = (double)__uint_as_float(prefix | 0x3FFu);
        candidate_window(vlo, vhi, mm, st, blockIdx.x == 0 && threadIdx.x == 0, blo, bhi);
    }
    double tlo, thi;
    tau_interval(vlo, vhi, mm, frac, tlo, thi);
    if constexpr (BR) {
        dbase = tau_defer_base(tlo, mm);
        if (blockIdx.x == 0 && threadIdx.x == 0) st->br_dbase = dbase;
    }
    float tin[W64], tout[W64];
#pragma unroll
    for (int w = 0; w < W64; ++w) {
        const int j = 64 * w + lane;
        tau_row_interval(tlo, thi, j < k ? margins[j] : 0.0, tin[w], tout[w]);
    }
    unsigned int below = 0;  // wave-uniform (a wave's entries are fewer than 2^32)
    const int64_t nrounds = (N + kPx - 1) / kPx;
    const int64_t nw = (int64_t)gridDim.x * 4;
    const int64_t R = (nrounds + nw - 1) / nw;  // rounds per wave
    const int64_t gw = (int64_t)blockIdx.x * 4 + wave;
    const int64_t r_end = (gw + 1) * R < nrounds ? (gw + 1) * R : nrounds;
    const int64_t region = R * kPx * k;  // entries of a wave's run of rounds
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->rg_waves = (unsigned int)nw;
        st->rg_size = (long long)region;
    }
    int64_t *creg = cand + gw * region, *dreg = didx + gw * region;
    unsigned int nc_w = 0, nd_w = 0;  // wave-uniform counts
    // entry base + lane (base wave-uniform) at place `at` of a region, d above it
    auto put = [&](int64_t *reg, uint32_t at, int64_t base, uint32_t d) {
        const uint64_t e = (uint64_t)base + (uint32_t)lane;
        *reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(reg) + 8u * at) = e | (uint64_t)d << kPackShift;
    };
    const bool row_live = 64 * (W64 - 1) + lane < k;
    const uint32_t key_and = row_live ? 0x7FFFFFFFu : 0u, key_or = row_live ? 0u : 0x7F800000u;
    const uint64_t rows = __ballot(row_live);  // of the last word
    // the keys of a round, loaded unconditionally (clamped indices: the loads
    // are in flight together; padding is replaced when the entry is used)
    auto load = [&](int64_t rd, uint32_t (&kk)[kPx][W64]) {
        const int64_t p0 = rd * kPx;
#pragma unroll
        for (int i = 0; i < kPx; ++i)
#pragma unroll
            for (int w = 0; w < W64; ++w) {
                const int j = 64 * w + lane;
                const int64_t pix = p0 + i;
                kk[i][w] = __float_as_uint(alpha[(pix < N ? pix : N - 1) * k + (j < k ? j : k - 1)]);
            }
    };
    uint32_t key[kPx][W64], nkey[kPx][W64];
    int64_t rd = gw * R;
    if (rd < r_end) load(rd, key);
    for (; rd < r_end; ++rd) {
        const int64_t p0 = rd * kPx;
        if (rd + 1 < r_end) load(rd + 1, nkey);  // next round in flight
        // lane l < kPx * W64 stores word (l / W64, l % W64), put there as the
        // words are formed (no array of ballots held in scalar registers)
        const int li = lane / W64, lw = lane - li * W64;
        int out_lo = 0, out_hi = 0;
#pragma unroll
        for (int i = 0; i < kPx; ++i) {
            if (p0 + i >= N) break;
#pragma unroll
            for (int w = 0; w < W64; ++w) {
                // rows past k get the key of +inf: not below, and out of every
                // interval within FP32, as a bracket's are (k_bracket_pick);
                // an interval that reaches past FP32 would take the key
                const uint64_t live = BR || w < W64 - 1 ? ~0ull : rows;
                const uint32_t x = w < W64 - 1 ? key[i][w] & 0x7FFFFFFFu : (key[i][w] & key_and) | key_or, d = x - blo;
                below += (unsigned int)__popcll(__builtin_amdgcn_uicmp(x, blo, kUlt));
                const unsigned long long cm = __builtin_amdgcn_uicmp(d, bhi - blo, kUle) & live;
                if (cm) {
                    if (__builtin_amdgcn_inverse_ballot_w64(cm)) put(creg, nc_w + lane_prefix(cm), (p0 + i) * k + 64 * w, BR ? d : 0u);
                    nc_w += (unsigned int)__popcll(cm);
                }
                const float f = __uint_as_float(x);
                const uint64_t inb = __builtin_amdgcn_fcmpf(f, tin[w], kOle) & live;
                out_lo = write_lane((int)(uint32_t)inb, i * W64 + w, out_lo);
                out_hi = write_lane((int)(uint32_t)(inb >> 32), i * W64 + w, out_hi);
                const unsigned long long dm = live & ~(inb | __builtin_amdgcn_fcmpf(f, tout[w], kOgt));  // NaN: deferred
                if (dm) {
                    if (__builtin_amdgcn_inverse_ballot_w64(dm)) put(dreg, nd_w + lane_prefix(dm), (p0 + i) * k + 64 * w, BR ? min(x - dbase, kPackMax) : 0u);
                    nd_w += (unsigned int)__popcll(dm);
                }
                // one entry at a time: keeps the ballots from piling up in
                // scalar registers
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const uint64_t outw = (uint64_t)(uint32_t)out_hi << 32 | (uint32_t)out_lo;
        if (lane < kPx * W64 && p0 + li < N) masks[(p0 + li) * W64 + lw] = outw;
#pragma unroll
        for (int i = 0; i < kPx; ++i)
#pragma unroll
            for (int w = 0; w < W64; ++w) key[i][w] = nkey[i][w];
    }
    if (lane == 0 && gw < nw) {
        ccnt[gw] = nc_w;
        dcnt[gw] = nd_w;
    }
    if (lane == 0) red[wave] = below;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    if (!BR && blockIdx.x == 0 && threadIdx.x == 0) st->nparts = gridDim.x;
}

// The listed entries against the exact tau, a lane per entry.  An entry whose
// rounded |a| is clear of tau by more than its row margin is decided at once;
// the wave's few within the margin (or NaN) are recomputed in FP64, eight at a
// time (exact_entry), and decided exactly.
__global__ __launch_bounds__(64) void k_median_mask_finish(const float *alpha, const float *rgb, int H, int W,
                                                           int p, const double *wmask, const float *omega, int k,
                                                           const int64_t *didx, const unsigned int *dcnt,
                                                           const int64_t *dcomp, const double *margins,
                                                           const TauState *st, uint64_t *masks,
                                                           const double *pstats) {
    constexpr int G = 64 / kExactLanes;
    extern __shared__ double s_exact[];  // exact_lds(p * p)
    __shared__ int64_t s_near[64];
    const int lane = threadIdx.x, grp = lane / kExactLanes, W64 = (k + 63) / 64;
    const double tau = st->tau;
    const bool packed = st->br_ok != 0;  // the list carries the keys
    const uint32_t dbase = st->br_dbase;
    ExactRun run;
    int64_t zero_pix = -1;  // the wave's
    auto set = [&](int64_t pix, int j) {
        atomicOr(reinterpret_cast<unsigned long long *>(masks + pix * W64 + (j >> 6)), 1ull << (j & 63));
    };
    // the wave's entries q0 .. q0 + width - 1 (width <= 64) of a list of cnt
    auto round = [&](const int64_t *lst, int64_t q0, int64_t cnt, int width) {
        const bool live = lane < width && q0 + lane < cnt;
        bool near = false;
        int64_t e = 0;
        if (live) {
            e = lst[q0 + lane];
            uint32_t d = 0;
            if (packed) {
                d = (uint32_t)((uint64_t)e >> kPackShift);
                e &= ((int64_t)1 << kPackShift) - 1;
            }
            const int64_t pix = e / k;
            const int j = (int)(e - pix * k);
            const double a = packed ? (double)__uint_as_float(dbase + d) : (double)fabsf(alpha[e]);
            const double m = margins[j];
            if (packed && d == kPackMax)
                near = true;
            else if (a <= tau - m)
                set(pix, j);
            else
                near = !(a > tau + m);  // within the margin, or NaN
            if (near && pix == zero_pix) {
                if (0.0 <= tau) set(pix, j);
                near = false;
            }
        }
        const unsigned long long nm = __ballot(near);
        if (!nm) return;
        if (near) s_near[__popcll(nm & ((1ull << lane) - 1ull))] = e;
        __builtin_amdgcn_wave_barrier();
        const int nn = (int)__popcll(nm);
        for (int i0 = 0; i0 < nn; i0 += G) {
            const bool on = i0 + grp < nn;
            const int64_t f = s_near[on ? i0 + grp : 0], pix = f / k;
            const int j = (int)(f - pix * k);
            const double v = run.entry(rgb, H, W, p, wmask, omega + (int64_t)j * p * p, pix, pstats,
                                       s_exact + grp * (p * p + 1), on);
            if (on && (lane & (kExactLanes - 1)) == 0 && fabs(v) <= tau) set(pix, j);
        }
        zero_pix = run.wave_zero();
        __builtin_amdgcn_wave_barrier();
    };
    const int64_t nd = (int64_t)st->n_d;
    if (nd <= kListCap) {
        // a short list spread over all waves, eight entries (one FP64 round)
        // at least each
        const int64_t share = (nd + gridDim.x - 1) / gridDim.x;
        const int width = share >= 64 ? 64 : share < G ? G : (int)((share + G - 1) / G * G);
        for (int64_t q = (int64_t)blockIdx.x * width; q < nd; q += (int64_t)gridDim.x * width)
            round(dcomp, q, nd, width);
        return;
    }
    const int64_t nw = (int64_t)st->rg_waves, region = (int64_t)st->rg_size;
    for (int64_t r = blockIdx.x; r < nw; r += gridDim.x)
        for (int64_t q = 0; q < (int64_t)dcnt[r]; q += 64) round(didx + r * region, q, dcnt[r], 64);
}

hipError_t median_mask_gather(const LaunchCtx &lc, const float *alpha, int64_t N, int k,
                              const double *max_margin, const double *margins, double frac, TauState *st,
                              int64_t *cand, unsigned int *ccnt, unsigned long long *parts, int64_t *didx,
                              unsigned int *dcnt, uint64_t *masks, const unsigned int *hist3) {
    if (N <= 0) return hipSuccess;
    // kRoundsPerWave rounds per wave (each prefetches the next), more where
    // the per-workgroup counts would not fit
    const int64_t blocks = median_gather_waves(N) / 4;
#define CS_MG_LAUNCH(WW)                                                                                    \
    hipLaunchKernelGGL((k_median_mask_gather<WW, false>), dim3((unsigned)blocks), dim3(256), 0, lc.stream, alpha, N, \
                       k, max_margin, margins, frac, st, cand, ccnt, parts, didx, dcnt, masks, hist3)
    switch ((k + 63) / 64) {
        case 1: CS_MG_LAUNCH(1); break;
        case 2: CS_MG_LAUNCH(2); break;
        case 3: CS_MG_LAUNCH(3); break;
        default: CS_MG_LAUNCH(4); break;
    }
#undef CS_MG_LAUNCH
    return hipGetLastError();
}

hipError_t median_bracket(const LaunchCtx &lc, const float *alpha, int64_t N, int k, const double *max_margin,
                          const double *margins, double frac, TauState *st, uint64_t *blist, int64_t *cand,
                          unsigned int *ccnt, unsigned long long *parts, int64_t *didx, unsigned int *dcnt,
                          uint64_t *masks, unsigned int *br_hist) {
    const int blocks = (int)(median_gather_waves(N) / 4);
    hipLaunchKernelGGL(k_bracket_sample, dim3(kSampleBlocks), dim3(1024), 0, lc.stream, alpha, N * k, br_hist);
    hipLaunchKernelGGL(k_bracket_pick, dim3(1), dim3(1024), 0, lc.stream, br_hist, max_margin, frac, st);
#define CS_BR_LAUNCH(WW)                                                                                           \
    hipLaunchKernelGGL((k_median_mask_gather<WW, true>), dim3((unsigned)blocks), dim3(256), 0, lc.stream, alpha, N, k, \
                       max_margin, margins, frac, st, (int64_t *)blist, ccnt, parts, didx, dcnt, masks, nullptr)
    switch ((k + 63) / 64) {
        case 1: CS_BR_LAUNCH(1); break;
        case 2: CS_BR_LAUNCH(2); break;
        case 3: CS_BR_LAUNCH(3); break;
        default: CS_BR_LAUNCH(4); break;
    }
#undef CS_BR_LAUNCH
    return median_bracket_list(lc, max_margin, st, blist, cand, ccnt, parts, br_hist);
}

hipError_t median_bracket_list(const LaunchCtx &lc, const double *max_margin, TauState *st, const uint64_t *blist,
                               int64_t *cand, unsigned int *ccnt, unsigned long long *parts, unsigned int *br_hist) {
    unsigned int *fine = br_hist + kBracketBins;
    hipLaunchKernelGGL(k_bracket_hist, dim3((unsigned)(lc.num_cu / 2)), dim3(1024), 0, lc.stream, blist, ccnt, st, fine);
    // (the list's counts are read and replaced by the wave that owns the region)
    hipLaunchKernelGGL(k_bracket_window, dim3((unsigned)lc.num_cu), dim3(256), 0, lc.stream, blist, ccnt, fine,
                       max_margin, st, parts, cand, ccnt);
    return hipGetLastError();
}

hipError_t median_patch_sample(const LaunchCtx &lc, const AnalyzeArgs &a, double frac, unsigned int *br_hist) {
    hipLaunchKernelGGL(k_select_setup, dim3(1), dim3(1024), 0, lc.stream, a);
    hipLaunchKernelGGL(k_patch_sample, dim3(kPatchSampleBlocks + 1), dim3(1024), 0, lc.stream, a, br_hist);
    hipLaunchKernelGGL(k_bracket_pick, dim3(1), dim3(1024), 0, lc.stream, br_hist, a.tau_max_margin, frac, a.tau_st);
    return hipGetLastError();
}

int64_t median_gather_waves(int64_t N) {
    int64_t blocks = (N + 4 * kPx * kRoundsPerWave - 1) / (4 * kPx * kRoundsPerWave);
    if (blocks > kGatherBlocks) blocks = kGatherBlocks;
    return 4 * blocks;
}

hipError_t median_mask_finish(const LaunchCtx &lc, const float *alpha, const float *rgb, int H, int W, int p,
                              const double *wmask, const float *omega, int k, const int64_t *didx,
                              const unsigned int *dcnt, const int64_t *dcomp, const double *margins,
                              const TauState *st, uint64_t *masks, const double *pstats) {
    const int64_t blocks = (int64_t)lc.num_cu * kExactWaves;
    hipLaunchKernelGGL(k_median_mask_finish, dim3((unsigned)blocks), dim3(64), exact_lds(p * p), lc.stream, alpha, rgb, H, W, p,
                       wmask, omega, k, didx, dcnt, dcomp, margins, st, masks, pstats);
    return hipGetLastError();
}

}  // namespace cs
