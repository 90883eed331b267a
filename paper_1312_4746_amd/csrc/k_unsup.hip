// Unsupervised data term on gfx950 (Sec. 3.1, unsupervised segmentation):
// colour classes by k-means on the pixels' colours, texture classes by
// k-medians on their co-support masks (texture similarity TSM = Hamming
// distance, component-wise median = majority), every (colour, texture) pair a
// segment class, and per pixel the class likelihoods in the form of
// eq:post_text, the data term the convex relaxation (with its label cost) then
// takes.
//
// k-means: the colour distances are FP64, summed in the order of the
// definition without contracted products, so the assignment decides as an
// FP64 evaluation does; the new centroids are FP64 means from partial sums
// added in a fixed order (deterministic).  k-medians: distances are popcounts
// and the medians integer counts, exact whatever the order.
//
// One launch assigns both clusterings and one moves both sets of centroids.
// These launches are short (481 x 321, 4 + 4 classes), so what bounds them is
// their own latency: serial chains and atomics on one address.  A wave turns
// 64 pixels' mask words by a 64 x 64 bit transpose (6 exchange steps), after
// which lane t counts bit t of every class with two popcounts, instead of one
// ballot and one scalar popcount per bit and class; the counts and colour sums
// stay in registers over the thread's pixels and leave as one partial per
// workgroup (no atomics: 603 per address cost 20 us); the update adds the
// partials with whole workgroups (by one thread per class it was 136 us).
// 481 x 321, ten iterations of 4 + 4 classes and the likelihoods: 1.93 -> 0.16 ms.
#include <type_traits>

#include "cs_internal.h"

namespace cs {

namespace {

constexpr int kUsMaxK = kUnsupMaxClasses;  // classes of one clustering
constexpr int kUsMaxWords = 4;      // 256 co-support bits

// Sum over the wave in lane 63: rows of 16 by shifts, then row 0 into row 1,
// rows 0-1 into rows 2-3 (the other lanes hold partial sums).
__device__ __forceinline__ double wave_sum_f64(double v) {
    auto add = [&](auto step) {
        constexpr int ctrl = decltype(step)::value;
        constexpr int rows = ctrl == 0x142 ? 0xa : ctrl == 0x143 ? 0xc : 0xf;
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)b, ctrl, rows, 0xf, true);
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(b >> 32), ctrl, rows, 0xf, true);
        v += __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };
    add(std::integral_constant<int, 0x111>{});  // row_shr 1, 2, 4, 8
    add(std::integral_constant<int, 0x112>{});
    add(std::integral_constant<int, 0x114>{});
    add(std::integral_constant<int, 0x118>{});
    add(std::integral_constant<int, 0x142>{});  // row_bcast 15, 31
    add(std::integral_constant<int, 0x143>{});
    return v;
}

}  // namespace

// ---- initial centroids (caller-given pixels) ----
__global__ __launch_bounds__(64) void k_us_init(UnsupArgs a, UnsupInit init) {
    const int t = threadIdx.x;
    const int64_t N = a.N;
    if (t < a.Kc) {
        const int64_t p = init.pix[t];
        for (int ch = 0; ch < 3; ++ch) a.ccent[t * 3 + ch] = (double)a.rgb[ch * N + p];
    }
    if (t < a.Kt) {
        const int64_t p = init.pix[a.Kc + t];
        for (int q = 0; q < a.nw; ++q) a.tcent[t * a.nw + q] = a.masks[p * a.nw + q];
    }
}

// ---- assignment of both clusterings and, with_sums, the partial sums ----
__device__ __forceinline__ uint32_t swz_xor(uint32_t v, int s) {
    switch (s) {  // ds_swizzle, bit mode: lane ^ s within 32 lanes
        case 16: return __builtin_amdgcn_ds_swizzle(v, 0x401f);
        case 8: return __builtin_amdgcn_ds_swizzle(v, 0x201f);
        case 4: return __builtin_amdgcn_ds_swizzle(v, 0x101f);
        case 2: return __builtin_amdgcn_ds_swizzle(v, 0x081f);
        default: return __builtin_amdgcn_ds_swizzle(v, 0x041f);
    }
}
// 64 x 64 bit transpose over the wave: bit i of lane j <-> bit j of lane i.
__device__ __forceinline__ void transpose64(uint32_t &lo, uint32_t &hi, int lane) {
    const auto p = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
    lo = p[0];
    hi = p[1];
    uint32_t mask = 0x0000ffffu;  // bits whose index has bit s clear
#pragma unroll
    for (int s = 16; s >= 1; s >>= 1) {
        const uint32_t olo = swz_xor(lo, s), ohi = swz_xor(hi, s);
        const bool up = lane & s;
        lo = up ? (lo & ~mask) | ((olo & ~mask) >> s) : (lo & mask) | ((olo & mask) << s);
        hi = up ? (hi & ~mask) | ((ohi & ~mask) >> s) : (hi & mask) | ((ohi & mask) << s);
        mask ^= mask << (s >> 1);
    }
}

// KC, KT: the class counts rounded up to 4 or 16.  cpart[(4 c + q) parts + b]:
// workgroup b's sums of r, g, b and pixels of colour class c; tpart[b][c nw 64
// + j]: its pixels of texture class c with bit j set; tsize[c parts + b]: its
// pixels of texture class c.
template <int KC, int KT>
__global__ __launch_bounds__(256) void k_us_assign(UnsupArgs a, int with_sums) {
#pragma clang fp contract(off)
    __shared__ double s_c[KC * 3];
    __shared__ uint64_t s_t[KT * kUsMaxWords];
    __shared__ double red[4][KC][4];
    __shared__ unsigned int s_cnt[KT * kUsMaxWords * 64], s_size[4][KT];
    const int64_t N = a.N;
    const int nw = a.nw, Kc = a.Kc, Kt = a.Kt;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < Kc * 3; i += 256) s_c[i] = a.ccent[i];
    for (int i = threadIdx.x; i < Kt * nw; i += 256) s_t[i] = a.tcent[i];
    __syncthreads();
    double sr[KC], sg[KC], sb[KC];
    int sn[KC];
    unsigned int cnt[KT][kUsMaxWords], size[KT];
#pragma unroll
    for (int c = 0; c < KC; ++c) sr[c] = sg[c] = sb[c] = 0.0, sn[c] = 0;
#pragma unroll
    for (int c = 0; c < KT; ++c) {
        size[c] = 0;
#pragma unroll
        for (int q = 0; q < kUsMaxWords; ++q) cnt[c][q] = 0;
    }
    // the same number of rounds for every lane (ballots)
    for (int64_t x0 = (int64_t)blockIdx.x * 256; x0 < N; x0 += (int64_t)gridDim.x * 256) {
        const int64_t x = x0 + threadIdx.x;
        const bool in = x < N;
        double r = 0, g = 0, b = 0;
        uint64_t m[kUsMaxWords] = {0, 0, 0, 0};
        if (in) {
            r = (double)a.rgb[x];
            g = (double)a.rgb[N + x];
            b = (double)a.rgb[2 * N + x];
#pragma unroll
            for (int q = 0; q < kUsMaxWords; ++q)
                if (q < nw) m[q] = a.masks[x * nw + q];
        }
        int best = 0, tbest = 0, td = 0;
        double bd = 0;
        for (int c = 0; c < Kc; ++c) {
            const double dr = r - s_c[3 * c], dg = g - s_c[3 * c + 1], db = b - s_c[3 * c + 2];
            const double d = (dr * dr + dg * dg) + db * db;
            if (c == 0 || d < bd) {
                bd = d;
                best = c;
            }
        }
        for (int c = 0; c < Kt; ++c) {
            int d = 0;
#pragma unroll
            for (int q = 0; q < kUsMaxWords; ++q)
                if (q < nw) d += __popcll(m[q] ^ s_t[c * nw + q]);
            if (c == 0 || d < td) {
                td = d;
                tbest = c;
            }
        }
        if (in) {
            a.clab[x] = best;
            a.tlab[x] = tbest;
        }
        if (!with_sums) continue;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const bool mine = in && best == c;
            sr[c] = sr[c] + (mine ? r : 0.0);
            sg[c] = sg[c] + (mine ? g : 0.0);
            sb[c] = sb[c] + (mine ? b : 0.0);
            sn[c] += __popcll(__ballot(mine));
        }
        uint64_t Cb[KT];  // the wave's pixels of each class
#pragma unroll
        for (int c = 0; c < KT; ++c) {
            Cb[c] = __ballot(in && tbest == c);
            size[c] += (unsigned int)__popcll(Cb[c]);
        }
#pragma unroll
        for (int q = 0; q < kUsMaxWords; ++q)
            if (q < nw) {
                uint32_t lo = (uint32_t)m[q], hi = (uint32_t)(m[q] >> 32);
                transpose64(lo, hi, lane);
#pragma unroll
                for (int c = 0; c < KT; ++c)
                    cnt[c][q] += __popc(lo & (uint32_t)Cb[c]) + __popc(hi & (uint32_t)(Cb[c] >> 32));
            }
    }
    if (!with_sums) return;
    for (int i = threadIdx.x; i < KT * kUsMaxWords * 64; i += 256) s_cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        if (c >= Kc) continue;
        const double vr = wave_sum_f64(sr[c]), vg = wave_sum_f64(sg[c]), vb = wave_sum_f64(sb[c]);
        if (lane == 63) {
            red[wave][c][0] = vr;
            red[wave][c][1] = vg;
            red[wave][c][2] = vb;
            red[wave][c][3] = (double)sn[c];
        }
    }
#pragma unroll
    for (int c = 0; c < KT; ++c) {
        if (c >= Kt) continue;
        if (lane == 0) s_size[wave][c] = size[c];
#pragma unroll
        for (int q = 0; q < kUsMaxWords; ++q)
            if (q < nw) atomicAdd(&s_cnt[(c * nw + q) * 64 + lane], cnt[c][q]);
    }
    __syncthreads();
    const int parts = gridDim.x;
    for (int i = threadIdx.x; i < Kc * 4; i += 256) {
        const int c = i >> 2, q = i & 3;
        a.cpart[(int64_t)i * parts + blockIdx.x] = ((red[0][c][q] + red[1][c][q]) + red[2][c][q]) + red[3][c][q];
    }
    for (int i = threadIdx.x; i < Kt * nw * 64; i += 256) a.tpart[(int64_t)blockIdx.x * Kt * nw * 64 + i] = s_cnt[i];
    for (int i = threadIdx.x; i < Kt; i += 256)
        a.tsize[(int64_t)i * parts + blockIdx.x] = s_size[0][i] + s_size[1][i] + s_size[2][i] + s_size[3][i];
}

// New centroids.  Workgroups 0 .. Kc - 1: colour class c, wave q adds the
// partials of component q (lanes strided, then a butterfly: a fixed order); a
// class without pixels keeps its centroid.  Then one per (texture class c,
// word q): bit j set iff 2 count >= size (the median of 0/1 values, a tie in).
__global__ __launch_bounds__(1024) void k_us_update(UnsupArgs a, int parts) {
#pragma clang fp contract(off)
    __shared__ double s_sum[4];
    __shared__ unsigned int s_cnt[16][64];
    __shared__ unsigned int s_n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)blockIdx.x < a.Kc) {
        const int c = blockIdx.x;
        if (wave < 4) {
            double s = 0.0;
#pragma unroll 8
            for (int p = lane; p < parts; p += 64) s = s + a.cpart[(int64_t)(4 * c + wave) * parts + p];
            s = wave_sum_f64(s);
            if (lane == 63) s_sum[wave] = s;
        }
        __syncthreads();
        if (threadIdx.x < 3 && s_sum[3] > 0.0) a.ccent[c * 3 + threadIdx.x] = s_sum[threadIdx.x] / s_sum[3];
        return;
    }
    const int i = (int)blockIdx.x - a.Kc, c = i / a.nw, q = i - c * a.nw;
    unsigned int n = 0;
#pragma unroll 16
    for (int p = wave; p < parts; p += 16) n += a.tpart[((int64_t)p * a.Kt * a.nw + i) * 64 + lane];
    s_cnt[wave][lane] = n;
    if (wave == 15) {
        unsigned int sz = 0;
#pragma unroll 8
        for (int p = lane; p < parts; p += 64) sz += a.tsize[(int64_t)c * parts + p];
        for (int off = 32; off >= 1; off >>= 1) sz += __shfl_xor(sz, off);
        if (lane == 0) s_n = sz;
    }
    __syncthreads();
    if (wave != 0) return;
    n = 0;
    for (int w = 0; w < 16; ++w) n += s_cnt[w][lane];
    const uint64_t word = __ballot(q * 64 + lane < a.k && 2ull * n >= (uint64_t)s_n);
    if (lane == 0 && s_n) a.tcent[c * a.nw + q] = word;
}

// ---- class likelihoods ----
// loglik[x][a Kt + b] = log P(I(x) | a) + log P(s_x | b): minus the distance
// (||I - mu_a||^2 / (2 sigma_c^2), TSM(x, c_b) / beta), normalised over all
// Kc Kt classes.
__global__ __launch_bounds__(256) void k_us_loglik(UnsupArgs a, float *loglik) {
#pragma clang fp contract(off)
    __shared__ double s_c[kUsMaxK * 3];
    __shared__ uint64_t s_t[kUsMaxK * kUsMaxWords];
    const int64_t N = a.N;
    const int nw = a.nw, Kc = a.Kc, Kt = a.Kt, L = Kc * Kt;
    for (int i = threadIdx.x; i < Kc * 3; i += 256) s_c[i] = a.ccent[i];
    for (int i = threadIdx.x; i < Kt * nw; i += 256) s_t[i] = a.tcent[i];
    __syncthreads();
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= N) return;
    const double r = (double)a.rgb[x], g = (double)a.rgb[N + x], b = (double)a.rgb[2 * N + x];
    const double two_s2 = 2.0 * a.sigma_c * a.sigma_c;
    double ec[kUsMaxK], et[kUsMaxK];
    double mc = 0, mt = 0;
    for (int c = 0; c < Kc; ++c) {
        const double dr = r - s_c[3 * c], dg = g - s_c[3 * c + 1], db = b - s_c[3 * c + 2];
        ec[c] = -(((dr * dr + dg * dg) + db * db) / two_s2);
        mc = c == 0 ? ec[c] : (ec[c] > mc ? ec[c] : mc);
    }
    uint64_t m[kUsMaxWords] = {0, 0, 0, 0};
    for (int q = 0; q < nw; ++q) m[q] = a.masks[x * nw + q];
    for (int c = 0; c < Kt; ++c) {
        int d = 0;
        for (int q = 0; q < nw; ++q) d += __popcll(m[q] ^ s_t[c * nw + q]);
        et[c] = -((double)d / a.beta);
        mt = c == 0 ? et[c] : (et[c] > mt ? et[c] : mt);
    }
    // normaliser over all classes, in class order (each exponential formed once)
    double xc[kUsMaxK], xt[kUsMaxK];
    for (int c = 0; c < Kc; ++c) xc[c] = exp(ec[c] - mc);
    for (int c = 0; c < Kt; ++c) xt[c] = exp(et[c] - mt);
    double sc = 0, st = 0;
    for (int i = 0; i < Kc; ++i)
        for (int j = 0; j < Kt; ++j) {
            sc = sc + xc[i];
            st = st + xt[j];
        }
    const double lc = mc + log(sc), lt = mt + log(st);
    float *out = loglik + x * L;
    if (Kt % 4 == 0 && (reinterpret_cast<uintptr_t>(loglik) & 15) == 0) {
        for (int i = 0; i < Kc; ++i)
            for (int j = 0; j < Kt; j += 4) {
                const double e = ec[i] - lc;
                *reinterpret_cast<float4 *>(out + i * Kt + j) =
                    make_float4((float)(e + (et[j] - lt)), (float)(e + (et[j + 1] - lt)),
                                (float)(e + (et[j + 2] - lt)), (float)(e + (et[j + 3] - lt)));
            }
        return;
    }
    for (int i = 0; i < Kc; ++i)
        for (int j = 0; j < Kt; ++j) out[i * Kt + j] = (float)((ec[i] - lc) + (et[j] - lt));
}

// ---- launchers ----
hipError_t launch_unsup_init(const LaunchCtx &lc, const UnsupArgs &a, const UnsupInit &init) {
    hipLaunchKernelGGL(k_us_init, dim3(1), dim3(64), 0, lc.stream, a, init);
    return hipGetLastError();
}

// Workgroups of an assignment: enough to fill the chip twice, few enough that
// their partials are added in a few loads per thread.
int unsup_parts(int64_t N) {
    const int64_t nb = (N + 255) / 256;
    return (int)(nb < 512 ? nb : 512);
}

hipError_t launch_unsup_step(const LaunchCtx &lc, const UnsupArgs &a, bool update) {
    const int parts = unsup_parts(a.N);
    const dim3 grid((unsigned)parts), block(256);
    if (a.Kc <= 4 && a.Kt <= 4)
        hipLaunchKernelGGL((k_us_assign<4, 4>), grid, block, 0, lc.stream, a, update ? 1 : 0);
    else if (a.Kc <= 4)
        hipLaunchKernelGGL((k_us_assign<4, 16>), grid, block, 0, lc.stream, a, update ? 1 : 0);
    else if (a.Kt <= 4)
        hipLaunchKernelGGL((k_us_assign<16, 4>), grid, block, 0, lc.stream, a, update ? 1 : 0);
    else
        hipLaunchKernelGGL((k_us_assign<16, 16>), grid, block, 0, lc.stream, a, update ? 1 : 0);
    if (update)
        hipLaunchKernelGGL(k_us_update, dim3((unsigned)(a.Kc + a.Kt * a.nw)), dim3(1024), 0, lc.stream, a, parts);
    return hipGetLastError();
}

hipError_t launch_unsup_loglik(const LaunchCtx &lc, const UnsupArgs &a, float *loglik) {
    const unsigned nb = (unsigned)((a.N + 255) / 256);
    hipLaunchKernelGGL(k_us_loglik, dim3(nb), dim3(256), 0, lc.stream, a, loglik);
    return hipGetLastError();
}

}  // namespace cs
