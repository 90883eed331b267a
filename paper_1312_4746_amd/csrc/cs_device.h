// Device helpers shared by the library's kernels (FP64 patch arithmetic in a
// fixed evaluation order, BF16 rounding).  Library-internal.
#pragma once
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cs_internal.h"

// lane l of old replaced by v
__device__ int write_lane(int v, int l, int old) __asm("llvm.amdgcn.writelane.i32");

namespace cs {

// Symmetric border reflection that repeats the edge pixel: -1 -> 0, n -> n-1.
__device__ __forceinline__ int reflect_idx(int i, int n) {
    return i < 0 ? -i - 1 : (i >= n ? 2 * n - i - 1 : i);
}

// Gray value, FP64, order (0.299 R + 0.587 G) + 0.114 B.
__device__ __forceinline__ double gray64_of(float r, float g, float b) {
#pragma clang fp contract(off)
    return (0.299 * (double)r + 0.587 * (double)g) + 0.114 * (double)b;
}
__device__ __forceinline__ double gray64(const float *rgb, int64_t N, int64_t idx) {
    return gray64_of(rgb[idx], rgb[N + idx], rgb[2 * N + idx]);
}

// Exact FP64 a_j = sum_t O_jt s_t of pixel pix (om = row j of O) by a group of
// kExactLanes lanes: the normalised Gaussian-masked gray patch rebuilt from
// the image in the oracle's operation order, q_t = w_t g_t, s_t = (q_t - mu) /
// sqrt(nu2) (0 when nu2 = 0), every sum sequential in t and no contraction.
// The lanes load and divide in parallel (buf: the group's n + 1 doubles of
// LDS), lane 0's sums are the serial part; with one lane per entry the chain of
// loads took 20 us however few the entries (1024 x 1024, 11 x 11, k = 242: the
// median's recompute 102 -> 35 us, the masks' last entries 77 -> 53 us).  mu =
// sum_t q_t / n and nu2 = sum_t (q_t - mu)^2 come from stats[2 pix], stats[2 pix
// + 1] (the analysis kernel's exact values, the same operations) when stats is
// non-null, else they are computed here.  Every lane of the wave takes part
// (live: the group has an entry); the group's lanes return the same value.  zero:
// the patch has nu2 = 0, so every entry of the pixel is 0.
constexpr int kExactLanes = 8;
// LDS of a wave's groups, n + 1 doubles each (an odd stride of banks), and waves
// per compute unit: sixteen fit up to 11 x 11 patches (with eight, 31000 entries of
// 121 went in two rounds: 44 us against 35)
inline size_t exact_lds(int n) { return sizeof(double) * (64 / kExactLanes) * (size_t)(n + 1); }
constexpr int kExactWaves = 16;
__device__ __forceinline__ double exact_entry(const float *rgb, int H, int W, int p, const double *wmask,
                                              const float *om, int64_t pix, const double *stats, double *buf,
                                              bool live, bool &zero) {
#pragma clang fp contract(off)
    const int64_t N = (int64_t)H * W;
    const int h = (p - 1) / 2, n = p * p, gl = threadIdx.x & (kExactLanes - 1);
    const int row = (int)(pix / W), col = (int)(pix - (int64_t)row * W);
    if (live)
        for (int t0 = gl; t0 < n; t0 += 4 * kExactLanes) {
            float r[4], g[4], b[4];
            double w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * kExactLanes < n ? t0 + u * kExactLanes : n - 1;
                const int y = t / p, x = t - y * p;
                const int64_t idx = (int64_t)reflect_idx(row + y - h, H) * W + reflect_idx(col + x - h, W);
                r[u] = rgb[idx];
                g[u] = rgb[N + idx];
                b[u] = rgb[2 * N + idx];
                w[u] = wmask[t];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (t0 + u * kExactLanes < n) buf[t0 + u * kExactLanes] = w[u] * gray64_of(r[u], g[u], b[u]);
        }
    __builtin_amdgcn_wave_barrier();  // a wave's LDS accesses complete in order
    double mu, nu2;
    if (stats) {
        mu = live ? stats[2 * pix] : 0.0;
        nu2 = live ? stats[2 * pix + 1] : 0.0;
    } else {
        double sum = 0.0;
        nu2 = 0.0;
        // every lane of the group the same sums (LDS broadcasts)
#pragma unroll 8
        for (int t = 0; t < n; ++t) sum = sum + buf[t];
        mu = sum / (double)n;
#pragma unroll 8
        for (int t = 0; t < n; ++t) {
            const double z = buf[t] - mu;
            nu2 = nu2 + z * z;
        }
    }
    const double nu = sqrt(nu2);
    if (live)
        for (int t = gl; t < n; t += kExactLanes) buf[t] = (double)om[t] * (nu2 == 0.0 ? 0.0 : (buf[t] - mu) / nu);
    __builtin_amdgcn_wave_barrier();
    double acc = 0.0;
#pragma unroll 8
    for (int t = 0; t < n; ++t) acc = acc + buf[t];
    __builtin_amdgcn_wave_barrier();
    zero = nu2 == 0.0;
    return zero ? 0.0 : acc;
}

// The same for a run of entries of which many are of one pixel: a zero patch is
// remembered (a black image has millions of such entries; each formed anew, 25
// instead of 4 ms at 1024 x 1024, k = 98).
struct ExactRun {
    int64_t zero_pix = -1;  // the group's
    __device__ __forceinline__ double entry(const float *rgb, int H, int W, int p, const double *wmask,
                                            const float *om, int64_t pix, const double *stats, double *buf, bool live) {
        const bool form = live && pix != zero_pix;
        if (!__any(form)) return 0.0;
        bool zero;
        const double v = exact_entry(rgb, H, W, p, wmask, om, pix, stats, buf, form, zero);
        if (form && zero) zero_pix = pix;
        return form ? v : 0.0;
    }
    // the zero patch that the wave's last group met, -1: none
    __device__ __forceinline__ int64_t wave_zero() const {
        const uint64_t z = (uint64_t)zero_pix;
        return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(z >> 32), 63) << 32 |
                         (uint32_t)__builtin_amdgcn_readlane((uint32_t)z, 63));
    }
};

// Per-row decision margin: the given absolute margin when >= 0, else the
// proven bound coef * ||O_j||_2 of the rounded analysed vector (unit-norm
// patch) with a relative safety factor for the FP64 evaluation of the bound
// itself and a tiny absolute term for flushed subnormal products.
__device__ __forceinline__ double row_margin(const float *omega, int j, int n, double margin, double coef) {
#pragma clang fp contract(off)
    if (margin >= 0.0) return margin;
    double ss = 0.0;
    for (int t = 0; t < n; ++t) {
        const double o = (double)omega[(int64_t)j * n + t];
        ss = ss + o * o;
    }
    return coef * sqrt(ss) * (1.0 + 0x1p-20) + 0x1p-100;
}

// Co-support at tau = frac * median|a| while the median is only known to lie in
// [v_lo, v_hi] up to the largest row margin mm: tau = fl(frac * median) is
// monotone in the median, so it lies in [tlo, thi] (both ends widened by the
// rounding of the bounds).
__device__ __forceinline__ void tau_interval(double vlo, double vhi, double mm, double frac, double &tlo,
                                             double &thi) {
    double mlo = vlo - mm;
    mlo = mlo > 0.0 ? nextafter(mlo, 0.0) : 0.0;
    const double mhi = nextafter(vhi + mm, INFINITY);
    tlo = mlo > 0.0 ? nextafter(frac * mlo, 0.0) : 0.0;
    thi = nextafter(frac * mhi, INFINITY);
}
// A row of margin m: rounded |a| <= tin is in, > tout is out, the rest is
// decided once tau is known.
__device__ __forceinline__ void tau_row_interval(double tlo, double thi, double m, float &tin, float &tout) {
    const double a = tlo - m, b = thi + m;
    tin = (float)a;
    if ((double)tin > a) tin = nextafterf(tin, -INFINITY);
    tout = (float)b;
    if ((double)tout < b) tout = nextafterf(tout, INFINITY);
}
// Float bits at or below every row's undecided entries.
__device__ __forceinline__ uint32_t tau_defer_base(double tlo, double mm) {
    const double a = tlo - mm;
    float fa = (float)a;
    if ((double)fa > a) fa = nextafterf(fa, -INFINITY);
    return fa > 0.0f ? __float_as_uint(fa) : 0u;
}
// Listed entries of a bracket: entry in the low bits, key less a base above
// (kPackMax: the key does not fit).
constexpr int kPackShift = 40;
constexpr uint32_t kPackMax = (1u << 24) - 1u;
// comparison predicates of the wave-mask builtins (LLVM's numbers)
constexpr int kUlt = 36, kUle = 37, kSgt = 38, kOgt = 2, kOle = 5;
// the set bits of m in lower lanes
__device__ __forceinline__ uint32_t lane_prefix(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Radix selection helpers (256-thread workgroups).
// The digit holding the remaining rank in a complete kHistBins-bin histogram
// (parallel prefix over the bins): the prefix with that digit set and the
// rank left inside it, returned to every thread.
__device__ __forceinline__ void tau_pick_digit(const unsigned int *hist, int shift, unsigned int prefix_in,
                                               unsigned long long rank_in, unsigned int &prefix_out,
                                               unsigned long long &rank_out) {
    constexpr int per = kHistBins / 256;
    __shared__ unsigned long long scan[256];
    __shared__ unsigned int s_pfx;
    __shared__ unsigned long long s_rank;
    const int t = threadIdx.x;
    unsigned int loc[per];
    unsigned long long sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        loc[i] = hist[t * per + i];
        sum += loc[i];
    }
    scan[t] = sum;
    if (t == 0) {
        s_pfx = prefix_in;
        s_rank = rank_in;
    }
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const unsigned long long v = t >= off ? scan[t - off] : 0ull;
        __syncthreads();
        scan[t] += v;
        __syncthreads();
    }
    const unsigned long long before = scan[t] - sum;
    if (rank_in >= before && rank_in < scan[t]) {
        unsigned long long rr = rank_in - before;
        for (int i = 0; i < per; ++i) {
            if (rr < loc[i]) {
                s_pfx = prefix_in | ((unsigned int)(t * per + i) << shift);
                s_rank = rr;
                break;
            }
            rr -= loc[i];
        }
    }
    __syncthreads();
    prefix_out = s_pfx;
    rank_out = s_rank;
}

// Set-up of a folded selection: per-row margins and their maximum (by one
// workgroup of nt threads, at least 256) ...
__device__ __forceinline__ void tau_setup_margins(const float *omega, int k, int n, double coef, double *margins,
                                                  double *max_margin, int nt) {
    __shared__ double red[16];
    const int t = threadIdx.x;
    double m = 0.0;
    if (t < k) margins[t] = m = row_margin(omega, t, n, -1.0, coef);
    for (int off = 1; off < 64; off <<= 1) m = fmax(m, __shfl_xor(m, off));
    if ((t & 63) == 0) red[t >> 6] = m;
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < nt / 64; ++w) m = fmax(m, red[w]);
        *max_margin = m;
    }
}
// ... and the state (digit 0: empty prefix, the target rank) and the cleared
// histograms.
__device__ __forceinline__ void tau_setup_state(TauState *st, unsigned int *hist3, int hist_words,
                                                unsigned long long rank0, int nt) {
    const int t = threadIdx.x;
    for (int i = t; i < hist_words; i += nt) hist3[i] = 0u;
    if (t == 0) {
        st->rank0 = rank0;
        st->rank = rank0;
        st->prefix = 0;
        for (int d = 0; d < 4; ++d) {
            st->pfx[d] = 0;
            st->rk[d] = rank0;
        }
        st->nparts = 0;
        st->below = 0;
        st->ncand = 0;
        st->n_d = 0;
        st->n_r = 0;
        st->lo = st->hi = 0.0;
        st->br_valid = st->br_ok = st->br_over = 0;
        st->median = 0.0;
        st->tau = 0.0;
    }
}

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// Two values to BF16, to nearest even, by the conversion instruction (the bits
// of bf16_rne for every finite value).
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{a, b}), bf16x2_t));
}
__device__ __forceinline__ short bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

}  // namespace cs
