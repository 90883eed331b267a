// Primal-dual iteration of the segmentation (Sec. 4.2) on image tiles held on
// chip, for FP32 and up to 16 labels; the scheme and its arithmetic are those
// stated in k_segment.hip, element for element.
//
// What bounds an iteration launched on its own is not its arithmetic but the
// trip of the whole state (u, u_bar, xi_x, xi_y, f: 56 MB at 481 x 321 and 10
// labels) through L2 and the launch itself, and every thread forms its
// neighbours' dual vectors again (three disc projections for one).  Here a
// workgroup holds a tile, one thread per pixel with the pixel's L labels in
// registers.  Right and left neighbours come from the wave by lane shifts (a
// wave is two rows of 32), the ones below and above from LDS (u_bar and xi_y),
// and each dual vector is projected once.
//
// Two forms.  k_pd_resident runs every iteration in one cooperative launch,
// the tiles exchanging their borders, where the image fits one tile per
// compute unit: 481 x 321 with 10 labels 25.4 -> 4.1 to 4.9 us per iteration (by
// the data: how often a wave's discs and simplex need their long way), with 16
// labels and a label cost 82 -> 7.4 us.  k_pd_tile serves larger images: it
// loads a 32 x 32 tile, runs S iterations (up to 8) and writes the pixels that
// are still right; an iteration at x reads u_bar at x + 1, x + W and the new xi
// at x - 1, x - W, so the valid square loses one pixel on each side per
// iteration and a tile yields (32 - 2 S)^2 pixels.  1024 x 1024: 16 labels 175
// -> 86 to 118 us by the data, 3 labels 51 -> 22 us per iteration; with a label cost
// (16 labels) 598 -> 341 us.  There the state's trip through HBM and the 1 tile per
// compute unit that 128 registers leave bound it.
//
// With a label cost the multipliers need sum_x mu of the whole image between
// iterations: k_pd_tile then runs one iteration a launch, every tile writes
// its sum per label, and every workgroup of the next launch adds the tiles'
// sums itself (one wave per label, fixed order); no atomics (603 FP64 atomics
// on one address per label were most of the 82 us).
#include "cs_internal.h"

namespace cs {

namespace {

constexpr int kTd = 32;  // tile side

__device__ __forceinline__ float lane_right(float v) {  // lane i gets lane i + 1
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_left(float v) {  // lane i gets lane i - 1
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}

// Square root and quotient correctly rounded, for operands whose intermediate
// steps neither overflow nor fall below the normal range (the guard below):
// the root by two Newton steps on the reciprocal root with fused remainders,
// the quotient by the same on the reciprocal (P. Markstein, IBM J. Res. Dev. 34,
// 1990).  The root is, from any estimate within a unit; the quotient by his
// theorem, the reciprocal after its step being correctly rounded for every
// significand (run on gfx950 over 2^-60 to 2^62).  So equal to sqrtf and to the
// division bit for bit in that range, at 9 and 8 instructions instead of about
// 40 for the two with scaling and special cases.
__device__ __forceinline__ float sqrt_rn(float x) {
    const float r0 = __builtin_amdgcn_rsqf(x);
    float s = x * r0, h = 0.5f * r0;
    const float e = fmaf(-h, s, 0.5f);
    h = fmaf(h, e, h);
    s = fmaf(s, e, s);
    return fmaf(fmaf(-s, s, x), h, s);
}
__device__ __forceinline__ float div_rn(float n, float d) {
    float y = __builtin_amdgcn_rcpf(d);
    y = fmaf(fmaf(-d, y, 1.0f), y, y);
    float q = n * y;
    q = fmaf(fmaf(-d, q, n), y, q);
    return fmaf(fmaf(-d, q, n), y, q);
}

// The L dual vectors of a pixel onto the disc of radius rad.  plain: the whole
// wave's radii lie where sqrt_rn and div_rn are exact; rad2: |q|^2 up to there
// is inside the disc whatever the rounding of the root, so a wave all of whose
// vectors are there needs neither root nor quotient.
template <int L>
__device__ __forceinline__ void project_discs(float (&px)[L], float (&py)[L], float rad, float rad2, bool plain) {
#pragma clang fp contract(off)
    if (plain) {
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float n2 = px[l] * px[l] + py[l] * py[l];
            if (__any(!(n2 <= rad2))) {
                const float n = sqrt_rn(n2);
                const float s = n > rad && !(n2 <= rad2) ? div_rn(rad, n) : 1.0f;
                px[l] = px[l] * s;
                py[l] = py[l] * s;
            }
        }
    } else {
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float n = sqrtf(px[l] * px[l] + py[l] * py[l]);
            const float s = n > rad ? rad / n : 1.0f;
            px[l] = px[l] * s;
            py[l] = py[l] * s;
        }
    }
}

// Michelot's projection of v[0..L) onto the simplex: theta, such that the
// projection is v[l] - theta where v[l] is not below thr, 0 elsewhere.  The
// coordinates in play are those not below any earlier theta, so the largest
// theta so far (thr) tells them; the first set leaves out what lies more than
// 1 below the maximum, which can never stay in play.  Sums run in label order.
template <int L>
__device__ __forceinline__ float simplex_theta_tile(const float (&v)[L], float &thr) {
#pragma clang fp contract(off)
    float mx = v[0];
#pragma unroll
    for (int l = 1; l < L; ++l) mx = fmaxf(mx, v[l]);
    float t = mx - 1.0f, theta = 0.0f;
    int cnt = 0;
    for (;;) {
        float s = 0.0f;
        int c = 0;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const bool on = !(v[l] < t);
            s = s + (on ? v[l] : 0.0f);
            c += on;
        }
        if (c == cnt) break;
        cnt = c;
        theta = div_rn(s - 1.0f, (float)c);
        t = theta > t ? theta : t;
    }
    thr = t;
    return theta;
}

// Sums over the wave of 16 values per lane, halves and rows swapped between
// registers so that every step adds two labels at once; lane 16 q + 15 ends
// with the sums of labels i + 4 (q & 1) + 8 (q >> 1) in x[i], i = 0..3.
__device__ __forceinline__ void wave_sums16(float (&x)[16]) {
    auto bits = [](float v) { return __builtin_bit_cast(unsigned int, v); };
    auto flt = [](unsigned int v) { return __builtin_bit_cast(float, v); };
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const auto p = __builtin_amdgcn_permlane32_swap(bits(x[i]), bits(x[i + 8]), false, false);
        x[i] = flt(p[0]) + flt(p[1]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto p = __builtin_amdgcn_permlane16_swap(bits(x[i]), bits(x[i + 4]), false, false);
        x[i] = flt(p[0]) + flt(p[1]);
    }
    // rows of 16 lanes: row_shr 1, 2, 4, 8
#define ROW_ADD(ctrl) \
    for (int i = 0; i < 4; ++i) \
        x[i] += flt((unsigned int)__builtin_amdgcn_update_dpp(0, (int)bits(x[i]), ctrl, 0xf, 0xf, true));
    ROW_ADD(0x111)
    ROW_ADD(0x112)
    ROW_ADD(0x114)
    ROW_ADD(0x118)
#undef ROW_ADD
}
// The FP64 value whose halves rows of 16 lanes hold, high, low, high, low: to
// both rows of a pair.
__device__ __forceinline__ double join_rows(uint32_t half) {
    const auto p = __builtin_amdgcn_permlane16_swap(half, half, false, false);
    return __builtin_bit_cast(double, (uint64_t)p[0] << 32 | p[1]);
}
// This lane's half of v (high in even rows of 16 lanes).
__device__ __forceinline__ uint32_t row_half(double v, int lane) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return (uint32_t)(lane & 16 ? b : b >> 32);
}

// The label of x[i] in this lane's row, after wave_sums16.
__device__ __forceinline__ int sums16_label(int i, int lane) { return i + 4 * ((lane >> 4) & 1) + 8 * (lane >> 5); }

}  // namespace

// Iterations t .. t + steps - 1 of one tile (steps <= S; with MDL both are 1).
template <int L, bool MDL>
__global__ __launch_bounds__(kTd *kTd) void k_pd_tile(PdArgs a, int t, int cur, int S, int steps, int tiles_x,
                                                      int ntiles) {
#pragma clang fp contract(off)
    __shared__ float s_ub[L][kTd * kTd];
    __shared__ float s_py[L][kTd * kTd];
    __shared__ float s_mb[L];
    constexpr bool kAhead = L <= (MDL ? 10 : 13);  // registers for all LDS reads at once
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int W = a.W, H = a.H;
    const int64_t N = a.N;
    const int nxt = cur ^ 1;
    // tiles per XCD in contiguous bands (workgroup b runs on XCD b mod 8)
    const int q8 = ntiles / 8, r8 = ntiles % 8, xcd = (int)blockIdx.x % 8, ib = (int)blockIdx.x / 8;
    const int tile = xcd < r8 ? xcd * (q8 + 1) + ib : r8 * (q8 + 1) + (xcd - r8) * q8 + ib;
    const int side = kTd - 2 * S;
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    const int lx = tid & (kTd - 1), ly = tid / kTd;
    const int c = tx * side + lx - S, r = ty * side + ly - S;
    const bool in = c >= 0 && c < W && r >= 0 && r < H;
    const bool mx = in && c < W - 1, my = in && r < H - 1;
    const bool own = in && lx >= S && lx < kTd - S && ly >= S && ly < kTd - S;
    const int x = in ? r * W + c : 0;
    const float s_xi = (float)a.sigma_xi, s_mu = (float)a.sigma_mu, t_u = (float)a.tau_u;

    float u[L], ub[L], px[L], py[L], f[L], mu[MDL ? L : 1];
    const float *F = (const float *)a.f;
    if (t == 0) {
        // the start state: u = u_bar = 1 / L, every multiplier 0
#pragma unroll
        for (int l = 0; l < L; ++l) {
            f[l] = F[l * N + x];
            u[l] = ub[l] = 1.0f / (float)L;
            px[l] = py[l] = 0.0f;
            if constexpr (MDL) mu[l] = 0.0f;
        }
    } else {
        const float *U = (const float *)a.u[cur], *UB = (const float *)a.ub[cur], *PX = (const float *)a.px[cur],
                    *PY = (const float *)a.py[cur];
        const float *MU = MDL ? (const float *)a.mu[cur] : nullptr;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            ub[l] = UB[l * N + x];
            px[l] = PX[l * N + x];
            py[l] = PY[l * N + x];
            if constexpr (MDL) mu[l] = MU[l * N + x];
        }
#pragma unroll
        for (int l = 0; l < L; ++l) {
            u[l] = U[l * N + x];
            f[l] = F[l * N + x];
        }
    }
    // radius of the dual disc, 0 outside the image (the dual vectors there are
    // and stay 0, which is what the divergence at the border takes)
    const float rad = in ? (float)(0.5 * a.lambda) * ((const float *)a.g)[x] : 0.0f;
    const bool plain = __all(!in || (rad > 1e-9f && rad < 1e9f));  // the wave's
    const float rad2 = rad * rad * (1.0f - 0x1p-20f);
    if constexpr (MDL) {
        // m^t and m_bar^t from the tiles' sums of mu^t (t = 0: m^0 = m_bar^0
        // = 1), one wave per label; workgroup 0 keeps m^t and the sum
        for (int l = wave; l < L; l += kTd * kTd / 64) {
            double sum = 0.0;
            if (t > 0) {
                const double *p = a.mpart + ((int64_t)(t & 1) * L + l) * ntiles;
                for (int i = lane; i < ntiles; i += 64) sum += p[i];
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
            }
            if (lane == 0) {
                double m, mprev;
                if (t == 0) {
                    m = mprev = a.mval[l];
                } else {
                    mprev = a.mval[(int64_t)(t - 1) * L + l];
                    m = mprev - a.tau_m * (a.nu + sum);
                    m = m < 0.0 ? 0.0 : (m > 1.0 ? 1.0 : m);
                    if (blockIdx.x == 0) a.mval[(int64_t)t * L + l] = m;
                }
                s_mb[l] = (float)(t == 0 ? m : 2.0 * m - mprev);
            }
        }
    }
#pragma unroll
    for (int l = 0; l < L; ++l) {
        if (!in) u[l] = ub[l] = px[l] = py[l] = f[l] = 0.0f;
        s_ub[l][tid] = ub[l];
    }
    __syncthreads();
    const int dn = (tid + kTd) & (kTd * kTd - 1), up = (tid - kTd) & (kTd * kTd - 1);
    const int last = MDL ? 0 : steps - 1;
    for (int it = 0; it <= last; ++it) {
        // dual step: xi = P(xi + sigma grad u_bar), every label's LDS read in
        // flight before the first disc test
        float gy[L];
        if constexpr (kAhead)
#pragma unroll
            for (int l = 0; l < L; ++l) gy[l] = s_ub[l][dn];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float ubr = lane_right(ub[l]);  // every lane takes part
            px[l] = px[l] + s_xi * (mx ? ubr - ub[l] : 0.0f);
            if constexpr (!kAhead) gy[l] = s_ub[l][dn];
            py[l] = py[l] + s_xi * (my ? gy[l] - ub[l] : 0.0f);
            if constexpr (MDL) {
                const float mn = mu[l] + s_mu * (s_mb[l] - ub[l]);
                mu[l] = mn < 0.0f ? mn : 0.0f;
            }
        }
        project_discs<L>(px, py, rad, rad2, plain);
#pragma unroll
        for (int l = 0; l < L; ++l) s_py[l][tid] = py[l];
        __syncthreads();
        // primal step
        if constexpr (kAhead)
#pragma unroll
            for (int l = 0; l < L; ++l) gy[l] = s_py[l][up];
        float v[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            float d = px[l] - lane_left(px[l]);
            d = d + py[l];
            if constexpr (!kAhead) gy[l] = s_py[l][up];
            d = d - gy[l];
            float step = -d + f[l];
            if constexpr (MDL) step = step - mu[l];
            v[l] = u[l] - t_u * step;
        }
        float thr;
        const float theta = simplex_theta_tile<L>(v, thr);
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float un = v[l] < thr ? 0.0f : v[l] - theta;
            ub[l] = 2.0f * un - u[l];
            u[l] = un;
        }
        if (it == last) break;
#pragma unroll
        for (int l = 0; l < L; ++l) s_ub[l][tid] = ub[l];
        __syncthreads();
    }
    if (own) {
        float *U = (float *)a.u[nxt], *UB = (float *)a.ub[nxt], *PX = (float *)a.px[nxt], *PY = (float *)a.py[nxt];
        float *MU = MDL ? (float *)a.mu[nxt] : nullptr;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            PX[l * N + x] = px[l];
            PY[l * N + x] = py[l];
            UB[l * N + x] = ub[l];
            U[l * N + x] = u[l];
            if constexpr (MDL) MU[l * N + x] = mu[l];
        }
    }
    if constexpr (MDL) {
        // the tile's sum of mu per label: the wave's lanes, then the waves in
        // order
        float sums[16];
#pragma unroll
        for (int l = 0; l < 16; ++l) sums[l] = l < L && own ? mu[l < L ? l : 0] : 0.0f;
        wave_sums16(sums);
        __syncthreads();
        float *red = &s_py[0][0];  // [wave][16]
        if ((lane & 15) == 15)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[wave * 16 + sums16_label(i, lane)] = sums[i];
        __syncthreads();
        if (tid < L) {
            double tot = 0.0;
            for (int w = 0; w < kTd * kTd / 64; ++w) tot = tot + (double)red[w * 16 + tid];
            a.mpart[((int64_t)((t + 1) & 1) * L + tid) * ntiles + tile] = tot;
        }
    }
}

// sum_x mu^T of each label from the last launch's tile sums (one wave each).
__global__ __launch_bounds__(64) void k_pd_msum(PdArgs a, int ntiles) {
    const int l = blockIdx.x;
    const double *p = a.mpart + ((int64_t)(a.iters & 1) * a.L + l) * ntiles;
    double sum = 0.0;
    for (int i = threadIdx.x; i < ntiles; i += 64) sum += p[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if (threadIdx.x == 0) a.msum[(int64_t)a.iters * a.L + l] = sum;
}

// ---- every iteration in one launch, the state on chip ----
// For images whose pixels fit the chip's registers (one tile per compute
// unit): tiles of 32 x th pixels, 30 x (th - 2) of them the tile's own and a
// ring of its neighbours' pixels around them.  A tile keeps the dual vectors
// of its ring's left column and top row itself (the same arithmetic on the
// same values as their owner), so an iteration needs only the neighbours' new
// u_bar: the owner of a border pixel stores it to global memory, and the ring
// thread of that pixel reads it there.  Each value travels in one 64-bit word
// with the number of its iteration, so a word that holds the awaited number
// holds its value and no further ordering is needed; two buffers alternate,
// and a tile can only be one iteration ahead of its neighbours (its next
// iteration needs theirs), so no word is overwritten before it was read.
// With a label cost the tiles' sums of mu travel the same way, each half of an
// FP64 value in a word of its own and a tile's words in a row, to one more
// workgroup, which adds them and sends the totals to every tile.
//
// The tiles wait for each other, so they have to be on the chip together: the
// launch is a cooperative one, and before its first iteration every workgroup
// waits until all have arrived (all_arrived).  Where that takes longer than
// a.arrive_ticks, as where another kernel keeps compute units for long, one of
// them decides that all leave without having written anything, the host sees it
// and runs k_pd_tile instead.  Once all have arrived, every later wait ends by
// itself; it still has an end of its own, kWaitPolls reads of its words (a look
// at the clock in the loop took 0.1 us of an iteration, 0.5 with a label cost): the tile's state becomes NaN, no wait follows, ctl[kPdCtlGaveUp] is set,
// and the launch ends.
//
// Every workgroup has an arrival word, and the first one reads them all (one
// counter for all, whose additions follow one another, took 15 us of a solve).
constexpr int kWaitPolls = 1 << 24;

__device__ __forceinline__ bool all_arrived(const PdArgs &a, int nthr) {
    __shared__ bool s_go;
    unsigned int *decided = a.ctl + kPdCtlDecided, *arrived = a.ctl + kPdCtlWords;
    const int tid = threadIdx.x, grid = gridDim.x;
    auto decision = [&]() { return __hip_atomic_load(decided, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto decide = [&](unsigned int v) {  // the first decision stands, and is told to the host
        unsigned int cur = 0;
        if (!__hip_atomic_compare_exchange_strong(decided, &cur, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT))
            return cur;
        *a.host_tag = v == 1u ? a.tag : -a.tag;  // (one store: nothing waits for it)
        return v;
    };
    const int64_t t0 = (int64_t)wall_clock64();
    auto late = [&]() { return (int64_t)wall_clock64() - t0 > a.arrive_ticks; };
    if (blockIdx.x == 0) {
        bool in = a.arrive_ticks >= 0;
        for (int i = tid ? tid : nthr; in && i < grid; i += nthr)
            while (in && !__hip_atomic_load(arrived + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                in = !decision() && !late();
        const bool all = __syncthreads_and(in);
        if (tid == 0) s_go = decide(all ? 1u : 2u) == 1u;
    } else if (tid == 0) {
        unsigned int d = a.arrive_ticks < 0 ? decide(2u) : 0u;
        __hip_atomic_store(arrived + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (!d) {
            d = decision();
            if (!d && late()) d = decide(2u);
            if (!d) __builtin_amdgcn_s_sleep(1);
        }
        s_go = d == 1u;
    }
    __syncthreads();
    return s_go;
}

__device__ __forceinline__ void put_word(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get_word(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Slot of border pixel (x, y) of a tile's own w x h pixels.
__device__ __forceinline__ int border_slot(int x, int y, int h) {
    constexpr int w = kTd - 2;
    return y == 0 ? x : y == h - 1 ? w + x : 2 * w + (x == 0 ? 0 : h - 2) + y - 1;
}

template <int L, bool MDL, int NT>
__global__ __launch_bounds__(NT) void k_pd_resident(PdArgs a, int th, int tiles_x, int ntiles) {
#pragma clang fp contract(off)
    constexpr int kIw = kTd - 2, kWaves = NT / 64;
    __shared__ float s_ub[L][NT];
    __shared__ float s_py[L][NT];
    constexpr bool kHoldF = !MDL || L <= 8;  // f in registers, else (the thread's own words) in LDS
    __shared__ float s_f[kHoldF ? 1 : L][NT];
    __shared__ float s_red[MDL ? kWaves : 1][16];
    __shared__ float s_mb[MDL ? 16 : 1];
    __shared__ double s_sum[MDL ? 2 : 1][kWaves][16];
    constexpr int kAhead = 5;  // pairs of tiles a wave reads together (two rounds for 240 tiles and 12 waves)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nthr = kTd * th, nwave = nthr / 64;
    const int W = a.W, H = a.H, ih = th - 2;
    const int64_t N = a.N;
    const int tile = (int)blockIdx.x, ty = tile / tiles_x, tx = tile - ty * tiles_x;
    const int lx = tid & (kTd - 1), ly = tid / kTd;
    const int c = tx * kIw + lx - 1, r = ty * ih + ly - 1;
    const bool in = c >= 0 && c < W && r >= 0 && r < H;
    const bool mx = in && c < W - 1, my = in && r < H - 1;
    const bool own = in && lx >= 1 && lx <= kIw && ly >= 1 && ly <= ih;
    const bool ring = in && !own;
    const int x = in ? r * W + c : 0;
    // exchange words: a tile's border pixels in slot order, L words each, so
    // that consecutive threads store and read consecutive words; this thread's
    // are tid, tid + nthr, tid + 2 nthr (the launch sees to it that these are
    // all): src and dst their places in s_ub, rd the word read (-1: none)
    const int per_tile = 2 * kIw + 2 * (ih - 2);
    const int64_t ebuf = (int64_t)ntiles * per_tile * L;
    int src[3], dst[3], rd[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int i = tid + k * nthr, q = i / L, l = i - q * L;
        {
            const int s2 = q - 2 * kIw, sx = q < kIw ? q : q < 2 * kIw ? q - kIw : s2 < ih - 2 ? 0 : kIw - 1;
            const int sy = q < kIw ? 0 : q < 2 * kIw ? ih - 1 : 1 + (s2 < ih - 2 ? s2 : s2 - (ih - 2));
            src[k] = q < per_tile ? l * NT + (sy + 1) * kTd + sx + 1 : -1;
        }
        {
            const int s2 = q - 2 * kTd, sx = q < kTd ? q : q < 2 * kTd ? q - kTd : (s2 & 1) * (kTd - 1);
            const int sy = q < kTd ? 0 : q < 2 * kTd ? th - 1 : 1 + (s2 >> 1);
            const int rc = tx * kIw + sx - 1, rr = ty * ih + sy - 1;
            const bool ok = q < 2 * kTd + 2 * (th - 2) && rc >= 0 && rc < W && rr >= 0 && rr < H;
            const int ox = ok ? rc / kIw : 0, oy = ok ? rr / ih : 0;
            rd[k] = ok ? ((oy * tiles_x + ox) * per_tile + border_slot(rc - ox * kIw, rr - oy * ih, ih)) * L + l : -1;
            dst[k] = ok ? l * NT + sy * kTd + sx : 0;
        }
    }
    // [2][tile][high, low][16] sums of mu, [2][high, low][16] their totals
    uint64_t *psum = a.exch + 2 * ebuf, *ptot = psum + 2 * 32 * (int64_t)ntiles;
    const int ml = lane & 15;  // the label of this lane's sums
    if (!all_arrived(a, nthr)) return;
    bool alive = a.wait_words;
    if constexpr (MDL) {
        if (tile == ntiles) {
            // the workgroup past the tiles adds the tiles' sums: a wave's load
            // has the words of two of them, a wave takes every nwave-th pair,
            // and the first wave adds the waves' sums
            for (int t = 0; t < a.iters; ++t) {
                const uint32_t tag = (uint32_t)t + 1u;
                const uint64_t *ps = psum + (int64_t)(t & 1) * 32 * ntiles;
                double s = 0.0;
                for (int i0 = 2 * wave; i0 < ntiles; i0 += 2 * kAhead * nwave) {  // (wave-uniform)
                    uint64_t w[kAhead];
                    bool got = false;
                    for (int n = 0; alive && !got; ++n) {
                        got = true;
#pragma unroll
                        for (int q = 0; q < kAhead; ++q) {
                            const int i = i0 + 2 * nwave * q + (lane >> 5);
                            w[q] = i < ntiles && ml < L ? get_word(ps + i * 32 + (lane & 31)) : (uint64_t)tag << 32;
                        }
#pragma unroll
                        for (int q = 0; q < kAhead; ++q) got &= (uint32_t)(w[q] >> 32) == tag;
                        alive = n < kWaitPolls;
                    }
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) s = s + join_rows(got ? (uint32_t)w[q] : 0x7ff80000u);
                }
                s = s + __shfl_xor(s, 32);
                if (lane < 16) s_sum[t & 1][wave][lane] = s;
                __syncthreads();
                if (wave != 0) continue;
                s = 0.0;
                for (int v = 0; v < nwave; ++v) s = s + s_sum[t & 1][v][ml];
                if (ml < L && lane < 32) put_word(ptot + (t & 1) * 32 + lane, (uint64_t)tag << 32 | row_half(s, lane));
                if (lane < L && t + 1 == a.iters) a.msum[(int64_t)a.iters * L + lane] = s;
            }
            if (!alive) a.ctl[kPdCtlGaveUp] = 1u;
            return;
        }
        for (int i = tid; i < kWaves * 16; i += nthr) (&s_red[0][0])[i] = 0.0f;
    }
    const float s_xi = (float)a.sigma_xi, s_mu = (float)a.sigma_mu, t_u = (float)a.tau_u;

    float u[L], ub[L], px[L], py[L], f[kHoldF ? L : 1], mu[MDL ? L : 1];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        // the start state: u = u_bar = 1 / L, every multiplier 0
        const float fl = in ? ((const float *)a.f)[l * N + x] : 0.0f;
        if constexpr (kHoldF)
            f[l] = fl;
        else
            s_f[l][tid] = fl;
        u[l] = ub[l] = in ? 1.0f / (float)L : 0.0f;
        px[l] = py[l] = 0.0f;
        if constexpr (MDL) mu[l] = 0.0f;
        s_ub[l][tid] = ub[l];
    }
    const float rad = in ? (float)(0.5 * a.lambda) * ((const float *)a.g)[x] : 0.0f;
    const bool plain = __all(!in || (rad > 1e-9f && rad < 1e9f));  // the wave's
    const float rad2 = rad * rad * (1.0f - 0x1p-20f);
    const int dn = tid + kTd < nthr ? tid + kTd : tid, up = tid >= kTd ? tid - kTd : tid;
    // of label ml: m^t (the first wave's) and m_bar^t
    double m = 1.0;
    float mb = 1.0f;
    __syncthreads();
    for (int t = 0; t < a.iters; ++t) {
        if (ring && t > 0)
#pragma unroll
            for (int l = 0; l < L; ++l) ub[l] = s_ub[l][tid];
        if constexpr (MDL)
            if (t > 0) mb = s_mb[ml];
        float gy[L];
#pragma unroll
        for (int l = 0; l < L; ++l) gy[l] = s_ub[l][dn];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float ubr = lane_right(ub[l]);
            px[l] = px[l] + s_xi * (mx ? ubr - ub[l] : 0.0f);
            py[l] = py[l] + s_xi * (my ? gy[l] - ub[l] : 0.0f);
            if constexpr (MDL) {
                const float mbl = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mb), l));
                const float mn = mu[l] + s_mu * (mbl - ub[l]);
                mu[l] = mn < 0.0f ? mn : 0.0f;
            }
        }
        project_discs<L>(px, py, rad, rad2, plain);
#pragma unroll
        for (int l = 0; l < L; ++l) s_py[l][tid] = py[l];
        if constexpr (MDL) {
            float sums[16];
#pragma unroll
            for (int l = 0; l < 16; ++l) sums[l] = l < L && own ? mu[l < L ? l : 0] : 0.0f;
            wave_sums16(sums);
            if ((lane & 15) == 15)
#pragma unroll
                for (int i = 0; i < 4; ++i) s_red[wave][sums16_label(i, lane)] = sums[i];
        }
        __syncthreads();
        if constexpr (MDL) {
            if (tid < 32 && ml < L) {
                double tot = 0.0;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) tot = tot + (double)s_red[w][ml];
                put_word(psum + ((int64_t)(t & 1) * ntiles + tile) * 32 + tid, (uint64_t)(t + 1) << 32 | row_half(tot, lane));
            }
        }
#pragma unroll
        for (int l = 0; l < L; ++l) gy[l] = s_py[l][up];
        float v[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            float d = px[l] - lane_left(px[l]);
            d = d + py[l];
            d = d - gy[l];
            float step = -d + (kHoldF ? f[kHoldF ? l : 0] : s_f[kHoldF ? 0 : l][tid]);
            if constexpr (MDL) step = step - mu[l];
            v[l] = u[l] - t_u * step;
        }
        float thr;
        const float theta = simplex_theta_tile<L>(v, thr);
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float un = v[l] < thr ? 0.0f : v[l] - theta;
            ub[l] = 2.0f * un - u[l];
            u[l] = un;
        }
        const bool more = t + 1 < a.iters;
        const uint32_t tag = (uint32_t)t + 1u;
        if (more) {
#pragma unroll
            for (int l = 0; l < L; ++l) s_ub[l][tid] = ub[l];
            __syncthreads();
            uint64_t *e = a.exch + (int64_t)(t & 1) * ebuf;
            const float *ub0 = &s_ub[0][0];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (src[k] >= 0)
                    put_word(e + (int64_t)tile * per_tile * L + tid + k * nthr,
                             (uint64_t)tag << 32 | __builtin_bit_cast(uint32_t, ub0[src[k]]));
        }
        // the neighbours' words and, with a label cost, in the first wave half a
        // total of label lane & 15 (every wave reading them and keeping an m of its
        // own, 13.6 us an iteration)
        if (more) {
            const uint64_t *e = a.exch + (int64_t)(t & 1) * ebuf;
            const uint64_t *pt = ptot + (t & 1) * 32 + (ml < L ? lane & 31 : 0);
            uint64_t w[3], sw = 0;
            bool got = false;
            for (int n = 0; alive && !got; ++n) {
#pragma unroll
                for (int k = 0; k < 3; ++k) w[k] = rd[k] >= 0 ? get_word(e + rd[k]) : (uint64_t)tag << 32;
                if (MDL && wave == 0) sw = get_word(pt);
                got = !MDL || wave != 0 || (uint32_t)(sw >> 32) == tag;
#pragma unroll
                for (int k = 0; k < 3; ++k) got &= (uint32_t)(w[k] >> 32) == tag;
                alive = n < kWaitPolls;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (rd[k] >= 0)
                    (&s_ub[0][0])[dst[k]] = got ? __builtin_bit_cast(float, (uint32_t)w[k]) : __builtin_nanf("");
            if (MDL && wave == 0) {
                double mn = m - a.tau_m * (a.nu + join_rows(got ? (uint32_t)sw : 0x7ff80000u));
                mn = mn < 0.0 ? 0.0 : (mn > 1.0 ? 1.0 : mn);
                if (tid < 16) s_mb[tid] = (float)(2.0 * mn - m);
                m = mn;
            }
        }
        __syncthreads();
    }
    if (!alive) a.ctl[kPdCtlGaveUp] = 1u;
    if (own) {
        float *U = (float *)a.u[1], *PX = (float *)a.px[1], *PY = (float *)a.py[1];
        float *MU = MDL ? (float *)a.mu[1] : nullptr;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            U[l * N + x] = u[l];
            PX[l * N + x] = px[l];
            PY[l * N + x] = py[l];
            if constexpr (MDL) MU[l * N + x] = mu[l];
        }
    }
}

// ---- launchers ----
static int64_t tiles_for(const PdArgs &a, int S) {
    const int side = kTd - 2 * S;
    return (int64_t)((a.W + side - 1) / side) * ((a.H + side - 1) / side);
}

// Iterations per launch: a tile costs about 2.5 iterations for its loads,
// stores and launch (one round of tiles at 10 labels: 16.1 us for one
// iteration, 22.8 for three), and the chip runs one tile per compute unit at a
// time, so the rounds of tiles decide.
int pd_tile_steps(const LaunchCtx &lc, const PdArgs &a) {
    if (a.mdl) return 1;
    int best = 1;
    double cost = 0.0;
    for (int S = 1; S <= 8; ++S) {
        const double rounds = (double)((tiles_for(a, S) + lc.num_cu - 1) / lc.num_cu);
        const double c = rounds * (S + 2.5) / S;
        if (S == 1 || c < cost) {
            best = S;
            cost = c;
        }
    }
    return best;
}

int64_t pd_tiles(const PdArgs &a, int S) { return tiles_for(a, S); }

template <bool MDL>
static void tile_launch(const LaunchCtx &lc, const PdArgs &a, int t, int cur, int S, int steps) {
    const int side = kTd - 2 * S, tiles_x = (a.W + side - 1) / side, nt = (int)tiles_for(a, S);
    const dim3 grid((unsigned)nt), block(kTd * kTd);
#define PD_TILE_CASE(n)                                                                                       \
    case n:                                                                                                   \
        hipLaunchKernelGGL((k_pd_tile<n, MDL>), grid, block, 0, lc.stream, a, t, cur, S, steps, tiles_x, nt); \
        break;
    switch (a.L) {
        PD_TILE_CASE(1) PD_TILE_CASE(2) PD_TILE_CASE(3) PD_TILE_CASE(4) PD_TILE_CASE(5) PD_TILE_CASE(6)
        PD_TILE_CASE(7) PD_TILE_CASE(8) PD_TILE_CASE(9) PD_TILE_CASE(10) PD_TILE_CASE(11) PD_TILE_CASE(12)
        PD_TILE_CASE(13) PD_TILE_CASE(14) PD_TILE_CASE(15) PD_TILE_CASE(16)
    }
#undef PD_TILE_CASE
}

hipError_t launch_pd_tile(const LaunchCtx &lc, const PdArgs &a, int t, int cur, int S, int steps) {
    if (a.mdl)
        tile_launch<true>(lc, a, t, cur, S, steps);
    else
        tile_launch<false>(lc, a, t, cur, S, steps);
    return hipGetLastError();
}

// Threads that a resident tile may have: 1024 where the state fits 128
// registers, else 768 (168 registers).
static constexpr int resident_threads(int L, bool mdl) { return L <= (mdl ? 5 : 12) ? 1024 : 768; }

// Rows of a resident tile: the fewest (the least work per compute unit and
// iteration) with which every tile has a compute unit; 0: the image is larger
// than the chip holds.
int pd_resident_rows(const LaunchCtx &lc, const PdArgs &a) {
    if (a.iters < 1) return 0;
    for (int th = 4; kTd * th <= resident_threads(a.L, a.mdl); th += 2) {
        if ((2 * kTd + 2 * (th - 2)) * a.L > 3 * kTd * th) continue;  // three exchange words a thread
        const int64_t nt = (int64_t)((a.W + kTd - 3) / (kTd - 2)) * ((a.H + th - 3) / (th - 2));
        if (nt + (a.mdl ? 1 : 0) <= lc.num_cu) return th;
    }
    return 0;
}

static int64_t resident_tiles(const PdArgs &a, int th) {
    return (int64_t)((a.W + kTd - 3) / (kTd - 2)) * ((a.H + th - 3) / (th - 2));
}

// Control words, then an arrival word per workgroup (an even number).
static size_t ctl_words(const PdArgs &a, int th) { return kPdCtlWords + (resident_tiles(a, th) + 2) / 2 * 2; }

size_t pd_resident_words(const PdArgs &a, int th) {
    const int per_tile = 2 * (kTd - 2) + 2 * (th - 4);
    return (size_t)resident_tiles(a, th) * 2 * (a.L * per_tile + (a.mdl ? 32 : 0)) + (a.mdl ? 2 * 32 : 0) +
           ctl_words(a, th) / 2;
}

unsigned int *pd_resident_ctl(const PdArgs &a, int th) {
    return (unsigned int *)(a.exch + pd_resident_words(a, th)) - ctl_words(a, th);
}

template <bool MDL>
static const void *resident_kernel(int L) {
#define PD_RES_CASE(n) \
    case n: return (const void *)&k_pd_resident<n, MDL, resident_threads(n, MDL)>;
    switch (L) {
        PD_RES_CASE(1) PD_RES_CASE(2) PD_RES_CASE(3) PD_RES_CASE(4) PD_RES_CASE(5) PD_RES_CASE(6)
        PD_RES_CASE(7) PD_RES_CASE(8) PD_RES_CASE(9) PD_RES_CASE(10) PD_RES_CASE(11) PD_RES_CASE(12)
        PD_RES_CASE(13) PD_RES_CASE(14) PD_RES_CASE(15) PD_RES_CASE(16)
    }
#undef PD_RES_CASE
    return nullptr;
}

hipError_t launch_pd_resident(const LaunchCtx &lc, const PdArgs &a, int th) {
    hipError_t e = launch_fill_u32(lc, (unsigned int *)a.exch, 2 * pd_resident_words(a, th), 0u);
    if (e != hipSuccess) return e;
    PdArgs arg = a;
    arg.ctl = pd_resident_ctl(a, th);
    int tiles_x = (a.W + kTd - 3) / (kTd - 2), nt = (int)resident_tiles(a, th);
    void *args[] = {&arg, &th, &tiles_x, &nt};
    e = hipLaunchCooperativeKernel(a.mdl ? resident_kernel<true>(a.L) : resident_kernel<false>(a.L),
                                   dim3((unsigned)(nt + (a.mdl ? 1 : 0))), dim3((unsigned)(kTd * th)), args, 0, lc.stream);
    // (for these the caller takes the other form)
    if (e == hipErrorCooperativeLaunchTooLarge || e == hipErrorNotSupported) (void)hipGetLastError();
    return e;
}

hipError_t launch_pd_msum(const LaunchCtx &lc, const PdArgs &a, int S) {
    hipLaunchKernelGGL(k_pd_msum, dim3((unsigned)a.L), dim3(64), 0, lc.stream, a, (int)tiles_for(a, S));
    return hipGetLastError();
}

}  // namespace cs
