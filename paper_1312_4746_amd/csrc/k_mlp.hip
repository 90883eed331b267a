// Learned surrogate of the data term on gfx950: a two-hidden-layer perceptron
// (GELU, 128 units) from a pixel's colour, normalised position and analysed
// vector (Sec. 2 a = O s of Sec. 3.1 patches) to its per-label
// log-likelihoods (the Sec. 3.1/3.2 data term), trained by Adam on exact
// targets.  Matrix products run on BF16 MFMA (v_mfma_f32_16x16x16_bf16 for
// training, 16x16x32 for inference) with FP32 accumulation; biases, GELU, the
// loss and Adam are FP32.
//
// Layout trick: every layer computes the TRANSPOSED product, units x rows.
// With A = weights (rows = units) and B = activations^T (columns = 16 batch
// rows), lane (g, j) of the result holds units 4g..4g+3 of batch row j, which
// is exactly the B-operand fragment (k = 4g..4g+3, column j) of the next
// layer.  So a 16-row tile flows through all layers in registers, and the
// backward pass reuses the same layout with the transposed weights as A.
//
// Weight gradients dW = delta^T act are reductions over the batch; the
// forward/backward kernel stores the BF16 activations and deltas of each
// 16-row tile as [unit][16 rows], so that the gradient kernel reads 4
// consecutive rows per lane for both MFMA operands and a wave's operand is 512
// consecutive bytes.  The gradient kernel adds its row chunks' partial sums in
// a fixed order (deterministic) and applies Adam to them itself.
//
// A training step is a short serial chain (batch 4096: one 16-row tile per
// compute unit), so what bounds it is latency, not the 0.8 GFLOP: every weight
// fragment of the forward and backward pass is requested before the first
// product, and the gradient's chunks meet in LDS instead of memory and a third
// launch.  Batch 4096, 103 inputs, 10 outputs: 36 -> 17.4 us of
// kernels per step (10.3 and 7.0; the gradient launch is bound by the 262 KB
// that a workgroup reads through its L1 and by the trip from the other XCDs).
#pragma clang fp contract(off)

#include <type_traits>

#include "cs_internal.h"
#include "cs_device.h"

namespace cs {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kClipNats = 20.0f;
constexpr float kAdamB1 = 0.9f, kAdamB2 = 0.999f, kAdamEps = 1e-8f;

// erf by the rational approximation 7.1.26 of Abramowitz and Stegun
// (Handbook of Mathematical Functions), |error| <= 1.5e-7: a polynomial in
// t = 1 / (1 + p |x|) times exp(-x^2), branch-free.  GELU(z) = z Phi(z) with
// Phi(z) = (1 + erf(z / sqrt 2)) / 2.
__device__ __forceinline__ float erf_as(float x) {
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
    float poly = fmaf(1.061405429f, t, -1.453152027f);
    poly = fmaf(poly, t, 1.421413741f);
    poly = fmaf(poly, t, -0.284496736f);
    poly = fmaf(poly, t, 0.254829592f);
    poly *= t;
    const float e = __builtin_amdgcn_exp2f(-ax * ax * 1.4426950408889634f);
    const float r = fmaf(-poly, e, 1.0f);
    return copysignf(r, x);
}
__device__ __forceinline__ float gelu(float z) { return z * fmaf(0.5f, erf_as(z * 0.70710678118654752f), 0.5f); }
// FP32 -> BF16 bit pattern, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ short to_bf16(float v) { return __builtin_bit_cast(short, (__bf16)v); }
__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * (1.0f + erf_as(z * 0.70710678118654752f)) +
           z * __builtin_amdgcn_exp2f(-0.5f * 1.4426950408889634f * z * z) * 0.39894228040143268f;
}

typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ s16x8 ld8(const short *p) { return *reinterpret_cast<const s16x8 *>(p); }
__device__ __forceinline__ s16x4 half8(s16x8 v, int i) {
    return i ? s16x4{v[4], v[5], v[6], v[7]} : s16x4{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void st4(short *p, s16x4 v) { *reinterpret_cast<s16x4 *>(p) = v; }
__device__ __forceinline__ s16x4 ld4(const short *p) { return *reinterpret_cast<const s16x4 *>(p); }
__device__ __forceinline__ f32x4 mfma(s16x4 a, s16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// BF16 weight copies in fragment order: the A fragments of MFMA step ks of
// the 16-row block hb, 8 bytes per lane (row 16 hb + j, columns 16 ks + 4 g ..
// +3 for lane 16 g + j), two steps per lane side by side, so that a wave's
// load is 1 KiB in a row (row-major weights cost a line per row and load).
// Place of element (row, col) of a matrix with np pairs of steps per block:
__device__ __forceinline__ int frag_at(int row, int col, int np) {
    return (((row >> 4) * np + (col >> 5)) * 64 + ((col >> 2) & 3) * 16 + (row & 15)) * 8 + ((col >> 4) & 1) * 4 +
           (col & 3);
}
// The 16 columns of W3^T (one step per block).
__device__ __forceinline__ int frag16_at(int row, int col) {
    return ((row >> 4) * 64 + (col >> 2) * 16 + (row & 15)) * 4 + (col & 3);
}
// Transposes a wave's 16 x 16 fragment within its quads: lane (g, 4 a + b)
// gives units 4 g .. +3 of row 4 a + b and gets unit 4 g + b of rows 4 a .. +3.
__device__ __forceinline__ s16x4 quad_transpose(s16x4 f, int lane) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = __builtin_bit_cast(u32x2, f);
    auto xor1 = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xb1, 0xf, 0xf, true); };
    auto xor2 = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4e, 0xf, 0xf, true); };
    // pairs: even lanes keep their first unit and take the neighbour's, odd
    // lanes the second (bytes of {other, own})
    const uint32_t sel = lane & 1 ? 0x03020706u : 0x05040100u;
    const uint32_t p = __builtin_amdgcn_perm(xor1(v[0]), v[0], sel), q = __builtin_amdgcn_perm(xor1(v[1]), v[1], sel);
    const bool high = lane & 2;
    const uint32_t o = xor2(high ? p : q);
    return __builtin_bit_cast(s16x4, high ? u32x2{o, q} : u32x2{p, o});
}

// Sum over the 16 lanes of a row (every lane gets it), in the order of a
// butterfly over lane bits 0, 1, 2, 3: quad permutes, then mirrors (all lanes
// of a quad, then of an 8-group, hold the same value).
__device__ __forceinline__ float row_sum16(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                     0xf, 0xf, true));
    };
    v += dpp(v, std::integral_constant<int, 0xb1>{});   // quad_perm 1 0 3 2
    v += dpp(v, std::integral_constant<int, 0x4e>{});   // quad_perm 2 3 0 1
    v += dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
    v += dpp(v, std::integral_constant<int, 0x140>{});  // row_mirror
    return v;
}

// ---- forward + backward of one batch (training and the gradient call) ----
// One workgroup per 16-row tile; wave w owns the hidden blocks 2w and 2w + 1
// (units 32w .. 32w + 31) of both hidden layers.  A layer's MFMA result
// fragments are the next layer's B operand for the same lane, so they pass
// between the waves through LDS as they are (lane l's fragment of block b at
// [b][l]); the input blocks, loaded by the waves in turn, pass the same way.
// The output layer and dY (16 outputs, one block) are computed by every wave
// alike; wave 0 writes them.  With one wave per SIMD nothing hides a load, so
// the weights of every layer (116 registers) are requested at the start.
__global__ __launch_bounds__(256) void k_mlp_fwdbwd(MlpTrainArgs a) {
    constexpr int kKs = kMlpMaxIn / 16;
    __shared__ s16x4 sh_x[kKs][64], sh_h1[8][64], sh_h2[8][64], sh_dz2[8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, j = lane & 15;
    const int wt = blockIdx.x;  // tile
    const int b0 = wt * 16;
    if (b0 >= a.B) return;  // uniform over the workgroup
    const int rb = b0 + j;
    const int nks = a.in_pad / 16, np = (nks + 1) / 2;
    const int32_t *ip = a.idx ? a.idx + rb : nullptr;
    const int32_t iv = ip ? *ip : rb;
    // weight fragments and biases (clamped steps past nks, not used)
    s16x8 w1[2][kKs / 2], w2[2][4], w3[4], w2t[2][4];
    s16x4 w3t[2];
    f32x4 bias1[2], bias2[2];
    float bias3[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int hb = 2 * wave + h;
#pragma unroll
        for (int k = 0; k < kKs / 2; ++k) w1[h][k] = ld8(a.W1f + ((hb * np + (k < np ? k : np - 1)) * 64 + lane) * 8);
#pragma unroll
        for (int k = 0; k < 4; ++k) w2[h][k] = ld8(a.W2f + ((hb * 4 + k) * 64 + lane) * 8);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) w3[k] = ld8(a.W3f + (k * 64 + lane) * 8);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int hb = 2 * wave + h;
        w3t[h] = ld4(a.W3Tf + (hb * 64 + lane) * 4);
#pragma unroll
        for (int k = 0; k < 4; ++k) w2t[h][k] = ld8(a.W2Tf + ((hb * 4 + k) * 64 + lane) * 8);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            bias1[h][r] = a.b1[16 * hb + 4 * g + r];
            bias2[h][r] = a.b2[16 * hb + 4 * g + r];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) bias3[r] = a.b3[4 * g + r < a.out ? 4 * g + r : 0];
    __builtin_amdgcn_sched_barrier(0);  // the weights are requested before the row index is waited for
    int64_t row = iv;
    row = row < 0 ? 0 : (row >= a.n_rows ? a.n_rows - 1 : row);  // memory-safe on bad input
    // inputs: this wave's blocks, four consecutive features per lane (zero
    // past in)
    f32x4 xv[kKs / 4];
#pragma unroll
    for (int q = 0; q < kKs / 4; ++q) {
        const int f0 = 16 * (wave + 4 * q) + 4 * g;
        const float *xr = a.x + row * a.in;
        if (16 * (wave + 4 * q) + 16 <= a.in) {
            __builtin_memcpy(&xv[q], xr + f0, 16);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) xv[q][r] = xr[f0 + r < a.in ? f0 + r : a.in - 1];
        }
    }
    float ell[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * g + r;
        ell[r] = a.ell[row * a.out + (o < a.out ? o : 0)];
    }
    s16x4 xo[kKs / 4];
#pragma unroll
    for (int q = 0; q < kKs / 4; ++q) {
        const int ks = wave + 4 * q;
#pragma unroll
        for (int r = 0; r < 4; ++r) xo[q][r] = to_bf16(16 * ks + 4 * g + r < a.in ? xv[q][r] : 0.0f);
        sh_x[ks][lane] = xo[q];
    }
    __syncthreads();
    // layer 1, own blocks
    s16x4 xb[kKs];
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) xb[ks] = sh_x[ks][lane];
    float z1[2][4], z2[2][4];
    s16x4 h1b[2], h2b[2];
    f32x4 acc1[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks)
        if (ks < nks)
#pragma unroll
            for (int h = 0; h < 2; ++h) acc1[h] = mfma(half8(w1[h][ks / 2], ks & 1), xb[ks], acc1[h]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z1[h][r] = acc1[h][r] + bias1[h][r];
            h1b[h][r] = to_bf16(gelu(z1[h][r]));
        }
        sh_h1[2 * wave + h][lane] = h1b[h];
    }
    __syncthreads();
    // layer 2, own blocks, from every block of layer 1
    f32x4 acc2[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
        const s16x4 hf = sh_h1[kb][lane];
#pragma unroll
        for (int h = 0; h < 2; ++h) acc2[h] = mfma(half8(w2[h][kb / 2], kb & 1), hf, acc2[h]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z2[h][r] = acc2[h][r] + bias2[h][r];
            h2b[h][r] = to_bf16(gelu(z2[h][r]));
        }
        sh_h2[2 * wave + h][lane] = h2b[h];
    }
    __syncthreads();
    // output layer (every wave): y^T = W3 h2^T
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) y = mfma(half8(w3[kb / 2], kb & 1), sh_h2[kb][lane], y);
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] += 4 * g + r < a.out ? bias3[r] : 0.0f;
    // clipped targets t = max(l, max_i l_i - 20); the row max over the four
    // lanes that share row j (lanes j, j+16, j+32, j+48)
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (4 * g + r >= a.out) ell[r] = -INFINITY;
        mx = fmaxf(mx, ell[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float scale = 2.0f / ((float)a.B * (float)a.out);
    float sq = 0.0f;
    float dy[4];
    s16x4 dyb;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * g + r;
        const float t = fmaxf(ell[r], mx - kClipNats);
        const float d = o < a.out ? y[r] - t : 0.0f;
        sq += d * d;
        dy[r] = scale * d;
        dyb[r] = to_bf16(dy[r]);
    }
    // dH2^T = W3^T dY^T (K = 16 outputs), dZ2 = dH2 * GELU'(z2), own blocks
    float dz2[2][4];
    s16x4 dz2b[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const f32x4 acc = mfma(w3t[h], dyb, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dz2[h][r] = acc[r] * gelu_grad(z2[h][r]);
            dz2b[h][r] = to_bf16(dz2[h][r]);
        }
        sh_dz2[2 * wave + h][lane] = dz2b[h];
    }
    __syncthreads();
    // dH1^T = W2^T dZ2^T, dZ1 = dH1 * GELU'(z1), own blocks
    float dz1[2][4];
    f32x4 accd[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
        const s16x4 df = sh_dz2[kb][lane];
#pragma unroll
        for (int h = 0; h < 2; ++h) accd[h] = mfma(half8(w2t[h][kb / 2], kb & 1), df, accd[h]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) dz1[h][r] = accd[h][r] * gelu_grad(z1[h][r]);
    // BF16 stores for the weight-gradient products, [tile][unit][row] (the
    // input blocks split over the waves): 4 rows of a unit per lane
    const int unit = 4 * g + (j & 3), r0 = j & 12;
#pragma unroll
    for (int q = 0; q < kKs / 4; ++q) {
        const int ks = wave + 4 * q;
        if (ks < nks)
            st4(a.Xt + ((int64_t)wt * a.in_pad + 16 * ks + unit) * 16 + r0, quad_transpose(xo[q], lane));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t u = ((int64_t)wt * kMlpHid + 16 * (2 * wave + h) + unit) * 16 + r0;
        s16x4 dz1b;
#pragma unroll
        for (int r = 0; r < 4; ++r) dz1b[r] = to_bf16(dz1[h][r]);
        st4(a.H1t + u, quad_transpose(h1b[h], lane));
        st4(a.H2t + u, quad_transpose(h2b[h], lane));
        st4(a.DZ2t + u, quad_transpose(dz2b[h], lane));
        st4(a.DZ1t + u, quad_transpose(dz1b, lane));
    }
    // bias gradients and squared error of the tile: sums over its 16 rows (FP32)
    float *bg = a.bgrad + (int64_t)wt * kMlpBiasStride;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        f32x4 s1, s2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s1[r] = row_sum16(dz1[h][r]);
            s2[r] = row_sum16(dz2[h][r]);
        }
        if (j == 0) {
            *reinterpret_cast<f32x4 *>(bg + 16 * (2 * wave + h) + 4 * g) = s1;
            *reinterpret_cast<f32x4 *>(bg + kMlpHid + 16 * (2 * wave + h) + 4 * g) = s2;
        }
    }
    if (wave == 0) {
        st4(a.DYt + ((int64_t)wt * kMlpOutPad + unit) * 16 + r0, quad_transpose(dyb, lane));
        f32x4 s3;
#pragma unroll
        for (int r = 0; r < 4; ++r) s3[r] = row_sum16(dy[r]);
        if (j == 0) *reinterpret_cast<f32x4 *>(bg + 2 * kMlpHid + 4 * g) = s3;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) sq += __shfl_xor(sq, off);
        if (lane == 0) a.lossp[wt] = sq;
    }
}

// ---- weight gradients and Adam (or gradient output) ----
// Adam update of parameter p with gradient g from its moments and value (read
// ahead by the caller), and its BF16 working copies.
__device__ __forceinline__ void adam_update(const MlpAdamArgs &a, int64_t p, float gsum, float m0, float v0, float w0) {
    if (a.grad_out) {
        a.grad_out[p] = gsum;
        return;
    }
    const float m = kAdamB1 * m0 + (1.0f - kAdamB1) * gsum;
    const float v = kAdamB2 * v0 + (1.0f - kAdamB2) * gsum * gsum;
    a.m[p] = m;
    a.v[p] = v;
    const float mhat = m / a.bc1, vhat = v / a.bc2;
    const float w = w0 - a.lr * mhat / (sqrtf(vhat) + kAdamEps);
    a.params[p] = w;
    const short wb = to_bf16(w);
    if (p < a.off_b1) {
        const int h = (int)p / a.in, i = (int)p - h * a.in;
        a.W1f[frag_at(h, i, (a.in_pad + 31) / 32)] = wb;
    } else if (p >= a.off_W2 && p < a.off_b2) {
        const int h = (int)((p - a.off_W2) / kMlpHid), k = (int)((p - a.off_W2) % kMlpHid);
        a.W2f[frag_at(h, k, 4)] = wb;
        a.W2Tf[frag_at(k, h, 4)] = wb;
    } else if (p >= a.off_W3 && p < a.off_b3) {
        const int o = (int)((p - a.off_W3) / kMlpHid), h = (int)((p - a.off_W3) % kMlpHid);
        a.W3f[frag_at(o, h, 4)] = wb;
        a.W3Tf[frag16_at(h, o)] = wb;
    }
}

// Sum over the lanes of a wave in a fixed order (butterfly), every lane gets it.
__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// The first workgroups take one 16 x 16 tile of a weight gradient each (tiles of
// one row block of the deltas on one XCD: workgroup w runs on XCD w mod 8).  Wave
// c takes the rows of chunk c (kc chunks, a chain of 16-row products in row
// order); the waves' partial sums meet in LDS and are added in chunk order by the
// thread that then updates the parameter.  The others add the per-tile bias
// gradients, 16 units each, and the last one the loss.
__global__ __launch_bounds__(1024) void k_mlp_grad_adam(MlpAdamArgs a, int wblocks) {
    __shared__ float s_part[16][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)blockIdx.x < wblocks) {
        const int g = lane >> 4, j = lane & 15;
        const int nks = a.in_pad / 16, t1 = 8 * nks, t2 = t1 + 64, tile = blockIdx.x;
        const short *Am, *Bm;
        int hb, ib, ncols, nrows, ua, ub;
        int64_t off;
        if (tile < t1) {          // dW1 = dZ1^T X
            hb = tile % 8; ib = tile / 8; Am = a.DZ1t; Bm = a.Xt; off = 0; ncols = a.in; nrows = kMlpHid;
            ua = kMlpHid; ub = a.in_pad;
        } else if (tile < t2) {   // dW2 = dZ2^T H1
            hb = (tile - t1) % 8; ib = (tile - t1) / 8; Am = a.DZ2t; Bm = a.H1t; off = a.off_W2; ncols = kMlpHid;
            nrows = kMlpHid; ua = kMlpHid; ub = kMlpHid;
        } else {                  // dW3 = dY^T H2
            hb = 0; ib = tile - t2; Am = a.DYt; Bm = a.H2t; off = a.off_W3; ncols = kMlpHid; nrows = a.out;
            ua = kMlpOutPad; ub = kMlpHid;
        }
        // this thread's parameter: row 16 hb + e / 16, column 16 ib + e % 16
        const int e = threadIdx.x, rr = 16 * hb + (e >> 4), cc = 16 * ib + (e & 15);
        const bool mine = e < 256 && rr < nrows && cc < ncols;
        const int64_t p = off + (int64_t)rr * ncols + cc;
        float m0 = 0.0f, v0 = 0.0f, w0 = 0.0f;
        if (mine && !a.grad_out) {
            m0 = a.m[p];
            v0 = a.v[p];
            w0 = a.params[p];
        }
        if (wave < a.kc) {
            const int chunk = a.ntiles / a.kc, k0 = wave * chunk;  // in 16-row tiles
            const short *ar = Am + ((int64_t)k0 * ua + 16 * hb + j) * 16 + 4 * g;
            const short *br = Bm + ((int64_t)k0 * ub + 16 * ib + j) * 16 + 4 * g;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            int k = 0;
            for (; k + 16 <= chunk; k += 16) {
                s16x4 av[16], bv[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    av[u] = ld4(ar + (int64_t)(k + u) * ua * 16);
                    bv[u] = ld4(br + (int64_t)(k + u) * ub * 16);
                }
#pragma unroll
                for (int u = 0; u < 16; ++u) acc = mfma(av[u], bv[u], acc);
            }
#pragma unroll 4
            for (; k < chunk; ++k) acc = mfma(ld4(ar + (int64_t)k * ua * 16), ld4(br + (int64_t)k * ub * 16), acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) s_part[wave][(4 * g + r) * 16 + j] = acc[r];
        }
        __syncthreads();
        if (!mine) return;
        float gsum = 0.0f;
        for (int c = 0; c < a.kc; ++c) gsum += s_part[c][e];
        adam_update(a, p, gsum, m0, v0, w0);
        return;
    }
    // 16 bias units per workgroup: thread (slot, unit) adds every 64th tile's
    // partial from its slot on, then wave w adds the 64 slots of unit w
    const int u0 = ((int)blockIdx.x - wblocks) * 16;
    const int nbias = 2 * kMlpHid + a.out;
    if (u0 >= 2 * kMlpHid + kMlpOutPad) {  // the workgroup past the units: the loss
        if (wave != 0 || !a.loss_out) return;
        float s = 0.0f;
#pragma unroll 4
        for (int t = lane; t < a.ntiles; t += 64) s += a.lossp[t];
        s = wave_sum_f32(s);
        if (lane == 0) *a.loss_out = s / ((float)a.B * (float)a.out);
        return;
    }
    const int u = u0 + wave;
    const bool mine = lane == 0 && u < nbias;
    const int64_t p = u < kMlpHid ? a.off_b1 + u : u < 2 * kMlpHid ? a.off_b2 + (u - kMlpHid) : a.off_b3 + (u - 2 * kMlpHid);
    float m0 = 0.0f, v0 = 0.0f, w0 = 0.0f;
    if (mine && !a.grad_out) {
        m0 = a.m[p];
        v0 = a.v[p];
        w0 = a.params[p];
    }
    const int slot = threadIdx.x >> 4, uu = threadIdx.x & 15;
    float s = 0.0f;
#pragma unroll 4
    for (int t = slot; t < a.ntiles; t += 64) s += a.bgrad[(int64_t)t * kMlpBiasStride + u0 + uu];
    s_part[uu][slot] = s;
    __syncthreads();
    s = wave_sum_f32(s_part[wave][lane]);
    if (mine) adam_update(a, p, s, m0, v0, w0);
}

// ---- exact fallback of the surrogate ----
// Pixels whose two largest surrogate outputs differ by less than `margin`
// nats are listed (list[*count ...]; *count is zero before): each thread
// tests kUncPer pixels, each wave compacts its flags by ballot, and one atomic
// per workgroup (not per wave: returning atomics on one address serialise
// across the chip) reserves the workgroup's slots.  The order of the list
// depends on the schedule; each listed pixel is recomputed on its own, so the
// results do not.
constexpr int kUncPer = 16;
__global__ __launch_bounds__(256) void k_mlp_uncertain(const float *y, int64_t n, int L, float margin,
                                                       int32_t *list, unsigned int *count) {
    __shared__ unsigned int s_wcnt[4], s_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * 256 * kUncPer + threadIdx.x;
    uint64_t ball[kUncPer];
    unsigned int wc = 0;
#pragma unroll
    for (int u = 0; u < kUncPer; ++u) {
        const int64_t i = p0 + (int64_t)u * 256;
        bool flag = false;
        if (i < n) {
            const float *r = y + i * L;
            float t1 = r[0], t2 = -INFINITY;
            for (int l = 1; l < L; ++l) {
                const float v = r[l];
                if (v > t1) {
                    t2 = t1;
                    t1 = v;
                } else if (v > t2) {
                    t2 = v;
                }
            }
            flag = L > 1 && !(t1 - t2 >= margin);  // NaN outputs are listed too
        }
        ball[u] = __ballot(flag);
        wc += (unsigned int)__popcll(ball[u]);
    }
    if (lane == 0) s_wcnt[wave] = wc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned int tot = s_wcnt[0] + s_wcnt[1] + s_wcnt[2] + s_wcnt[3];
        s_base = tot ? atomicAdd(count, tot) : 0u;
    }
    __syncthreads();
    unsigned int off = s_base;
    for (int w = 0; w < wave; ++w) off += s_wcnt[w];
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int u = 0; u < kUncPer; ++u) {
        if ((ball[u] >> lane) & 1ull) list[off + __popcll(ball[u] & lt)] = (int32_t)(p0 + (int64_t)u * 256);
        off += (unsigned int)__popcll(ball[u]);
    }
}

// out[list[i]][l] = ex[i][l] for the m listed rows of L values.
__global__ __launch_bounds__(256) void k_mlp_scatter_rows(const float *ex, const int32_t *list, int64_t m, int L,
                                                          float *out) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= m * L) return;
    const int64_t i = t / L;
    const int l = (int)(t - i * L);
    out[(int64_t)list[i] * L + l] = ex[t];
}

hipError_t launch_mlp_uncertain(const LaunchCtx &lc, const float *y, int64_t n, int L, float margin, int32_t *list,
                                unsigned int *count) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_uncertain, dim3((unsigned)((n + 256 * kUncPer - 1) / (256 * kUncPer))), dim3(256), 0,
                       lc.stream, y, n, L, margin, list, count);
    return hipGetLastError();
}

hipError_t launch_mlp_scatter_rows(const LaunchCtx &lc, const float *ex, const int32_t *list, int64_t m, int L,
                                   float *out) {
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_scatter_rows, dim3((unsigned)((m * L + 255) / 256)), dim3(256), 0, lc.stream, ex, list,
                       m, L, out);
    return hipGetLastError();
}

// BF16 working copies of the master FP32 parameters (padding stays zero).
__global__ __launch_bounds__(256) void k_mlp_convert(MlpAdamArgs a) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= a.P) return;
    const short wb = to_bf16(a.params[p]);
    if (p < a.off_b1) {
        const int h = (int)(p / a.in), i = (int)(p % a.in);
        a.W1f[frag_at(h, i, (a.in_pad + 31) / 32)] = wb;
    } else if (p >= a.off_W2 && p < a.off_b2) {
        const int h = (int)((p - a.off_W2) / kMlpHid), k = (int)((p - a.off_W2) % kMlpHid);
        a.W2f[frag_at(h, k, 4)] = wb;
        a.W2Tf[frag_at(k, h, 4)] = wb;
    } else if (p >= a.off_W3 && p < a.off_b3) {
        const int o = (int)((p - a.off_W3) / kMlpHid), h = (int)((p - a.off_W3) % kMlpHid);
        a.W3f[frag_at(o, h, 4)] = wb;
        a.W3Tf[frag16_at(h, o)] = wb;
    }
}

// ---- inference: persistent workgroups, BF16 weights staged once in LDS ----
// Uses v_mfma_f32_16x16x32_bf16 (K = 32 per instruction).  A layer's result
// holds units 4g..4g+3 of each 16-unit block in lane (g, j); the K = 32 step
// over blocks 2s and 2s+1 takes the B fragment [block 2s units 4g..4g+3,
// block 2s+1 units 4g..4g+3] and the matching weight columns in the same
// (permuted) order, so no data moves between lanes.
//
// The first layer's B fragment of lane (g, j) is features 32 ks + 8 g .. +7 of
// row j, read straight from global memory.  The kernel orders a surrogate
// input [r, g, b, col, row, a_0..a_{k-1}] as [a_0..a_{k-1}, 0 ..., r, g, b,
// col, row] (the five leading features in the last five of the 128 slots;
// the first layer's weight columns are permuted to match when they are staged
// in LDS), so a window below k is two 16-byte loads and the window that holds
// k takes clamped element loads.  Explicit rows x of more than five features
// take the same order, so both forms round alike; narrower rows keep theirs.
// Two 12-wave workgroups per CU (76 VGPRs, six waves per SIMD) hide the
// input loads without a prefetch; the hidden activations are evaluated as
// twice the GELU (gelu2x), 12 VALU instructions each, which is what bounds
// the kernel.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kInfWaves = 12;          // waves per workgroup; two workgroups per CU (weights in LDS twice)
constexpr int kInfBlocksPerCu = 2;
constexpr int kInfNT = 1;              // 16-pixel tiles per wave and round (each weight fragment read feeds kInfNT products)
constexpr int kInfRows = 16 * kInfNT;  // pixels per wave and round
constexpr int kInfIn = 128;            // input features padded to whole K = 32 steps
constexpr int kInfKs = kInfIn / 32;
constexpr int kInfLd = kMlpHid + 8;    // LDS row stride (elements) of the weights

__device__ __forceinline__ f32x4 mfma32(s16x8 a, s16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}
__device__ __forceinline__ s16x8 cat4(s16x4 lo, s16x4 hi) {
    return s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}
// Twice the GELU with the erf approximation above: 2 GELU(z) = z + |z| erf(|z|
// / sqrt 2) = z + |z| (1 - P(t) e^{-z^2/2}), t = 1 / (1 + p |z| / sqrt 2) --
// 12 instructions.  The factor 2 is exact and is undone by halving the next
// layer's (BF16) weights, which is exact too.
__device__ __forceinline__ float gelu2x(float z) {
    const float az = fabsf(z);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, az, 1.0f));
    float q = fmaf(1.061405429f, t, -1.453152027f);
    q = fmaf(q, t, 1.421413741f);
    q = fmaf(q, t, -0.284496736f);
    q = fmaf(q, t, 0.254829592f);
    const float e = __builtin_amdgcn_exp2f((z * z) * (-0.5f * 1.4426950408889634f));
    return fmaf(az, fmaf(-(q * t), e, 1.0f), z);
}
__device__ __forceinline__ short half_bf16(short w) {
    return to_bf16(0.5f * __builtin_bit_cast(float, (uint32_t)(uint16_t)w << 16));
}

__global__ __launch_bounds__(64 * kInfWaves) __attribute__((amdgpu_waves_per_eu(kInfWaves * kInfBlocksPerCu / 4))) void k_mlp_infer(MlpInferArgs a) {
    __shared__ __align__(16) short sW1[kMlpHid * kInfLd];
    __shared__ __align__(16) short sW2[kMlpHid * kInfLd];
    __shared__ __align__(16) short sW3[kMlpOutPad * kInfLd];
    __shared__ __align__(16) float sb[2 * kMlpHid + kMlpOutPad];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;
    // head: the five leading features go to slots kInfIn-5 .. kInfIn-1, the
    // w features after them to slots 0 .. w-1 (source rows of stride ld)
    const bool rows_x = a.x != nullptr;
    const bool head = !rows_x || a.in > 5;
    const int w = rows_x ? (head ? a.in - 5 : a.in) : a.k;
    const int ld = rows_x ? a.in : a.k;
    const float *src0 = rows_x ? a.x + (head ? 5 : 0) : a.alpha;
    for (int e = tid; e < kMlpHid * kInfLd / 8; e += 64 * kInfWaves) *reinterpret_cast<s16x8 *>(sW1 + 8 * e) = s16x8{};
    __syncthreads();
    // 8 weights of a row per lane, in fragment order
    const int np = (a.in_pad + 31) / 32;
    for (int e = tid; e < 8 * np * 64; e += 64 * kInfWaves) {
        const s16x8 v = ld8(a.W1f + 8 * e);
        const int l = e & 63, blk = e >> 6, hb = blk / np, kp = blk - hb * np;
        short *dst = sW1 + (16 * hb + (l & 15)) * kInfLd;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            // kernel feature of network column nc
            const int nc = 32 * kp + 16 * (q >> 2) + 4 * (l >> 4) + (q & 3);
            if (nc < a.in) dst[!head ? nc : nc < 5 ? kInfIn - 5 + nc : nc - 5] = v[q];
        }
    }
    // the hidden layers hold twice their activations (gelu2x): halved weights
    auto stage = [&](short *dst0, const short *src, int blocks) {
        for (int e = tid; e < blocks * 4 * 64; e += 64 * kInfWaves) {
            const s16x8 v = ld8(src + 8 * e);
            const int l = e & 63, blk = e >> 6;
            short *dst = dst0 + (16 * (blk >> 2) + (l & 15)) * kInfLd + 32 * (blk & 3) + 4 * (l >> 4);
#pragma unroll
            for (int q = 0; q < 8; ++q) dst[16 * (q >> 2) + (q & 3)] = half_bf16(v[q]);
        }
    };
    stage(sW2, a.W2f, 8);
    stage(sW3, a.W3f, 1);
    for (int e = tid; e < 2 * kMlpHid + kMlpOutPad; e += 64 * kInfWaves)
        sb[e] = e < kMlpHid ? a.b1[e] : e < 2 * kMlpHid ? a.b2[e - kMlpHid] : (e - 2 * kMlpHid < a.out ? a.b3[e - 2 * kMlpHid] : 0.f);
    __syncthreads();
    const int ks1 = head ? kInfKs : (a.in + 31) / 32;
    const int64_t ngrp = (a.n + kInfRows - 1) / kInfRows;
    const int64_t N = (int64_t)a.H * a.W;
    const float sx = a.W > 1 ? 1.0f / (float)(a.W - 1) : 0.0f, sy = a.H > 1 ? 1.0f / (float)(a.H - 1) : 0.0f;
    // raw inputs of the round: features 32 ks + 8 g .. +7 of row 16 tt + j
    float raw[kInfNT][kInfKs][8];
    // Windows of the K steps below kf lie below w for every lane; the window
    // of step kf may cross w (its elements at or past w become zero).  The
    // source is read through a buffer resource that ends at the round's last
    // valid element, so rows past the end read zero.
    const int kf = w >> 5;
    const int voff = (j * ld + 8 * g) * 4;
    auto fetch = [&](int64_t t) {
        if (t >= ngrp) return;
        const int64_t p0 = t * kInfRows;
        const int rows = (int)(a.n - p0 < kInfRows ? a.n - p0 : kInfRows);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(src0 + p0 * ld), (short)0, ((rows - 1) * ld + w) * 4, 0x00020000);
#pragma unroll
        for (int tt = 0; tt < kInfNT; ++tt) {
            const int vo = voff + 16 * tt * ld * 4;  // the range check covers the vector offset only
#pragma unroll
            for (int ks = 0; ks < kInfKs; ++ks) {
                if (ks < kf) {
                    const f32x4 lo = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo + 128 * ks, 0, 0));
                    const f32x4 hi = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo + 128 * ks + 16, 0, 0));
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        raw[tt][ks][c] = lo[c];
                        raw[tt][ks][4 + c] = hi[c];
                    }
                } else if (ks == kf) {
                    // opaque copies: keeps the compiler from hoisting 8 offsets
                    // and 8 lane masks per K step out of the loop
                    int o = vo + 128 * ks, nv = w - 32 * ks - 8 * g;
                    __asm__ volatile("" : "+v"(o), "+v"(nv));
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        const float v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, o + 4 * c, 0, 0));
                        raw[tt][ks][c] = c < nv ? v : 0.0f;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 8; ++c) raw[tt][ks][c] = 0.0f;
                }
            }
            int64_t row = p0 + 16 * tt + j;
            if (row > a.n - 1) row = a.n - 1;  // rows past the end repeat the last (their outputs are not written)
            if (head) {
                float hv[5];
                if (rows_x) {
#pragma unroll
                    for (int c = 0; c < 5; ++c) hv[c] = a.x[row * a.in + c];
                } else {
                    const int pix = (int)row;  // images hold fewer than 2^31 pixels
                    const int prow = pix / a.W;
                    hv[0] = a.rgb[pix];
                    hv[1] = a.rgb[N + pix];
                    hv[2] = a.rgb[2 * N + pix];
                    hv[3] = (float)(pix - prow * a.W) * sx;
                    hv[4] = (float)prow * sy;
                }
#pragma unroll
                for (int c = 0; c < 5; ++c)
                    if (g == 3) raw[tt][kInfKs - 1][3 + c] = hv[c];
            }
        }
    };
    int64_t t = (int64_t)blockIdx.x * kInfWaves + wave;
    for (; t < ngrp; t += (int64_t)gridDim.x * kInfWaves) {
        const int64_t p0 = t * kInfRows;
        const int np = (int)(a.n - p0 < kInfRows ? a.n - p0 : kInfRows);
        fetch(t);
        s16x8 xb[kInfNT][kInfKs];
#pragma unroll
        for (int tt = 0; tt < kInfNT; ++tt)
#pragma unroll
            for (int ks = 0; ks < kInfKs; ++ks)
#pragma unroll
                for (int c = 0; c < 8; ++c) xb[tt][ks][c] = to_bf16(raw[tt][ks][c]);
        // layer 1 (kernel feature order, natural K: features 32 ks + 8 g .. +7)
        s16x4 h1b[kInfNT][8];
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) {
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(sb + 16 * hb + 4 * g);
            f32x4 acc[kInfNT];
#pragma unroll
            for (int tt = 0; tt < kInfNT; ++tt) acc[tt] = bias;
            const short *wr = sW1 + (16 * hb + j) * kInfLd + 8 * g;
#pragma unroll
            for (int ks = 0; ks < kInfKs; ++ks)
                if (ks < ks1) {
                    const s16x8 wf = *reinterpret_cast<const s16x8 *>(wr + 32 * ks);
#pragma unroll
                    for (int tt = 0; tt < kInfNT; ++tt) acc[tt] = mfma32(wf, xb[tt][ks], acc[tt]);
                }
#pragma unroll
            for (int tt = 0; tt < kInfNT; ++tt)
#pragma unroll
                for (int r = 0; r < 4; ++r) h1b[tt][hb][r] = to_bf16(gelu2x(acc[tt][r]));
            // every block: keeps the weight loads of later blocks from piling
            // up in VGPRs
            __builtin_amdgcn_sched_barrier(0);
        }
        // layer 2 (permuted K order over block pairs)
        s16x4 h2b[kInfNT][8];
#pragma unroll
        for (int hb = 0; hb < 8; ++hb) {
            const f32x4 bias = *reinterpret_cast<const f32x4 *>(sb + kMlpHid + 16 * hb + 4 * g);
            f32x4 acc[kInfNT];
#pragma unroll
            for (int tt = 0; tt < kInfNT; ++tt) acc[tt] = bias;
            const short *wr = sW2 + (16 * hb + j) * kInfLd + 4 * g;
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
                const s16x8 wf = cat4(ld4(wr + 32 * s2), ld4(wr + 32 * s2 + 16));
#pragma unroll
                for (int tt = 0; tt < kInfNT; ++tt)
                    acc[tt] = mfma32(wf, cat4(h1b[tt][2 * s2], h1b[tt][2 * s2 + 1]), acc[tt]);
            }
#pragma unroll
            for (int tt = 0; tt < kInfNT; ++tt)
#pragma unroll
                for (int r = 0; r < 4; ++r) h2b[tt][hb][r] = to_bf16(gelu2x(acc[tt][r]));
            __builtin_amdgcn_sched_barrier(0);
        }
        const f32x4 bias3 = *reinterpret_cast<const f32x4 *>(sb + 2 * kMlpHid + 4 * g);
        f32x4 y[kInfNT];
#pragma unroll
        for (int tt = 0; tt < kInfNT; ++tt) y[tt] = bias3;
        {
            const short *wr = sW3 + j * kInfLd + 4 * g;
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
                const s16x8 wf = cat4(ld4(wr + 32 * s2), ld4(wr + 32 * s2 + 16));
#pragma unroll
                for (int tt = 0; tt < kInfNT; ++tt)
                    y[tt] = mfma32(wf, cat4(h2b[tt][2 * s2], h2b[tt][2 * s2 + 1]), y[tt]);
            }
        }
#pragma unroll
        for (int tt = 0; tt < kInfNT; ++tt)
            if (16 * tt + j < np)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int o = 4 * g + r;
                    if (o < a.out) a.y[(p0 + 16 * tt + j) * a.out + o] = y[tt][r];
                }
    }
}

// Surrogate inputs of listed pixels: [r, g, b, col/(W-1), row/(H-1), a_0..a_{k-1}].
__global__ __launch_bounds__(256) void k_mlp_features(const float *rgb, int H, int W, const float *alpha, int k,
                                                       const int32_t *pix, int64_t n, float *x) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int in = 5 + k;
    if (e >= n * in) return;
    const int64_t r = e / in;
    const int f = (int)(e - r * in);
    const int64_t p = pix[r];
    const int64_t N = (int64_t)H * W;
    float v;
    if (f < 3) v = rgb[f * N + p];
    else if (f == 3) v = W > 1 ? (float)(p % W) * (1.0f / (float)(W - 1)) : 0.0f;
    else if (f == 4) v = H > 1 ? (float)(p / W) * (1.0f / (float)(H - 1)) : 0.0f;
    else v = alpha[p * k + (f - 5)];
    x[e] = v;
}

// Output bias b3_i = mean over the rows of the clipped target
// t_i = max(l_i, max_j l_j - 20), FP64 sums: per workgroup (a thread takes a
// row's every label, so a row is read once; one workgroup per label read every
// row 16 times over, 35 us for 8192 rows), then the workgroups' sums in a
// fixed order.
__global__ __launch_bounds__(256) void k_mlp_target_sums(const float *ell, int64_t n, int out, double *part) {
    __shared__ double red[4][kMlpOutPad];
    double s[kMlpOutPad];
#pragma unroll
    for (int o = 0; o < kMlpOutPad; ++o) s[o] = 0.0;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256) {
        float v[kMlpOutPad];
#pragma unroll
        for (int o = 0; o < kMlpOutPad; ++o) v[o] = ell[r * out + (o < out ? o : 0)];
        float mx = v[0];
#pragma unroll
        for (int o = 1; o < kMlpOutPad; ++o) mx = fmaxf(mx, v[o]);
#pragma unroll
        for (int o = 0; o < kMlpOutPad; ++o) s[o] += (double)fmaxf(v[o], mx - kClipNats);
    }
#pragma unroll
    for (int o = 0; o < kMlpOutPad; ++o) {
        if (o >= out) continue;
        double t = s[o];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][o] = t;
    }
    __syncthreads();
    const int o = threadIdx.x;
    if (o < out) part[(int64_t)o * gridDim.x + blockIdx.x] = ((red[0][o] + red[1][o]) + red[2][o]) + red[3][o];
}
__global__ __launch_bounds__(64) void k_mlp_bias_mean(const double *part, int nparts, int64_t n, float *b3) {
    double s = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 64) s += part[(int64_t)blockIdx.x * nparts + i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (threadIdx.x == 0) b3[blockIdx.x] = (float)(s / (double)n);
}

constexpr int kTargetParts = 256;
static unsigned target_parts(int64_t n) { return (unsigned)(n < 256 * kTargetParts ? (n + 255) / 256 : kTargetParts); }
size_t mlp_bias_mean_bytes(int out) { return sizeof(double) * (size_t)out * kTargetParts; }
hipError_t launch_mlp_bias_mean(const LaunchCtx &lc, const float *ell, int64_t n, int out, double *part, float *b3) {
    const unsigned parts = target_parts(n);
    hipLaunchKernelGGL(k_mlp_target_sums, dim3(parts), dim3(256), 0, lc.stream, ell, n, out, part);
    hipLaunchKernelGGL(k_mlp_bias_mean, dim3((unsigned)out), dim3(64), 0, lc.stream, part, (int)parts, n, b3);
    return hipGetLastError();
}

hipError_t launch_mlp_fwdbwd(const LaunchCtx &lc, const MlpTrainArgs &a) {
    const int tiles = a.B / 16;  // one workgroup per 16-row tile
    hipLaunchKernelGGL(k_mlp_fwdbwd, dim3((unsigned)tiles), dim3(256), 0, lc.stream, a);
    return hipGetLastError();
}
hipError_t launch_mlp_grad_adam(const LaunchCtx &lc, const MlpAdamArgs &a) {
    const int wblocks = 8 * (a.in_pad / 16) + 64 + 8;      // 16 x 16 tiles of the three weight gradients
    const int bblocks = (2 * kMlpHid + kMlpOutPad) / 16 + 1;  // 16 bias units each, then the loss
    hipLaunchKernelGGL(k_mlp_grad_adam, dim3((unsigned)(wblocks + bblocks)), dim3(1024), 0, lc.stream, a, wblocks);
    return hipGetLastError();
}
hipError_t launch_mlp_convert(const LaunchCtx &lc, const MlpAdamArgs &a) {
    hipLaunchKernelGGL(k_mlp_convert, dim3((unsigned)((a.P + 255) / 256)), dim3(256), 0, lc.stream, a);
    return hipGetLastError();
}
hipError_t launch_mlp_infer(const LaunchCtx &lc, const MlpInferArgs &a) {
    const int64_t ngrp = (a.n + kInfRows - 1) / kInfRows;
    int64_t blocks = (int64_t)lc.num_cu * kInfBlocksPerCu;
    if (blocks > (ngrp + kInfWaves - 1) / kInfWaves) blocks = (ngrp + kInfWaves - 1) / kInfWaves;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)blocks), dim3(64 * kInfWaves), 0, lc.stream, a);
    return hipGetLastError();
}
hipError_t launch_mlp_features(const LaunchCtx &lc, const float *rgb, int H, int W, const float *alpha, int k,
                               const int32_t *pix, int64_t n, float *x) {
    const int64_t total = n * (5 + k);
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_features, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, lc.stream, rgb, H, W,
                       alpha, k, pix, n, x);
    return hipGetLastError();
}

}  // namespace cs
