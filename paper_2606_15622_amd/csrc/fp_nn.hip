// fp_nn.hip -- learned closure: BF16 MFMA inference and training of the surrogate MLP.
//
// Network (the surrogate of Sec. "Phase 1-2"/"Phase 3": standardised inputs and
// outputs, dense layers): 32 -> 128 -> 128 -> 128 -> 16 with SiLU; 27 features of the
// theta-normalised moments and 9 normalised coefficients, zero padded.  All products are
// v_mfma_f32_32x32x16_bf16 (BF16 operands, FP32 accumulation).
//
// Operand layouts of the 32x32x16 MFMA (wave64, lane l, half h = l / 32):
//   A (32 x 16):  lane holds A[l % 32][8h + i], i = 0..7
//   B (16 x 32):  lane holds B[8h + i][l % 32]
//   D (32 x 32):  lane holds D[8(j/4) + 4h + j%4][l % 32], j = 0..15
// Inference computes H_out^T = W H_in^T with the batch (cells) along the MFMA columns,
// so a lane keeps one cell through all layers.  The rows of a layer's output that a
// lane holds are exactly the k-slots it must feed into the next layer's B operand once
// the next weight matrix has its columns permuted by
//   pi(16 s + 8 h + i) = 16 s + 8 floor(i/4) + 4 h + i % 4,
// so activations never leave the registers between layers.  The permuted BF16 weights
// are stored fragment-major ([tile][k-step][lane][8]) and live in LDS.
#include "fp_closure_dev.h"
#include "fp_mlp_dev.h"

#include <algorithm>
#include <mutex>
#include <string>

namespace fpg {

constexpr int NF = 32, NH = 128, NO = 16;
constexpr int OFF_W1 = 0, OFF_B1 = 4096, OFF_W2 = 4224, OFF_B2 = 20608, OFF_W3 = 20736,
              OFF_B3 = 37120, OFF_W4 = 37248, OFF_B4 = 39296, OFF_XM = 39312, OFF_XS = 39344,
              OFF_YM = 39376, OFF_YS = 39392, N_PARAMS = 39408, N_TRAIN = 39312;
// BF16 fragment image
constexpr int IMG_L1 = 0, IMG_L2 = 4096, IMG_L3 = 20480, IMG_L4 = 36864, IMG_BF = 40960;
// FP32 section after the image: b1 b2 b3 b4 x_mean x_std y_mean y_std
constexpr int SEC_B1 = 0, SEC_B2 = 128, SEC_B3 = 256, SEC_B4 = 384, SEC_XM = 400, SEC_XS = 432,
              SEC_YM = 464, SEC_YS = 480, SEC_N = 496;

__device__ __forceinline__ int perm_k(int K) {
    const int s = K >> 4, h = (K >> 3) & 1, i = K & 7;
    return 16 * s + 8 * (i >> 2) + 4 * h + (i & 3);
}

// inference: z * sigmoid(z) with the hardware exp2 and reciprocal (about 1 ulp; the
// result is rounded to bfloat16 right after)
__device__ __forceinline__ float silu_fast(float z) {
    constexpr float LOG2E = 1.4426950408889634f;
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-LOG2E * z));
}
// training: a = silu(z) = z / (1 + e^-z) and its derivative d, both from one exponential and
// one reciprocal.  The quotients take Markstein's steps to a correctly rounded division (IBM J.
// Res. Dev. 34, 1990: reciprocal, one Newton step, two residual corrections by fused
// multiply-adds) without scaling extreme operands: the divisor is at least 1, and beyond 2^126
// both results are below 1e-35
__device__ __forceinline__ float quotient(float x, float d, float r) {
    float q = x * r;
    q = __builtin_fmaf(__builtin_fmaf(-d, q, x), r, q);
    q = __builtin_fmaf(__builtin_fmaf(-d, q, x), r, q);
    return __builtin_amdgcn_div_fixupf(q, d, x);   // infinities and NaN
}
__device__ __forceinline__ void silu_and_derivative(float z, float& a, float& d) {
    const float u = 1.0f + __expf(-z);
    float r = __builtin_amdgcn_rcpf(u);
    r = __builtin_fmaf(__builtin_fmaf(-u, r, 1.0f), r, r);
    a = quotient(z, u, r);
    const float s = quotient(1.0f, u, r);
    d = s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------------------
// pack FP32 parameters into the permuted BF16 fragment image + FP32 section
__global__ void nn_pack_kernel(const float* __restrict__ p, __bf16* __restrict__ img,
                               float* __restrict__ sec) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < IMG_BF) {
        int layer, base, ks_n;
        if (t < IMG_L2) { layer = 1; base = IMG_L1; ks_n = 2; }
        else if (t < IMG_L3) { layer = 2; base = IMG_L2; ks_n = 8; }
        else if (t < IMG_L4) { layer = 3; base = IMG_L3; ks_n = 8; }
        else { layer = 4; base = IMG_L4; ks_n = 8; }
        const int e = t - base;
        const int i = e & 7, lane = (e >> 3) & 63, frag = e >> 9;
        const int ks = frag % ks_n, mt = frag / ks_n;
        const int m = mt * 32 + (lane & 31), h = lane >> 5;
        const int K = ks * 16 + 8 * h + i;
        float v = 0.0f;
        if (layer == 1) v = p[OFF_W1 + m * NF + K];
        else if (layer == 2) v = p[OFF_W2 + m * NH + perm_k(K)];
        else if (layer == 3) v = p[OFF_W3 + m * NH + perm_k(K)];
        else v = m < NO ? p[OFF_W4 + m * NH + perm_k(K)] : 0.0f;
        img[t] = (__bf16)v;
    }
    if (t < SEC_N) {
        float v;
        if (t < SEC_B2) v = p[OFF_B1 + t];
        else if (t < SEC_B3) v = p[OFF_B2 + t - SEC_B2];
        else if (t < SEC_B4) v = p[OFF_B3 + t - SEC_B3];
        else if (t < SEC_XM) v = p[OFF_B4 + t - SEC_B4];
        else if (t < SEC_XS) v = p[OFF_XM + t - SEC_XM];
        else if (t < SEC_YM) v = p[OFF_XS + t - SEC_XS];
        else if (t < SEC_YS) v = p[OFF_YM + t - SEC_YM];
        else v = p[OFF_YS + t - SEC_YS];
        sec[t] = v;
    }
}

// features of one cell (FP64 in, FP32 out), index K in 0..31:
// [P/th - I (6), T/th^1.5 (10), R/th^2 - 5 I (6), W/th^2.5 (3), eps_hat, log10 N, 0...]
__device__ __forceinline__ void cell_features(const double* m, double eps_hat, float f[32]) {
    const double th = m[M_TH];
    const double i1 = 1.0 / th, i15 = i1 / sqrt(th), i2 = i1 * i1, i25 = i2 / sqrt(th);
    const double d6[6] = {1, 0, 0, 1, 0, 1};
#pragma unroll
    for (int q = 0; q < 6; ++q) f[q] = (float)(m[M_P + q] * i1 - d6[q]);
#pragma unroll
    for (int q = 0; q < 10; ++q) f[6 + q] = (float)(m[M_T + q] * i15);
#pragma unroll
    for (int q = 0; q < 6; ++q) f[16 + q] = (float)(m[M_R + q] * i2 - 5.0 * d6[q]);
#pragma unroll
    for (int q = 0; q < 3; ++q) f[22 + q] = (float)(m[M_W + q] * i25);
    f[25] = (float)eps_hat;
    f[26] = (float)log10(m[M_N]);
#pragma unroll
    for (int q = 27; q < 32; ++q) f[q] = 0.0f;
}

// the 16 features lane half h feeds into the first layer: f[q] = feature 8h + q (q < 8)
// and 16 + 8h + (q - 8) (q >= 8); the same arithmetic as cell_features, with only the
// moments that half needs loaded (17 of them for h = 0, 11 for h = 1)
__device__ __forceinline__ void half_features(const double* __restrict__ m, int h, double eps_hat,
                                              float f[16]) {
    const double th = m[M_TH];
    const double i1 = 1.0 / th, i15 = i1 / sqrt(th), i2 = i1 * i1, i25 = i2 / sqrt(th);
    // feature K -> (moment index, scale: 0 = 1/th 1 = th^-1.5 2 = th^-2 3 = th^-2.5,
    // offset), for K < 25
    auto fea = [&](int K, bool hi) -> float {
        if (K < 6) return (float)(m[M_P + K] * i1 - ((K == 0 || K == 3 || K == 5) ? 1.0 : 0.0));
        if (K < 16) return (float)(m[M_T + K - 6] * i15);
        if (K < 22) {
            const int q = K - 16;
            return (float)(m[M_R + q] * i2 - ((q == 0 || q == 3 || q == 5) ? 5.0 : 0.0));
        }
        if (K < 25) return (float)(m[M_W + K - 22] * i25);
        if (K == 25) return (float)eps_hat;
        if (K == 26) return hi ? (float)log10(m[M_N]) : 0.0f;
        return 0.0f;
    };
    if (h == 0) {
#pragma unroll
        for (int q = 0; q < 16; ++q) f[q] = fea(q < 8 ? q : 16 + q - 8, false);
    } else {
#pragma unroll
        for (int q = 0; q < 16; ++q) f[q] = fea(q < 8 ? 8 + q : 24 + q - 8, true);
    }
}

// ---------------------------------------------------------------------------------------
// fused inference: standardised outputs y_std[cell][16] (entries 9..15 zero)
// 16 waves per workgroup share one LDS copy of the weights (82 KB: one workgroup per
// CU), i.e. 4 waves per SIMD, so that one wave's SiLU epilogue (VALU) overlaps another's
// MFMAs; every wave keeps at most 128 registers (VGPRs and AGPRs together)
constexpr int NN_BLOCK = 1024;

// Inverted dropout of the hidden activations for the sensitivity probe: activation row u
// of cell k in pass t is kept if word u % 4 of Philox4x32-10 at counter
// (k, t, PURPOSE_DROPOUT, 32 (layer - 1) + u / 4) is at least keep_min (= floor(p 2^32)),
// and then scaled by 1 / (1 - p); no dropout when drop is null.
// DROP: inverted dropout after the SiLU; bit 16 mt + 4 jq + i of keep set <=> the lane's
// output row 32 mt + 8 jq + 4 h + i is kept (and scaled)
template <int KS, bool DROP = false>
__device__ __forceinline__ void nn_layer(const __bf16* __restrict__ img_l, const float* __restrict__ bias,
                                         const bf16x8 (&bin)[8], bf16x8 (&bout)[8], int lane,
                                         uint64_t keep = 0, float scale = 1.0f) {
    const int h = lane >> 5;
    // two of the four 32-row output tiles at a time (32 accumulator registers live)
#pragma unroll
    for (int mp = 0; mp < 4; mp += 2) {
        // accumulators start from the bias: output row u = 32 mt + 8 (j / 4) + 4 h + j % 4,
        // four consecutive rows per 16-byte LDS read
        f32x16 acc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int jq = 0; jq < 4; ++jq) {
                const float4 bq = *(const float4*)(bias + (mp + t) * 32 + 8 * jq + 4 * h);
                acc[t][4 * jq + 0] = bq.x;
                acc[t][4 * jq + 1] = bq.y;
                acc[t][4 * jq + 2] = bq.z;
                acc[t][4 * jq + 3] = bq.w;
            }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const bf16x8 a = *(const bf16x8*)(img_l + (((mp + t) * KS + s) * 64 + lane) * 8);
                acc[t] = mfma32(a, bin[s], acc[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if constexpr (DROP) {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const float a = silu_fast(acc[t][j]);
                    bout[2 * (mp + t) + (j >> 3)][j & 7] =
                        (__bf16)(((keep >> (16 * (mp + t) + j)) & 1) ? a * scale : 0.0f);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    bout[2 * (mp + t) + (j >> 3)][j & 7] = (__bf16)silu_fast(acc[t][j]);
            }
        }
    }
}

__global__ __launch_bounds__(NN_BLOCK) void nn_infer_kernel(int32_t ncell, const double* __restrict__ mom,
                                                             double eps_hat,
                                                             const __bf16* __restrict__ gimg,
                                                             const float* __restrict__ gsec,
                                                             float* __restrict__ yout) {
    __shared__ __attribute__((aligned(16))) __bf16 img[IMG_BF];
    __shared__ __attribute__((aligned(16))) float sec[SEC_N];
    for (int t = threadIdx.x; t < IMG_BF / 8; t += NN_BLOCK)
        ((bf16x8*)img)[t] = ((const bf16x8*)gimg)[t];
    for (int t = threadIdx.x; t < SEC_N; t += NN_BLOCK) sec[t] = gsec[t];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, n = lane & 31;
    const int32_t ntiles = (ncell + 31) / 32;
    // consecutive tiles go to different workgroups: few tiles spread over the CUs before two
    // share one (a tile issues 1622 vector instructions, 8.1 k busy cycles, 960 of them for its
    // SiLU).  The checked closure of 1000 / 40 000 / 200 704 cells takes 17.4 / 24 / 57 us; with 16 consecutive tiles to a workgroup it took 28 / 34 / 65.  At 1e6 cells, where
    // every wave has its 7 or 8 tiles either way, no difference
    for (int32_t tile = blockIdx.x + gridDim.x * wave; tile < ntiles; tile += gridDim.x * (NN_BLOCK / 64)) {
        // the weight fragments are read from LDS inside every tile: keep the compiler from
        // hoisting them out of the loop (80 fragments would not fit in the registers)
        __asm__ volatile("" ::: "memory");
        const int32_t cell = tile * 32 + n;
        const bool valid = cell < ncell;
        float f[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) f[q] = 0.0f;
        if (valid) {
            const double* mr = mom + (int64_t)cell * MOM;
            if (mr[M_N] > 1.0 && mr[M_TH] > 0.0) half_features(mr, h, eps_hat, f);
        }
        bf16x8 b0[8], b1[8];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int K = 16 * s + 8 * h + i;
                b0[s][i] = (__bf16)((f[8 * s + i] - sec[SEC_XM + K]) / sec[SEC_XS + K]);
            }
        nn_layer<2>(img + IMG_L1, sec + SEC_B1, b0, b1, lane);
        nn_layer<8>(img + IMG_L2, sec + SEC_B2, b1, b0, lane);
        nn_layer<8>(img + IMG_L3, sec + SEC_B3, b0, b1, lane);
        f32x16 acc = f32x16{};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const bf16x8 a = *(const bf16x8*)(img + IMG_L4 + (s * 64 + lane) * 8);
            acc = mfma32(a, b1[s], acc);
        }
        // rows 0..3 and 8 live in half 0 (j = 0..3, 4), rows 4..7 in half 1 (j = 0..3)
        float o[9];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float mine = acc[j];
            const float other = __shfl_xor(mine, 32, 64);
            o[j] = mine;
            o[4 + j] = other;
        }
        o[8] = acc[4];
        if (valid && h == 0) {
            float* dst = yout + (int64_t)cell * NO;
#pragma unroll
            for (int q = 0; q < 9; ++q) dst[q] = o[q] + sec[SEC_B4 + q];
#pragma unroll
            for (int q = 9; q < 16; ++q) dst[q] = 0.0f;
        }
    }
}

// ---------------------------------------------------------------------------------------
// coefficient-sensitivity probe (Sec. "Heuristic coefficient-sensitivity probe"): npass
// forward passes with inverted dropout on the three hidden layers; per cell the standard
// deviation (1/npass) over the passes of each de-standardised normalised coefficient, and
// sens[cell] = (|sigma_C| over the six stress coefficients, |sigma_Gamma| over the three
// heat-flux ones); cells without features (N <= 1 or theta <= 0) get zeros.  Each wave
// keeps its 32 cells' inputs and runs every pass; the sums of the deviations from the
// first pass are FP64 (no cancellation).
constexpr int SENS_BLOCK = 512;

__global__ __launch_bounds__(SENS_BLOCK) void nn_sense_kernel(int32_t ncell, const double* __restrict__ mom,
                                                              double eps_hat, const __bf16* __restrict__ gimg,
                                                              const float* __restrict__ gsec, int32_t npass,
                                                              uint64_t seed, uint32_t keep_min, float scale,
                                                              double* __restrict__ sens) {
    __shared__ __attribute__((aligned(16))) __bf16 img[IMG_BF];
    __shared__ __attribute__((aligned(16))) float sec[SEC_N];
    for (int t = threadIdx.x; t < IMG_BF / 8; t += SENS_BLOCK)
        ((bf16x8*)img)[t] = ((const bf16x8*)gimg)[t];
    for (int t = threadIdx.x; t < SEC_N; t += SENS_BLOCK) sec[t] = gsec[t];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, n = lane & 31;
    const int32_t ntiles = (ncell + 31) / 32;
    for (int32_t tile = blockIdx.x * (SENS_BLOCK / 64) + wave; tile < ntiles;
         tile += gridDim.x * (SENS_BLOCK / 64)) {
        __asm__ volatile("" ::: "memory");
        const int32_t cell = tile * 32 + n;
        const bool valid = cell < ncell;
        float f[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) f[q] = 0.0f;
        bool feat = false;
        if (valid) {
            const double* mr = mom + (int64_t)cell * MOM;
            feat = mr[M_N] > 1.0 && mr[M_TH] > 0.0;
            if (feat) half_features(mr, h, eps_hat, f);
        }
        bf16x8 bin[2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int K = 16 * s + 8 * h + i;
                bin[s][i] = (__bf16)((f[8 * s + i] - sec[SEC_XM + K]) / sec[SEC_XS + K]);
            }
        double y0[9], s1[9], s2[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) y0[q] = s1[q] = s2[q] = 0.0;
        for (int32_t t = 0; t < npass; ++t) {
            __asm__ volatile("" ::: "memory");  // keeps the weight reads inside the pass
            bf16x8 b0[8], b1[8];
            b0[0] = bin[0];
            b0[1] = bin[1];
            // masks of the lane's 64 rows of each hidden layer: row 32 mt + 8 jq + 4 h + i
            // of layer l is decided by word i of the draw with sub 32 (l-1) + 8 mt + 2 jq + h
            uint64_t km[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                uint64_t m = 0;
#pragma unroll 1
                for (int g = 0; g < 16; ++g) {
                    const uint4 r = draw(seed, (uint32_t)cell, (uint32_t)t, PURPOSE_DROPOUT,
                                         32u * (uint32_t)l + 2u * (uint32_t)g + (uint32_t)h);
                    const uint64_t b = (uint64_t)(r.x >= keep_min) | ((uint64_t)(r.y >= keep_min) << 1) |
                                       ((uint64_t)(r.z >= keep_min) << 2) |
                                       ((uint64_t)(r.w >= keep_min) << 3);
                    m |= b << (4 * g);
                }
                km[l] = m;
            }
            nn_layer<2, true>(img + IMG_L1, sec + SEC_B1, b0, b1, lane, km[0], scale);
            nn_layer<8, true>(img + IMG_L2, sec + SEC_B2, b1, b0, lane, km[1], scale);
            nn_layer<8, true>(img + IMG_L3, sec + SEC_B3, b0, b1, lane, km[2], scale);
            f32x16 acc = f32x16{};
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const bf16x8 a = *(const bf16x8*)(img + IMG_L4 + (s * 64 + lane) * 8);
                acc = mfma32(a, b1[s], acc);
            }
            float o[9];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float mine = acc[j];
                const float other = __shfl_xor(mine, 32, 64);
                o[j] = mine;
                o[4 + j] = other;
            }
            o[8] = acc[4];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const double y = (double)(o[q] + sec[SEC_B4 + q]) * (double)sec[SEC_YS + q] +
                                 (double)sec[SEC_YM + q];
                if (t == 0) y0[q] = y;
                const double dy = y - y0[q];
                s1[q] += dy;
                s2[q] += dy * dy;
            }
        }
        if (valid && h == 0) {
            double vc = 0.0, vg = 0.0;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const double m = s1[q] / (double)npass;
                const double var = fmax(s2[q] / (double)npass - m * m, 0.0);
                if (q < 6) vc += var;
                else vg += var;
            }
            sens[(int64_t)cell * 2] = feat ? sqrt(vc) : 0.0;
            sens[(int64_t)cell * 2 + 1] = feat ? sqrt(vg) : 0.0;
        }
    }
}

// ---------------------------------------------------------------------------------------
// training: the weights are packed to bfloat16 fragments (forward and transposed), one kernel
// takes tiles of samples through the forward pass, the loss, the backward pass and the
// weight gradients, and one kernel adds the workgroups' partial sums (and applies Adam).
//
// fragments of 64 lanes x 8 values: F1..F4 the forward A operands (rows = output units), T4
// T3 T2 the backward ones (rows = input units, inner dimension = output units)
constexpr int FR_F1 = 0, FR_F2 = 8, FR_F3 = 40, FR_F4 = 72, FR_T4 = 80, FR_T3 = 84, FR_T2 = 116,
              FR_N = 148;
// one workgroup's partial gradient: 40 tiles of 32 x 32 in accumulator order (W2 and W3 16
// each, tile 4 mt + kt; W1 by mt; W4 by kt, its rows 16..31 unused), then b1 b2 b3 b4
constexpr int GT_W2 = 0, GT_W3 = 16, GT_W1 = 32, GT_W4 = 36, GT_N = 40;
constexpr int GROW = GT_N * 1024 + 3 * NH + NO;
constexpr int TRAIN_MAX_WG = 256;   // one workgroup per CU

__global__ __launch_bounds__(64) void nn_train_pack_kernel(const float* __restrict__ p, __bf16* __restrict__ img) {
    const int f = blockIdx.x, lane = threadIdx.x, c = lane & 31, h = lane >> 5;
    bf16x8 v;
    if (f < FR_T4) {
        const bool first = f < FR_F2, last = f >= FR_F4;
        const int ks = first ? 2 : 8, base = first ? FR_F1 : (f < FR_F3 ? FR_F2 : (last ? FR_F4 : FR_F3));
        const int off = first ? OFF_W1 : (f < FR_F3 ? OFF_W2 : (last ? OFF_W4 : OFF_W3));
        const int K = first ? NF : NH, m = ((f - base) / ks) * 32 + c, k0 = ((f - base) % ks) * 16 + 8 * h;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)(last && m >= NO ? 0.0f : p[off + m * K + k0 + i]);
    } else {
        const bool last = f < FR_T3;
        const int ks = last ? 1 : 8, base = last ? FR_T4 : (f < FR_T2 ? FR_T3 : FR_T2);
        const int off = last ? OFF_W4 : (f < FR_T2 ? OFF_W3 : OFF_W2);
        const int k = ((f - base) / ks) * 32 + c, m0 = ((f - base) % ks) * 16 + 8 * h;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)p[off + (m0 + i) * NH + k];
    }
    *(bf16x8*)(img + (f * 64 + lane) * 8) = v;
}

// D tile of the wave's 32 units and 32 samples: A fragments in registers, B from the
// sample-major image
template <int KS>
__device__ __forceinline__ f32x16 tile_product(const bf16x8 (&a)[KS], const __bf16* hin, int stride, int n, int h) {
    f32x16 acc = f32x16{};
#pragma unroll
    for (int s = 0; s < KS; ++s) acc = mfma32(a[s], *(const bf16x8*)(hin + n * stride + 16 * s + 8 * h), acc);
    return acc;
}

template <int CT, int KIND>
struct TrainShared {
    static constexpr int NS = 32 * CT;   // samples of a tile
    // row strides (bfloat16): 16-byte rows that start on different banks
    static constexpr int SI = NF + 8, SH = NH + 8, SO = NO + 8, ST = NS + 8;
    __attribute__((aligned(16))) __bf16 hn[2][NS * SH];    // sample-major: H1 H2 H3, then dZ3 dZ2
    __attribute__((aligned(16))) __bf16 h0n[NS * SI];
    __attribute__((aligned(16))) __bf16 h0t[NF * ST];      // unit-major
    __attribute__((aligned(16))) __bf16 ht[3][NH * ST];    // H1 H2 H3
    __attribute__((aligned(16))) __bf16 dzt[2][NH * ST];   // dZ3, dZ2, dZ1
    // KIND 1: the tile's systems wait in dzt, unused until the backward pass, and here
    static constexpr int SYS_MORE = KIND ? NS * 90 - NH * ST / 2 : 1;
    double sys_more[SYS_MORE];
    __attribute__((aligned(16))) __bf16 dyt[NO * ST];      // dY, rows 9..15 zero
    __attribute__((aligned(16))) __bf16 dyn[NS * SO];
    float yf[NS * 17];                                     // Y, then dY in columns 0..8
    float eh[NS];                                          // feature 25, eps_hat
    __attribute__((aligned(16))) float bias[3 * NH + NO];  // b1 b2 b3 b4
    __attribute__((aligned(16))) float xm[NF], xs[NF];
    float ym[NO], ys[NO];
};

// Forward, loss, backward and weight gradients of B samples, tile by tile.  A workgroup has
// four waves per 32 samples: wave (ct, rt) computes units 32 rt .. of samples 32 ct .. in
// every layer.  Activations pass from layer to layer through LDS (sample-major), stay there
// unit-major for the weight gradients, and the pre-activations' derivatives stay in
// registers; every wave keeps a quarter (CT = 1) or an eighth of the weight gradient's 40
// tiles in accumulators over all of its workgroup's tiles, so that no activation and no
// back-propagated gradient goes to memory.
// Bound by the vector work of the activations (1950 instructions per wave and tile with CT = 2,
// 0.42 of the kernel's time at 200,000 samples, and 2350 with CT = 1, against 66 MFMA), by the
// waits at its barriers and, for a single tile, by the chain of nine dependent phases.  A kernel
// per layer with activations, gradients and FP32 pre-activations in memory, per-lane weight
// conversions and one thread per bias took 1548 us for an Adam step at batch 4096 and 2658 us
// at 200,000 (residual loss); this takes 24.5 and 201 us (the kernel itself 21 and 190).
//   KIND 0: mean over samples of sum_o (y_o - t_o)^2 on standardised targets
//   KIND 1: mean of |A y - b|^2 of the normalised closure system with y the de-standardised
//           output (sys[n] = A row-major (81) then b (9), FP64)
template <int CT, int KIND>
__global__ __launch_bounds__(256 * CT) void nn_train_kernel(int64_t B, const float* __restrict__ p,
                                                            const __bf16* __restrict__ img,
                                                            const float* __restrict__ feats,
                                                            const float* __restrict__ T,
                                                            const double* __restrict__ sys,
                                                            float* __restrict__ part,
                                                            double* __restrict__ lpart) {
    using S = TrainShared<CT, KIND>;
    constexpr int NS = S::NS, BLOCK = 256 * CT, KT = 4 / CT, ITEMS = (NS * 9 + BLOCK - 1) / BLOCK;
    __shared__ S sm;
    int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: fragment bases in SGPRs
    const int rt = wave & 3, ct = wave >> 2;
    int n = ct * 32 + c;
    const double invB = 1.0 / (double)B;
    for (int t = tid; t < NO * S::ST; t += BLOCK) sm.dyt[t] = (__bf16)0.0f;
    for (int t = tid; t < NS * S::SO; t += BLOCK) sm.dyn[t] = (__bf16)0.0f;
    for (int t = tid; t < NH; t += BLOCK) {
        sm.bias[t] = p[OFF_B1 + t];
        sm.bias[NH + t] = p[OFF_B2 + t];
        sm.bias[2 * NH + t] = p[OFF_B3 + t];
    }
    if (tid < NF) {
        sm.xm[tid] = p[OFF_XM + tid];
        sm.xs[tid] = p[OFF_XS + tid];
    }
    if (tid < NO) {
        sm.bias[3 * NH + tid] = p[OFF_B4 + tid];
        sm.ym[tid] = p[OFF_YM + tid];
        sm.ys[tid] = p[OFF_YS + tid];
    }

    // this thread's four inputs of a tile: sample tid / 8, features 4 (tid % 8) .. (samples
    // from B on read the last one's; their output gradients are zero)
    float fx[4];
    auto load_inputs = [&](int64_t n0) {
        const float* f = feats + min(n0 + (tid >> 3), B - 1) * NF + (tid & 7) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) fx[e] = f[e];
    };
    f32x16 g2[KT], g3[KT], gx[2 / CT];   // gx: W1 tile rt and W4 tile rt (CT = 1), else one of them
#pragma unroll
    for (int t = 0; t < KT; ++t) g2[t] = g3[t] = f32x16{};
#pragma unroll
    for (int t = 0; t < 2 / CT; ++t) gx[t] = f32x16{};
    float bs[3] = {0.0f, 0.0f, 0.0f};   // bias gradients: the lane's unit row_sums() names
    float b4 = 0.0f;
    double loss = 0.0;

    // acc += dZ^T H over the tile's samples: the lane's row of a and column of b (unit-major)
    auto wgrad = [&](f32x16& acc, const __bf16* a, int row, const __bf16* b, int col) {
#pragma unroll
        for (int s = 0; s < 2 * CT; ++s)
            acc = mfma32(*(const bf16x8*)(a + row * S::ST + 16 * s + 8 * h),
                         *(const bf16x8*)(b + col * S::ST + 16 * s + 8 * h), acc);
    };
    // hidden layer: activation to both images, derivative kept
    auto activate = [&](const f32x16& acc, const float* bias, float (&d)[16], __bf16* hs, __bf16* hu) {
        float a[16];
#pragma unroll
        for (int jq = 0; jq < 4; ++jq) {
            const float4 b = *(const float4*)(bias + rt * 32 + 8 * jq + 4 * h);
            const float bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float z = acc[4 * jq + e] + bb[e];
                silu_and_derivative(z, a[4 * jq + e], d[4 * jq + e]);
                // computed here, not put off to the backward pass with its operands kept
                __asm__ volatile("" : "+v"(d[4 * jq + e]));
            }
        }
        put_tile<true>(hs, S::SH, hu, S::ST, n, rt * 32, h, a);
    };
    auto backward = [&](auto inner, const f32x16& acc, const float (&d)[16], float& b, __bf16* zs, __bf16* zu) {
        float dz[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            dz[j] = acc[j] * d[j];
        }
        b += row_sums(dz, lane);
        put_tile<decltype(inner)::value>(zs, S::SH, zu, S::ST, n, rt * 32, h, dz);
    };

    const int64_t tiles = (B + NS - 1) / NS;
    lds_barrier();
    load_inputs((int64_t)blockIdx.x * NS);
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t n0 = tile * NS;
        // the weight fragments are read in every tile: not hoisted out of the loop (they
        // would not fit in the registers)
        __asm__ volatile("" ::: "memory");
        // and neither are the LDS addresses (a register each; spilled, they would be reloaded
        // one wait at a time): the lane numbers they come from look new in every tile
        __asm__ volatile("" : "+v"(tid), "+v"(lane), "+v"(h), "+v"(c), "+v"(n));
        bf16x8 w1[2], w[8], t4[1];
        load_frags<2>(img, FR_F1 + rt * 2, lane, w1);
        {
            const int in_n = tid >> 3, in_k = (tid & 7) * 4;
            const float4 m4 = *(const float4*)(sm.xm + in_k), s4 = *(const float4*)(sm.xs + in_k);
            const float xm[4] = {m4.x, m4.y, m4.z, m4.w}, xs[4] = {s4.x, s4.y, s4.z, s4.w};
            bf16x4 q;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                q[e] = (__bf16)((fx[e] - xm[e]) / xs[e]);
                sm.h0t[(in_k + e) * S::ST + in_n] = q[e];
            }
            *(bf16x4*)(sm.h0n + in_n * S::SI + in_k) = q;
            if (KIND == 1 && in_k == 24) sm.eh[in_n] = fx[1];
        }
        // item it of the loss: sample it / 9 of the tile, output it % 9
        float tv[ITEMS];
        if constexpr (KIND == 0) {
#pragma unroll
            for (int u = 0; u < ITEMS; ++u) {
                const int it = min(tid + u * BLOCK, NS * 9 - 1), i = it / 9;
                tv[u] = T[min(n0 + i, B - 1) * NO + (it - 9 * i)];
            }
        }
        // the tile's systems (read once, in order): to LDS while the first layers run
        constexpr int SQ = KIND ? (NS * 90 + BLOCK - 1) / BLOCK : 1;
        double sq[SQ];
        if constexpr (KIND == 1) {
#pragma unroll
            for (int u = 0; u < SQ; ++u) sq[u] = sys[min(n0 * 90 + tid + u * BLOCK, B * 90 - 1)];
        }
        double* const systems = (double*)sm.dzt[0];   // [sample][90], on into sys_more
        lds_barrier();
        float d1[16], d2[16], d3[16];
        // each layer's fragments are loaded while the layer before it goes through its
        // activations (some 2000 cycles of vector work)
        f32x16 acc = tile_product<2>(w1, sm.h0n, S::SI, n, h);
        load_frags<8>(img, FR_F2 + rt * 8, lane, w);
        activate(acc, sm.bias, d1, sm.hn[0], sm.ht[0]);
        lds_barrier();
        acc = tile_product<8>(w, sm.hn[0], S::SH, n, h);
        load_frags<8>(img, FR_F3 + rt * 8, lane, w);
        activate(acc, sm.bias + NH, d2, sm.hn[1], sm.ht[1]);
        if constexpr (KIND == 1) {
#pragma unroll
            for (int u = 0; u < SQ; ++u)
                if (tid + u * BLOCK < NS * 90) systems[tid + u * BLOCK] = sq[u];
        }
        lds_barrier();
        acc = tile_product<8>(w, sm.hn[1], S::SH, n, h);
        if (rt == 0) load_frags<8>(img, FR_F4, lane, w);
        activate(acc, sm.bias + 2 * NH, d3, sm.hn[0], sm.ht[2]);
        lds_barrier();
        if (rt == 0) {
            acc = tile_product<8>(w, sm.hn[0], S::SH, n, h);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int o = 8 * (j >> 2) + 4 * h + (j & 3);
                sm.yf[n * 17 + o] = acc[j] + sm.bias[3 * NH + o];
            }
        }
        load_frags<1>(img, FR_T4 + rt, lane, t4);
        load_frags<8>(img, FR_T3 + rt * 8, lane, w);
        lds_barrier();
        // loss and dL/dY
        auto put_dy = [&](int i, int o, float d) {
            sm.yf[i * 17 + o] = d;
            sm.dyn[i * S::SO + o] = (__bf16)d;
            sm.dyt[o * S::ST + i] = (__bf16)d;
        };
        if constexpr (KIND == 0) {
#pragma unroll
            for (int u = 0; u < ITEMS; ++u) {
                const int it = tid + u * BLOCK, i = it / 9, o = it - 9 * i;
                if (it >= NS * 9) continue;
                float d = 0.0f;
                if (n0 + i < B) {
                    const double t = ((double)tv[u] - sm.ym[o]) / sm.ys[o];
                    const double e = (double)sm.yf[i * 17 + o] - t;
                    loss += e * e;
                    d = (float)(2.0 * e * invB);
                }
                put_dy(i, o, d);
            }
        } else {
            // r = A y - b a row per thread, then dL/dy = 2 A^T r a column per thread (a
            // partial last round only in its waves)
            double* rr = (double*)sm.hn[1];
#pragma unroll
            for (int u = 0; u < ITEMS; ++u) {
                const int it = tid + u * BLOCK, i = it / 9, o = it - 9 * i;
                if (it >= NS * 9 || n0 + i >= B) continue;
                const double e5 = 5.0 * (double)sm.eh[i];
                const double* A = systems + i * 90;
                double t = -A[81 + o];
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    double y = (double)sm.yf[i * 17 + k] * sm.ys[k] + sm.ym[k];
                    if (k == 0 || k == 3 || k == 5) y += e5;
                    t = fma(A[o * 9 + k], y, t);
                }
                rr[it] = t;
                loss += t * t;
            }
            lds_barrier();
#pragma unroll
            for (int u = 0; u < ITEMS; ++u) {
                const int it = tid + u * BLOCK, i = it / 9, o = it - 9 * i;
                if (it >= NS * 9) continue;
                float d = 0.0f;
                if (n0 + i < B) {
                    const double* A = systems + i * 90;
                    double g = 0.0;
#pragma unroll
                    for (int k = 0; k < 9; ++k) g = fma(A[k * 9 + o], rr[9 * i + k], g);
                    d = (float)(2.0 * g * invB * sm.ys[o]);
                }
                put_dy(i, o, d);
            }
        }
        lds_barrier();
        backward(std::true_type{}, tile_product<1>(t4, sm.dyn, S::SO, n, h), d3, bs[2], sm.hn[1], sm.dzt[0]);
        if (wave == 0) {
            // the output bias: lane = output + 16 x quarter of the tile's samples
#pragma unroll
            for (int i = 0; i < NS / 4; ++i) b4 += sm.yf[((lane >> 4) * (NS / 4) + i) * 17 + (lane & 15)];
        }
        load_inputs((tile + gridDim.x) * NS);
        lds_barrier();
        acc = tile_product<8>(w, sm.hn[1], S::SH, n, h);
        load_frags<8>(img, FR_T2 + rt * 8, lane, w);
        backward(std::true_type{}, acc, d2, bs[1], sm.hn[0], sm.dzt[1]);
        if (CT == 1 || ct == 1) wgrad(gx[2 / CT - 1], sm.dyt, c & 15, sm.ht[2], rt * 32 + c);
#pragma unroll
        for (int t = 0; t < KT; ++t) wgrad(g3[t], sm.dzt[0], rt * 32 + c, sm.ht[1], (ct * KT + t) * 32 + c);
        lds_barrier();
        backward(std::false_type{}, tile_product<8>(w, sm.hn[0], S::SH, n, h), d1, bs[0], (__bf16*)nullptr, sm.dzt[0]);
#pragma unroll
        for (int t = 0; t < KT; ++t) wgrad(g2[t], sm.dzt[1], rt * 32 + c, sm.ht[0], (ct * KT + t) * 32 + c);
        lds_barrier();
        if (CT == 1 || ct == 0) wgrad(gx[0], sm.dzt[0], rt * 32 + c, sm.h0t, c);
        lds_barrier();
    }

    float* out = part + (int64_t)blockIdx.x * GROW;
    auto put_tile = [&](int t, const f32x16& g) {
#pragma unroll
        for (int jq = 0; jq < 4; ++jq)
            *(float4*)(out + t * 1024 + jq * 256 + lane * 4) =
                make_float4(g[4 * jq], g[4 * jq + 1], g[4 * jq + 2], g[4 * jq + 3]);
    };
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        put_tile(GT_W2 + rt * 4 + ct * KT + t, g2[t]);
        put_tile(GT_W3 + rt * 4 + ct * KT + t, g3[t]);
    }
    if (CT == 1) {
        put_tile(GT_W1 + rt, gx[0]);
        put_tile(GT_W4 + rt, gx[2 / CT - 1]);
    } else {
        put_tile((ct == 0 ? GT_W1 : GT_W4) + rt, gx[0]);
    }
    // biases: over the wave's 32 samples, then the waves of the same units; loss: over all
    float* bl = sm.yf;
    if (!(lane & 16)) {
        const int j = lane & 15;
#pragma unroll
        for (int l = 0; l < 3; ++l) bl[ct * 3 * NH + l * NH + rt * 32 + 8 * (j >> 2) + 4 * h + (j & 3)] = bs[l];
    }
    double* ll = (double*)sm.dzt[1];
    ll[tid] = loss;
    b4 += __shfl_xor(b4, 16, 64);
    b4 += __shfl_xor(b4, 32, 64);
    lds_barrier();
    for (int t = tid; t < 3 * NH; t += BLOCK) out[GT_N * 1024 + t] = CT == 1 ? bl[t] : bl[t] + bl[3 * NH + t];
    if (tid < NO) out[GT_N * 1024 + 3 * NH + tid] = tid < 9 ? b4 : 0.0f;
    for (int s = BLOCK / 2; s > 0; s >>= 1) {
        if (tid < s) ll[tid] += ll[tid + s];
        lds_barrier();
    }
    if (tid == 0) lpart[blockIdx.x] = ll[0];
}

// grad = the workgroups' partial sums added in order (16 ranges of rows by 16 waves, then the
// ranges), a float4 of four values per lane; with ADAM the parameters are updated as well.
// The last workgroup adds the loss.
constexpr int RED_R = 16, RED_BLOCK = 64 * RED_R;
template <bool ADAM>
__global__ __launch_bounds__(RED_BLOCK) void nn_reduce_kernel(int rows, const float* __restrict__ part,
                                                              const double* __restrict__ lpart, int64_t B,
                                                              float* __restrict__ grad, float* __restrict__ loss,
                                                              AdamArgs ad) {
    const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x >= 64) return;
        double s = 0.0;
        for (int i = lane; i < rows; i += 64) s += lpart[i];
        s = group_sum<64>(s);
        if (lane == 0) *loss = (float)(s / (double)B);
        return;
    }
    __shared__ float4 red[RED_R][64];
    const int f4 = blockIdx.x * 64 + lane;
    const bool in = f4 < GROW / 4;
    // parameter of the lane's first value, the stride to the next ones, and whether they exist
    int q, st = 1;
    bool live = in;
    if (f4 < GT_N * 256) {
        const int t = f4 >> 8, row = 8 * ((f4 >> 6) & 3) + 4 * (lane >> 5), col = lane & 31;
        st = NH;
        if (t < GT_W1) q = (t < GT_W3 ? OFF_W2 : OFF_W3) + (((t & 15) >> 2) * 32 + row) * NH + (t & 3) * 32 + col;
        else if (t < GT_W4) q = OFF_W1 + ((t - GT_W1) * 32 + row) * (st = NF) + col;
        else {
            q = OFF_W4 + row * NH + (t - GT_W4) * 32 + col;
            live = row < NO;
        }
    } else {
        const int i = (f4 - GT_N * 256) * 4;
        q = i < NH ? OFF_B1 + i : (i < 2 * NH ? OFF_B2 + i - NH : (i < 3 * NH ? OFF_B3 + i - 2 * NH : OFF_B4 + i - 3 * NH));
    }
    float pq[4], mq[4], vq[4];
    if (ADAM && r == 0 && live) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pq[e] = ad.p[q + e * st];
            mq[e] = ad.m[q + e * st];
            vq[e] = ad.v[q + e * st];
        }
    }
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (in) {
        const int r1 = (r + 1) * rows / RED_R;
#pragma unroll 8
        for (int i = r * rows / RED_R; i < r1; ++i) {
            const float4 v = *(const float4*)(part + (int64_t)i * GROW + f4 * 4);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
    }
    red[r][lane] = s;
    __syncthreads();
    if (r != 0 || !live) return;
#pragma unroll
    for (int i = 1; i < RED_R; ++i) {
        const float4 v = red[i][lane];
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    }
    const float g[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        grad[q + e * st] = g[e];
        if (ADAM) adam_one(ad, q + e * st, g[e], mq[e], vq[e], pq[e]);
    }
}

__global__ void nn_adam_kernel(AdamArgs a, const float* __restrict__ g) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < N_TRAIN) adam_one(a, q, g[q], a.m[q], a.v[q], a.p[q]);
}

// features of a batch of moment records (raw, unstandardised) for training
__global__ void nn_features_kernel(int64_t n, const double* __restrict__ mom, double eps_hat,
                                   float* __restrict__ feats) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    double m[31];
#pragma unroll
    for (int i = 0; i < 31; ++i) m[i] = mom[c * MOM + i];
    float f[32];
    cell_features(m, eps_hat, f);
#pragma unroll
    for (int q = 0; q < 32; ++q) feats[c * NF + q] = f[q];
}

// normalised targets of a batch of update records
__global__ void nn_targets_kernel(int64_t n, const double* __restrict__ rec, double eps_hat,
                                  float* __restrict__ tg) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const double* r = rec + c * REC;
    const double tau = r[R_TAU], sth = sqrt(r[R_TH]);
    const double d6[6] = {1, 0, 0, 1, 0, 1};
#pragma unroll
    for (int q = 0; q < 6; ++q) tg[c * NO + q] = (float)(r[R_C + q] * tau - 5.0 * eps_hat * d6[q]);
#pragma unroll
    for (int q = 0; q < 3; ++q) tg[c * NO + 6 + q] = (float)(r[R_G + q] * tau * sth);
#pragma unroll
    for (int q = 9; q < NO; ++q) tg[c * NO + q] = 0.0f;
}

// normalised closure system (A row-major, then b) of a batch of moment records
__global__ void nn_system_kernel(int64_t n, const double* __restrict__ mom, double eps_hat,
                                 double* __restrict__ sys) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    double m[31];
#pragma unroll
    for (int i = 0; i < 31; ++i) m[i] = mom[c * MOM + i];
    CellSystem s;
    build_system(m, eps_hat, s);
    double* d = sys + c * 90;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
#pragma unroll
        for (int k = 0; k < 9; ++k) d[i * 9 + k] = s.a[i][k];
        d[81 + i] = s.a[i][9];
    }
}

}  // namespace fpg

// =========================================================================================
using namespace fpg;

struct fp_nn {
    fp_ctx* ctx = nullptr;
    int64_t max_batch = 0;
    __bf16* img = nullptr;
    float* sec = nullptr;
    float* ybuf = nullptr;   // [ncell][16] standardised outputs of the last inference
    // training scratch: weight fragments, partial gradients and losses of the workgroups
    __bf16* timg = nullptr;
    float *part = nullptr, *grad = nullptr;
    double* lpart = nullptr;
};

template <typename T>
static bool nalloc(T** p, size_t count) {
    return hipMalloc((void**)p, sizeof(T) * (count ? count : 1)) == hipSuccess;
}

// ---- scratch of fp_closure_nn_noalloc --------------------------------------------------
// The standardised network outputs pass from the network kernel to the check kernel through
// this file-scope array instead of the handle's buffer: every GPU the library runs on holds
// one copy of FP_NN_NOALLOC_CELLS x 16 floats (16 MiB) until the process ends.  In host code
// the name `scratch` is a host-side stand-in, not a device address: fp_nn_create looks up
// the address of the current device's copy once per device (hipGetSymbolAddress) and keeps
// it in scratch_dev[device]; host code uses only that pointer.
static __device__ __align__(256) float scratch[(size_t)FP_NN_NOALLOC_CELLS * NO];
constexpr int SCRATCH_DEVICES = 64;
static std::mutex scratch_mu;
static float* scratch_dev[SCRATCH_DEVICES] = {};

// With the context's device current: look up that device's copy of the array once.
static int scratch_setup(fp_ctx* c) {
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (c->device < 0 || c->device >= SCRATCH_DEVICES) return FP_EINVAL;
    if (scratch_dev[c->device]) return FP_OK;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return FP_EDEVICE;
    scratch_dev[c->device] = (float*)ptr;
    return FP_OK;
}

static float* scratch_of(const fp_ctx* c) {
    std::lock_guard<std::mutex> lock(scratch_mu);
    return (c->device >= 0 && c->device < SCRATCH_DEVICES) ? scratch_dev[c->device] : nullptr;
}

extern "C" int fp_nn_create(fp_ctx* c, int64_t max_batch, fp_nn** out) {
    if (!c || !out || max_batch < 0 || max_batch > ((int64_t)1 << 26)) return FP_EINVAL;
    *out = nullptr;
    {
        int cur = -1;
        if (hipGetDevice(&cur) != hipSuccess) return set_err(c, FP_EDEVICE, "fp_nn_create: hipGetDevice failed");
        if (cur != c->device && hipSetDevice(c->device) != hipSuccess)
            return set_err(c, FP_EDEVICE, "fp_nn_create: hipSetDevice failed");
        const int rc = scratch_setup(c);
        if (cur != c->device) (void)hipSetDevice(cur);
        if (rc) return set_err(c, rc, "fp_nn_create: no address for the no-allocation scratch");
    }
    fp_nn* n = new (std::nothrow) fp_nn();
    if (!n) return FP_ENOMEM;
    n->ctx = c;
    n->max_batch = max_batch;
    // the most workgroups of any batch up to max_batch
    const size_t rows = (size_t)std::min<int64_t>(TRAIN_MAX_WG, (max_batch + 31) / 32);
    bool ok = nalloc(&n->img, IMG_BF) && nalloc(&n->sec, SEC_N) && nalloc(&n->ybuf, (size_t)c->ncell * NO);
    if (ok && max_batch > 0)
        ok = nalloc(&n->timg, FR_N * 512) && nalloc(&n->part, rows * GROW) && nalloc(&n->grad, N_PARAMS) &&
             nalloc(&n->lpart, rows);
    if (!ok) {
        fp_nn_destroy(n);
        return FP_ENOMEM;
    }
    *out = n;
    return FP_OK;
}

extern "C" void fp_nn_destroy(fp_nn* n) {
    if (!n) return;
    (void)hipDeviceSynchronize();
    for (void* p : {(void*)n->img, (void*)n->sec, (void*)n->ybuf, (void*)n->timg, (void*)n->part, (void*)n->grad,
                    (void*)n->lpart})
        (void)hipFree(p);
    delete n;
}

extern "C" int fp_nn_load(fp_ctx* c, fp_nn* n, const float* params, hipStream_t s) {
    if (!c || !n || !params || n->ctx != c) return set_err(c, FP_EINVAL, "fp_nn_load: bad argument");
    hipLaunchKernelGGL(nn_pack_kernel, dim3((IMG_BF + 255) / 256), dim3(256), 0, s, params, n->img,
                       n->sec);
    return check_launch(c, "fp_nn_load");
}

namespace fpg {
int launch_closure_nn(fp_ctx* c, const float* ynn, const float* ysec, double tol_abs,
                      double tol_rel, double relax, const double* mom, double* rec, int32_t* status,
                      hipStream_t s);
}

// network kernel into ybuf ([ncell][16] floats), then the check / de-normalisation kernel
static int closure_nn(fp_ctx* c, const fp_nn* n, const double* mom, double* rec, int32_t* status,
                      double tol_abs, double tol_rel, double relax, float* ybuf, const char* what,
                      hipStream_t s) {
    if (!c || !n || !mom || !rec || !status || n->ctx != c || !(tol_abs >= 0) || !(tol_rel >= 0) ||
        !(relax > 0.0 && relax <= 1.0))
        return set_err(c, FP_EINVAL, std::string(what) + ": bad argument");
    if (c->cfg.moment_order == 3 && tol_abs != INFINITY)
        return set_err(c, FP_EINVAL, std::string(what) + ": the check needs moments through fifth order");
    const int32_t ntiles = (c->ncell + 31) / 32;
    const int grid = std::min(ntiles, 256);   // one workgroup per CU, each loops over its tiles
    hipLaunchKernelGGL(nn_infer_kernel, dim3(grid), dim3(NN_BLOCK), 0, s, c->ncell, mom,
                       c->cfg.eps_hat, (const __bf16*)n->img, (const float*)n->sec, ybuf);
    int rc = check_launch(c, what);
    if (rc) return rc;
    return launch_closure_nn(c, ybuf, n->sec + SEC_YM, tol_abs, tol_rel, relax, mom, rec, status, s);
}

extern "C" int fp_closure_nn(fp_ctx* c, const fp_nn* n, const double* mom, double* rec,
                             int32_t* status, double tol_abs, double tol_rel, double relax,
                             hipStream_t s) {
    if (!c || !n) return set_err(c, FP_EINVAL, "fp_closure_nn: bad argument");
    return closure_nn(c, n, mom, rec, status, tol_abs, tol_rel, relax, n->ybuf, "fp_closure_nn", s);
}

extern "C" int fp_closure_nn_noalloc(fp_ctx* c, const fp_nn* n, const double* mom, double* rec,
                                     int32_t* status, double tol_abs, double tol_rel, double relax,
                                     hipStream_t s) {
    if (!c || !n) return set_err(c, FP_EINVAL, "fp_closure_nn_noalloc: bad argument");
    if (c->ncell > FP_NN_NOALLOC_CELLS)
        return set_err(c, FP_EINVAL, "fp_closure_nn_noalloc: more cells than FP_NN_NOALLOC_CELLS (" +
                                         std::to_string(c->ncell) + " > " +
                                         std::to_string(FP_NN_NOALLOC_CELLS) + ")");
    float* y = scratch_of(c);
    if (!y) return set_err(c, FP_EINVAL, "fp_closure_nn_noalloc: no scratch on this device");
    return closure_nn(c, n, mom, rec, status, tol_abs, tol_rel, relax, y, "fp_closure_nn_noalloc", s);
}

extern "C" int fp_nn_infer(fp_ctx* c, const fp_nn* n, const double* mom, float* y, hipStream_t s) {
    if (!c || !n || !mom || !y || n->ctx != c) return set_err(c, FP_EINVAL, "fp_nn_infer: bad argument");
    if (c->ncell == 0) return FP_OK;
    const int32_t ntiles = (c->ncell + 31) / 32;
    const int grid = std::min(ntiles, 256);
    hipLaunchKernelGGL(nn_infer_kernel, dim3(grid), dim3(NN_BLOCK), 0, s, c->ncell, mom, c->cfg.eps_hat,
                       (const __bf16*)n->img, (const float*)n->sec, y);
    return check_launch(c, "fp_nn_infer");
}

extern "C" int fp_nn_sensitivity(fp_ctx* c, const fp_nn* n, const double* mom, int32_t npass,
                                 double p, uint64_t seed, double* sens, hipStream_t s) {
    if (!c || !n || !mom || !sens || n->ctx != c || npass < 1 || !(p >= 0.0 && p < 1.0))
        return set_err(c, FP_EINVAL, "fp_nn_sensitivity: bad argument");
    const int32_t ntiles = (c->ncell + 31) / 32;
    int grid = (ntiles + SENS_BLOCK / 64 - 1) / (SENS_BLOCK / 64);
    if (grid > 512) grid = 512;
    const uint32_t keep_min = (uint32_t)std::floor(p * 4294967296.0);
    hipLaunchKernelGGL(nn_sense_kernel, dim3(grid), dim3(SENS_BLOCK), 0, s, c->ncell, mom,
                       c->cfg.eps_hat, (const __bf16*)n->img, (const float*)n->sec, npass, seed,
                       keep_min, (float)(1.0 / (1.0 - p)), sens);
    return check_launch(c, "fp_nn_sensitivity");
}

extern "C" int fp_nn_outputs(fp_ctx* c, const fp_nn* n, float* y, hipStream_t s) {
    if (!c || !n || !y) return set_err(c, FP_EINVAL, "fp_nn_outputs: bad argument");
    if (hipMemcpyAsync(y, n->ybuf, sizeof(float) * (size_t)c->ncell * NO, hipMemcpyDeviceToDevice,
                       s) != hipSuccess)
        return set_err(c, FP_EDEVICE, "fp_nn_outputs: copy failed");
    return FP_OK;
}

extern "C" int fp_nn_features(fp_ctx* c, const double* mom, int64_t n, float* feats, hipStream_t s) {
    if (!c || !mom || !feats || n < 0) return set_err(c, FP_EINVAL, "fp_nn_features: bad argument");
    if (n == 0) return FP_OK;
    hipLaunchKernelGGL(nn_features_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, mom,
                       c->cfg.eps_hat, feats);
    return check_launch(c, "fp_nn_features");
}

extern "C" int fp_nn_targets(fp_ctx* c, const double* rec, int64_t n, float* targets, hipStream_t s) {
    if (!c || !rec || !targets || n < 0) return set_err(c, FP_EINVAL, "fp_nn_targets: bad argument");
    if (n == 0) return FP_OK;
    hipLaunchKernelGGL(nn_targets_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, rec,
                       c->cfg.eps_hat, targets);
    return check_launch(c, "fp_nn_targets");
}

extern "C" int fp_closure_build(fp_ctx* c, const double* mom, int64_t n, double* sys, hipStream_t s) {
    if (!c || !mom || !sys || n < 0) return set_err(c, FP_EINVAL, "fp_closure_build: bad argument");
    if (n == 0) return FP_OK;
    hipLaunchKernelGGL(nn_system_kernel, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, s, n, mom,
                       c->cfg.eps_hat, sys);
    return check_launch(c, "fp_closure_build");
}

// gradient (and, with ad, the Adam step on it); the arguments are checked
static int train_launch(fp_ctx* c, fp_nn* n, const float* params, const float* feats, const float* targets,
                        const double* sys, int64_t B, int32_t loss_kind, float* grad, float* loss,
                        const AdamArgs* ad, const char* what, hipStream_t s) {
    hipLaunchKernelGGL(nn_train_pack_kernel, dim3(FR_N), dim3(64), 0, s, params, n->timg);
    // tiles of 32 samples while they fit on the CUs at once (the shorter chain per workgroup),
    // else of 64, a workgroup per CU: eight waves hide each other's latencies, and the
    // partial gradients (165 KB a workgroup, written and read back) grow no further.  Just
    // below and above the line: 38.7 us at 8192 samples, 40.8 us at 16,384
    const bool small = B <= 32 * TRAIN_MAX_WG;
    const int rows = small ? (int)((B + 31) / 32) : (int)std::min<int64_t>(TRAIN_MAX_WG, (B + 63) / 64);
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(rows), dim3(small ? 256 : 512), 0, s, B, params, (const __bf16*)n->timg, feats,
                           targets, sys, n->part, n->lpart);
    };
    if (loss_kind == 0) launch(small ? nn_train_kernel<1, 0> : nn_train_kernel<2, 0>);
    else launch(small ? nn_train_kernel<1, 1> : nn_train_kernel<2, 1>);
    const dim3 rgrid((GROW / 4 + 63) / 64 + 1);
    if (ad)
        hipLaunchKernelGGL(nn_reduce_kernel<true>, rgrid, dim3(RED_BLOCK), 0, s, rows, (const float*)n->part,
                           (const double*)n->lpart, B, grad, loss, *ad);
    else
        hipLaunchKernelGGL(nn_reduce_kernel<false>, rgrid, dim3(RED_BLOCK), 0, s, rows, (const float*)n->part,
                           (const double*)n->lpart, B, grad, loss, AdamArgs{});
    return check_launch(c, what);
}

static bool grad_args(const fp_ctx* c, const fp_nn* n, const float* params, const float* feats, const float* targets,
                      const double* sys, int64_t B, int32_t loss_kind, const float* grad, const float* loss) {
    return c && n && params && feats && grad && loss && B > 0 && B <= n->max_batch &&
           (loss_kind == 0 || loss_kind == 1) && (loss_kind != 0 || targets) && (loss_kind != 1 || sys);
}

extern "C" int fp_nn_grad(fp_ctx* c, fp_nn* n, const float* params, const float* feats,
                          const float* targets, const double* sys, int64_t B, int32_t loss_kind,
                          float* grad, float* loss, hipStream_t s) {
    if (!grad_args(c, n, params, feats, targets, sys, B, loss_kind, grad, loss))
        return set_err(c, FP_EINVAL, "fp_nn_grad: bad argument");
    return train_launch(c, n, params, feats, targets, sys, B, loss_kind, grad, loss, nullptr, "fp_nn_grad", s);
}

extern "C" int fp_nn_adam(fp_ctx* c, float* params, const float* grad, float* m, float* v,
                          int64_t t, float lr, hipStream_t s) {
    if (!c || !params || !grad || !m || !v || t < 1 || !(lr >= 0.0f))
        return set_err(c, FP_EINVAL, "fp_nn_adam: bad argument");
    hipLaunchKernelGGL(nn_adam_kernel, dim3((N_TRAIN + 255) / 256), dim3(256), 0, s, adam_args(params, m, v, t, lr),
                       grad);
    return check_launch(c, "fp_nn_adam");
}

extern "C" int fp_nn_train_step(fp_ctx* c, fp_nn* n, float* params, float* m, float* v, int64_t t,
                                float lr, const float* feats, const float* targets, const double* sys,
                                int64_t B, int32_t loss_kind, float* loss, hipStream_t s) {
    if (!n) return set_err(c, FP_EINVAL, "fp_nn_train_step: bad argument");
    if (!grad_args(c, n, params, feats, targets, sys, B, loss_kind, n->grad, loss))
        return set_err(c, FP_EINVAL, "fp_nn_grad: bad argument");
    if (!m || !v || t < 1 || !(lr >= 0.0f)) {
        // as the two calls would: the gradient and the loss, then the refusal
        const int rc = train_launch(c, n, params, feats, targets, sys, B, loss_kind, n->grad, loss, nullptr,
                                    "fp_nn_grad", s);
        return rc ? rc : set_err(c, FP_EINVAL, "fp_nn_adam: bad argument");
    }
    const AdamArgs ad = adam_args(params, m, v, t, lr);
    return train_launch(c, n, params, feats, targets, sys, B, loss_kind, n->grad, loss, &ad, "fp_nn_train_step", s);
}
