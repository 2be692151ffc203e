// fp_mlp_dev.h -- device pieces shared by the MFMA kernels of the two networks: the 32 x 32
// x 16 bfloat16 product, the LDS images of an output tile, and barriers that order LDS only.
//
// Operand layouts of the 32x32x16 MFMA (wave64, lane l, half h = l / 32):
//   A (32 x 16):  lane holds A[l % 32][8h + i], i = 0..7
//   B (16 x 32):  lane holds B[8h + i][l % 32]
//   D (32 x 32):  lane holds D[8(j/4) + 4h + j%4][l % 32], j = 0..15
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace fpg {

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// workgroup barrier for data that passes through LDS: waits for LDS operations only, so that
// global loads issued before it (the next layer's weights) stay in flight across it
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// the same within a wave, for data that its lanes exchange through LDS: nothing to wait for (a
// wave's LDS operations are done in order), but the compiler keeps the order too
__device__ __forceinline__ void lds_wave_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// the lane's 16 values of a 32 x 32 output tile (rows = units r0 .., columns = samples), as
// bfloat16, into the sample-major image s[sample][unit] (the next product's B operand; only
// with SAMPLE_MAJOR) and the unit-major image t[unit][sample] (the operands of the weight gradients,
// whose inner dimension is the sample)
template <bool SAMPLE_MAJOR>
__device__ __forceinline__ void put_tile(__bf16* s, int ss, __bf16* t, int ts, int n, int r0, int h,
                                         const float (&v)[16]) {
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
        const int row = r0 + 8 * jq + 4 * h;
        bf16x4 q;
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = (__bf16)v[4 * jq + e];
        if constexpr (SAMPLE_MAJOR) *(bf16x4*)(s + n * ss + row) = q;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[(row + e) * ts + n] = q[e];
    }
}

// KS consecutive fragments of 64 lanes x 8 values, from fragment f0
template <int KS>
__device__ __forceinline__ void load_frags(const __bf16* __restrict__ img, int f0, int lane, bf16x8 (&a)[KS]) {
#pragma unroll
    for (int s = 0; s < KS; ++s) a[s] = *(const bf16x8*)(img + ((f0 + s) * 64 + lane) * 8);
}

// sums over the 32 samples (columns) of the lane's 16 rows of a D tile: every exchange halves
// the rows a lane keeps; lane l ends with row j = l % 16 of its half (twice: lanes l, l ^ 16)
__device__ __forceinline__ float row_sums(const float (&v)[16], int lane) {
    float a[8], b[4], c[2];
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = (b3 ? v[i + 8] : v[i]) + __shfl_xor(b3 ? v[i] : v[i + 8], 8, 64);
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (b2 ? a[i + 4] : a[i]) + __shfl_xor(b2 ? a[i] : a[i + 4], 4, 64);
#pragma unroll
    for (int i = 0; i < 2; ++i) c[i] = (b1 ? b[i + 2] : b[i]) + __shfl_xor(b1 ? b[i] : b[i + 2], 2, 64);
    float s = (b0 ? c[1] : c[0]) + __shfl_xor(b0 ? c[0] : c[1], 1, 64);
    return s + __shfl_xor(s, 16, 64);
}

// Adam (Kingma and Ba) on one trainable parameter, FP32 master weights
struct AdamArgs {
    float *p, *m, *v;
    float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ void adam_one(const AdamArgs& a, int64_t q, float gq, float mq, float vq, float pq) {
    mq = a.b1 * mq + (1.0f - a.b1) * gq;
    vq = a.b2 * vq + (1.0f - a.b2) * gq * gq;
    a.m[q] = mq;
    a.v[q] = vq;
    a.p[q] = pq - a.lr * (mq / a.c1) / (sqrtf(vq / a.c2) + a.eps);
}

inline AdamArgs adam_args(float* params, float* m, float* v, int64_t t, float lr) {
    return {params, m, v, lr, 0.9f, 0.999f, 1e-8f, (float)(1.0 - pow(0.9, (double)t)),
            (float)(1.0 - pow(0.999, (double)t))};
}

}  // namespace fpg
