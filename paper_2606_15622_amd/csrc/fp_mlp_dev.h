// fp_mlp_dev.h -- device pieces shared by the MFMA kernels of the two networks: the 32 x 32
// x 16 bfloat16 product, the LDS images of an output tile, and barriers that order LDS only.
//
// Operand layouts of the 32x32x16 MFMA (wave64, lane l, half h = l / 32):
//   A (32 x 16):  lane holds A[l % 32][8h + i], i = 0..7
//   B (16 x 32):  lane holds B[8h + i][l % 32]
//   D (32 x 32):  lane holds D[8(j/4) + 4h + j%4][l % 32], j = 0..15
#pragma once
#include <hip/hip_runtime.h>

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

}  // namespace fpg
