// The f32 identity that the fused decoder rests on, for the test that holds it:
// one or two lanes a workgroup run on the vector ALU, as fmaf in increasing k,
// the chains that the encoder runs on v_mfma_f32_16x16x4_f32.  Not part of the
// public ABI.
#include <string>

#include "boa_internal.h"
#include "device_common.h"

namespace boa {
// Problem blockIdx.x: A [16][K], B [16][K] -> A B^T by either unit, [16][16].
__global__ __launch_bounds__(64) void k_f32_chain(const float* __restrict__ A, const float* __restrict__ B, int K,
                                                  float* __restrict__ by_mfma, float* __restrict__ by_fma) {
    const int li = threadIdx.x & 15, lk = threadIdx.x >> 4;
    const long long p = blockIdx.x;
    A += p * 16 * K;
    B += p * 16 * K;
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < K; k += 4)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(A[li * K + k + lk], B[li * K + k + lk], acc, 0, 0, 0);
    for (int rr = 0; rr < 4; ++rr) {
        const int row = 4 * lk + rr;
        float v = 0.0f;
        for (int k = 0; k < K; ++k) v = fmaf(A[row * K + k], B[li * K + k], v);
        by_mfma[p * 256 + row * 16 + li] = acc[rr];
        by_fma[p * 256 + row * 16 + li] = v;
    }
}
}  // namespace boa

// n problems, K a multiple of 4; device pointers; waits for `stream`.
extern "C" int boa_test_f32_chain(const float* d_A, const float* d_B, uint32_t n, uint32_t K, float* d_mfma,
                                  float* d_fma, void* stream) {
    if (!d_A || !d_B || !d_mfma || !d_fma || n == 0 || K == 0 || K % 4 || K > 4096 || n > (1u << 20))
        return boa::set_error(BOA_E_ARG, "bad argument");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(boa::k_f32_chain, dim3(n), dim3(64), 0, s, d_A, d_B, (int)K, d_mfma, d_fma);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e == hipSuccess ? BOA_OK : boa::set_error(BOA_E_DEVICE, hipGetErrorString(e));
}
