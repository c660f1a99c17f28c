// The rank-r projection as a side job of a product kernel (gemm_direct.hip, gemm_big_kernel.h).
#pragma once
#include "device_common.h"

namespace mlr {

struct ProjectArgs {
    const uint16_t *act;          // [M][C]
    const float *F;               // forward A [C][r], backward B [r][C]
    int M, C, r;
};

// The projection of 16 activation rows over contraction elements [k0, k1) (multiples of 8), the waves
// of the workgroup sharing its steps: sum act[row][c] F(c, j) on the matrix cores, the fp32 factor
// split exactly into three bfloat16 terms (binary16 activations into two).  The wave's own sums for factor columns 16 g ...
template <bool F_IS_A, bool F16, int NWAVES>
__device__ __forceinline__ f32x4 project_wave(const ProjectArgs &d, int row0, int k0, int k1, int g) {
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int i = lane & 15, cs = lane >> 4, r = d.r;
    const int row = row0 + i < d.M ? row0 + i : d.M - 1;
    const uint16_t *arow = d.act + (size_t)row * d.C;
    const int steps = (k1 - k0 + 31) / 32;
    const int s0 = steps * wave / NWAVES, s1 = steps * (wave + 1) / NWAVES;
    const int j = g * 16 + i;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    constexpr int UNR = 4;
    for (int st = s0; st < s1; st += UNR) {
        uint4 av[UNR];
        float f[UNR][8];
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
            const int c = k0 + (st + q) * 32 + cs * 8;
            const bool ok = st + q < s1 && c < k1;
            av[q] = make_uint4(0, 0, 0, 0);
            if (ok) av[q] = *reinterpret_cast<const uint4 *>(arow + c);
#pragma unroll
            for (int e = 0; e < 8; ++e) f[q][e] = 0.f;
            if (ok && j < r) {
                if (F_IS_A) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[q][e] = d.F[(size_t)(c + e) * r + j];
                } else {
                    const float4 q0 = *reinterpret_cast<const float4 *>(d.F + (size_t)j * d.C + c);
                    const float4 q1 = *reinterpret_cast<const float4 *>(d.F + (size_t)j * d.C + c + 4);
                    f[q][0] = q0.x; f[q][1] = q0.y; f[q][2] = q0.z; f[q][3] = q0.w;
                    f[q][4] = q1.x; f[q][5] = q1.y; f[q][6] = q1.z; f[q][7] = q1.w;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
            if (st + q >= s1) break;      // wave-uniform
            uint32_t p[3][4];
            split3(f[q], p[0], p[1], p[2]);
            const uint32_t ar[4] = {av[q].x, av[q].y, av[q].z, av[q].w};
            uint32_t a2[2][4];
            if (F16) split_f16x8(ar, a2[0], a2[1]);
#pragma unroll
            for (int h = 0; h < (F16 ? 2 : 1); ++h) {
                bf16x8 x, y;
                __builtin_memcpy(&x, F16 ? a2[h] : ar, 16);
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    __builtin_memcpy(&y, p[t], 16);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, acc, 0, 0, 0);
                }
            }
        }
    }
    return acc;
}
// ... into LDS (`red`: NWAVES * RG * 256 floats), and, a barrier later, their sum over the waves: P[row][j].
__device__ __forceinline__ void project_leave(const f32x4 &acc, int g, int RG, float *red) {
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((wave * RG + g) * 4 + v) * 64 + lane] = acc[v];
}
template <int NWAVES>
__device__ __forceinline__ void project_sum(const ProjectArgs &d, int row0, int RG, float *dst, const float *red) {
    for (int x = threadIdx.x; x < RG * 256; x += NWAVES * 64) {
        const int g = x >> 8, v = (x >> 6) & 3, l = x & 63;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NWAVES; ++w) sum += red[((w * RG + g) * 4 + v) * 64 + l];
        const int prow = row0 + 4 * (l >> 4) + v, j = g * 16 + (l & 15);
        if (prow < d.M && j < d.r) dst[(size_t)prow * d.r + j] = sum;
    }
}
// All of it.  Ends with every thread past its reads of `red`.
template <bool F_IS_A, bool F16, int NWAVES>
__device__ __forceinline__ void project_rows(const ProjectArgs &d, int row0, int k0, int k1, float *dst, float *red) {
    const int RG = (d.r + 15) >> 4;
    for (int g = 0; g < RG; ++g) project_leave(project_wave<F_IS_A, F16, NWAVES>(d, row0, k0, k1, g), g, RG, red);
    __syncthreads();
    project_sum<NWAVES>(d, row0, RG, dst, red);
    __syncthreads();
}

}  // namespace mlr
