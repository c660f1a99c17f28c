// Round-to-nearest group quantizer and packer: the quantizer side (the black-box Q of
// ModuLoRA Section 2.2) in its simplest form, the round-to-nearest baseline of the paper's
// quantizer ablation.  W float32 [N][K] -> packed codes, binary16 scales, uint8 zero points in
// the layout the layer kernels read.  Every decision is taken in IEEE float32 (correctly
// rounded subtract / divide, round half to even), so the result is defined bit for bit:
//     lo = min(group, 0), hi = max(group, 0)
//     scale = smallest binary16 >= max((hi - lo) / (2^b - 1), 2^-14)
//     zero  = clamp(rne(-lo / scale), 0, 2^b - 1)
//     q     = clamp(rne(w / scale) + zero, 0, 2^b - 1)
// Bound by reading W.  The usual groups (32, 64, 128 or 256 inputs) take one pass: a tile of W
// stays in registers from its statistics to its codes (rtn_fused_kernel).  Other groups, up to a
// whole row, do not fit a workgroup's registers and take two passes: group statistics (a workgroup
// per row and run of groups, float4 loads along K), then quantize + pack (64 x 64 tiles: loads
// coalesced along K, codes turned through LDS, words stored coalesced along N).
#include <hip/hip_fp16.h>

#include "launch.h"

namespace mlr {

namespace {

__device__ __forceinline__ uint16_t f16_bits_round_up(float x) {
    const __half h = __float2half_rn(x);
    uint16_t bits = __half_as_ushort(h);
    if (__half2float(h) < x) bits += 1;   // positive finite: the next bit pattern is the next value
    return bits;
}

__device__ __forceinline__ float f16_bits_to_float(uint16_t bits) { return __half2float(__ushort_as_half(bits)); }

// ---- one pass: statistics, codes and bitstream of a tile held in registers -----------
// Measured at 22016 x 8192, 3 bits, group 128: 131 us a call (790 MB read and written at 6.0 TB/s; a
// large copy reaches 4.8); as two passes over W, each at 4 TB/s, it took 357.
// A workgroup takes 64 rows x TK inputs (TK = 128, or 256 for groups of 256): a thread holds 8 (16)
// float4, whose loads are all issued first; a group is 8, 16, 32 or 64 adjacent lanes of one load, so
// its range is a cross-lane reduction.  The tile's rows are wide enough (512 bytes) for the memory
// and 128 inputs few enough registers (52) for eight workgroups on a compute unit.  256 inputs take 86, which
// leaves five, and reach almost the same rate: 137 us at that size with groups of 256 (421 in two passes).
//
// The quotient w / s is not divided out per element (ten instructions each): with inv = 1 / s off
// by an ulp, t = w inv is within 2^-22 + 2^-23 (relative) of the rounded quotient, and
// |t| < 2^b <= 16, so the two round to the same integer unless t lies within 16 (2^-22 + 2^-23) <
// 2^-17 of a half-integer.  Within 2^-16 of one the wave divides (1 % of the loads of random weights).
constexpr int FR = 64;                 // rows of a tile
constexpr float HALF_BAND = 0.5f - 0x1p-16f;

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// minimum / maximum over LPG adjacent lanes, in every one of them
template <int LPG>
__device__ __forceinline__ void reduce_range(float &lo, float &hi) {
    lo = fminf(lo, dpp<0xB1>(lo)); hi = fmaxf(hi, dpp<0xB1>(hi));        // quad_perm 1,0,3,2
    lo = fminf(lo, dpp<0x4E>(lo)); hi = fmaxf(hi, dpp<0x4E>(hi));        // quad_perm 2,3,0,1
    lo = fminf(lo, dpp<0x141>(lo)); hi = fmaxf(hi, dpp<0x141>(hi));      // row_half_mirror
    if (LPG >= 16) { lo = fminf(lo, dpp<0x140>(lo)); hi = fmaxf(hi, dpp<0x140>(hi)); }   // row_mirror
    if (LPG >= 32) { lo = fminf(lo, __shfl_xor(lo, 16)); hi = fmaxf(hi, __shfl_xor(hi, 16)); }
    if (LPG >= 64) { lo = fminf(lo, __shfl_xor(lo, 32)); hi = fmaxf(hi, __shfl_xor(hi, 32)); }
}

template <int BITS, int LPG>           // LPG: lanes (float4) per group
__global__ __launch_bounds__(256) void rtn_fused_kernel(QuantArgs a) {
    constexpr int TK = LPG == 64 ? 256 : 128, RL = TK / 4;       // inputs of a tile, lanes per row
    constexpr int RPW = 64 / RL, NL = FR / (4 * RPW);            // rows of a wave's load, loads per thread
    constexpr int GT = TK / (4 * LPG);                           // groups of a tile's row
    constexpr int CROW = RL + 8;                                 // LDS row stride: 16-byte aligned, rows on other banks
    __shared__ __attribute__((aligned(16))) uint16_t codes[FR][CROW];   // four codes (4 BITS bits) each
    __shared__ uint16_t sc[GT][FR];
    __shared__ uint8_t zp[GT][FR];
    typedef float vec4 __attribute__((ext_vector_type(4)));
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int k0 = blockIdx.x * TK, n0 = blockIdx.y * FR;
    const int f4 = lane & (RL - 1), k = k0 + 4 * f4;
    const int row0 = wave * (FR / 4) + (RPW == 2 ? lane >> 5 : 0);
    const bool k_ok = k < a.K;                                   // a whole group is inside or outside
    const float *src = a.W + (k_ok ? k : 0);
    vec4 w[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int n = n0 + row0 + i * RPW < a.N ? n0 + row0 + i * RPW : a.N - 1;
        w[i] = __builtin_nontemporal_load(reinterpret_cast<const vec4 *>(src + (size_t)n * a.K));
    }
    constexpr float maxq = (float)((1 << BITS) - 1);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int nl = row0 + i * RPW;
        // zero is always inside the range
        float lo = fminf(fminf(fminf(w[i].x, w[i].y), fminf(w[i].z, w[i].w)), 0.f);
        float hi = fmaxf(fmaxf(fmaxf(w[i].x, w[i].y), fmaxf(w[i].z, w[i].w)), 0.f);
        reduce_range<LPG>(lo, hi);
        const uint16_t sbits = f16_bits_round_up(fmaxf(__fdiv_rn(__fsub_rn(hi, lo), maxq), 6.103515625e-05f));
        const float s = f16_bits_to_float(sbits), inv = __builtin_amdgcn_rcpf(s);
        float q[4], zq = -lo * inv, off = 0.f;
        const float rz = rintf(zq);
        off = fabsf(zq - rz);
        zq = rz;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float tq = w[i][e] * inv;
            q[e] = rintf(tq);
            off = fmaxf(off, fabsf(tq - q[e]));
        }
        if (off > HALF_BAND) {
            zq = rintf(__fdiv_rn(-lo, s));
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = rintf(__fdiv_rn(w[i][e], s));
        }
        zq = fminf(fmaxf(zq, 0.f), maxq);
        // the four codes side by side: at most 16 bits, exact in float32
        float packed = 0.f;
#pragma unroll
        for (int e = 3; e >= 0; --e) packed = __builtin_fmaf(packed, (float)(1 << BITS), fminf(fmaxf(q[e] + zq, 0.f), maxq));
        codes[nl][f4] = (uint16_t)packed;
        if (f4 % LPG == 0) {
            sc[f4 / LPG][nl] = sbits;
            zp[f4 / LPG][nl] = (uint8_t)zq;
        }
    }
    __syncthreads();
    const int nl = t & (FR - 1), n = n0 + nl;
    if (n >= a.N) return;
#pragma unroll
    for (int blk = wave; blk < TK / 32; blk += 4) {               // one 32-code block of one row per thread
        if (k0 + 32 * blk >= a.K) break;
        const uint4 c4 = *reinterpret_cast<const uint4 *>(&codes[nl][blk * 8]);
        const uint32_t piece2[4] = {c4.x, c4.y, c4.z, c4.w};
        uint32_t out[BITS];
#pragma unroll
        for (int j = 0; j < BITS; ++j) out[j] = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t p = c & 1 ? piece2[c / 2] >> 16 : piece2[c / 2] & 0xFFFFu;
            const int pos = c * 4 * BITS, wd = pos >> 5, sh = pos & 31;
            out[wd] |= p << sh;
            if (sh + 4 * BITS > 32) out[wd + 1] |= p >> (32 - sh);
        }
        uint32_t *dst = a.qweight + (size_t)(k0 / 32 + blk) * BITS * a.N + n;
#pragma unroll
        for (int j = 0; j < BITS; ++j) dst[(size_t)j * a.N] = out[j];
    }
    const int g0 = k0 / (4 * LPG);
    for (int gi = wave; gi < GT; gi += 4) {
        if (k0 + gi * 4 * LPG >= a.K) break;
        a.scales[(size_t)(g0 + gi) * a.N + n] = sc[gi][nl];
        a.zeros[(size_t)(g0 + gi) * a.N + n] = zp[gi][nl];
    }
}

template <int LPG>
hipError_t launch_fused(const QuantArgs &a, hipStream_t stream) {
    constexpr int TK = LPG == 64 ? 256 : 128;
    const dim3 grid((a.K + TK - 1) / TK, (a.N + FR - 1) / FR);
    switch (a.bits) {
        case 2: launch_kernel("rtn_fused", rtn_fused_kernel<2, LPG>, grid, dim3(256), 0, stream, a); break;
        case 3: launch_kernel("rtn_fused", rtn_fused_kernel<3, LPG>, grid, dim3(256), 0, stream, a); break;
        default: launch_kernel("rtn_fused", rtn_fused_kernel<4, LPG>, grid, dim3(256), 0, stream, a); break;
    }
    return hipGetLastError();
}

// ---- two passes, pass 1: scales and zero points --------------------------------------------------
// grid (N, runs of groups); a workgroup covers `gpb` whole groups of row n (gpb * g <= 1024
// floats, one float4 per thread) or, for g > 1024, one group in several sweeps.
__global__ __launch_bounds__(256) void rtn_stats_kernel(QuantArgs a, int gpb) {
    __shared__ float mn[256], mx[256];
    const int t = threadIdx.x, n = blockIdx.x;
    const int g = a.group, G = a.K / g;
    const int g_first = blockIdx.y * gpb;
    int ngroups = G - g_first;
    if (ngroups > gpb) ngroups = gpb;
    const int floats = ngroups * g;
    const float *row = a.W + (size_t)n * a.K + (size_t)g_first * g;
    float lo = 0.f, hi = 0.f;            // zero is always inside the range
    for (int i = 4 * t; i < floats; i += 1024) {
        const float4 v = *reinterpret_cast<const float4 *>(row + i);
        lo = fminf(fminf(lo, v.x), fminf(fminf(v.y, v.z), v.w));
        hi = fmaxf(fmaxf(hi, v.x), fmaxf(fmaxf(v.y, v.z), v.w));
    }
    mn[t] = lo;
    mx[t] = hi;
    __syncthreads();
    if (t >= ngroups) return;
    // entries of local group t: one float4 per thread when the run fits one sweep, else all
    int e0 = 0, e1 = 256;
    if (floats <= 1024) { e0 = t * (g / 4); e1 = e0 + g / 4; }
    lo = 0.f; hi = 0.f;
    for (int e = e0; e < e1; ++e) { lo = fminf(lo, mn[e]); hi = fmaxf(hi, mx[e]); }
    const float maxq = (float)((1 << a.bits) - 1);
    const float raw = __fdiv_rn(__fsub_rn(hi, lo), maxq);
    const uint16_t sbits = f16_bits_round_up(fmaxf(raw, 6.103515625e-05f));
    const float s = f16_bits_to_float(sbits);
    const float z = fminf(fmaxf(rintf(__fdiv_rn(-lo, s)), 0.f), maxq);
    const size_t o = (size_t)(g_first + t) * a.N + n;
    a.scales[o] = sbits;
    a.zeros[o] = (uint8_t)z;
}

// ---- pass 2: codes and bitstream -----------------------------------------------------
constexpr int QT = 64;            // tile: 64 output columns x 64 inputs (two 32-code blocks)
constexpr int QROW = QT / 4 + 1;  // LDS row stride in words (4 codes per word), padded

template <int BITS>
__global__ __launch_bounds__(256) void rtn_pack_kernel(QuantArgs a) {
    __shared__ uint32_t codes[QT][QROW];
    const int t = threadIdx.x;
    const int n0 = blockIdx.x * QT, k0 = blockIdx.y * QT;
    const float maxq = (float)((1 << BITS) - 1);
    const int f4 = t & 15, k = k0 + 4 * f4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int nl = (t >> 4) + 16 * i, n = n0 + nl;
        uint32_t packed4 = 0;
        if (n < a.N && k < a.K) {
            const float4 w = *reinterpret_cast<const float4 *>(a.W + (size_t)n * a.K + k);
            const size_t go = (size_t)(k / a.group) * a.N + n;
            const float s = f16_bits_to_float(a.scales[go]);
            const float z = (float)a.zeros[go];
            const float wv[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float q = fminf(fmaxf(rintf(__fdiv_rn(wv[e], s)) + z, 0.f), maxq);
                packed4 |= (uint32_t)q << (8 * e);
            }
        }
        codes[nl][f4] = packed4;
    }
    __syncthreads();
    if (t >= 2 * QT) return;
    const int nl = t & (QT - 1), blk = t >> 6;    // one 32-code block of one column per thread
    const int n = n0 + nl, kb = k0 + 32 * blk;
    if (n >= a.N || kb >= a.K) return;
    uint32_t out[BITS];
#pragma unroll
    for (int j = 0; j < BITS; ++j) out[j] = 0;
#pragma unroll
    for (int c = 0; c < 32; ++c) {
        const uint32_t q = (codes[nl][blk * 8 + c / 4] >> (8 * (c % 4))) & 0xFFu;
        const int pos = c * BITS, wd = pos >> 5, sh = pos & 31;
        out[wd] |= q << sh;
        if (sh + BITS > 32) out[wd + 1] |= q >> (32 - sh);
    }
    uint32_t *dst = a.qweight + (size_t)(kb / 32) * BITS * a.N + n;
#pragma unroll
    for (int j = 0; j < BITS; ++j) dst[(size_t)j * a.N] = out[j];
}

}  // namespace

hipError_t launch_quantize_rtn(const QuantArgs &a, hipStream_t stream) {
    switch (a.group) {
        case 32: return launch_fused<8>(a, stream);
        case 64: return launch_fused<16>(a, stream);
        case 128: return launch_fused<32>(a, stream);
        case 256: return launch_fused<64>(a, stream);
        default: break;
    }
    const int G = a.K / a.group;
    int gpb = 1024 / a.group;
    if (gpb < 1) gpb = 1;
    launch_kernel("rtn_stats", rtn_stats_kernel, dim3(a.N, (G + gpb - 1) / gpb), dim3(256), 0, stream, a, gpb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid((a.N + QT - 1) / QT, (a.K + QT - 1) / QT);
    switch (a.bits) {
        case 2: launch_kernel("rtn_pack", rtn_pack_kernel<2>, grid, dim3(256), 0, stream, a); break;
        case 3: launch_kernel("rtn_pack", rtn_pack_kernel<3>, grid, dim3(256), 0, stream, a); break;
        default: launch_kernel("rtn_pack", rtn_pack_kernel<4>, grid, dim3(256), 0, stream, a); break;
    }
    return hipGetLastError();
}

}  // namespace mlr
