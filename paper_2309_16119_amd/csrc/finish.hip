// The second launch of the products that are cut into slices of the contraction and keep the adapter out
// of it (gemm_direct.hip; smallm.hip for a rank over 8): sum of the slices' fp32 results and of the parts
// of the rank-r projection, the adapter term s P F of eq. (3), the bias, one rounding to 16 bits.
//
// Bound by trips to memory: everything a workgroup needs -- its tile of the factor, the projection's parts and
// the first slices -- is on its way before the first of it is waited for, and the factor's tile goes through
// LDS, where the rows of the workgroup share it.  (With the parts summed one element after the other and the
// factor fetched eight rows at a time the same launch took, in us: 16 x 4096, r = 16 / 64 7.1 / 13.0, now 5.9 / 6.8;
// 16 x 22016, r = 64 12.0, now 6.8; 24 x 2048, r = 16 11.7, now 7.8; 240 x 14720, r = 64 45, now 23.)
#include "gemm_common.h"

namespace mlr {

// Bias, adapter term (l; already in y where ADDED) and rounding of eight adjacent outputs.
template <bool BWD, bool F16, bool ADDED = false>
__device__ __forceinline__ void finish_store(const FinishArgs &d, int m, int col, float (&y)[8], const float (&l)[8]) {
    if (F16 && !BWD && d.bias16 != nullptr) {               // the frozen layer's bias: forward only
        const uint4 bw = *reinterpret_cast<const uint4 *>(d.bias16 + col);
        const uint32_t w4[4] = {bw.x, bw.y, bw.z, bw.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            y[2 * q] += half_bits_to_float((uint16_t)(w4[q] & 0xFFFFu));
            y[2 * q + 1] += half_bits_to_float((uint16_t)(w4[q] >> 16));
        }
    }
    if (!ADDED) {
#pragma unroll
        for (int c = 0; c < 8; ++c) y[c] = __builtin_fmaf(d.lora_scale, l[c], y[c]);
    }
    const uint4 o = make_uint4(pack_pair<F16>(y[0], y[1]), pack_pair<F16>(y[2], y[3]), pack_pair<F16>(y[4], y[5]), pack_pair<F16>(y[6], y[7]));
    *reinterpret_cast<uint4 *>(d.out + (size_t)m * d.Cout + col) = o;
}

// R: columns of rank that there is room for (0, 8, 16, 32, 64).  ROWS x COLS outputs, eight of a row per thread, in SG
// groups of threads that share the slices and the rank and meet in LDS.
// DEEP: everything in flight at once, at two waves a SIMD.
template <bool BWD, bool F16, int R, int ROWS, int SG, bool DEEP>
__global__ __launch_bounds__(256, DEEP ? 2 : (R <= 16 ? 6 : 4)) void finish_kernel(FinishArgs d) {
    constexpr int COLS = 2048 / ROWS / SG, PS = R + 4;
    constexpr int F4 = R > 0 ? (R * COLS / 4 + 255) / 256 : 1;       // float4 of the factor's tile per thread
    constexpr int P_SLOTS = R > 0 ? ROWS * R / 4 : 1;                // float4 of the projection's rows
    constexpr int P4 = (P_SLOTS + 255) / 256, GROUPS = P_SLOTS < 256 ? 256 / P_SLOTS : 1;
    constexpr int PB = (DEEP ? 16 : R <= 16 ? 4 : 8) / P4, SB = DEEP ? 8 : 4;      // in flight: parts per slot, slices
    __shared__ __attribute__((aligned(16))) float Fs[R > 0 ? R * COLS + COLS / 2 : 4], Ps[R > 0 ? GROUPS * ROWS * PS : 4];      // [group of parts][row]
    __shared__ __attribute__((aligned(16))) float4 Ys[SG > 1 ? (SG - 1) * 2 * (256 / SG) : 1];
    const int tid = threadIdx.x, r = d.r, M = d.M, Cout = d.Cout;
    const int m0 = blockIdx.y * ROWS, c0 = blockIdx.x * COLS;
    const int sg = uniform(tid / (256 / SG)), row = tid % (256 / SG) / (COLS / 8), cl = tid % (COLS / 8) * 8, m = m0 + row, col = c0 + cl;
    const bool mine = m < M && col < Cout;                            // Cout is a multiple of 8: all eight or none
    const int rows = M - m0 < ROWS ? M - m0 : ROWS, cols = Cout - c0 < COLS ? Cout - c0 : COLS;
    const bool quads = (r & 3) == 0;
    auto row_of = [&](int x) { return (int)__umulhi((uint32_t)x, d.r_magic); };      // x / r; the magic is 0 for r = 1
    auto split_index = [&](int x, int &q, int &j) {
        q = r > 1 ? row_of(x) : x;
        j = x - q * r;
    };

    const float *src = d.slices + (mine ? (size_t)m * Cout + col : (size_t)0);
    float4 v0[SB], v1[SB];
    auto load_slices = [&](int q0) {
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if ((q0 + u) * SG + sg < d.split) {
                v0[u] = *reinterpret_cast<const float4 *>(src + (size_t)((q0 + u) * SG + sg) * d.slice_stride);
                v1[u] = *reinterpret_cast<const float4 *>(src + (size_t)((q0 + u) * SG + sg) * d.slice_stride + 4);
            }
    };
    load_slices(0);
    // forward: F [r][Cout], its tile [j][COLS]; backward: F [Cout][r], whose tile is one run of floats
    float4 f[F4];
    if (R > 0) {
#pragma unroll
        for (int q = 0; q < F4; ++q) {
            const int x = q * 256 + tid;
            f[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!BWD) {
                const int j = x / (COLS / 4), c = x % (COLS / 4) * 4;
                if (j < r && c < cols) f[q] = *reinterpret_cast<const float4 *>(d.F + (size_t)j * Cout + c0 + c);
            } else if (4 * x < cols * r) {                            // cols is a multiple of 8
                f[q] = *reinterpret_cast<const float4 *>(d.F + (size_t)c0 * r + 4 * x);
            }
        }
    }
    // the projection's rows m0 ... as one run of floats per part (parts are padded to whole float4)
    const int p_slot = tid % P_SLOTS, p_group = tid / P_SLOTS;
    const float *psrc = d.ppart + (size_t)m0 * r;
    float4 p[P4][PB];
    auto load_parts = [&](int s0) {
#pragma unroll
        for (int t = 0; t < P4; ++t)
#pragma unroll
            for (int u = 0; u < PB; ++u) {
                const int x = 4 * (p_slot + 256 * t), s = (s0 + u) * GROUPS + p_group;
                p[t][u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (x < rows * r && s < d.parts) p[t][u] = *reinterpret_cast<const float4 *>(psrc + (size_t)s * d.part_stride + x);
            }
    };
    if (R > 0) load_parts(0);
    float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto add_slices = [&](int q0) {
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if ((q0 + u) * SG + sg < d.split) {
                y[0] += v0[u].x; y[1] += v0[u].y; y[2] += v0[u].z; y[3] += v0[u].w;
                y[4] += v1[u].x; y[5] += v1[u].y; y[6] += v1[u].z; y[7] += v1[u].w;
            }
    };
    float l[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (R > 0) {
        // backward: a column's r values side by side, four floats after every eighth column so that the threads of a
        // row, eight columns apart, meet different banks
        auto bwd_at = [&](int c, int quad) { return (c >> 3) * (8 * R + 4) + (c & 7) * R + 4 * quad; };
#pragma unroll
        for (int q = 0; q < F4; ++q) {
            const int x = q * 256 + tid;
            if (!BWD) {
                if (R * COLS / 4 % 256 == 0 || x < R * COLS / 4) *reinterpret_cast<float4 *>(Fs + 4 * x) = f[q];
            } else if (4 * x < cols * r) {
                int c, j;
                split_index(4 * x, c, j);
                if (quads) {
                    *reinterpret_cast<float4 *>(Fs + bwd_at(c, j >> 2)) = f[q];
                } else {
                    const float f4[4] = {f[q].x, f[q].y, f[q].z, f[q].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        Fs[bwd_at(c, j >> 2) + (j & 3)] = f4[e];
                        if (++j == r) { j = 0; ++c; }
                    }
                }
            }
        }
        if (!quads) {                                                 // zeros that fill up the last quad
            for (int x = tid; x < COLS * 4; x += 256)
                if (BWD && (r & 3) + (x & 3) < 4) Fs[bwd_at(x >> 2, r >> 2) + (r & 3) + (x & 3)] = 0.f;
            for (int x = tid; x < GROUPS * ROWS * 4; x += 256)
                if ((r & 3) + (x & 3) < 4) Ps[(x >> 2) * PS + r + (x & 3)] = 0.f;
        }
        float4 sum[P4];
#pragma unroll
        for (int t = 0; t < P4; ++t) sum[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int s0 = 0; s0 * GROUPS < d.parts; s0 += PB) {
            if (s0 > 0) load_parts(s0);
#pragma unroll
            for (int t = 0; t < P4; ++t)
#pragma unroll
                for (int u = 0; u < PB; ++u) { sum[t].x += p[t][u].x; sum[t].y += p[t][u].y; sum[t].z += p[t][u].z; sum[t].w += p[t][u].w; }
        }
#pragma unroll
        for (int t = 0; t < P4; ++t) {
            const int x = 4 * (p_slot + 256 * t);
            if (x >= rows * r) continue;
            const float s4[4] = {sum[t].x, sum[t].y, sum[t].z, sum[t].w};
            int q, j;
            split_index(x, q, j);
            float *dst = Ps + p_group * (ROWS * PS);
            if (quads) {
                *reinterpret_cast<float4 *>(dst + q * PS + j) = sum[t];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (x + e < rows * r) dst[q * PS + j] = s4[e];
                    if (++j == r) { j = 0; ++q; }
                }
            }
        }
        __syncthreads();
        if (blockIdx.x == 0 && d.P_out != nullptr)
            for (int x = tid; x < rows * r; x += 256) {
                int q, j;
                split_index(x, q, j);
                float o = Ps[q * PS + j];
#pragma unroll
                for (int g = 1; g < GROUPS; ++g) o += Ps[(g * ROWS + q) * PS + j];
                d.P_out[(size_t)m0 * r + x] = o;
            }
        for (int j = 4 * sg; j < r; j += 4 * SG) {
            float4 pj = *reinterpret_cast<const float4 *>(Ps + row * PS + j);
#pragma unroll
            for (int g = 1; g < GROUPS; ++g) {
                const float4 o = *reinterpret_cast<const float4 *>(Ps + (g * ROWS + row) * PS + j);
                pj.x += o.x; pj.y += o.y; pj.z += o.z; pj.w += o.w;
            }
            const float p4[4] = {pj.x, pj.y, pj.z, pj.w};
            if (!BWD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (j + e >= r) break;
                    const float4 a = *reinterpret_cast<const float4 *>(Fs + (j + e) * COLS + cl), b = *reinterpret_cast<const float4 *>(Fs + (j + e) * COLS + cl + 4);
                    l[0] = __builtin_fmaf(p4[e], a.x, l[0]); l[1] = __builtin_fmaf(p4[e], a.y, l[1]);
                    l[2] = __builtin_fmaf(p4[e], a.z, l[2]); l[3] = __builtin_fmaf(p4[e], a.w, l[3]);
                    l[4] = __builtin_fmaf(p4[e], b.x, l[4]); l[5] = __builtin_fmaf(p4[e], b.y, l[5]);
                    l[6] = __builtin_fmaf(p4[e], b.z, l[6]); l[7] = __builtin_fmaf(p4[e], b.w, l[7]);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float4 a = *reinterpret_cast<const float4 *>(Fs + bwd_at(cl + c, j >> 2));
                    l[c] = __builtin_fmaf(p4[0], a.x, l[c]);
                    l[c] = __builtin_fmaf(p4[1], a.y, l[c]);
                    l[c] = __builtin_fmaf(p4[2], a.z, l[c]);
                    l[c] = __builtin_fmaf(p4[3], a.w, l[c]);
                }
            }
        }
    }
    add_slices(0);
    for (int q0 = SB; q0 * SG < d.split; q0 += SB) { load_slices(q0); add_slices(q0); }
    if (SG > 1) {
        const int t = tid % (256 / SG);
#pragma unroll
        for (int c = 0; c < 8; ++c) y[c] = __builtin_fmaf(d.lora_scale, l[c], y[c]);
        if (sg > 0) {
            Ys[((sg - 1) * 2 + 0) * (256 / SG) + t] = make_float4(y[0], y[1], y[2], y[3]);
            Ys[((sg - 1) * 2 + 1) * (256 / SG) + t] = make_float4(y[4], y[5], y[6], y[7]);
        }
        __syncthreads();
        if (sg > 0) return;
#pragma unroll
        for (int g = 0; g < SG - 1; ++g) {
            const float4 a = Ys[(g * 2 + 0) * (256 / SG) + t], b = Ys[(g * 2 + 1) * (256 / SG) + t];
            y[0] += a.x; y[1] += a.y; y[2] += a.z; y[3] += a.w;
            y[4] += b.x; y[5] += b.y; y[6] += b.z; y[7] += b.w;
        }
    }
    if (!mine) return;
    finish_store<BWD, F16, (SG > 1)>(d, m, col, y, l);
}

// The same for a rank of 1 to 8 where many workgroups fill the chip: 32 rows x 64 columns, eight of a row per thread, one element of
// the projection and two of the factor's tile per thread, so that registers leave eight waves a SIMD and the first
// slices, the factor and eight parts are all on their way at once.  Bound by that trip and the slices' bytes.
// us in finish_kernel (R = 8) / here, forward and backward: 512 x 4096, r = 8 6.1 / 5.6 and 6.0 / 5.6, binary16 6.2 / 5.7 and
// 5.9 / 5.5; 200 x 8192 5.4 / 5.0 and 5.4 / 5.0; 1000 x 4096, r = 5 7.2 / 5.9 and 8.3 / 6.0; 1024 x 6656, r = 8 13.7 /
// 13.7 and 14.4 / 13.6.
template <bool BWD, bool F16>
__global__ __launch_bounds__(256) void finish_low_rank_kernel(FinishArgs d) {
    constexpr int R = 8, PARTS = 8, SB = 4, FS = BWD ? 68 : 64;      // 68: a column's r values, written at once, meet different banks
    __shared__ __attribute__((aligned(16))) float Ps[32 * R], Fs[R * FS];      // [32][r], [r][64]
    const int tid = threadIdx.x, r = d.r, M = d.M, Cout = d.Cout;
    const int m0 = blockIdx.y * 32, c0 = blockIdx.x * 64;
    const int m = m0 + (tid >> 3), cl = (tid & 7) * 8, col = c0 + cl;
    const int rows = M - m0 < 32 ? M - m0 : 32, cols = Cout - c0 < 64 ? Cout - c0 : 64;
    const bool mine = m < M && col < Cout;                // Cout is a multiple of 8: all eight or none
    const float *src = d.slices + (mine ? (size_t)m * Cout + col : (size_t)0);
    float4 v0[SB], v1[SB];
    auto load_slices = [&](int q0) {
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if (q0 + u < d.split) {
                v0[u] = *reinterpret_cast<const float4 *>(src + (size_t)(q0 + u) * d.slice_stride);
                v1[u] = *reinterpret_cast<const float4 *>(src + (size_t)(q0 + u) * d.slice_stride + 4);
            }
    };
    float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto add_slices = [&](int q0) {
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if (q0 + u < d.split) {
                y[0] += v0[u].x; y[1] += v0[u].y; y[2] += v0[u].z; y[3] += v0[u].w;
                y[4] += v1[u].x; y[5] += v1[u].y; y[6] += v1[u].z; y[7] += v1[u].w;
            }
    };
    load_slices(0);
    float f[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int x = tid + 256 * h;
        f[h] = 0.f;
        if (!BWD) {
            if ((x >> 6) < r && (x & 63) < cols) f[h] = d.F[(size_t)(x >> 6) * Cout + c0 + (x & 63)];
        } else if (x < cols * r) {                        // one run of floats
            f[h] = d.F[(size_t)c0 * r + x];
        }
    }
    const bool has_p = tid < rows * r;
    const float *psrc = d.ppart + (size_t)m0 * r + (has_p ? tid : 0);
    float p[PARTS], sum = 0.f;
#pragma unroll
    for (int s = 0; s < PARTS; ++s) p[s] = s < d.parts ? psrc[(size_t)s * d.part_stride] : 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int x = tid + 256 * h;
        if (!BWD) {
            Fs[(x >> 6) * FS + (x & 63)] = f[h];
        } else if (x < cols * r) {
            const int c = r > 1 ? (int)__umulhi((uint32_t)x, d.r_magic) : x;
            Fs[(x - c * r) * FS + c] = f[h];
        }
    }
#pragma unroll
    for (int s = 0; s < PARTS; ++s) sum += p[s];
#pragma unroll 8
    for (int s = PARTS; s < d.parts; ++s) sum += psrc[(size_t)s * d.part_stride];
    if (has_p) {
        Ps[tid] = sum;
        if (blockIdx.x == 0 && d.P_out != nullptr) d.P_out[(size_t)m0 * r + tid] = sum;
    }
    __syncthreads();
    add_slices(0);
    for (int q0 = SB; q0 < d.split; q0 += SB) { load_slices(q0); add_slices(q0); }
    if (!mine) return;
    float l[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < r; ++j) {
        const float pj = Ps[(tid >> 3) * r + j];
        const float4 a = *reinterpret_cast<const float4 *>(Fs + j * FS + cl), b = *reinterpret_cast<const float4 *>(Fs + j * FS + cl + 4);
        l[0] = __builtin_fmaf(pj, a.x, l[0]); l[1] = __builtin_fmaf(pj, a.y, l[1]);
        l[2] = __builtin_fmaf(pj, a.z, l[2]); l[3] = __builtin_fmaf(pj, a.w, l[3]);
        l[4] = __builtin_fmaf(pj, b.x, l[4]); l[5] = __builtin_fmaf(pj, b.y, l[5]);
        l[6] = __builtin_fmaf(pj, b.z, l[6]); l[7] = __builtin_fmaf(pj, b.w, l[7]);
    }
    finish_store<BWD, F16>(d, m, col, y, l);
}

namespace {
template <bool BWD, bool F16, int ROWS, int SG, bool DEEP>
hipError_t launch_finish_rows(const char *name, const FinishArgs &d, hipStream_t stream) {
    constexpr int COLS = 2048 / ROWS / SG;
    const dim3 grid((d.Cout + COLS - 1) / COLS, (d.M + ROWS - 1) / ROWS);
    if (d.r == 0) launch_kernel(name, finish_kernel<BWD, F16, 0, ROWS, SG, DEEP>, grid, 256, 0, stream, d);
    else if (d.r <= 8) {
        if constexpr (DEEP) launch_kernel(name, finish_kernel<BWD, F16, 8, ROWS, SG, DEEP>, grid, 256, 0, stream, d);
        else launch_kernel(name, finish_low_rank_kernel<BWD, F16>, grid, 256, 0, stream, d);      // ROWS is 32, COLS 64
    }
    else if (d.r <= 16) launch_kernel(name, finish_kernel<BWD, F16, 16, ROWS, SG, DEEP>, grid, 256, 0, stream, d);
    else if (d.r <= 32) launch_kernel(name, finish_kernel<BWD, F16, 32, ROWS, SG, DEEP>, grid, 256, 0, stream, d);
    else launch_kernel(name, finish_kernel<BWD, F16, 64, ROWS, SG, DEEP>, grid, 256, 0, stream, d);
    return hipGetLastError();
}
template <int ROWS, int SG, bool DEEP>
hipError_t launch_finish_any(const char *name, const FinishArgs &d, bool backward, bool f16, hipStream_t stream) {
    if (f16) return backward ? launch_finish_rows<true, true, ROWS, SG, DEEP>(name, d, stream) : launch_finish_rows<false, true, ROWS, SG, DEEP>(name, d, stream);
    return backward ? launch_finish_rows<true, false, ROWS, SG, DEEP>(name, d, stream) : launch_finish_rows<false, false, ROWS, SG, DEEP>(name, d, stream);
}
}  // namespace

// Up to 16 rows: the narrowest tile that leaves no more workgroups than fit the chip at two waves a SIMD (16 rows,
// r = 16 / 64, us with 32, 64 and 128 columns: 4096 wide 5.9, 7.6, 10.5 / 6.8, 8.9, 13.3; 11008 wide 5.0, 5.3, 7.2 / 6.1,
// 6.6, 9.8; 22016 wide 7.2, 5.1, 5.5 / 9.1, 6.8, 8.9; 40960 wide 9.5, 7.6, 5.7 / 11.6, 10.3, 9.1).
// More: many workgroups need registers for four to six waves a SIMD more than they need every load in flight
// (512 x 4096, r = 8: 8.4 us deep, 6.2 not, 5.6 in the kernel for low ranks); few wait for their trips (24 x 2048, r = 16: 7.8 us deep, 12.2 not).
hipError_t launch_finish(const char *name, FinishArgs d, bool backward, bool f16, hipStream_t stream) {
    d.r_magic = d.r > 1 ? (uint32_t)((1ull << 32) / d.r) + 1u : 0u;      // x / r by one multiply-high, x < 2^13, r <= 64
    if (d.M <= 16) {
        if (d.Cout <= 32 * 512) return launch_finish_any<16, 4, true>(name, d, backward, f16, stream);
        if (d.Cout <= 64 * 512) return launch_finish_any<16, 2, true>(name, d, backward, f16, stream);
        return launch_finish_any<16, 1, true>(name, d, backward, f16, stream);
    }
    if (((long)d.Cout + 63) / 64 * ((d.M + 31) / 32) <= 512) return launch_finish_any<32, 1, true>(name, d, backward, f16, stream);
    return launch_finish_any<32, 1, false>(name, d, backward, f16, stream);
}

}  // namespace mlr
