// The rank-r adapter side of the layer (Section 3.1 eq. (3) and Section 3.1.1 of the
// ModuLoRA paper): the skinny projections  XA = X A  and  dYBt = dY B^T, the adapter
// gradients  dA = s X^T dYBt  and  dB = s XA^T dY, and the preparation of the
// "extended contraction" operands with which the tile GEMM adds the adapter term
// s (X A) B inside its MFMA loop.
//
// All of these are bound by one streaming pass over X or dY, and all run on the matrix cores, the
// fp32 operand (the factor, or P) split exactly into three bfloat16 terms.
#include "device_common.h"
#include "launch.h"

namespace mlr {

// Extended operands, segments of r elements.  Three segments (bfloat16 outputs): (hi,hi,lo) on the
// activation side and (hi,lo,hi) on the weight side of a two-way split, so that the dot product is
// hi*hi + hi*lo + lo*hi ~= (hi+lo)*(hi+lo) to about 2^-16 relative.  Six segments (binary16 outputs):
// the products of a three-way split down to 2^-16 of the first, (0,0,1,1,0,2) against (0,1,0,1,2,0); the
// three parts, each rounded to nearest, carry all 24 bits, and what is left out is at most 2^-24 of a product and of
// either sign: an fp32 multiply's own rounding (over 4 M pairs near a power of two, where it is largest: at most
// 2^-24.1, 2^-26.5 rms; 2^-24.0 and 2^-24.8 rounded to fp32; with truncated parts 2^-21.1 and all of one sign).
// An infinity or NaN stands in the first segment only: an infinite factor or projection then gives
// the infinity that the definition gives, as in the kernels that add the term in fp32 (finish.hip), not the
// NaN of inf - inf or inf * 0.
__device__ __forceinline__ uint16_t ext_part(float v, int segment, int segments, bool weight_side) {
    const int part = ((segments == 3 ? (weight_side ? 0x010 : 0x100) : weight_side ? 0x021010 : 0x201100) >> (4 * segment)) & 15;
    const uint32_t bits = __float_as_uint(v);
    const bool finite = (bits & 0x7F800000u) != 0x7F800000u;
    uint16_t hi = float_to_bf16_bits(v);
    if (finite && (hi & 0x7FFFu) == 0x7F80u) hi = (uint16_t)(bits >> 16);      // rounded past the largest bfloat16
    const float r1 = v - bf16_bits_to_float(hi);
    const uint16_t mid = float_to_bf16_bits(r1), lo = float_to_bf16_bits(r1 - bf16_bits_to_float(mid));
    const uint16_t value = part == 0 ? hi : part == 1 ? mid : lo;
    return finite || segment == 0 ? value : (uint16_t)0;
}

// ---------------------------------------------------------------------------
// Projection: P[m][j] = sum_c act[m][c] F(c, j) on the matrix cores.  A workgroup owns 16 rows;
// its waves split the contraction and meet in LDS.  act is bfloat16 already; the fp32 factor is
// split on the fly into three bfloat16 terms (hi + mid + lo carry all 24 significand bits), so
// three 16x16x32 MFMAs per step give the fp32-exact products, accumulated in fp32.
// Lane l = 16 cs + i: activation row i / factor column i, contraction elements 8 cs .. 8 cs + 7
// of the step.  Extra workgroups (blockIdx.x >= row blocks) write the weight-side extension.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bf16x8 regs_to_bf16x8(const uint32_t r[4]) {
    bf16x8 v;
    __builtin_memcpy(&v, r, 16);
    return v;
}

// Eight consecutive elements (one 16-byte store) of the weight-side extension w_ext [Cw][RE]:
// row c holds the segments of the r factor values of that row (ext_part()) and zero padding.
// Unit u = c * (RE / 8) + chunk, consecutive threads take consecutive units: the stores are
// contiguous, and the loads of a wave touch a few dozen adjacent rows c (from B [r][Cw]: runs of
// adjacent floats in up to eight rows j; from A [Cw][r]: adjacent floats of a row).
__device__ __forceinline__ void write_w_ext_unit(const DownArgs &a, size_t u) {
    const int r = a.r, per_row = a.RE >> 3;
    const int c = (int)(u / per_row), e0 = (int)(u % per_row) * 8;
    float src[8];
    int seg[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = e0 + q;
        seg[q] = e / r;
        const int j = e - seg[q] * r;
        src[q] = seg[q] < a.segments ? (a.w_from_A ? a.Wsrc[(size_t)c * r + j] : a.Wsrc[(size_t)j * a.Cw + c]) : 0.f;
    }
    uint32_t o[4];
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
        const uint32_t lo16 = seg[q] < a.segments ? ext_part(src[q], seg[q], a.segments, true) : 0u;
        const uint32_t hi16 = seg[q + 1] < a.segments ? ext_part(src[q + 1], seg[q + 1], a.segments, true) : 0u;
        o[q >> 1] = lo16 | (hi16 << 16);
    }
    *reinterpret_cast<uint4 *>(a.w_ext + u * 8) = make_uint4(o[0], o[1], o[2], o[3]);
}

// One element of a projection (column j, 0 .. 15 at least): P and, where it is asked for, its place in
// every segment of the activation-side extension; the threads past the rank write the zeros that pad it.
__device__ __forceinline__ void store_projection(const DownArgs &a, int m, int j, float p) {
    const int r = a.r;
    if (j < r) a.P[(size_t)m * r + j] = p;
    if (a.act_ext == nullptr) return;
    uint16_t *ext = a.act_ext + (size_t)m * a.RE;
    if (j < r) {
        const float v = a.lora_scale * p;
        for (int seg = 0; seg < a.segments; ++seg) ext[seg * r + j] = ext_part(v, seg, a.segments, false);
    }
    // (at most 15 zeros: RE is the segments' length rounded up to 16)
    if (j < 16 && a.segments * r + j < a.RE) ext[a.segments * r + j] = 0;
}

// ROWT: 16-row tiles per workgroup (they share every factor operand); UNR: steps whose loads
// are issued together before any of them is used.
// ACT_F16: the activations are binary16; each operand is split exactly into two bfloat16 ones.
template <int RG, int ROWT, bool F_IS_A, bool ACT_F16>
__global__ __launch_bounds__(1024) void lora_down_kernel(DownArgs a, int row_blocks, int split, Cut cut /* of the steps of 32 over slices and waves */) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];   // [waves][ROWT][RG][256] partial tiles
    constexpr int UNR = ROWT > 1 ? 2 : (RG == 1 ? 4 : (RG == 2 ? 2 : 1));
    constexpr int ROWS = 16 * ROWT;
    const int tid = threadIdx.x, nthreads = blockDim.x;
    const int r = a.r;

    if ((int)blockIdx.x >= row_blocks) {
        if (blockIdx.y != 0) return;
        // weight-side extension, one 16-byte unit per thread
        const size_t u = (size_t)(blockIdx.x - row_blocks) * nthreads + tid;
        if (u < (size_t)a.Cw * (a.RE >> 3)) write_w_ext_unit(a, u);
        return;
    }

    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthreads >> 6;
    const int i = lane & 15, cs = lane >> 4;
    const int m0 = blockIdx.x * ROWS;
    const uint16_t *arow[ROWT];
#pragma unroll
    for (int t = 0; t < ROWT; ++t) {
        int row = m0 + 16 * t + i;
        if (row > a.M - 1) row = a.M - 1;
        arow[t] = a.act + (size_t)row * a.C;
    }
    // the contraction is cut over (blockIdx.y, wave)
    const int s_begin = (int)cut.begin(blockIdx.y * nwaves + wave), s_end = (int)cut.begin(blockIdx.y * nwaves + wave + 1);

    f32x4 acc[ROWT][RG];
#pragma unroll
    for (int t = 0; t < ROWT; ++t)
#pragma unroll
        for (int g = 0; g < RG; ++g) acc[t][g] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int st = s_begin; st < s_end; st += UNR) {
        uint4 av[UNR][ROWT];
        float f[UNR][RG][8];
        // all loads of UNR steps first
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
            const int c = (st + q) * 32 + cs * 8;       // C is a multiple of 8: the chunk is all in or all out
            const bool c_ok = st + q < s_end && c < a.C;
#pragma unroll
            for (int t = 0; t < ROWT; ++t) {
                av[q][t] = make_uint4(0, 0, 0, 0);
                if (c_ok) av[q][t] = *reinterpret_cast<const uint4 *>(arow[t] + c);
            }
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int j = g * 16 + i;
#pragma unroll
                for (int e = 0; e < 8; ++e) f[q][g][e] = 0.f;
                if (c_ok && j < r) {
                    if (F_IS_A) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) f[q][g][e] = a.Fm[(size_t)(c + e) * r + j];
                    } else {
                        const float4 q0 = *reinterpret_cast<const float4 *>(a.Fm + (size_t)j * a.C + c);
                        const float4 q1 = *reinterpret_cast<const float4 *>(a.Fm + (size_t)j * a.C + c + 4);
                        f[q][g][0] = q0.x; f[q][g][1] = q0.y; f[q][g][2] = q0.z; f[q][g][3] = q0.w;
                        f[q][g][4] = q1.x; f[q][g][5] = q1.y; f[q][g][6] = q1.z; f[q][g][7] = q1.w;
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < UNR; ++q)
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                uint32_t hi[4], mid[4], lo[4];
                split3(f[q][g], hi, mid, lo);
                const bf16x8 bh = regs_to_bf16x8(hi), bm = regs_to_bf16x8(mid), bl = regs_to_bf16x8(lo);
#pragma unroll
                for (int t = 0; t < ROWT; ++t) {
                    const uint32_t ar[4] = {av[q][t].x, av[q][t].y, av[q][t].z, av[q][t].w};
                    if (ACT_F16) {
                        uint32_t ah[4], al[4];
                        split_f16x8(ar, ah, al);
                        const bf16x8 aop = regs_to_bf16x8(ah), aop2 = regs_to_bf16x8(al);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bh, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bm, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bl, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop2, bh, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop2, bm, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop2, bl, acc[t][g], 0, 0, 0);
                    } else {
                        const bf16x8 aop = regs_to_bf16x8(ar);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bh, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bm, acc[t][g], 0, 0, 0);
                        acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bl, acc[t][g], 0, 0, 0);
                    }
                }
            }
    }

    // D register v of lane (i, cs): row 4 cs + v, column i.  Partial tiles -> LDS -> sum over the waves.
    constexpr int TILES = ROWT * RG;
#pragma unroll
    for (int t = 0; t < ROWT; ++t)
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) lds_f[((wave * TILES + t * RG + g) * 4 + v) * 64 + lane] = acc[t][g][v];
    __syncthreads();
    for (int x = tid; x < TILES * 256; x += nthreads) {
        const int tile = x >> 8, prow = 16 * (tile / RG) + ((x >> 4) & 15), j = (tile % RG) * 16 + (x & 15);
        const int v = (x >> 4) & 3, l = 16 * ((x >> 6) & 3) + (x & 15);      // where the tile's element stands in LDS
        float sum = 0.f;
        for (int w = 0; w < nwaves; ++w) sum += lds_f[((w * TILES + tile) * 4 + v) * 64 + l];
        if (split > 1)   // a slice of the contraction: leave the tile for lora_down_finish_kernel
            a.partials[((size_t)blockIdx.y * row_blocks + blockIdx.x) * (TILES * 256) + prow * (16 * RG) + j] = sum;
        else if (m0 + prow < a.M)
            store_projection(a, m0 + prow, j, sum);
    }
}

// The same projection for many rows or a large rank (lora_down_plan()): a workgroup owns 64 rows (a tile of
// 16 per wave) and one of `split` slices of the contraction, which it walks in chunks of 128.  The factor's
// chunk is split into its three parts once per workgroup, into LDS, and every wave multiplies from there;
// the activations and factor values of two further chunks are on their way to registers meanwhile.
// Bound by a chunk's chain of split, barrier, LDS reads and MFMAs -- 1.05 us for a workgroup alone on its compute
// unit at r <= 16, 1.6 at 32, 2.3 at 64 -- into which the unit's other workgroups fall; workgroups of eight
// waves were no quicker anywhere.
constexpr int DOWN_WAVES = 4;
constexpr int DOWN_CHUNK = 128;      // contraction elements of one chunk
template <int RG, bool F_IS_A, bool ACT_F16>
__global__ __launch_bounds__(DOWN_WAVES * 64) void lora_down_tile_kernel(DownArgs a, int row_blocks, int split, Cut cut /* of the chunks over the slices */) {
    constexpr int NW = DOWN_WAVES;
    constexpr int KC = DOWN_CHUNK, ROW = KC * 2 + 16;           // bytes of an LDS row: 16 lanes of a 16-byte read meet 64 banks
    constexpr int COLS = 16 * RG, PLANE = COLS * ROW;
    constexpr int UNITS = (COLS * (KC / 8) + NW * 64 - 1) / (NW * 64);   // (column, eight elements) units per thread
    __shared__ __attribute__((aligned(16))) unsigned char planes[3 * PLANE];
    const int tid = threadIdx.x, r = a.r, C = a.C;
    // (workgroups behind the last slice write the weight-side extension: a row of them beside every slice, of which all but
    // one return at once, made a call of 1082 x 19584, r = 8, four thousand outputs, 25 us long instead of 17)
    if ((int)blockIdx.y >= split) {
        const size_t u = ((size_t)(blockIdx.y - split) * row_blocks + blockIdx.x) * (NW * 64) + tid;
        if (u < (size_t)a.Cw * (a.RE >> 3)) write_w_ext_unit(a, u);
        return;
    }
    const int lane = tid & 63, wave = uniform(tid >> 6), i = lane & 15, cs = lane >> 4;
    const int m0 = (blockIdx.x * NW + wave) * 16;
    const uint16_t *arow = a.act + (size_t)(m0 + i < a.M ? m0 + i : a.M - 1) * C + 8 * cs;
    const int ch0 = (int)cut.begin(blockIdx.y), ch1 = (int)cut.begin(blockIdx.y + 1);

    struct Chunk {
        uint4 x[KC / 32];
        float f[UNITS][8];
    };
    // column and octet of a unit: neighbouring lanes read neighbouring floats of the factor
    auto unit_at = [&](int q, int &j, int &o) {
        const int u = q * (NW * 64) + tid;
        j = F_IS_A ? u % COLS : u / (KC / 8);
        o = F_IS_A ? u / COLS : u % (KC / 8);
        return COLS * (KC / 8) % (NW * 64) == 0 || u < COLS * (KC / 8);
    };
    auto load = [&](Chunk &k, int ch) {
#pragma unroll
        for (int s = 0; s < KC / 32; ++s) {
            const int c = ch * KC + 32 * s;              // C is a multiple of 8: a lane's eight are all in or all out
            k.x[s] = make_uint4(0, 0, 0, 0);
            if (c + 8 * cs < C) k.x[s] = *reinterpret_cast<const uint4 *>(arow + c);
        }
#pragma unroll
        for (int q = 0; q < UNITS; ++q) {
            int j, o;
            const bool mine = unit_at(q, j, o);
            const int c = ch * KC + 8 * o;
#pragma unroll
            for (int e = 0; e < 8; ++e) k.f[q][e] = 0.f;
            if (mine && j < r && c < C) {
                if (F_IS_A) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) k.f[q][e] = a.Fm[(size_t)(c + e) * r + j];
                } else {
                    const float4 q0 = *reinterpret_cast<const float4 *>(a.Fm + (size_t)j * C + c);
                    const float4 q1 = *reinterpret_cast<const float4 *>(a.Fm + (size_t)j * C + c + 4);
                    k.f[q][0] = q0.x; k.f[q][1] = q0.y; k.f[q][2] = q0.z; k.f[q][3] = q0.w;
                    k.f[q][4] = q1.x; k.f[q][5] = q1.y; k.f[q][6] = q1.z; k.f[q][7] = q1.w;
                }
            }
        }
    };
    f32x4 acc[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    Chunk set[2];                                        // two chunks on their way: a trip to memory is longer than a chunk
    load(set[0], ch0);
    load(set[1], ch0 + 1 < ch1 ? ch0 + 1 : ch0);
    for (int c2 = ch0; c2 < ch1; c2 += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ch = c2 + h;
            if (ch >= ch1) break;
            Chunk &k = set[h];
            if (ch > ch0) __syncthreads();               // every wave has read the chunk before
#pragma unroll
            for (int q = 0; q < UNITS; ++q) {
                int j, o;
                if (!unit_at(q, j, o)) continue;
                uint32_t p[3][4];
                split3(k.f[q], p[0], p[1], p[2]);
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    *reinterpret_cast<uint4 *>(planes + t * PLANE + j * ROW + o * 16) = make_uint4(p[t][0], p[t][1], p[t][2], p[t][3]);
            }
            uint4 x[KC / 32];
#pragma unroll
            for (int s = 0; s < KC / 32; ++s) x[s] = k.x[s];
            if (ch + 2 < ch1) load(k, ch + 2);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < KC / 32; ++s) {
                const uint32_t ar[4] = {x[s].x, x[s].y, x[s].z, x[s].w};
                uint32_t ah[4], al[4];
                if (ACT_F16) split_f16x8(ar, ah, al);
                const bf16x8 hi = regs_to_bf16x8(ACT_F16 ? ah : ar), lo = regs_to_bf16x8(ACT_F16 ? al : ar);
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        const bf16x8 b = *reinterpret_cast<const bf16x8 *>(planes + t * PLANE + (16 * g + i) * ROW + s * 64 + cs * 16);
                        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, b, acc[g], 0, 0, 0);
                        if (ACT_F16) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, b, acc[g], 0, 0, 0);
                    }
            }
        }
    }
    // D register v of lane (i, cs): row 4 cs + v, column 16 g + i
    if (split > 1) {
        float *part = a.partials + (((size_t)blockIdx.y * row_blocks + blockIdx.x) * NW + wave) * (256 * RG);
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[(4 * cs + v) * COLS + 16 * g + i] = acc[g][v];
        return;
    }
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (m0 + 4 * cs + v < a.M) store_projection(a, m0 + 4 * cs + v, 16 * g + i, acc[g][v]);
}

// Second stage when the contraction was split over workgroups: add the slices' tiles of 16 rows
// in slice order, write P and the activation-side extension.  One workgroup per 16 rows; the
// partials of a first-stage workgroup hold its ROWT tiles one after the other.  Bound by its chain of
// loads: every element of a thread is summed side by side, eight slices at a time.
template <int RG>
__global__ __launch_bounds__(256) void lora_down_finish_kernel(DownArgs a, int row_blocks, int split, int rowt) {
    const int tid = threadIdx.x, m0 = blockIdx.x * 16;
    const int rb = blockIdx.x / rowt, tile = blockIdx.x % rowt;
    const size_t wg_floats = (size_t)rowt * 256 * RG, stride = (size_t)row_blocks * wg_floats;
    const float *src = a.partials + (size_t)rb * wg_floats + (size_t)tile * (256 * RG) + tid;
    constexpr int SB = 8;
    float sum[RG];
#pragma unroll
    for (int q = 0; q < RG; ++q) sum[q] = 0.f;
    for (int y = 0; y < split; y += SB) {
        float v[SB][RG];
#pragma unroll
        for (int u = 0; u < SB; ++u)
#pragma unroll
            for (int q = 0; q < RG; ++q) v[u][q] = y + u < split ? src[(size_t)(y + u) * stride + 256 * q] : 0.f;
#pragma unroll
        for (int u = 0; u < SB; ++u)
#pragma unroll
            for (int q = 0; q < RG; ++q)
                if (y + u < split) sum[q] += v[u][q];
    }
#pragma unroll
    for (int q = 0; q < RG; ++q) {
        const int x = tid + 256 * q, prow = x / (16 * RG), j = x % (16 * RG);
        if (m0 + prow < a.M) store_projection(a, m0 + prow, j, sum[q]);
    }
}

template <int RG, int ROWT>
static hipError_t launch_down_rg(const DownArgs &a, const DownPlan &plan, hipStream_t stream) {
    constexpr int ROWS = 16 * ROWT;
    const int row_blocks = (a.M + ROWS - 1) / ROWS;
    const int nwaves = plan.nwaves, nthreads = nwaves * 64, split = plan.split;
    const int w_blocks = a.w_ext ? (int)(((size_t)a.Cw * (a.RE / 8) + nthreads - 1) / nthreads) : 0;
    const size_t lds = (size_t)(nwaves * RG * ROWT * 256) * sizeof(float);
    const dim3 grid(row_blocks + w_blocks, split);
    const Cut cut = make_cut((a.C + 31) / 32, split * nwaves);
    if constexpr (RG == 2 && ROWT == 4) {
        // long calls of such a rank go by tiles, but for a bfloat16 forward call with little scratch (lora_down_row_bytes())
        if (a.act_f16 || !a.f_is_A) return hipErrorInvalidValue;
        launch_kernel("lora_down", lora_down_kernel<RG, ROWT, true, false>, grid, nthreads, lds, stream, a, row_blocks, split, cut);
    } else if (a.act_f16) {
        if (a.f_is_A)
            launch_kernel("lora_down", lora_down_kernel<RG, ROWT, true, true>, grid, nthreads, lds, stream, a, row_blocks, split, cut);
        else
            launch_kernel("lora_down", lora_down_kernel<RG, ROWT, false, true>, grid, nthreads, lds, stream, a, row_blocks, split, cut);
    } else if (a.f_is_A) {
        launch_kernel("lora_down", lora_down_kernel<RG, ROWT, true, false>, grid, nthreads, lds, stream, a, row_blocks, split, cut);
    } else {
        launch_kernel("lora_down", lora_down_kernel<RG, ROWT, false, false>, grid, nthreads, lds, stream, a, row_blocks, split, cut);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || split <= 1) return e;
    launch_kernel("lora_down_finish", lora_down_finish_kernel<RG>, (a.M + 15) / 16, 256, 0, stream, a, row_blocks, split, ROWT);
    return hipGetLastError();
}

template <int RG>
static hipError_t launch_down_tiles(const DownArgs &a, const DownPlan &plan, hipStream_t stream) {
    const int row_blocks = (a.M + 16 * DOWN_WAVES - 1) / (16 * DOWN_WAVES), split = plan.split;
    const int w_blocks = a.w_ext ? (int)(((size_t)a.Cw * (a.RE / 8) + DOWN_WAVES * 64 - 1) / (DOWN_WAVES * 64)) : 0;
    const dim3 grid(row_blocks, split + (w_blocks + row_blocks - 1) / row_blocks);
    const Cut cut = make_cut((a.C + DOWN_CHUNK - 1) / DOWN_CHUNK, split);
    if (a.act_f16) {
        if (a.f_is_A) launch_kernel("lora_down", lora_down_tile_kernel<RG, true, true>, grid, DOWN_WAVES * 64, 0, stream, a, row_blocks, split, cut);
        else launch_kernel("lora_down", lora_down_tile_kernel<RG, false, true>, grid, DOWN_WAVES * 64, 0, stream, a, row_blocks, split, cut);
    } else if (a.f_is_A) {
        launch_kernel("lora_down", lora_down_tile_kernel<RG, true, false>, grid, DOWN_WAVES * 64, 0, stream, a, row_blocks, split, cut);
    } else {
        launch_kernel("lora_down", lora_down_tile_kernel<RG, false, false>, grid, DOWN_WAVES * 64, 0, stream, a, row_blocks, split, cut);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || split <= 1) return e;
    launch_kernel("lora_down_finish", lora_down_finish_kernel<RG>, (a.M + 15) / 16, 256, 0, stream, a, row_blocks, split, DOWN_WAVES);
    return hipGetLastError();
}

hipError_t launch_lora_down(const DownArgs &a, hipStream_t stream) {
    DownPlan plan = lora_down_plan(a.M, a.C, a.r);
    if (down_plan_bytes(plan, a.M, a.r) > a.partials_bytes) plan = lora_down_row_plan(a.M, a.C, a.r);
    if (plan.tiles) {
        switch ((a.r + 15) / 16) {
            case 1: return launch_down_tiles<1>(a, plan, stream);
            case 2: return launch_down_tiles<2>(a, plan, stream);
            case 3: return launch_down_tiles<3>(a, plan, stream);
            default: return launch_down_tiles<4>(a, plan, stream);
        }
    }
    if (plan.rowt == 4) {
        if (a.r <= 16) return launch_down_rg<1, 4>(a, plan, stream);
        return launch_down_rg<2, 4>(a, plan, stream);
    }
    if (a.r <= 16) return launch_down_rg<1, 1>(a, plan, stream);
    if (a.r <= 32) return launch_down_rg<2, 1>(a, plan, stream);
    if (a.r <= 48) return launch_down_rg<3, 1>(a, plan, stream);
    return launch_down_rg<4, 1>(a, plan, stream);
}

// ---------------------------------------------------------------------------
// Adapter gradients (Section 3.1.1), both in one launch:
//   dA[k][j] = s * sum_m X[m][k]  dYBt[m][j]      dB[j][n] = s * sum_m XA[m][j] dY[m][n]
// on the matrix cores: per 32 rows, P^T (16 adapter columns x 32 rows; P = dYBt or XA, its fp32
// values split exactly into three bfloat16 parts) times a 32-row block of X or dY.
//
// Bound by the read of X and dY.  On the vector ALUs (64 multiply-adds per row and lane at r = 16)
// it was bound by those instead: 30 + 4 us (the 4 a second launch that added row chunks) at
// 2048 x (4096 + 11008), r = 16, 20 + 4 at 777 x (11008 + 4096), 96 + 7 at 2048 x 16384, r = 64; now 14,
// 9.5 and 26 us.  247 MB at 4096 x (8192 + 22016), r = 8: 47 + 4 -> 47 us, 5.3 TB/s.
//
// A lane loads CPL adjacent columns of the eight rows that it holds of the contraction, so 16 lanes
// read 32 CPL contiguous bytes of a row; column c + q of the eight rows is then gathered with four
// byte permutes and is the MFMA's right operand as it stands -- no transposed load, no LDS.  The
// waves of a workgroup take blocks of 32 rows in turn and add their sums in LDS at the end, so one
// workgroup can own a block of columns over all rows and write the gradient itself.
//   CPL   4 (128-byte pieces; twice the workgroups): the data of a few thousand rows come out of the
//         last-level cache and what counts is the number of compute units that pull (6656 x 2, M = 1024:
//         7.9 us against 9.4).  8 (256-byte pieces) from 128 MB on, where HBM does the work (247 MB:
//         47 us against 55; r = 32: 55 against 72), for r <= 32; beyond that eight columns'
//         accumulators leave too few waves (r = 64 at 2048 x 16384: 26 us against 43).
//         From 257 rows on (16 waves) registers let two workgroups share a compute unit only at CPL 4, r <= 16,
//         bfloat16; the others run 256 workgroups at a time, and 257 ... 512 blocks of 64 columns as two
//         rounds: there 8 goes from the first row past 256 on (binary16, r = 8, 8192 + 8320 columns: M = 256 5.6
//         against 6.1 us, 400 10.4 -> 8.3, 1536 21.8 -> 18.0, 3000 39.1 -> 30.5; 8192 + 22016: M = 256 5.9 against 6.5,
//         1024 17.6 -> 16.2; more blocks, 22016 x 2: M = 1024 25.1 against 27.3; not binary16 with r > 16, where
//         it is up to 7 % the slower from 1280 rows on).  So it does where 129 ... 170 blocks of 64 columns allow
//         one chunk of rows, but half as many of 128 three (binary16, 4096 + 4224 columns, M = 4096: 25.0 -> 21.1).
//   rows  in chunks that leave partials for a reduction launch (4 us) where the columns are too
//         few to occupy the chip and at least 1024 rows remain to each: 256 + 256 columns, M = 4096:
//         14.4 -> 6.4 + 4.1 us; 2048 + 2048: 16.3 -> 9.3 + 4.2; a chunk of 512 rows gains less than
//         the launch costs (4096 + 11008, M = 2048: 14.4 -> 13.0 + 4.0).
//         Where the blocks leave compute units idle in the last round of 256: up to five chunks where the
//         rounds that they save, at 4.5 TB/s, outweigh the second launch and its partials and enough rows
//         remain.  8192 + 8320 columns (129 blocks), M = 8192: one chunk 53.0 us, three 48.1; binary16 72.4,
//         five 59.6; M = 16384: 135 and 152, five 104 and 113; r = 64 at M = 4096: 75.8, three 65.0; r = 8,
//         too few rows: 26.7, three 28.5.  6144 + 6144 columns, M = 16384: two chunks 84.7, five 80.0.
//         Over 656 timed shapes of 4096 ... 44032 columns and 1536 ... 16384 rows the choice is on average
//         3 % slower than the best of the eight or sixteen timed (one or two widths, one to eight chunks).
// No atomics (device-scope fp32 atomics bypass the per-XCD L2 and are slow), no zero-fill.
// ---------------------------------------------------------------------------
GradGeom grad_geom(int M, int K, int N, int r, bool f16) {
    GradGeom g;
    g.rg = r > 0 ? (r + 15) / 16 : 1;
    const bool pair = !f16 && g.rg == 1;             // two workgroups of CPL 4 share a compute unit
    const int blocks4 = (K + 63) / 64 + (N + 63) / 64;
    const bool wide = (size_t)M * ((size_t)K + N) * 2 >= (size_t)128 << 20 ||
                      (!pair && ((blocks4 > 256 && blocks4 <= 512 && M > 256 && !(f16 && g.rg == 2)) || (blocks4 > 128 && blocks4 <= 170 && M >= 3 * 960)));
    g.cpl = g.rg <= 2 && wide ? 8 : 4;
    const int wcols = 16 * g.cpl;
    g.cols_a = (K + wcols - 1) / wcols;
    g.cols_b = (N + wcols - 1) / wcols;
    const int blocks = g.cols_a + g.cols_b, fewest = !pair && g.cpl == 8 ? 960 : 1024;
    int chunks = 256 / blocks;
    if (chunks > M / fewest) chunks = M / fewest;
    if (chunks < 1) chunks = 1;
    if (!(pair && g.cpl == 4)) {
        const double bytes = (double)M * ((double)K + N) * 2.0;
        const auto us = [&](int c) {                 // rounds of 256 workgroups, and what a second launch adds
            const long n = (long)blocks * c;
            return bytes / 4.5e6 * (double)((n + 255) / 256 * 256) / (double)n + (c > 1 ? 4.0 + c * ((double)K + N) * r * 8.0 / 4.0e6 : 0.0);
        };
        for (int c = chunks + 1; c <= 5 && M / c >= (pair ? 2048 : 1365); ++c)
            if (us(c) < us(chunks)) chunks = c;
    }
    const int rows = ((M + chunks - 1) / chunks + 31) / 32 * 32;
    g.rows_per_block = rows;
    g.chunks = (M + rows - 1) / rows;
    const int most = g.rg * g.cpl <= 8 ? 16 : 8;     // their sums meet in at most 64 KB of LDS
    g.nwaves = 1;
    while (g.nwaves < most && g.nwaves * 32 < rows) g.nwaves *= 2;
    g.partial_floats = (size_t)g.chunks * (size_t)(K + N) * (size_t)(r > 0 ? r : 0);
    return g;
}

// RG: groups of 16 adapter columns; CPL: adjacent columns of X / dY per lane; F16: the activations are
// binary16 (paper-literal path) instead of bfloat16.
template <int RG, int CPL, bool F16>
__global__ __launch_bounds__(RG * CPL <= 8 ? 1024 : 512) void lora_grad_partial_kernel(GradPairArgs a, GradGeom g) {
    extern __shared__ __attribute__((aligned(16))) float red[];   // [nwaves / 2][CPL * RG * 4][64]
    typedef uint32_t words_t __attribute__((ext_vector_type(CPL / 2)));
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int i = lane & 15, cs = lane >> 4;
    const bool is_a = (int)blockIdx.x < g.cols_a;
    const uint16_t *__restrict__ act = is_a ? a.X : a.dY;
    const float *__restrict__ P = is_a ? a.dYBt : a.XA;   // [M][r]
    const int C = is_a ? a.K : a.N, r = a.r;
    const int c = (is_a ? blockIdx.x : blockIdx.x - g.cols_a) * (16 * CPL) + CPL * i;
    const bool col_ok = c < C;                            // C is a multiple of 8: all CPL columns or none
    const int m_begin = blockIdx.y * g.rows_per_block;
    const int m_end = m_begin + g.rows_per_block < a.M ? m_begin + g.rows_per_block : a.M;
    const uint16_t *col = act + (col_ok ? c : 0);

    f32x4 acc[CPL][RG];
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
        for (int t = 0; t < RG; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int mb = m_begin + 32 * wave; mb < m_end; mb += 32 * nwaves) {
        const int m8 = mb + 8 * cs;                       // this lane's eight rows of the contraction
        words_t x[8];
        float p[RG][8];
        if (mb + 32 <= m_end) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = *reinterpret_cast<const words_t *>(col + (size_t)(m8 + e) * C);
#pragma unroll
            for (int t = 0; t < RG; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    p[t][e] = 0.f;
                    if (16 * t + i < r) p[t][e] = P[(size_t)(m8 + e) * r + 16 * t + i];
                }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] = words_t(0u);
                if (m8 + e < m_end) x[e] = *reinterpret_cast<const words_t *>(col + (size_t)(m8 + e) * C);
            }
#pragma unroll
            for (int t = 0; t < RG; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    p[t][e] = 0.f;
                    if (16 * t + i < r && m8 + e < m_end) p[t][e] = P[(size_t)(m8 + e) * r + 16 * t + i];
                }
        }
        bf16x8 ph[RG], pm[RG], pl[RG];
#pragma unroll
        for (int t = 0; t < RG; ++t) {
            uint32_t hi[4], mid[4], lo[4];
            split3(p[t], hi, mid, lo);
            ph[t] = regs_to_bf16x8(hi);
            pm[t] = regs_to_bf16x8(mid);
            pl[t] = regs_to_bf16x8(lo);
        }
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            uint32_t b[4];                                // column c + q of the eight rows
#pragma unroll
            for (int e = 0; e < 4; ++e)
                b[e] = __builtin_amdgcn_perm(x[2 * e + 1][q / 2], x[2 * e][q / 2], q & 1 ? 0x07060302u : 0x05040100u);
            if (F16) {
                uint32_t bh[4], bl[4];
                split_f16x8(b, bh, bl);
                const bf16x8 oh = regs_to_bf16x8(bh), ol = regs_to_bf16x8(bl);
#pragma unroll
                for (int t = 0; t < RG; ++t) {
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph[t], oh, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pm[t], oh, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl[t], oh, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph[t], ol, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pm[t], ol, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl[t], ol, acc[q][t], 0, 0, 0);
                }
            } else {
                const bf16x8 o = regs_to_bf16x8(b);
#pragma unroll
                for (int t = 0; t < RG; ++t) {
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ph[t], o, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pm[t], o, acc[q][t], 0, 0, 0);
                    acc[q][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl[t], o, acc[q][t], 0, 0, 0);
                }
            }
        }
    }

    // An infinity has no exact split (inf - inf is NaN) and meets the zero parts of the other operand
    // (inf * 0).  A wave that finds a NaN among its sums adds its rows again with fp32 multiply-adds, which
    // give what the definition does (every dY NaN, 4096 x (8192 + 22016), r = 8: 161 us a call instead of 42).
    bool nan = false;
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
        for (int t = 0; t < RG; ++t)             // a compare tells of two sums whether either is NaN
            nan |= __builtin_isunordered(acc[q][t][0], acc[q][t][1]) | __builtin_isunordered(acc[q][t][2], acc[q][t][3]);
    if (__builtin_expect(__any(nan), 0)) {
#pragma unroll
        for (int q = 0; q < CPL; ++q)
#pragma unroll
            for (int t = 0; t < RG; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        int c_again = c;
        asm("" : "+v"(c_again));                         // addresses of its own: none stays alive for it in the loop above
        const uint16_t *col_again = act + (c_again < C ? c_again : 0);
        for (int mb = m_begin + 32 * wave; mb < m_end; mb += 32 * nwaves)
            for (int m = mb; m < mb + 32 && m < m_end; ++m) {
                const words_t x = *reinterpret_cast<const words_t *>(col_again + (size_t)m * C);
#pragma unroll
                for (int t = 0; t < RG; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int j = 16 * t + 4 * cs + v;       // the layout of the sums, see below
                        const float p = j < r ? P[(size_t)m * r + j] : 0.f;
#pragma unroll
                        for (int q = 0; q < CPL; ++q) {
                            const uint32_t bits = q & 1 ? x[q / 2] >> 16 : x[q / 2] & 0xFFFFu;
                            const float xq = F16 ? half_bits_to_float((uint16_t)bits) : __uint_as_float(bits << 16);
                            acc[q][t][v] = __builtin_fmaf(xq, p, acc[q][t][v]);
                        }
                    }
            }
    }

    // the waves' sums meet in LDS, half of the waves handing theirs to the other half at a time
    constexpr int FL = CPL * RG * 4;
    for (int half = nwaves >> 1; half > 0; half >>= 1) {
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int q = 0; q < CPL; ++q)
#pragma unroll
                for (int t = 0; t < RG; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[((wave - half) * FL + (q * RG + t) * 4 + v) * 64 + lane] = acc[q][t][v];
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int q = 0; q < CPL; ++q)
#pragma unroll
                for (int t = 0; t < RG; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[q][t][v] += red[(wave * FL + (q * RG + t) * 4 + v) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave != 0 || !col_ok) return;
    // a single row chunk is the whole sum: finish here (scale, accumulate flag) in the outputs
    // themselves, which have the layout of a partial, and skip the reduction launch
    const bool direct = g.chunks == 1;
    float *part = a.partials + (size_t)blockIdx.y * ((size_t)(a.K + a.N) * r);
    const bool add_old = direct && a.accumulate;
    const float scale = direct ? a.lora_scale : 1.0f;
    // accumulator register v of this lane: adapter column 16 t + 4 cs + v, activation column c + q
    if (is_a) {
        float *base = (direct ? a.dA : part) + (size_t)c * r;
#pragma unroll
        for (int q = 0; q < CPL; ++q)
#pragma unroll
            for (int t = 0; t < RG; ++t) {
                const int j = 16 * t + 4 * cs;
                float *dst = base + (size_t)q * r + j;
                if ((r & 3) == 0) {
                    if (j < r) {
                        float4 o = make_float4(scale * acc[q][t][0], scale * acc[q][t][1], scale * acc[q][t][2], scale * acc[q][t][3]);
                        if (add_old) {
                            const float4 old = *reinterpret_cast<const float4 *>(dst);
                            o.x += old.x; o.y += old.y; o.z += old.z; o.w += old.w;
                        }
                        *reinterpret_cast<float4 *>(dst) = o;
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (j + v < r) dst[v] = add_old ? dst[v] + scale * acc[q][t][v] : scale * acc[q][t][v];
                }
            }
    } else {
        float *base = (direct ? a.dB : part + (size_t)a.K * r) + c;
#pragma unroll
        for (int t = 0; t < RG; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = 16 * t + 4 * cs + v;
                if (j >= r) continue;
#pragma unroll
                for (int q = 0; q < CPL; q += 4) {
                    float4 o = make_float4(scale * acc[q][t][v], scale * acc[q + 1][t][v], scale * acc[q + 2][t][v], scale * acc[q + 3][t][v]);
                    float4 *dst = reinterpret_cast<float4 *>(base + (size_t)j * a.N + q);
                    if (add_old) {
                        const float4 old = *dst;
                        o.x += old.x; o.y += old.y; o.z += old.z; o.w += old.w;
                    }
                    *dst = o;
                }
            }
    }
}

// out = (accumulate ? out : 0) + s * sum over chunks; 4 consecutive elements per thread.
__global__ __launch_bounds__(256) void lora_grad_reduce_kernel(GradPairArgs a, int chunks) {
    const size_t n_a = (size_t)a.K * a.r, n = n_a + (size_t)a.N * a.r;
    const size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (e >= n) return;
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    const float *p = a.partials + e;
    int q = 0;
    for (; q + 4 <= chunks; q += 4) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4 *>(p + (size_t)(q + u) * n);
#pragma unroll
        for (int u = 0; u < 4; ++u) { sum.x += v[u].x; sum.y += v[u].y; sum.z += v[u].z; sum.w += v[u].w; }
    }
    for (; q < chunks; ++q) {
        const float4 v = *reinterpret_cast<const float4 *>(p + (size_t)q * n);
        sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    float4 *dst = reinterpret_cast<float4 *>(e < n_a ? a.dA + e : a.dB + (e - n_a));
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.accumulate) o = *dst;
    o.x = __builtin_fmaf(a.lora_scale, sum.x, o.x);
    o.y = __builtin_fmaf(a.lora_scale, sum.y, o.y);
    o.z = __builtin_fmaf(a.lora_scale, sum.z, o.z);
    o.w = __builtin_fmaf(a.lora_scale, sum.w, o.w);
    *dst = o;
}

template <int RG, int CPL>
static hipError_t launch_grad(const GradPairArgs &a, const GradGeom &g, hipStream_t stream) {
    const dim3 grid(g.cols_a + g.cols_b, g.chunks);
    const size_t lds = (size_t)(g.nwaves / 2) * CPL * RG * 4 * 64 * sizeof(float);
    if (a.f16) launch_kernel("lora_grad", lora_grad_partial_kernel<RG, CPL, true>, grid, g.nwaves * 64, lds, stream, a, g);
    else launch_kernel("lora_grad", lora_grad_partial_kernel<RG, CPL, false>, grid, g.nwaves * 64, lds, stream, a, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || g.chunks == 1) return e;
    const size_t n = (size_t)(a.K + a.N) * a.r;
    launch_kernel("lora_grad_reduce", lora_grad_reduce_kernel, (unsigned)((n / 4 + 255) / 256), 256, 0, stream, a, g.chunks);
    return hipGetLastError();
}

hipError_t launch_lora_grad_pair(const GradPairArgs &a, hipStream_t stream) {
    const GradGeom g = grad_geom(a.M, a.K, a.N, a.r, a.f16 != 0);
    switch (g.rg) {
        case 1: return g.cpl == 8 ? launch_grad<1, 8>(a, g, stream) : launch_grad<1, 4>(a, g, stream);
        case 2: return g.cpl == 8 ? launch_grad<2, 8>(a, g, stream) : launch_grad<2, 4>(a, g, stream);
        case 3: return launch_grad<3, 4>(a, g, stream);
        default: return launch_grad<4, 4>(a, g, stream);
    }
}

}  // namespace mlr
