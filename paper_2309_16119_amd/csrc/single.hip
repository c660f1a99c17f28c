// The forward call of a handful of tokens through a small layer in one launch.
//
// The streaming kernels (smallm.hip) cut the contraction into slices so that every compute unit reads a share of the
// packed weight, and a second launch adds the slices and the adapter term.  For a small layer both launches are
// mostly their own start and end (4 us each, with a product of less than one).  Here a workgroup owns 16 or 64
// output columns and the whole contraction, which its eight waves share: they meet in LDS, and the rank-r projection of
// the rows is computed by every workgroup for itself beside the product -- that repeated work is what bounds the size of
// the layer (single_wins()).  Same arithmetic as smallm.hip: the codes themselves enter the matrix cores, weights are never
// rounded to 16 bits, the projection is exact products summed in fp32.  Bound by one trip to memory for everything (all of a
// wave's first units are on their way before the first is waited for) and the start of the launch.
// Measured, us of a call's kernels with two launches / here (8 tokens or fewer): 256 x 2304, r = 8 9.6 / 4.1; 768 x 2432
// 9.2 / 5.3; 1024 x 2048 8.9 / 6.0; 2048 x 1200 9.6 / 6.3; 512 x 11008, r = 64 11.6 / 11.0; 256 x 17000, r = 8 11.1 / 9.
// (Backward the same plan lost: a workgroup needs 128 columns, so few of them each dequantize their columns' whole
// contraction: 512 x 2304 8.4 / 12.7 us, 256 x 512 8.3 / 7.2.)
#include "gemm_common.h"
#include "launch.h"
#include "small_codes.h"

namespace mlr {

namespace single {
constexpr int NWAVES = 8, THREADS = NWAVES * 64;
}

struct SingleDev {
    LayerView w;
    const uint16_t *act;       // [M][K]
    const float *A, *B;        // [K][r], [r][N]
    int M, r;
    float lora_scale;
    uint16_t *out;
    float *P_out;              // [M][r] or NULL
    const uint16_t *zeros16, *bias16;
    uint32_t spg_plus, spg_magic;      // quantization group of a step, (step + plus) * magic / 2^32
};

// Sum of the waves' parts of the projection: P[row][16 RG], row stride 16 RG + 4, and its hand-off by the first workgroup.
template <int RG>
__device__ __forceinline__ void single_projection(const SingleDev &d, const float *red, float *Ps) {
    using namespace single;
    constexpr int PS = 16 * RG + 4;
    for (int x = threadIdx.x; x < RG * 256; x += THREADS) {
        const int g = x >> 8, v = (x >> 6) & 3, l = x & 63;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NWAVES; ++w) sum += red[((w * RG + g) * 4 + v) * 64 + l];
        const int row = 4 * (l >> 4) + v, j = g * 16 + (l & 15);
        Ps[row * PS + j] = sum;
        if (blockIdx.x == 0 && d.P_out != nullptr && row < d.M && j < d.r) d.P_out[(size_t)row * d.r + j] = sum;
    }
}

// D += act F for one operand of 16-bit activations and the fp32 factor values that belong to it, products exact
template <bool F16>
__device__ __forceinline__ f32x4 single_project(const uint32_t a[4], const float f[8], f32x4 acc) {
    uint32_t p[3][4], h[2][4];
    split3(f, p[0], p[1], p[2]);
    if (F16) split_f16x8(a, h[0], h[1]);
#pragma unroll
    for (int x = 0; x < (F16 ? 2 : 1); ++x)
#pragma unroll
        for (int t = 0; t < 3; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sm::as_bf16x8(F16 ? h[x] : a), sm::as_bf16x8(p[t]), acc, 0, 0, 0);
    return acc;
}

// A unit is 32 contraction elements, one MFMA deep: four bits, a word of each lane group (lane l = 16 j + i: column(s)
// of i, lane group j); two bits, half of the 16 codes of its word; three bits, one of the four 8-code chunks of its
// 32-code block.  Wave w takes units w, w + 8, ..., U of them in flight.  Columns of a workgroup: 16 CT, CT adjacent ones per lane.
template <int BITS, bool F16, int RG, int CT>
__global__ __launch_bounds__(single::THREADS, 2) void single_kernel(SingleDev d) {
    using namespace single;
    using NF = sm::Num<F16>;
    constexpr int NC = sm::Geo<BITS>::NC, NWORDS = BITS == 3 ? 2 : 1, U = RG == 1 ? 4 : 2, R = 16 * RG, PS = R + 4;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *red_y = smem, *red_p = red_y + NWAVES * CT * 256, *Ps = red_p + NWAVES * RG * 256, *Bs = Ps + 16 * PS;      // Bs [R][16 CT]
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int i = lane & 15, j = lane >> 4, K = d.w.K, N = d.w.N, r = d.r, M = d.M;
    const int n0 = blockIdx.x * 16 * CT;
    int n = n0 + CT * i;
    if (n > N - CT) n = N - CT;                     // N is a multiple of 8; stores are masked
    const uint16_t *xrow = d.act + (size_t)(i < M ? i : M - 1) * K;      // rows past M repeat the last one, never stored
    const int units = K / 32;

    // the adapter's rows at these columns, on their way first and needed last
    constexpr int B4 = (R * 4 * CT + THREADS - 1) / THREADS;
    float4 bq[B4];
#pragma unroll
    for (int q = 0; q < B4; ++q) {
        const int x = q * THREADS + tid, row = x / (4 * CT), c = n0 + x % (4 * CT) * 4;
        bq[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row < r && c < N) bq[q] = *reinterpret_cast<const float4 *>(d.B + (size_t)row * N + c);
    }
    struct Stage {
        uint32_t w[NWORDS][CT], x[4], sc[(CT + 1) / 2], z[F16 ? (CT + 1) / 2 : 1];
        float f[RG][8];
    };
    auto load = [&](Stage &s, int u) {
        if (u > units - 1) u = units - 1;
        const int step = u / NC, c = u % NC;
        const uint32_t *row = d.w.qweight + (size_t)(4 * step + j) * sm::Geo<BITS>::WORDS * N + n;
        const int lo = BITS == 3 ? (24 * c) >> 5 : 0;
        auto words_at = [&](uint32_t *dst, const uint32_t *src) {
            if (CT == 1) dst[0] = *src;
            else {
                const uint4 v = *reinterpret_cast<const uint4 *>(src);
                dst[0] = v.x; dst[1] = v.y; dst[CT > 2 ? 2 : 0] = v.z; dst[CT > 3 ? 3 : 0] = v.w;
            }
        };
        words_at(s.w[0], row + (size_t)lo * N);
        if (BITS == 3) words_at(s.w[NWORDS - 1], row + (size_t)(lo < 2 ? lo + 1 : 2) * N);
        const int k = BITS == 4 ? 32 * u + 8 * j : BITS == 3 ? 128 * step + 32 * j + 8 * c : 64 * step + 16 * j + 4 * c;
        if (BITS == 2) {
            const uint2 a = *reinterpret_cast<const uint2 *>(xrow + k), b = *reinterpret_cast<const uint2 *>(xrow + k + 8);
            s.x[0] = a.x; s.x[1] = a.y; s.x[2] = b.x; s.x[3] = b.y;
        } else {
            const uint4 a = *reinterpret_cast<const uint4 *>(xrow + k);
            s.x[0] = a.x; s.x[1] = a.y; s.x[2] = a.z; s.x[3] = a.w;
        }
        const size_t g = (size_t)__umulhi((uint32_t)step + d.spg_plus, d.spg_magic) * N + n;
        auto halves_at = [&](uint32_t *dst, const uint16_t *src) {
            if (CT == 1) dst[0] = *src;
            else {
                const uint2 v = *reinterpret_cast<const uint2 *>(src);
                dst[0] = v.x; dst[CT > 2 ? 1 : 0] = v.y;
            }
        };
        halves_at(s.sc, d.w.scales + g);
        if (F16) halves_at(s.z, d.zeros16 + g);
        else s.z[0] = CT == 1 ? (uint32_t)d.w.zeros[g] : *reinterpret_cast<const uint32_t *>(d.w.zeros + g);
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const int col = 16 * q + i;
            const float *f = d.A + (size_t)k * r + (col < r ? col : 0);
#pragma unroll
            for (int e = 0; e < 8; ++e) s.f[q][e] = r > 0 ? f[(size_t)(e < 4 ? e : (BITS == 2 ? 4 + e : e)) * r] : 0.f;
        }
    };
    const uint32_t ones4[4] = {NF::ONES, NF::ONES, NF::ONES, NF::ONES}, offs4[4] = {NF::MAGIC3, NF::MAGIC3, NF::MAGIC3, NF::MAGIC3};
    const bf16x8 ones = sm::as_bf16x8(ones4), offs = sm::as_bf16x8(offs4);
    const sm::CodeMasks masks = sm::make_masks<BITS, F16>();
    f32x4 y[CT], P[RG];
#pragma unroll
    for (int t = 0; t < CT; ++t) y[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < RG; ++q) P[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const Stage &s, int u) {
        // elements 0 .. 3 and 4 .. 7 of the lane side by side, as the code registers pair them
        uint32_t a4[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) a4[p] = __builtin_amdgcn_perm(s.x[2 + (p >> 1)], s.x[p >> 1], p & 1 ? 0x07060302u : 0x05040100u);
        const bf16x8 a = sm::as_bf16x8(a4);
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        const f32x4 xsum = sm::mma<F16>(a, ones, zero4), off = BITS == 3 ? sm::mma<F16>(a, offs, zero4) : xsum;
        f32x4 start;      // minus what the operands' offsets add
#pragma unroll
        for (int v = 0; v < 4; ++v) start[v] = BITS == 3 ? -off[v] : -NF::OFFSET * off[v];
        const int c = u % NC;
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const uint32_t x = BITS == 4 ? s.w[0][t] : BITS == 2 ? s.w[0][t] >> (8 * c) : __builtin_amdgcn_alignbit(s.w[NWORDS - 1][t], s.w[0][t], (24 * c) & 31);
            uint32_t o[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int sh = BITS == 3 ? 3 * p - 4 : BITS * p;
                o[p] = sm::and_or(sh < 0 ? x << (-sh) : x >> (sh < 0 ? 0 : sh), masks.field, masks.magic);
            }
            const f32x4 qx = sm::mma<F16>(a, sm::as_bf16x8(o), start);
            const float scale = half_bits_to_float((uint16_t)(s.sc[t >> 1] >> (16 * (t & 1))));
            const float z = F16 ? half_bits_to_float((uint16_t)(s.z[F16 ? t >> 1 : 0] >> (16 * (t & 1)))) : (float)((s.z[0] >> (8 * t)) & 0xFFu);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (F16) y[t][v] = __builtin_fmaf(scale, qx[v], __builtin_fmaf(z, xsum[v], y[t][v]));
                else y[t][v] = __builtin_fmaf(scale, __builtin_fmaf(-z, xsum[v], qx[v]), y[t][v]);
            }
        }
        if (r > 0) {
#pragma unroll
            for (int q = 0; q < RG; ++q) {
                const bool mine = 16 * q + i < r;
                float f[8];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    f[2 * p] = mine ? s.f[q][p] : 0.f;
                    f[2 * p + 1] = mine ? s.f[q][p + 4] : 0.f;
                }
                P[q] = single_project<F16>(a4, f, P[q]);
            }
        }
    };
    Stage st[U];
#pragma unroll
    for (int q = 0; q < U; ++q) load(st[q], wave + NWAVES * q);
#pragma unroll
    for (int q = 0; q < B4; ++q)
        if (q * THREADS + tid < R * 4 * CT) *reinterpret_cast<float4 *>(Bs + 4 * (q * THREADS + tid)) = bq[q];
    for (int u = wave; u < units; u += NWAVES * U) {
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (u + NWAVES * q < units) {
                compute(st[q], u + NWAVES * q);
                load(st[q], u + NWAVES * (q + U));
            }
    }
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) red_y[((wave * CT + t) * 4 + v) * 64 + lane] = y[t][v];
#pragma unroll
    for (int q = 0; q < RG; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) red_p[((wave * RG + q) * 4 + v) * 64 + lane] = P[q][v];
    __syncthreads();
    single_projection<RG>(d, red_p, Ps);
    __syncthreads();
    // two adjacent columns of a row: T threads side by side share the waves' sums and the rank
    constexpr int T = 4 / CT;
    const int part = tid % T, pair = tid / T, m = pair / (8 * CT), c0 = 2 * (pair % (8 * CT)), v = m & 3;
    float o[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int t = (c0 + h) % CT, l = 16 * (m >> 2) + (c0 + h) / CT;
        float sum = 0.f, ad = 0.f;
#pragma unroll
        for (int w = 0; w < NWAVES / T; ++w) sum += red_y[(((part * (NWAVES / T) + w) * CT + t) * 4 + v) * 64 + l];
        if (r > 0) {
#pragma unroll 8
            for (int q = 0; q < R / T; ++q) ad = __builtin_fmaf(Ps[m * PS + part * (R / T) + q], Bs[(part * (R / T) + q) * 16 * CT + c0 + h], ad);
        }
        o[h] = __builtin_fmaf(d.lora_scale, ad, sum);
        if (T > 1) o[h] += __shfl_xor(o[h], 1, 64);
        if (T > 2) o[h] += __shfl_xor(o[h], 2, 64);
    }
    const int col = n0 + c0;
    if (part != 0 || m >= M || col >= N) return;
    if (F16 && d.bias16 != nullptr) {
        const uint32_t b = *reinterpret_cast<const uint32_t *>(d.bias16 + col);
        o[0] += half_bits_to_float((uint16_t)(b & 0xFFFFu));
        o[1] += half_bits_to_float((uint16_t)(b >> 16));
    }
    *reinterpret_cast<uint32_t *>(d.out + (size_t)m * N + col) = sm::pack16<F16>(o[0], o[1]);
}

namespace {
template <int BITS, bool F16, int RG, int CT>
hipError_t launch_single_ct(const SingleDev &d, hipStream_t stream) {
    constexpr int R = 16 * RG;
    constexpr size_t LDS = (size_t)(single::NWAVES * (CT + RG) * 256 + 16 * (R + 4) + R * 16 * CT) * 4;
    auto kern = single_kernel<BITS, F16, RG, CT>;
    static bool configured[64] = {};
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void *>(kern), LDS, configured);
    if (e != hipSuccess) return e;
    launch_kernel(F16 ? "f16_stream_fwd_single" : "stream_fwd_single", kern, (d.w.N + 16 * CT - 1) / (16 * CT), single::THREADS, LDS, stream, d);
    return hipGetLastError();
}
template <int BITS, bool F16, int RG>
hipError_t launch_single_rg(const SingleDev &d, bool wide, hipStream_t stream) {
    return wide ? launch_single_ct<BITS, F16, RG, 4>(d, stream) : launch_single_ct<BITS, F16, RG, 1>(d, stream);
}
template <int BITS, bool F16>
hipError_t launch_single_bits(const SingleDev &d, bool wide, hipStream_t stream) {
    if (d.r <= 16) return launch_single_rg<BITS, F16, 1>(d, wide, stream);
    return d.r <= 32 ? launch_single_rg<BITS, F16, 2>(d, wide, stream) : launch_single_rg<BITS, F16, 4>(d, wide, stream);
}
template <bool F16>
hipError_t launch_single_any(const SingleDev &d, bool wide, hipStream_t stream) {
    switch (d.w.bits) {
        case 2: return launch_single_bits<2, F16>(d, wide, stream);
        case 3: return launch_single_bits<3, F16>(d, wide, stream);
        default: return launch_single_bits<4, F16>(d, wide, stream);
    }
}
}  // namespace

namespace {
// Estimated time of the launch in microseconds; `units`: of 256 contraction elements, one unit of every wave; `rounds`:
// workgroups per compute unit.  Fits (13 and 11 % rms) to 1060 timed layers of 256 to 4096 x 256 to 22016, r = 0 to 64.
double single_us(const LayerView &w, int r, bool f16, bool wide) {
    const double units = w.K / 256.0, rg = (double)(r > 32 ? 4 : (r + 15) / 16), h = f16 ? rg : 0.0, three = w.bits == 3 ? 1.0 : 0.0;
    const int workgroups = wide ? (w.N + 63) / 64 : (w.N + 15) / 16;
    const double more = workgroups > 256 ? workgroups / 256.0 - 1.0 : 0.0;
    if (wide)
        return 4.02 + units * (0.36 + 0.13 * three + 0.40 * rg + 0.17 * h) +
               more * (9.98 + 2.88 * rg + units * (2.58 + 1.40 * three + 0.99 * rg + 0.63 * h));
    return 3.63 + units * (0.23 + 0.07 * three + 0.36 * rg + 0.13 * h) + more * (0.60 + 1.06 * rg + units * (0.35 + 0.05 * three + 0.30 * rg + 0.09 * h));
}
}  // namespace

bool single_wins(const LayerView &w, int M, int r, bool f16) {
    if (M > 15 || w.K > 4096) return false;
    const double two = 9.2 + 0.177e-6 * ((double)w.K * w.N * w.bits / 8) + 0.35 * ((r + 15) / 16) + 0.23 * w.K / 1024;
    const double narrow = single_us(w, r, f16, false), wide = single_us(w, r, f16, true);
    return 1.1 * (narrow < wide ? narrow : wide) < two;
}

hipError_t launch_single(const SmallArgs &a, hipStream_t stream) {
    SingleDev d;
    d.w = a.w;
    d.act = a.act;
    d.A = a.A; d.B = a.B;
    d.M = a.M; d.r = a.r;
    d.lora_scale = a.lora_scale;
    d.out = a.out; d.P_out = a.P_out;
    d.zeros16 = a.zeros16; d.bias16 = a.bias16;
    const uint32_t spg = (uint32_t)(a.w.group / (a.w.bits == 4 ? 32 : a.w.bits == 2 ? 64 : 128));      // steps per group
    d.spg_plus = spg > 1 ? 0u : 1u;
    d.spg_magic = spg > 1 ? (uint32_t)((1ull << 32) / spg) + 1u : 0xFFFFFFFFu;
    const bool wide = single_us(a.w, a.r, a.f16, true) < single_us(a.w, a.r, a.f16, false);
    return a.f16 ? launch_single_any<true>(d, wide, stream) : launch_single_any<false>(d, wide, stream);
}

}  // namespace mlr
