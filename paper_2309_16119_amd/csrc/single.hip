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
#include <cmath>

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
    uint32_t bpg_plus, bpg_magic;      // quantization group of a 32-code block, (block + plus) * magic / 2^32
};

// Sum of the waves' parts of the projection: P[row][16 RG], row stride 16 RG + 4, and its hand-off by the first column of workgroups.
template <int RG, int RT>
__device__ __forceinline__ void single_projection(const SingleDev &d, int m0, const float *red, float *Ps) {
    using namespace single;
    constexpr int PS = 16 * RG + 4;
    for (int x = threadIdx.x; x < RT * RG * 256; x += THREADS) {
        const int g = x >> 8, v = (x >> 6) & 3, l = x & 63;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NWAVES; ++w) sum += red[((w * RT * RG + g) * 4 + v) * 64 + l];
        const int row = 16 * (g / RG) + 4 * (l >> 4) + v, j = g % RG * 16 + (l & 15);
        Ps[row * PS + j] = sum;
        if (blockIdx.x == 0 && d.P_out != nullptr && m0 + row < d.M && j < d.r) d.P_out[(size_t)(m0 + row) * d.r + j] = sum;
    }
}

// A unit is 32 contraction elements, one MFMA deep: lane l = 16 j + i holds the column(s) of i and quarter j of their 32-code
// block.  Wave w takes units w, w + 8, ..., U of them in flight.  A workgroup owns 16 RT rows and 16 CT columns, CT adjacent ones
// per lane.  ROUND: the weight is dequantized and rounded to 16 bits as in every kernel for more tokens than the
// streaming ones take; otherwise the codes are multiplied as they are and the affine part applied to each unit's sums.
template <int BITS, bool F16, bool ROUND, int RG, int RT, int CT>
__global__ __launch_bounds__(single::THREADS, 2) void single_kernel(SingleDev d) {
    using namespace single;
    using NF = sm::Num<F16>;
    constexpr int NWORDS = BITS == 3 ? 2 : 1, U = RG == 1 && RT * CT <= 4 ? 4 : 2, R = 16 * RG, PS = R + 4;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *red_y = smem, *red_p = red_y + NWAVES * RT * CT * 256, *Ps = red_p + NWAVES * RT * RG * 256, *Bs = Ps + 16 * RT * PS;      // Bs [R][16 CT]
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int i = lane & 15, j = lane >> 4, K = d.w.K, N = d.w.N, r = d.r, M = d.M;
    const int n0 = blockIdx.x * 16 * CT, m0 = blockIdx.y * 16 * RT;
    int n = n0 + CT * i;
    if (n > N - CT) n = N - CT;                     // N is a multiple of 8; stores are masked
    const uint16_t *xrow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {                  // rows past M repeat the last one, never stored
        const int m = m0 + 16 * t + i;
        xrow[t] = d.act + (size_t)(m < M ? m : M - 1) * K + 8 * j;
    }
    const int units = K / 32;
    // word row(s) of quarter j inside a block, and the shift that brings its 8 codes to bit 0
    const int lo = BITS == 4 ? j : BITS == 2 ? j >> 1 : (24 * j) >> 5, hi = lo < 2 ? lo + 1 : 2;
    const uint32_t shift = BITS == 4 ? 0u : BITS == 2 ? 16u * (j & 1) : (24u * j) & 31u;

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
        uint32_t w[NWORDS][CT], sc[(CT + 1) / 2], z[F16 ? (CT + 1) / 2 : 1];
        uint4 x[RT];
        float f[RG][8];
    };
    auto load = [&](Stage &s, int u) {
        if (u > units - 1) u = units - 1;
        const uint32_t *block = d.w.qweight + (size_t)u * BITS * N + n;
        auto words_at = [&](uint32_t *dst, const uint32_t *src) {
            if (CT == 1) dst[0] = *src;
            else {
                const uint4 v = *reinterpret_cast<const uint4 *>(src);
                dst[0] = v.x; dst[CT > 1 ? 1 : 0] = v.y; dst[CT > 2 ? 2 : 0] = v.z; dst[CT > 3 ? 3 : 0] = v.w;
            }
        };
        words_at(s.w[0], block + (size_t)lo * N);
        if (BITS == 3) words_at(s.w[NWORDS - 1], block + (size_t)hi * N);
#pragma unroll
        for (int t = 0; t < RT; ++t) s.x[t] = *reinterpret_cast<const uint4 *>(xrow[t] + 32 * u);
        const size_t g = (size_t)__umulhi((uint32_t)u + d.bpg_plus, d.bpg_magic) * N + n;
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
        if (r == 0) return;
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const float *f = d.A + (size_t)(32 * u + 8 * j) * r + (16 * q + i < r ? 16 * q + i : 0);
#pragma unroll
            for (int e = 0; e < 8; ++e) s.f[q][e] = f[(size_t)e * r];
        }
    };
    const uint32_t ones4[4] = {NF::ONES, NF::ONES, NF::ONES, NF::ONES}, offs4[4] = {NF::MAGIC3, NF::MAGIC3, NF::MAGIC3, NF::MAGIC3};
    const bf16x8 ones = sm::as_bf16x8(ones4), offs = sm::as_bf16x8(offs4);
    const sm::CodeMasks masks = sm::make_masks<BITS, F16>();
    const DqMasks dq_masks = make_dq_masks<BITS>();
    f32x4 y[RT][CT], P[RT][RG];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
        for (int c = 0; c < CT; ++c) y[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < RG; ++q) P[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto compute = [&](const Stage &s) {
        // elements p and p + 4 of the lane side by side, as the code registers pair them
        uint32_t a4[RT][4];
        f32x4 xsum[RT], start[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const uint32_t xw[4] = {s.x[t].x, s.x[t].y, s.x[t].z, s.x[t].w};
#pragma unroll
            for (int p = 0; p < 4; ++p) a4[t][p] = __builtin_amdgcn_perm(xw[2 + (p >> 1)], xw[p >> 1], p & 1 ? 0x07060302u : 0x05040100u);
            if (!ROUND) {
                const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
                xsum[t] = sm::mma<F16>(sm::as_bf16x8(a4[t]), ones, zero4);
                const f32x4 off = BITS == 3 ? sm::mma<F16>(sm::as_bf16x8(a4[t]), offs, zero4) : xsum[t];
#pragma unroll
                for (int v = 0; v < 4; ++v) start[t][v] = BITS == 3 ? -off[v] : -NF::OFFSET * off[v];      // minus what the operands' offsets add
            }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const uint32_t x = BITS == 4 ? s.w[0][c] : BITS == 2 ? s.w[0][c] >> shift : __builtin_amdgcn_alignbit(s.w[NWORDS - 1][c], s.w[0][c], shift);
            const uint32_t codes = unit_codes<BITS>(x, 0x0C010C00u);      // codes p and p + 4 at bits BITS p (+ 4: three bits) of either half
            const uint32_t scale16 = s.sc[c >> 1] >> (16 * (c & 1)), z = F16 ? s.z[F16 ? c >> 1 : 0] >> (16 * (c & 1)) : s.z[0] >> (8 * c);
            uint32_t o[4];
            if (ROUND) {
                const DqPair dq = make_dq_pair<BITS, F16>(scale16, z);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const half16x2 h = unit_pair<BITS, F16>(codes, BITS * p, dq_masks);
                    o[p] = pack_pair_cvt<F16>(dq_lo<F16>(h, dq), dq_hi<F16>(h, dq));
                }
#pragma unroll
                for (int t = 0; t < RT; ++t) y[t][c] = sm::mma<F16>(sm::as_bf16x8(a4[t]), sm::as_bf16x8(o), y[t][c]);
            } else {
#pragma unroll
                for (int p = 0; p < 4; ++p) o[p] = sm::and_or(codes >> (BITS * p), masks.field, masks.magic);
                const float scale = half_bits_to_float((uint16_t)scale16);
                const float zero = F16 ? half_bits_to_float((uint16_t)z) : (float)(z & 0xFFu);
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    const f32x4 qx = sm::mma<F16>(sm::as_bf16x8(a4[t]), sm::as_bf16x8(o), start[t]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (F16) y[t][c][v] = __builtin_fmaf(scale, qx[v], __builtin_fmaf(zero, xsum[t][v], y[t][c][v]));
                        else y[t][c][v] = __builtin_fmaf(scale, __builtin_fmaf(-zero, xsum[t][v], qx[v]), y[t][c][v]);
                    }
                }
            }
        }
        if (r == 0) return;
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const bool mine = 16 * q + i < r;
            float f[8];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                f[2 * p] = mine ? s.f[q][p] : 0.f;
                f[2 * p + 1] = mine ? s.f[q][p + 4] : 0.f;
            }
            uint32_t p3[3][4];
            split3(f, p3[0], p3[1], p3[2]);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                uint32_t h[2][4];
                if (F16) split_f16x8(a4[t], h[0], h[1]);
#pragma unroll
                for (int x = 0; x < (F16 ? 2 : 1); ++x)
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        P[t][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sm::as_bf16x8(F16 ? h[x] : a4[t]), sm::as_bf16x8(p3[e]), P[t][q], 0, 0, 0);
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
                compute(st[q]);
                load(st[q], u + NWAVES * (q + U));
            }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) red_y[(((wave * RT + t) * CT + c) * 4 + v) * 64 + lane] = y[t][c][v];
#pragma unroll
        for (int q = 0; q < RG; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) red_p[(((wave * RT + t) * RG + q) * 4 + v) * 64 + lane] = P[t][q][v];
    }
    __syncthreads();
    single_projection<RG, RT>(d, m0, red_p, Ps);
    __syncthreads();
    // two adjacent columns of a row: T threads side by side share the waves' sums and the rank
    constexpr int T = 4 / CT;
    const int part = tid % T, pair = tid / T, c0 = 2 * (pair % (8 * CT)), v = (pair / (8 * CT)) & 3, col = n0 + c0;
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int m = 16 * t + pair / (8 * CT);
        float o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = (c0 + h) % CT, l = 16 * ((m >> 2) & 3) + (c0 + h) / CT;
            float sum = 0.f, ad = 0.f;
#pragma unroll
            for (int w = 0; w < NWAVES / T; ++w) sum += red_y[((((part * (NWAVES / T) + w) * RT + t) * CT + c) * 4 + v) * 64 + l];
            if (r > 0) {
#pragma unroll 8
                for (int q = 0; q < R / T; ++q) ad = __builtin_fmaf(Ps[m * PS + part * (R / T) + q], Bs[(part * (R / T) + q) * 16 * CT + c0 + h], ad);
            }
            o[h] = __builtin_fmaf(d.lora_scale, ad, sum);
            if (T > 1) o[h] += __shfl_xor(o[h], 1, 64);
            if (T > 2) o[h] += __shfl_xor(o[h], 2, 64);
        }
        if (part != 0 || m0 + m >= M || col >= N) continue;
        if (F16 && d.bias16 != nullptr) {
            const uint32_t b = *reinterpret_cast<const uint32_t *>(d.bias16 + col);
            o[0] += half_bits_to_float((uint16_t)(b & 0xFFFFu));
            o[1] += half_bits_to_float((uint16_t)(b >> 16));
        }
        *reinterpret_cast<uint32_t *>(d.out + (size_t)(m0 + m) * N + col) = sm::pack16<F16>(o[0], o[1]);
    }
}

namespace {
template <int BITS, bool F16, bool ROUND, int RG, int RT, int CT>
hipError_t launch_single_ct(const SingleDev &d, hipStream_t stream) {
    constexpr int R = 16 * RG;
    constexpr size_t LDS = (size_t)(single::NWAVES * RT * (CT + RG) * 256 + 16 * RT * (R + 4) + R * 16 * CT) * 4;
    auto kern = single_kernel<BITS, F16, ROUND, RG, RT, CT>;
    static bool configured[64] = {};
    const hipError_t e = ensure_lds_limit(reinterpret_cast<const void *>(kern), LDS, configured);
    if (e != hipSuccess) return e;
    const dim3 grid((d.w.N + 16 * CT - 1) / (16 * CT), (d.M + 16 * RT - 1) / (16 * RT));
    launch_kernel(ROUND ? (F16 ? "f16_gemm_fwd_single" : "gemm_fwd_single") : (F16 ? "f16_stream_fwd_single" : "stream_fwd_single"), kern, grid,
                  single::THREADS, LDS, stream, d);
    return hipGetLastError();
}
template <int BITS, bool F16, int RG>
hipError_t launch_single_rg(const SingleDev &d, bool round, bool wide, hipStream_t stream) {
    if (round) return wide ? launch_single_ct<BITS, F16, true, RG, 2, 4>(d, stream) : launch_single_ct<BITS, F16, true, RG, 2, 1>(d, stream);
    return wide ? launch_single_ct<BITS, F16, false, RG, 1, 4>(d, stream) : launch_single_ct<BITS, F16, false, RG, 1, 1>(d, stream);
}
template <int BITS, bool F16>
hipError_t launch_single_bits(const SingleDev &d, bool round, bool wide, hipStream_t stream) {
    if (d.r <= 16) return launch_single_rg<BITS, F16, 1>(d, round, wide, stream);
    return d.r <= 32 ? launch_single_rg<BITS, F16, 2>(d, round, wide, stream) : launch_single_rg<BITS, F16, 4>(d, round, wide, stream);
}
template <bool F16>
hipError_t launch_single_any(const SingleDev &d, bool round, bool wide, hipStream_t stream) {
    switch (d.w.bits) {
        case 2: return launch_single_bits<2, F16>(d, round, wide, stream);
        case 3: return launch_single_bits<3, F16>(d, round, wide, stream);
        default: return launch_single_bits<4, F16>(d, round, wide, stream);
    }
}
}  // namespace

// Estimated time of the launch in microseconds: its start, the units that a wave takes in turn, and the same again for
// every workgroup more than one per compute unit.  Fits (9 to 15 % rms) to 1060 timed layers of 256 to 4096 x 256 to
// 22016 with up to 15 tokens, and 1425 of up to 2^23 weights with 16 ... 2500 (round), r = 0 to 64, both conventions.
static double single_us(const LayerView &w, int M, int r, bool f16, bool round, bool wide) {
    const double units = w.K / 256.0, rg = (double)(r > 32 ? 4 : (r + 15) / 16), h = f16 ? rg : 0.0, three = w.bits == 3 ? 1.0 : 0.0;
    const int columns = wide ? (w.N + 63) / 64 : (w.N + 15) / 16;
    const double workgroups = (double)columns * (round ? (M + 31) / 32 : 1);
    double more = workgroups > 256.0 ? workgroups / 256.0 - 1.0 : 0.0;
    if (round && (wide || rg > 2.0)) more = std::ceil(more);      // their LDS leaves room for one workgroup per compute unit
    if (round) {
        if (wide)
            return 5.42 + (r > 16 ? 1.18 : 0.0) + units * (0.383 + 0.621 * rg + 0.198 * h) +
                   more * (2.06 + 1.85 * rg + units * (0.811 + 0.244 * rg + 0.336 * h));
        return 5.68 + units * (0.313 + 0.383 * rg + 0.192 * h) + more * (2.87 + 0.646 * rg + units * (0.578 + 0.241 * rg + 0.146 * h));
    }
    if (wide)
        return 4.02 + units * (0.36 + 0.13 * three + 0.40 * rg + 0.17 * h) +
               more * (9.98 + 2.88 * rg + units * (2.58 + 1.40 * three + 0.99 * rg + 0.63 * h));
    return 3.63 + units * (0.23 + 0.07 * three + 0.36 * rg + 0.13 * h) + more * (0.60 + 1.06 * rg + units * (0.35 + 0.05 * three + 0.30 * rg + 0.09 * h));
}

// In place of the two streaming launches.  (Sixteen tokens, a full tile, keep the two launches that the streaming
// kernels' tests name, though the times do not cross there.)
bool single_wins(const LayerView &w, int M, int r, bool f16) {
    if (M > 15 || w.K > 4096) return false;
    const double two = 9.2 + 0.177e-6 * ((double)w.K * w.N * w.bits / 8) + 0.35 * ((r + 15) / 16) + 0.23 * w.K / 1024;
    const double narrow = single_us(w, M, r, f16, false, false), wide = single_us(w, M, r, f16, false, true);
    return 1.1 * (narrow < wide ? narrow : wide) < two;
}
// In place of a product and its projection or second launch, whose estimate is `us`: over the 1425 layers above a
// call's kernels take 1.37x less time on average (256 x 488, 252 tokens, us 11.4 -> 6.3; 1024 x 640, 40 tokens 15.5 -> 9.6; on the other
// side 512 x 4096, 300 tokens 14.4 and 20).
bool single_beats(int K, int N, int M, int r, bool f16, double us) {
    if (K > 2304 || (size_t)K * N >= ((size_t)1 << 23)) return false;
    LayerView w{};
    w.K = K; w.N = N;
    const double narrow = single_us(w, M, r, f16, true, false), wide = single_us(w, M, r, f16, true, true);
    return 1.05 * (narrow < wide ? narrow : wide) < us;
}

hipError_t launch_single(const SmallArgs &a, bool round, hipStream_t stream) {
    SingleDev d;
    d.w = a.w;
    d.act = a.act;
    d.A = a.A; d.B = a.B;
    d.M = a.M; d.r = a.r;
    d.lora_scale = a.lora_scale;
    d.out = a.out; d.P_out = a.P_out;
    d.zeros16 = a.zeros16; d.bias16 = a.bias16;
    const uint32_t bpg = (uint32_t)(a.w.group / 32);      // blocks per group
    d.bpg_plus = bpg > 1 ? 0u : 1u;
    d.bpg_magic = bpg > 1 ? (uint32_t)((1ull << 32) / bpg) + 1u : 0xFFFFFFFFu;
    const bool wide = single_us(a.w, a.M, a.r, a.f16, round, true) < single_us(a.w, a.M, a.r, a.f16, round, false);
    return a.f16 ? launch_single_any<true>(d, round, wide, stream) : launch_single_any<false>(d, round, wide, stream);
}

}  // namespace mlr
