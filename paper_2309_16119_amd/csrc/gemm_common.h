// Pieces shared by the tile GEMM kernels: tile order, the per-launch device
// arguments and small address helpers.
#pragma once
#include "device_common.h"
#include "launch.h"

namespace mlr {

struct TileCoord {
    int tm, tc;
};

// XCD-aware tile order: consecutive workgroup ids go round-robin over the 8 XCDs, so
// give each XCD a contiguous run of tiles, and walk tiles row-block-fastest inside a
// run so that neighbours on one XCD share the weight tile (and its L2 lines).
__device__ __forceinline__ TileCoord tile_of_block(int bid, int tiles_m, int tiles_c) {
    const int total = tiles_m * tiles_c;
    const int per_xcd = (total + 7) / 8;
    int t = (bid % 8) * per_xcd + bid / 8;
    TileCoord tc;
    if (t >= total) { tc.tm = -1; tc.tc = -1; return tc; }
    tc.tc = t / tiles_m;
    tc.tm = t % tiles_m;
    return tc;
}

// Row block and column block of a linear tile index when the tiles are walked in bands of
// BAND row blocks, row-block-fastest inside a band: the ~32 tiles of consecutive index that
// one XCD runs at a time then span BAND activation panels and 32 / BAND weight panels.  An
// activation panel is 16 / bits times the bytes of a weight panel, so few rows and many
// columns keep the bytes that XCD pulls through its L2 lowest (2 rows: about a third of what
// a whole column of 16 row blocks costs).
template <int BAND>
__device__ __forceinline__ TileCoord banded_tile(int tile, int tiles_m, int tiles_c) {
    const int full = (tiles_m / BAND) * BAND * tiles_c;     // tiles in whole bands
    TileCoord tc;
    if (tile < full) {
        const int band = tile / (BAND * tiles_c), r = tile - band * (BAND * tiles_c);
        tc.tc = r / BAND;
        tc.tm = band * BAND + r % BAND;
    } else {
        const int rows = tiles_m % BAND, r = tile - full;   // the last, narrower band
        tc.tc = r / rows;
        tc.tm = (tiles_m / BAND) * BAND + r % rows;
    }
    return tc;
}

struct GemmDev {
    GemmArgs a;
    int tiles_m, tiles_c;
    // group index of a 32-code block: blk / (group/32), as one multiply-high with
    // magic = floor(2^32 / d) + 1 (exact for blk, d < 2^15); d == 1 is passed through
    uint32_t blocks_per_group, blocks_per_group_magic;
    __device__ __forceinline__ uint32_t group_of_block(uint32_t blk) const {
        return blocks_per_group == 1 ? blk : __umulhi(blk, blocks_per_group_magic);
    }
};



inline GemmDev make_gemm_dev(const GemmArgs &a, int MT, int CT) {
    const int Cout = a.backward ? a.w.K : a.w.N;
    GemmDev d;
    d.a = a;
    d.tiles_m = (a.M + MT - 1) / MT;
    d.tiles_c = (Cout + CT - 1) / CT;
    d.blocks_per_group = (uint32_t)(a.w.group / 32);
    d.blocks_per_group_magic = d.blocks_per_group > 1 ? (uint32_t)((1ull << 32) / d.blocks_per_group) + 1u : 0u;
    return d;
}

// Raise the dynamic-LDS limit of a kernel once per device (not a stream operation, but
// keep it out of the steady state and out of graph captures after the first call).
inline hipError_t ensure_lds_limit(const void *kernel, size_t lds_bytes, bool *configured /*[64]*/) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64 || !configured[dev]) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) configured[dev] = true;
    }
    return hipSuccess;
}

// One direct global->LDS load of 16 bytes per lane: lane i's data lands at
// lds_base + 16 i (lds_base wave-uniform, in M0).
__device__ __forceinline__ void load_to_lds_16(const void *gbase_uniform, uint32_t voff_bytes, uint32_t lds_base_uniform) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_base_uniform), "v"(voff_bytes), "s"(gbase_uniform)
                 : "memory");
}

// Register loads issued from inline assembly (uniform base + per-lane byte offset).  The
// compiler does not know that they are in flight: every consumer must sit behind
// wait_loads(), which also ties the destination registers so that no use can be moved
// ahead of the wait.  This keeps the compiler from sprinkling conservative vmcnt waits
// (which would also wait for the direct loads) through the MFMA phase.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void aload_b32(uint32_t &dst, const void *base, uint32_t voff) {
    asm volatile("global_load_dword %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(base) : "memory");
}
__device__ __forceinline__ void aload_u16(uint32_t &dst, const void *base, uint32_t voff) {
    asm volatile("global_load_ushort %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(base) : "memory");
}
__device__ __forceinline__ void aload_u8(uint32_t &dst, const void *base, uint32_t voff) {
    asm volatile("global_load_ubyte %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(base) : "memory");
}
__device__ __forceinline__ void aload_b64(u32x2 &dst, const void *base, uint32_t voff) {
    asm volatile("global_load_dwordx2 %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(base) : "memory");
}
__device__ __forceinline__ void aload_b128(u32x4 &dst, const void *base, uint32_t voff) {
    asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(voff), "s"(base) : "memory");
}

// Two fp32 values rounded to nearest even into a pair of 16-bit floats, `lo` in the low half:
// bfloat16, or binary16 for the layer in the paper's own storage convention.
typedef _Float16 half16x2 __attribute__((ext_vector_type(2)));
template <bool F16>
__device__ __forceinline__ uint32_t pack_pair(float lo, float hi) {
    if (!F16) return pack_bf16x2(lo, hi);
    const half16x2 v = {(_Float16)lo, (_Float16)hi};
    uint32_t u;
    __builtin_memcpy(&u, &v, sizeof u);
    return u;
}

// Quarter j (0..3) of a 32-code block held in BITS words: its 8 codes dequantized with one
// (scale, bias) into 8 bfloat16 (or binary16), code 8 j in the low half of out[0].
template <int BITS, bool F16 = false>
__device__ __forceinline__ void dequant_quarter(const uint32_t *w, int j, const DqConst &c, uint32_t out[4]) {
    if (BITS == 4) {
        const uint32_t lo = w[j] & 0x0F0F0F0Fu, hi = (w[j] >> 4) & 0x0F0F0F0Fu;
#pragma unroll
        for (int i = 0; i < 4; ++i)   // codes 2i (byte i of lo) and 2i+1 (byte i of hi)
            out[i] = pack_pair<F16>(dq_value((lo >> (8 * i)) & 0xFFu, c), dq_value((hi >> (8 * i)) & 0xFFu, c));
    } else if (BITS == 2) {
        const uint32_t h = w[j >> 1] >> (16 * (j & 1));   // 8 codes in the low 16 bits
        const uint32_t even = h & 0x3333u, odd = (h >> 2) & 0x3333u;   // nibble n: code 2n / 2n+1
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[i] = pack_pair<F16>(dq_value((even >> (4 * i)) & 0xFu, c), dq_value((odd >> (4 * i)) & 0xFu, c));
    } else {
        const uint32_t chunk = block_chunk<BITS>(w, j);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[i] = pack_pair<F16>(dq_value(chunk_code<BITS>(chunk, 2 * i), c), dq_value(chunk_code<BITS>(chunk, 2 * i + 1), c));
    }
}

// The same quarter by fewer and cheaper instructions.  A code OR-ed into the mantissa of a binary16
// power of two whose unit in that bit is one is that power of two plus the code, two codes per
// instruction: (w >> s & fields) | magic.  The multiply-add then reads either half as it stands:
//   (q - zero) scale = (2^m + q) scale - (2^m + zero) scale,
// and with zero <= 255 and 2^m of 64 or 1024 the second product has at most 22 significant bits, so
// both it and the result are exact, as they are in dq_value().  A wave's extract, convert and
// multiply-add cost 4 issue cycles each (measured; plain shifts, ANDs and fp32 multiply-adds 2):
// 14 per 3-bit code that way, 9.5 this way; the 256 x 256 kernel 1252 -> 1216 us forward and 1218 ->
// 1196 backward at 4096 x 8192 x 22016 (3 bits), 172 -> 165 and 158 -> 153 at 2048 x 4096 x 11008 (4 bits),
// 86 -> 83 both ways at 1024 x 6656 x 6656 (2 bits).  (In the producer waves of the 128 x 64 kernel it
// measured slower, 75 -> 79 us a step: they wait for LDS, and two rows per store pass conflict.)  Binary16 layers add their zero point, whose sum with
// the power of two would round: there the power of two is taken off first (exact).
struct DqPair {
    _Float16 scale, z;   // z: the binary16 zero point that is added (F16)
    float lo, hi;        // addend of the codes in the low and in the high halves (integer zero points)
};
struct DqMasks {
    uint32_t fields, magic;      // in registers of their own: one v_and_or_b32 instead of two instructions with literals
};
template <int BITS, bool IN_REGS = true>
__device__ __forceinline__ DqMasks make_dq_masks() {
    DqMasks m;
    m.fields = BITS == 4 ? 0x000F000Fu : (BITS == 2 ? 0x00030003u : 0x00070070u);
    m.magic = BITS == 3 ? 0x64005400u : 0x64006400u;       // 1024.0 twice; 3 bits: 1024.0, 64.0 (low field at bits 4-6)
    if (IN_REGS) {
        asm volatile("" : "+s"(m.fields));
        asm volatile("" : "+v"(m.magic));
    }
    return m;
}
template <int BITS, bool F16>
__device__ __forceinline__ DqPair make_dq_pair(uint32_t scale_bits, uint32_t zero_bits) {
    DqPair c;
    const uint16_t sb = (uint16_t)scale_bits;
    __builtin_memcpy(&c.scale, &sb, 2);
    if (F16) {
        const uint16_t zb = (uint16_t)zero_bits;
        __builtin_memcpy(&c.z, &zb, 2);
        c.lo = c.hi = 0.f;
    } else {
        c.z = (_Float16)0.0f;
        const float s = (float)c.scale, z = (float)(zero_bits & 0xFFu);
        c.hi = -(1024.0f + z) * s;
        c.lo = BITS == 3 ? -(64.0f + z) * s : c.hi;
    }
    return c;
}
// a pair's two weights in fp32, the products exact: one v_fma_mix_f32 each, with the halves as they stand
template <bool F16>
__device__ __forceinline__ float dq_lo(half16x2 h, const DqPair &c) {
    return __builtin_fmaf((float)h.x, (float)c.scale, F16 ? (float)c.z : c.lo);
}
template <bool F16>
__device__ __forceinline__ float dq_hi(half16x2 h, const DqPair &c) {
    return __builtin_fmaf((float)h.y, (float)c.scale, F16 ? (float)c.z : c.hi);
}
// Codes p (low half) and p + 4 (high half) of quarter j, as they enter the multiply-add.
template <int BITS, bool F16>
__device__ __forceinline__ half16x2 quarter_pair(const uint32_t *w, int j, int p, const DqMasks &m) {
    uint32_t x;
    if (BITS == 4) {
        x = w[j] >> (4 * p);
    } else if (BITS == 2) {
        // the quarter's two bytes side by side, one per half
        x = __builtin_amdgcn_perm(0u, w[j >> 1], (j & 1) ? 0x0C030C02u : 0x0C010C00u) >> (2 * p);
    } else {
        const int sh = 24 * j + 3 * p - 4;       // stream bit that lands at register bit 0
        if (sh < 0) x = w[0] << (-sh);
        else if ((sh & 31) == 0) x = w[sh >> 5];
        else if ((sh >> 5) == 2) x = w[2 % BITS] >> (sh & 31);
        else if ((sh & 31) + 19 <= 32) x = w[sh >> 5] >> (sh & 31);
        else x = __builtin_amdgcn_alignbit(w[((sh >> 5) + 1) % BITS], w[sh >> 5], sh & 31);
    }
    x = (x & m.fields) | m.magic;
    half16x2 h;
    __builtin_memcpy(&h, &x, 4);
    if (F16) h -= half16x2{(_Float16)(BITS == 3 ? 64.0f : 1024.0f), (_Float16)1024.0f};
    return h;
}
// The same for the eight codes of one weight column inside a word (the backward kernels' units): `y`
// from unit_codes(), pass p (any lane's own order) by its right shift BITS * p.
template <int BITS>
__device__ __forceinline__ uint32_t unit_codes(uint32_t chunk_or_word, uint32_t two_bit_bytes) {
    if (BITS == 2) return __builtin_amdgcn_perm(0u, chunk_or_word, two_bit_bytes);
    return BITS == 3 ? chunk_or_word << 4 : chunk_or_word;
}
template <int BITS, bool F16>
__device__ __forceinline__ half16x2 unit_pair(uint32_t y, uint32_t shift, const DqMasks &m) {
    const uint32_t x = ((y >> shift) & m.fields) | m.magic;
    half16x2 h;
    __builtin_memcpy(&h, &x, 4);
    if (F16) h -= half16x2{(_Float16)(BITS == 3 ? 64.0f : 1024.0f), (_Float16)1024.0f};
    return h;
}
// Two fp32 values rounded to nearest even into a pair of 16-bit floats by ONE conversion: the fences
// keep the compiler from folding a binary16 conversion into the multiply-adds (v_fma_mixlo_f16 takes
// 8 cycles a value, v_fma_mix_f32 and half of v_cvt_pk_f16_f32 take 6).
template <bool F16>
__device__ __forceinline__ uint32_t pack_pair_cvt(float lo, float hi) {
    if (F16) asm("" : "+v"(lo), "+v"(hi));
    return pack_pair<F16>(lo, hi);
}
template <int BITS, bool F16>
__device__ __forceinline__ void dequant_quarter_pairs(const uint32_t *w, int j, const DqPair &c, const DqMasks &m, uint32_t out[4]) {
    float v[8];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const half16x2 h = quarter_pair<BITS, F16>(w, j, p, m);
        v[p] = dq_lo<F16>(h, c);
        v[p + 4] = dq_hi<F16>(h, c);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = pack_pair_cvt<F16>(v[2 * i], v[2 * i + 1]);
}

// gemm_big.hip, gemm_big_192.hip: the 8-wave variants of 256, 192 and 128 rows by 256 columns
hipError_t launch_gemm_big(const GemmArgs &a, hipStream_t stream);
// gemm_mid.hip: 128x64 tiles for grids of about one tile per CU, producer and consumer waves
hipError_t launch_gemm_mid(const GemmArgs &a, hipStream_t stream);

}  // namespace mlr
