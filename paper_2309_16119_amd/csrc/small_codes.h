// A packed code as half of an operand register: device code shared by the kernels for a handful of tokens
// (smallm.hip, single.hip).  The header of smallm.hip describes the arithmetic.
#pragma once
#include "gemm_common.h"

namespace mlr {

namespace sm {
// Number format of the activations and of the operands built from the codes: bfloat16, or binary16
// for the layer in the paper's own storage convention (F16).  A b-bit field OR-ed into the mantissa
// of a power of two whose unit in the last place is one gives that power of two plus the code:
// bfloat16 128.0 (7 mantissa bits), binary16 1024.0 (10 mantissa bits); with the field four bits up,
// bfloat16 8.0 or binary16 64.0.
template <bool F16> struct Num {
    static constexpr uint32_t MAGIC = F16 ? 0x64006400u : 0x43004300u;    // two 1024.0 / two 128.0
    static constexpr uint32_t MAGIC3 = F16 ? 0x64005400u : 0x43004100u;   // (64.0, 1024.0) / (8.0, 128.0): 3-bit forward, low field at bits 4-6
    static constexpr uint32_t ONES = F16 ? 0x3C003C00u : 0x3F803F80u;     // two 1.0
    static constexpr float OFFSET = F16 ? 1024.0f : 128.0f;
};
constexpr uint32_t MAGIC = Num<false>::MAGIC;
constexpr uint32_t MAGIC3 = Num<false>::MAGIC3;
constexpr uint32_t ONES = Num<false>::ONES;
typedef _Float16 half16x8 __attribute__((ext_vector_type(8)));

// D = A B + C on a 16 x 16 x 32 tile, operands given as four registers of 16-bit pairs
template <bool F16>
__device__ __forceinline__ f32x4 mma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
    if (F16) {
        half16x8 x, y;
        __builtin_memcpy(&x, &a, 16);
        __builtin_memcpy(&y, &b, 16);
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, c, 0, 0, 0);
    }
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// two fp32 -> a pair of 16-bit floats (round to nearest even), `lo` in the low half
template <bool F16>
__device__ __forceinline__ uint32_t pack16(float lo, float hi) {
    return pack_pair<F16>(lo, hi);
}
// a stored 16-bit float -> fp32 (exact)
template <bool F16>
__device__ __forceinline__ float widen16(uint32_t bits16) {
    return F16 ? half_bits_to_float((uint16_t)bits16) : __uint_as_float(bits16 << 16);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const uint32_t r[4]) {
    bf16x8 v;
    __builtin_memcpy(&v, r, 16);
    return v;
}
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 q) {
    bf16x8 v;
    __builtin_memcpy(&v, &q, 16);
    return v;
}

// (x & mask) | magic.  A VOP3 instruction of this ISA takes no literal, so with literal
// constants the compiler emits v_and + v_or; callers pass mask and magic as opaque
// register values (see opaque_sgpr / opaque_vgpr) and get one v_and_or_b32.  The
// instruction itself is left to the compiler: hand-written VALU assembly next to MFMAs is
// not covered by the compiler's hazard handling.
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t magic) {
    return (x & mask) | magic;
}
__device__ __forceinline__ uint32_t opaque_sgpr(uint32_t v) {
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ uint32_t opaque_vgpr(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}
struct CodeMasks {
    uint32_t field, magic;        // field mask of a register pair, 2 x 128.0
};

// chunks (8 codes) per step of a lane group, and codes per wave step
template <int BITS> struct Geo {
    static constexpr int NC = BITS == 4 ? 1 : (BITS == 2 ? 2 : 4);   // MFMA calls per wave step
    static constexpr int WORDS = BITS == 4 ? 1 : (BITS == 2 ? 1 : 3); // packed words per lane-group step
    static constexpr int KSTEP = 32 * NC;                             // codes per wave step
};

template <int BITS, bool F16>
__device__ __forceinline__ CodeMasks make_masks() {
    CodeMasks m;
    m.field = opaque_sgpr(BITS == 4 ? 0x000F000Fu : (BITS == 2 ? 0x00030003u : 0x00070070u));
    m.magic = opaque_vgpr(BITS == 3 ? Num<F16>::MAGIC3 : Num<F16>::MAGIC);
    return m;
}

// The 8 operand values (4 registers) of call c from the words of one lane-group step.
template <int BITS>
__device__ __forceinline__ void codes_to_operand(const uint32_t *w, int c, const CodeMasks &m, uint32_t o[4]) {
    if (BITS == 4) {
        // reg p = (code p, code p+4)
#pragma unroll
        for (int p = 0; p < 4; ++p) o[p] = and_or(w[0] >> (4 * p), m.field, m.magic);
    } else if (BITS == 2) {
        // word of 16 codes; call c, reg p = (code 4c+p, code 4c+p+8)
#pragma unroll
        for (int p = 0; p < 4; ++p) o[p] = and_or(w[0] >> (2 * (4 * c + p)), m.field, m.magic);
    } else {
        // 24-bit chunk c of the 96-bit block (stream bits 24c .. 24c+23); reg p = (code p,
        // code p+4): code p must land at bits 4-6, i.e. the chunk shifted right by 3p - 4, and
        // code p+4 (12 bits further up) then sits at bits 16-18.  The shift is folded into the
        // extraction of the chunk from the words (one funnel shift or plain shift per register).
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int sh = 24 * c + 3 * p - 4;       // stream bit that lands at register bit 0
            uint32_t x;
            if (sh < 0) x = w[0] << (-sh);
            else if ((sh & 31) == 0) x = w[sh >> 5];
            else if ((sh >> 5) == 2) x = w[2] >> (sh & 31);
            else x = __builtin_amdgcn_alignbit(w[(sh >> 5) + 1], w[sh >> 5], sh & 31);
            o[p] = and_or(x, m.field, m.magic);
        }
    }
}

}  // namespace sm

// One element of the projection of binary16 activations over contraction elements [k0, k1) (multiples of 8), in plain
// fp32.  An infinity has no exact split (inf - inf is NaN) and meets the zero parts of the other operand (inf * 0): where
// the matrix cores' sum of a row and a factor column is NaN, it is added again by this, which gives what the definition
// does.  (An infinite activation is no rarity in binary16.)  Only such calls pay: us of the launch without / with every
// activation NaN 16 x 22016, r = 64 27 / 81; 16 x 8192, r = 8 19.5 / 18.4; 2048 x 2048, 15 tokens, r = 8 in one launch 9 / 49.
template <bool F_IS_A>
__device__ __forceinline__ float project_f16_again(const uint16_t *row, const float *F, int C, int r, int j, int k0, int k1) {
    float sum = 0.f;
#pragma unroll 1
    for (int c = k0; c < k1; c += 8) {
        const uint4 x = *reinterpret_cast<const uint4 *>(row + c);
        const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
            sum = __builtin_fmaf(half_bits_to_float((uint16_t)(xw[e >> 1] >> (16 * (e & 1)))), F_IS_A ? F[(size_t)(c + e) * r + j] : F[(size_t)j * C + c + e], sum);
    }
    return sum;
}

}  // namespace mlr
