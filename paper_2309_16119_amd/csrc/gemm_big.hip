// The large-M kernel (gemm_big_kernel.h) with tiles of 256 and of 128 rows, and what launches all of them.
#include "gemm_big_kernel.h"

namespace mlr {

template <int BITS, bool F16, int MT>
static hipError_t launch_big_dir(const GemmArgs &a, const BigPlan &plan, hipStream_t stream, const SlicedPlan *sliced, const BigSide &side) {
    return a.backward ? launch_big_mt<BITS, true, F16, MT>(a, plan, stream, sliced, side) : launch_big_mt<BITS, false, F16, MT>(a, plan, stream, sliced, side);
}
template <int BITS, bool F16>
static hipError_t launch_big_bits(const GemmArgs &a, const BigPlan &plan, hipStream_t stream, const SlicedPlan *sliced, const BigSide &side) {
    return plan.mt == 128 ? launch_big_dir<BITS, F16, 128>(a, plan, stream, sliced, side) : launch_big_dir<BITS, F16, 256>(a, plan, stream, sliced, side);
}
template <bool F16>
static hipError_t launch_big_any(const GemmArgs &a, const BigPlan &plan, hipStream_t stream, const SlicedPlan *sliced, const BigSide &side) {
    switch (a.w.bits) {
        case 2: return launch_big_bits<2, F16>(a, plan, stream, sliced, side);
        case 3: return launch_big_bits<3, F16>(a, plan, stream, sliced, side);
        default: return launch_big_bits<4, F16>(a, plan, stream, sliced, side);
    }
}
static hipError_t launch_big(const GemmArgs &a, bool f16, const BigPlan &plan, hipStream_t stream, const SlicedPlan *sliced, const BigSide &side) {
    if (plan.mt == 192) return launch_big_192(a, f16, plan, stream);
    return f16 ? launch_big_any<true>(a, plan, stream, sliced, side) : launch_big_any<false>(a, plan, stream, sliced, side);
}
static BigPlan plan_of(const GemmArgs &a) { return big_plan(a.M, a.backward ? a.w.N : a.w.K, a.backward ? a.w.K : a.w.N); }

hipError_t launch_gemm_big(const GemmArgs &a, hipStream_t stream) { return launch_big(a, false, plan_of(a), stream, nullptr, BigSide{}); }
hipError_t launch_gemm_big_f16(const GemmArgs &a, hipStream_t stream) { return launch_big(a, true, plan_of(a), stream, nullptr, BigSide{}); }

hipError_t launch_sliced(const SmallArgs &s, bool backward, hipStream_t stream) {
    const int C = backward ? s.w.N : s.w.K, Cout = backward ? s.w.K : s.w.N;
    const SlicedPlan p = sliced_plan(s.M, C, Cout, s.r, s.f16);
    if (p.parts < 1) return hipErrorInvalidValue;     // callers asked product_route() first
    GemmArgs g{};
    g.w = s.w; g.backward = backward; g.act = s.act; g.M = s.M; g.out = s.out;
    g.zeros16 = s.zeros16; g.bias16 = s.bias16;
    g.partials = static_cast<float *>(s.ws);
    BigSide side{};
    side.F = backward ? s.B : s.A;
    side.ppart = reinterpret_cast<float *>(static_cast<char *>(s.ws) + p.slices_bytes(s.M, Cout));
    side.r = s.r; side.parts = p.parts; side.part_stride = SlicedPlan::part_stride(s.M, s.r);
    const int row_tiles = (s.M + 15) / 16;
    side.row_tiles_magic = row_tiles > 1 ? (uint32_t)((1ull << 32) / row_tiles) + 1u : 0u;      // items < 2^16
    const hipError_t e = launch_big(g, s.f16, p.big, stream, &p, side);
    if (e != hipSuccess) return e;
    FinishArgs f{};
    f.slices = g.partials; f.slice_stride = (size_t)s.M * Cout; f.split = p.big.split; f.M = s.M; f.Cout = Cout;
    f.ppart = side.ppart; f.part_stride = side.part_stride; f.parts = p.parts; f.r = s.r;
    f.F = backward ? s.A : s.B; f.bias16 = s.bias16; f.lora_scale = s.lora_scale; f.out = s.out; f.P_out = s.P_out;
    return launch_finish(big_name(p.big.mt, backward, s.f16, true), f, backward, s.f16, stream);
}

}  // namespace mlr
