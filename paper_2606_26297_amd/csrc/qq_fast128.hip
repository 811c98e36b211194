// qq_fast128.hip -- complex128 pass kernels, one launch per pass, one kernel instantiation per pass
// kind and qubit-set geometry (bodies in qq_passes128.h).
#include "qq_passes128.h"

namespace qq {
namespace {

using namespace dev;

// One workgroup per (state b, workgroup slot g); FP64 partial sums per slot.
template <int KIND, bool HIGH, bool FULL, bool PART>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(KIND >= FK_LASTG ? 2 : KIND == FK_MID ? 4 : 3)))
fast_pass128(const p128::Args a)
{
    constexpr int NSLOT = passes::kind_slots<KIND>();
    using W = typename std::conditional<passes::kind_states<KIND>() == 2, double2, double>::type;
    __shared__ W lds[kLdsSlots];
    __shared__ double s_red[kThreads / 64][4];

    const int t = threadIdx.x;
    int b, g;
    block_coords(a.B, a.G, b, g);
    double acc[3] = {0.0, 0.0, 0.0};
    if constexpr (KIND == FK_FIRST) {
        // the later passes' layer coefficients, one thread per layer
        if (g == 0 && t < a.p) {
            double sb, cb;
            sincos(a.params[((size_t)b * a.p + t) * 2 + 1], &sb, &cb);
            a.pre[(size_t)b * a.p + t] = make_double2(cb, sb);
        }
    }
    const p128::Coef f = p128::coef<KIND>(a, b);
    p128::pass_body<KIND, HIGH, FULL, PART>(a, lds, acc, t, b, g, f);

    if constexpr (NSLOT > 0) {
        const int lane = t & 63, wave = t >> 6;
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) {
            double xs = acc[s];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) xs += __shfl_xor(xs, d, 64);
            if (lane == 0) s_red[wave][s] = xs;
        }
        __syncthreads();
        if (t < NSLOT)
            a.partial[(size_t)(a.slot_base + t) * a.slot_stride + (size_t)b * a.G + g] =
                (s_red[0][t] + s_red[1][t]) + (s_red[2][t] + s_red[3][t]);
    }
}

// n <= 12: one workgroup per parameter set runs its whole evaluation and writes the results.
template <int NS, typename DT>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
single128(const SingleArgs a)
{
    using W = typename std::conditional<NS == 2, double2, double>::type;
    __shared__ W lds[kLdsSlots];
    __shared__ double s_red[kThreads / 64];
    __shared__ double2 s_cs[QQ_MAX_P];
    const int b = blockIdx.x;
    const p128::Single e = {a.n, a.p, a.amp0, a.params + (size_t)b * 2 * a.p, a.diag};
    double2 *psi = a.psi ? static_cast<double2 *>(a.psi) + ((size_t)b << a.n) : nullptr;
    p128::single_eval<NS, DT>(e, lds, s_red, s_cs, threadIdx.x, psi,
                              [&](int o, double v) __attribute__((always_inline)) {
                                  if (o == 0) a.out.energy[(size_t)b * a.out.estride] = v * a.escale;
                                  else a.out.grad[(size_t)b * a.out.gstride + (o - 1)] = v * (2.0 * a.escale);
                              });
}

template <int KIND, bool HIGH, bool FULL>
hipError_t launch_geom(const p128::Args &a, bool part, hipStream_t s)
{
    const dim3 grid((unsigned)(a.B * a.G)), block(kThreads);
    if constexpr (KIND == FK_FIRST || KIND == FK_TURN || KIND == FK_BTURN) {
        if (part) {
            hipLaunchKernelGGL((fast_pass128<KIND, HIGH, FULL, true>), grid, block, 0, s, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((fast_pass128<KIND, HIGH, FULL, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <int KIND>
hipError_t launch_kind(const p128::Args &a, bool high, bool part, hipStream_t s)
{
    if (!high) return launch_geom<KIND, false, true>(a, part, s);
    return a.active == 0x0ff0 ? launch_geom<KIND, true, true>(a, part, s) : launch_geom<KIND, true, false>(a, part, s);
}

}  // namespace

hipError_t launch_fast_pass128(int kind, bool high, const FastPassParams &pp, hipStream_t s)
{
    // full high sets keep 32-bit lane offsets: (15 + 3 * 2^pos8) amplitudes of 16 bytes (pos8 is at
    // most 24 for n <= 34)
    if (high && pp.active == 0x0ff0 && ((15ull + (3ull << pp.pos8)) * 16ull) >> 32) return hipErrorInvalidValue;
    p128::Args a;
    a.B = pp.B;
    a.G = pp.G;
    a.p = pp.p;
    a.k = pp.k;
    a.tiles = pp.tiles;
    a.pos4 = pp.pos4;
    a.pos8 = pp.pos8;
    a.w1 = pp.w1;
    a.w2 = pp.w2;
    a.active = pp.active;
    a.store_psi = pp.store_psi;
    a.slot_base = pp.slot_base;
    a.slot_stride = pp.slot_stride;
    a.amp0 = pp.amp0;
    a.params = pp.params;
    a.psi = static_cast<double2 *>(pp.psi);
    a.lam = static_cast<double2 *>(pp.lam);
    a.state_stride = pp.state_stride;
    a.partial = pp.partial;
    a.blocked = pp.blocked;
    a.cq = pp.cq;
    a.ctab = pp.ctab;
    a.cthr = pp.cthr;
    a.pre = static_cast<double2 *>(pp.pre);
    a.ltab = pp.ltab;
    a.lthr = pp.lthr;
    a.xtab = pp.xtab;
    a.xthr = pp.xthr;
    switch (kind) {
    case FK_FIRST: return launch_kind<FK_FIRST>(a, high, pp.part != 0, s);
    case FK_MID: return launch_kind<FK_MID>(a, high, pp.part != 0, s);
    case FK_TURN: return launch_kind<FK_TURN>(a, high, pp.part != 0, s);
    case FK_LAST: return launch_kind<FK_LAST>(a, high, pp.part != 0, s);
    case FK_LASTG: return launch_kind<FK_LASTG>(a, high, pp.part != 0, s);
    case FK_BMID: return launch_kind<FK_BMID>(a, high, pp.part != 0, s);
    case FK_BTURN: return launch_kind<FK_BTURN>(a, high, pp.part != 0, s);
    case FK_BLAST: return launch_kind<FK_BLAST>(a, high, pp.part != 0, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_single128(const SingleArgs &a, int B, bool grad, int diag_type, hipStream_t s)
{
    const dim3 grid((unsigned)B), block(kThreads);
#define QQ_SINGLE128(DT)                                                              \
    if (grad) hipLaunchKernelGGL((single128<2, DT>), grid, block, 0, s, a);           \
    else hipLaunchKernelGGL((single128<1, DT>), grid, block, 0, s, a)
    switch (diag_type) {
    case DIAG_F64: QQ_SINGLE128(double); break;
    case DIAG_I32: QQ_SINGLE128(int32_t); break;
    default: QQ_SINGLE128(int16_t); break;
    }
#undef QQ_SINGLE128
    return hipGetLastError();
}

}  // namespace qq
