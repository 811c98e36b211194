// qq_passes128.h -- complex128 tile-pass bodies specialised per pass kind.
//
// The pass kinds, tiles, thread layouts and cost tables are those of the complex64 bodies
// (qq_passes.h) with FP64 amplitudes: a pass streams tiles of 2^12 amplitudes through registers
// (256 threads x 16 amplitudes of 16 bytes per state), with the operation sequence and the layouts
// fixed at compile time.  Used by the per-pass kernels and by the persistent complex128 launch.
//
// Mixer: RX(2 beta) = cos(beta) I - i sin(beta) X applied as it stands, two products and two FMAs per
// amplitude and qubit (the FP64 vector rate leaves room for them: about 280 lane operations per
// amplitude pair of the heaviest kind, against 500 in the time its 64 bytes take).
//
// What bounds them: HBM bandwidth for states beyond the caches.  Two states of a tile take 128
// VGPRs, so the two-state kinds run two workgroups per compute unit; the transposes go through LDS in
// one round of 16-byte words (69.6 KB per workgroup, two workgroups fit the 160 KB).  The
// operation-list kernel that served these passes before kept one workgroup per compute unit (its
// layouts and masks were run-time values) and read the stored diagonal.  Measured at n = 22, four
// states: adjoint passes 450 -> 252 us (low set) and 305 us (high sets) for 1 GiB, forward ones 250 -> 106
// and 128 us for 0.5 GiB; 4.5 to 5.4 TB/s at n = 25 and 28 against 4.7 of a large copy.  Alternating
// blocks of psi and lambda (as in complex64) changed nothing at n = 25 and slowed the seed pass at n = 28
// (4.07 -> 4.64 ms), so the two stay apart.
#pragma once

#include "qq_passes.h"

namespace qq {
namespace p128 {

using namespace dev;
using passes::opaque_u64;
using passes::RegCost;
using passes::reg_cost;
using passes::reg_cost_form;
using passes::RegQ;
using passes::tab_load;
using passes::TabVals;
using passes::u32x4;

// exp(-i theta): theta reduced modulo pi/2 by a two-term Cody-Waite reduction with FMAs, then the Taylor
// polynomials of sine (to x^17) and cosine (to x^16) on [-pi/4, pi/4], whose remainders there are below
// 1e-19 and 3e-18.  The rounding of theta * 2 / pi leaves the remainder up to |theta| 2^-52 outside that
// interval, so it is reduced once more (by j = 0, which changes nothing, up to about |theta| = 2^44; the low
// part of j pi / 2 is below the first step's own rounding) and bounded; the result keeps modulus 1 for every
// finite theta.  Straight-line: a branch to this step spills the two-state kinds.
__device__ __forceinline__ void cos_sin(double th, double &c, double &s)
{
    const double k = rint(th * (4.0 * QQ_INV_TWO_PI));
    double x = fma(-k, 0.25 * QQ_TWO_PI_LO, fma(-k, 0.25 * QQ_TWO_PI_HI, th));
    const double j = rint(x * (4.0 * QQ_INV_TWO_PI));
    x = fma(-j, 0.25 * QQ_TWO_PI_HI, x);
    x = fabs(x) > 0.8 ? 0.0 : x;  // beyond 2^96 or so; a NaN stays
    const int q = (int)(k - 4.0 * rint(0.25 * k)) + (int)j;  // k + j modulo 4 in the low bits
    const double y = x * x;
    double ps = 1.0 / 355687428096000.0;
    ps = fma(ps, y, -1.0 / 1307674368000.0);
    ps = fma(ps, y, 1.0 / 6227020800.0);
    ps = fma(ps, y, -1.0 / 39916800.0);
    ps = fma(ps, y, 1.0 / 362880.0);
    ps = fma(ps, y, -1.0 / 5040.0);
    ps = fma(ps, y, 1.0 / 120.0);
    ps = fma(ps, y, -1.0 / 6.0);
    const double sx = fma(x * y, ps, x);
    double pc = 1.0 / 20922789888000.0;
    pc = fma(pc, y, -1.0 / 87178291200.0);
    pc = fma(pc, y, 1.0 / 479001600.0);
    pc = fma(pc, y, -1.0 / 3628800.0);
    pc = fma(pc, y, 1.0 / 40320.0);
    pc = fma(pc, y, -1.0 / 720.0);
    pc = fma(pc, y, 1.0 / 24.0);
    // 1 - y/2 + y^2 pc with the rounding of 1 - y/2 carried along
    const double h = 0.5 * y, w = 1.0 - h;
    const double cx = w + fma(y * y, pc, (1.0 - w) - h);
    const double a = (q & 1) ? cx : sx, b = (q & 1) ? sx : cx;
    s = (q & 2) ? -a : a;
    c = ((q + 1) & 2) ? -b : b;
}

// State amplitudes are streamed once per pass: non-temporal 16-byte accesses through a wave-uniform
// 64-bit base and a per-lane offset.
template <typename O>
__device__ __forceinline__ double2 gld(uint64_t sbase, O voff)
{
    const u32x4 u =
        __builtin_nontemporal_load(reinterpret_cast<const u32x4 __attribute__((address_space(1))) *>(sbase + voff));
    return make_double2(__hiloint2double((int)u.y, (int)u.x), __hiloint2double((int)u.w, (int)u.z));
}
template <typename O>
__device__ __forceinline__ void gst(uint64_t sbase, O voff, double2 x)
{
    u32x4 u;
    u.x = (uint32_t)__double2loint(x.x);
    u.y = (uint32_t)__double2hiint(x.x);
    u.z = (uint32_t)__double2loint(x.y);
    u.w = (uint32_t)__double2hiint(x.y);
    __builtin_nontemporal_store(u, reinterpret_cast<u32x4 __attribute__((address_space(1))) *>(sbase + voff));
}

// Transpose between two layouts.  Two-state kinds: one round of 16-byte words through 69.6 KB of LDS
// (two workgroups per compute unit, which their registers allow).  One-state kinds: the real parts,
// then the imaginary parts, through 34.8 KB (room for the three workgroups per compute unit that the registers
// of the kinds with a phase or an energy allow, and the four of the middle pass).
template <int FROM, int TO>
__device__ __forceinline__ void xpose(double2 *lds, double2 (&v)[kRegs], int t)
{
    __syncthreads();
    double2 *p = lds + slot_base<FROM>(t);
#pragma unroll
    for (int r = 0; r < kRegs; ++r) p[slot_stride<FROM>() * r] = v[r];
    __syncthreads();
    const double2 *q = lds + slot_base<TO>(t);
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[r] = q[slot_stride<TO>() * r];
}
template <int FROM, int TO>
__device__ __forceinline__ void xpose(double *lds, double2 (&v)[kRegs], int t)
{
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        __syncthreads();
        lds_put<FROM>(lds, v, t, c);
        __syncthreads();
        lds_get<TO>(lds, v, t, c);
    }
}

// RX(2 beta) on register bit K.
template <int K>
__device__ __forceinline__ void bf(double2 (&v)[kRegs], double c, double s)
{
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        if (r & (1 << K)) continue;
        const double2 a = v[r], b = v[r | (1 << K)];
        v[r] = make_double2(fma(c, a.x, s * b.y), fma(c, a.y, -(s * b.x)));
        v[r | (1 << K)] = make_double2(fma(c, b.x, s * a.y), fma(c, b.y, -(s * a.x)));
    }
    QQ_STAGE_FENCE();
}

// sum over the register pairs of bit K of Im(conj(l_r) a_{r|2^K} + conj(l_{r|2^K}) a_r), in four chains
template <int K>
__device__ __forceinline__ double xexp(const double2 (&a)[kRegs], const double2 (&l)[kRegs])
{
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        if (r & (1 << K)) continue;
        const int q = r | (1 << K);
        s0 = fma(l[r].x, a[q].y, s0);
        s1 = fma(-l[r].y, a[q].x, s1);
        s2 = fma(l[q].x, a[r].y, s2);
        s3 = fma(-l[q].y, a[r].x, s3);
    }
    QQ_STAGE_FENCE();
    return (s0 + s1) + (s2 + s3);
}

// Mixer on the four register bits; ON: every bit active, else the bits of `mask` (the identity on the
// others, selected in scalar registers).
template <int NS, int ST, bool GB, bool ON>
__device__ __forceinline__ void group(double2 (&v)[NS][kRegs], int mask, double c, double s, double &gacc)
{
    if constexpr (!ON)
        if (mask == 0) return;
#define QQ_BIT128(K)                                                              \
    {                                                                             \
        const double ck = ON || (mask & (1 << K)) ? c : 1.0;                      \
        const double sk = ON || (mask & (1 << K)) ? s : 0.0;                      \
        if constexpr (GB) {                                                       \
            const double x = xexp<K>(v[0], v[NS - 1]);                            \
            gacc += ON || (mask & (1 << K)) ? x : 0.0;                            \
        }                                                                         \
        if constexpr (ST & 1) bf<K>(v[0], ck, sk);                                \
        if constexpr (NS > 1 && (ST & 2)) bf<K>(v[NS - 1], ck, sk);               \
    }
    QQ_BIT128(0)
    QQ_BIT128(1)
    QQ_BIT128(2)
    QQ_BIT128(3)
#undef QQ_BIT128
}

template <int FROM, int TO, int NS, int ST, typename W>
__device__ __forceinline__ void xpose_all(W *lds, double2 (&v)[NS][kRegs], int t)
{
    if constexpr (ST & 1) xpose<FROM, TO>(lds, v[0], t);
    if constexpr (NS > 1 && (ST & 2)) xpose<FROM, TO>(lds, v[NS - 1], t);
}

// One mixer operation on the active tile bits from layout FROM (2 or 1) to the other one; GB:
// accumulate sum_q Im<lambda|X_q|psi> (both states live).
template <bool HIGH, bool FULL, int FROM, int NS, int ST, bool GB, typename W>
__device__ __forceinline__ void mix_op(W *lds, double2 (&v)[NS][kRegs], int t, int active, double c, double s,
                                       double &gacc)
{
    int am = 0;
    if constexpr (!FULL) {
        // opaque here, so the selects are formed at each use instead of held across the tile loop
        am = __builtin_amdgcn_readfirstlane(active);
        asm volatile("" : "+s"(am));
    }
    constexpr int A = FROM, Z = 3 - FROM;
    const int ma = (am >> (4 * A)) & 15, mz = (am >> (4 * Z)) & 15;
    group<NS, ST, GB, FULL>(v, ma, c, s, gacc);
    if constexpr (!HIGH) {
        xpose_all<A, 0, NS, ST>(lds, v, t);
        group<NS, ST, GB, FULL>(v, am & 15, c, s, gacc);
        xpose_all<0, Z, NS, ST>(lds, v, t);
    } else {
        xpose_all<A, Z, NS, ST>(lds, v, t);
    }
    group<NS, ST, GB, FULL>(v, mz, c, s, gacc);
}

// Arguments of one pass (fields as in passes::FastArgs; the cost always comes from the tables).
struct Args {
    int B, G, p, k;
    uint64_t tiles;
    int pos4, pos8, w1, w2, active;
    int store_psi;
    int slot_base, slot_stride;
    double amp0;
    const double *params;
    double2 *psi;
    double2 *lam;
    uint64_t state_stride;
    double *partial;
    int blocked;
    const double *cq;
    const double *ctab;
    const double *cthr;
    double2 *pre;  // [B][p]: (cos, sin) of beta_k, written by the first pass (per-pass kernels)
    const double *ltab, *lthr, *xtab, *xthr;  // PART: the QPU-local parts' and the cross part's
};

// The layer constants of a pass: (cos, sin) of the first and the second mixer, gamma of its phase.
struct Coef {
    double c1, s1, c2, s2, gam;
};

// From the (cos, sin) of the kind's own layer k and, where it has a second mixer of another layer, of that one.
template <int KIND>
__device__ __forceinline__ Coef coef_of(double2 first, double2 second, const double *x, int k)
{
    Coef f{};
    f.c1 = first.x;
    f.s1 = KIND >= FK_BMID ? -first.y : first.y;
    f.gam = passes::phase_gamma<KIND>(x, k);
    if constexpr (KIND == FK_TURN) {
        f.c2 = second.x;
        f.s2 = second.y;
    } else if constexpr (KIND == FK_LASTG) {
        f.c2 = first.x;
        f.s2 = -first.y;
    } else if constexpr (KIND == FK_BTURN) {
        f.c2 = second.x;
        f.s2 = -second.y;
    }
    return f;
}
// In a per-pass kernel: from the first pass's (cos, sin) per layer (the first pass itself forms its own).
template <int KIND>
__device__ __forceinline__ Coef coef(const Args &a, int b)
{
    const double *x = a.params + (size_t)b * 2 * a.p;
    const int k = a.k;
    auto cs = [&](int layer) {
        if constexpr (KIND != FK_FIRST) {
            const auto *q = (const double __attribute__((address_space(4))) *)(a.pre + (size_t)b * a.p + layer);
            return make_double2(q[0], q[1]);
        } else {
            double s, c;
            sincos(x[2 * layer + 1], &s, &c);
            return make_double2(c, s);
        }
    };
    const double2 first = cs(KIND == FK_FIRST ? 0 : k);
    double2 second = make_double2(0.0, 0.0);
    if constexpr (KIND == FK_TURN) second = cs(k + 1);
    if constexpr (KIND == FK_BTURN) second = cs(k - 1);
    return coef_of<KIND>(first, second, x, k);
}

// The tile loop of one pass kind (the kinds' operations are listed in qq_passes.h).
// PART: phases by the QPU-local parts together and the cross part, one rotation by the sum of their two
// quadratic forms (the operation-list kernel took a gathered read, a sine and a cosine per QPU and amplitude:
// n = 20, eight sets, three QPUs, p = 3, gradient 3.62 -> 0.79 ms).
template <int KIND, bool HIGH, bool FULL, bool PART, typename W>
__device__ __forceinline__ void pass_body(const Args &a, W *lds, double (&acc)[3], int t, int b, int g,
                                          const Coef &f)
{
    constexpr int NS = passes::kind_states<KIND>();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t lane_lo = t & 15, lane_hi = (t >> 4) & 3;
    // partial high sets: the upper run of n >= 31 puts a lane's layout-1 offset beyond 32 bits
    using O1 = typename std::conditional<HIGH && !FULL, uint64_t, uint32_t>::type;
    const O1 vs2 = ((O1)lane_lo + ((O1)lane_hi << a.pos4)) * (O1)16;
    const O1 vs1 = ((O1)lane_lo + ((O1)lane_hi << a.pos8)) * (O1)16;
    const uint64_t w2 = (uint64_t)wave << (a.pos4 + 2), w1 = (uint64_t)wave << (a.pos8 + 2);
    const uint64_t psi_a = (uint64_t)(a.psi + (size_t)b * a.state_stride);
    const uint64_t lam_a = (uint64_t)(a.lam + (size_t)b * a.state_stride);
    double2 v[NS][kRegs];

    uint64_t t_begin = (uint64_t)g, t_end = a.tiles, t_step = (uint64_t)a.G;
    if (a.blocked) {
        const uint64_t per = a.tiles / (uint64_t)a.G;
        t_begin = (uint64_t)g * per;
        t_end = t_begin + per;
        t_step = 1;
    }
    for (uint64_t tile = t_begin; tile < t_end; tile += t_step) {
        uint64_t base;
        if constexpr (HIGH) base = tile_base(tile, a.pos4, a.pos8, a.w1, a.w2);
        else base = tile << kTileBits;
        // register strides, opaque per use so their multiples are formed in scalar registers there
        const uint64_t ss2 = opaque_u64(1ull << a.pos8), ss1 = opaque_u64(1ull << a.pos4);
        const uint64_t sb2 = base + w2, sb1 = base + w1;
        RegQ *cq = (RegQ *)a.cq;
        TabVals tv, xv;
        RegCost rc;
        auto tab = [&]() {
            tab_load(tv, (PART ? a.ltab : a.ctab) + tile * kCostRow, (PART ? a.lthr : a.cthr) + 8 * t, t, wave);
            if constexpr (PART) tab_load(xv, a.xtab + tile * kCostRow, a.xthr + 8 * t, t, wave);
        };
        auto form = [&]() {
            if constexpr (PART) {
                tv.lane += xv.lane;
                tv.wave += xv.wave;
#pragma unroll
                for (int j = 0; j < 4; ++j) tv.reg[j] += xv.reg[j];
#pragma unroll
                for (int j = 0; j < 5; ++j) tv.thr[j] += xv.thr[j];
            }
            reg_cost_form(rc, tv);
        };
        auto load = [&](uint64_t arr, double2 (&x)[kRegs]) {
#pragma unroll
            for (int r = 0; r < kRegs; ++r) x[r] = gld<O1>(arr + (sb2 + r * ss2) * 16, vs2);
        };
        auto store2 = [&](uint64_t arr, const double2 (&x)[kRegs]) {
            const uint64_t ss = opaque_u64(ss2);
#pragma unroll
            for (int r = 0; r < kRegs; ++r) gst<O1>(arr + (sb2 + r * ss) * 16, vs2, x[r]);
        };
        auto store1 = [&](uint64_t arr, const double2 (&x)[kRegs]) {
            const uint64_t ss = opaque_u64(ss1);
#pragma unroll
            for (int r = 0; r < kRegs; ++r) gst<O1>(arr + (sb1 + r * ss) * 16, vs1, x[r]);
        };
        double unused = 0.0;
        if constexpr (KIND == FK_FIRST) {
            tab();
            form();
#pragma unroll
            for (int r = 0; r < kRegs; ++r) {
                double c, s;
                cos_sin(f.gam * reg_cost(rc, cq, r), c, s);
                v[0][r] = make_double2(a.amp0 * c, -(a.amp0 * s));
                __builtin_amdgcn_sched_barrier(0);
            }
            mix_op<HIGH, FULL, 2, 1, 1, false>(lds, v, t, a.active, f.c1, f.s1, unused);
            store1(psi_a, v[0]);
        } else if constexpr (KIND == FK_MID || KIND == FK_TURN || KIND == FK_LAST) {
            load(psi_a, v[0]);
            if constexpr (KIND != FK_MID) tab();
            mix_op<HIGH, FULL, 2, 1, 1, false>(lds, v, t, a.active, f.c1, f.s1, unused);
            if constexpr (KIND == FK_MID) {
                store1(psi_a, v[0]);
            } else if constexpr (KIND == FK_TURN) {
                form();
#pragma unroll
                for (int r = 0; r < kRegs; ++r) {
                    double c, s;
                    cos_sin(f.gam * reg_cost(rc, cq, r), c, s);
                    rot_phase<double>(v[0][r], c, s);
                    __builtin_amdgcn_sched_barrier(0);
                }
                mix_op<HIGH, FULL, 1, 1, 1, false>(lds, v, t, a.active, f.c2, f.s2, unused);
                store2(psi_a, v[0]);
            } else {
                form();
                double e = 0.0;
#pragma unroll
                for (int r = 0; r < kRegs; ++r)
                    e = fma(fma(v[0][r].x, v[0][r].x, v[0][r].y * v[0][r].y), reg_cost(rc, cq, r), e);
                acc[0] += e;
                if (a.store_psi) store1(psi_a, v[0]);
            }
        } else if constexpr (KIND == FK_LASTG) {
            load(psi_a, v[0]);
            tab();
            mix_op<HIGH, FULL, 2, 2, 1, false>(lds, v, t, a.active, f.c1, f.s1, unused);
            form();
            double e = 0.0;
#pragma unroll
            for (int r = 0; r < kRegs; ++r) {
                const double cz = reg_cost(rc, cq, r);
                e = fma(fma(v[0][r].x, v[0][r].x, v[0][r].y * v[0][r].y), cz, e);
                v[1][r] = make_double2(cz * v[0][r].x, cz * v[0][r].y);
            }
            acc[0] += e;
            mix_op<HIGH, FULL, 1, 2, 3, true>(lds, v, t, a.active, f.c2, f.s2, acc[1]);
            store2(lam_a, v[1]);
        } else {
            load(psi_a, v[0]);
            load(lam_a, v[1]);
            if constexpr (KIND != FK_BMID) tab();
            mix_op<HIGH, FULL, 2, 2, 3, true>(lds, v, t, a.active, f.c1, f.s1, acc[0]);
            if constexpr (KIND == FK_BMID) {
                store1(psi_a, v[0]);
                store1(lam_a, v[1]);
            } else {
                form();
                double gg = 0.0;
#pragma unroll
                for (int r = 0; r < kRegs; ++r) {
                    const double cz = reg_cost(rc, cq, r);
                    const double2 ps = v[0][r], la = v[1][r];
                    gg = fma(cz, fma(la.x, ps.y, -(la.y * ps.x)), gg);
                    if constexpr (KIND == FK_BTURN) {
                        double c, s;
                        cos_sin(f.gam * cz, c, s);
                        rot_phase<double>(v[0][r], c, -s);
                        rot_phase<double>(v[1][r], c, -s);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[1] += gg;
                if constexpr (KIND == FK_BTURN) {
                    mix_op<HIGH, FULL, 1, 2, 3, true>(lds, v, t, a.active, f.c2, f.s2, acc[2]);
                    store2(psi_a, v[0]);
                    store2(lam_a, v[1]);
                }
            }
        }
    }
}

// ---- problems with n <= 12: the whole evaluation of one parameter set in one tile -------------------
// The tile holds 2^(12-n) identical copies of the state (tile bits n..11 are never mixed and the
// diagonal is read at z & (2^n - 1)), so tile sums are 2^(12-n) times the state's sums.  Layer k's
// mixer runs from layout 2 to 1 for even k and back for odd k; the layers are taken in pairs so that
// every layout is fixed at compile time.  One workgroup per parameter set: the latency of its serial
// chain bounds it (about 700 FP64 operations per thread and layer forwards).
struct Single {
    int n, p;
    double amp0;
    const double *x;   // the set's 2p parameters
    const void *diag;
};

// C of an index; the loaded integer is opaque (16-bit loads were otherwise paired across registers and
// spilled 140 of them).
template <typename DT>
__device__ __forceinline__ double single_cost(const DT *diag, uint32_t i)
{
    if constexpr (std::is_same<DT, double>::value) return diag[i];
    int c = diag[i];
    asm("" : "+v"(c));
    return (double)c;
}

template <int L, int NS, typename DT, typename W>
__device__ __forceinline__ void single_layer(W *lds, double2 (&v)[NS][kRegs], const Single &a, uint32_t mask, int t,
                                             double gam, double2 cs)
{
    asm volatile("" : "+v"(t));  // addresses formed here, not held across the layer loop
    const DT *diag = static_cast<const DT *>(a.diag);
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        double c, s;
        cos_sin(gam * single_cost(diag, (uint32_t)lidx<L>(t, r) & mask), c, s);
        rot_phase<double>(v[0][r], c, s);
        if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    double unused = 0.0;
    mix_op<false, false, L, NS, 1, false>(lds, v, t, (int)mask, cs.x, cs.y, unused);
}

// Adjoint step of a layer: inverse mixer with the beta-derivative from the layout the forward layer ended
// in back to L, then the gamma-derivative and the un-phase (harmless after layer 0).
template <int L, typename DT, typename W>
__device__ __forceinline__ void single_back(W *lds, double2 (&v)[2][kRegs], const Single &a, uint32_t mask, int t,
                                            double gam, double2 cs, double &gb, double &gg)
{
    asm volatile("" : "+v"(t));
    gb = gg = 0.0;
    mix_op<false, false, 3 - L, 2, 3, true>(lds, v, t, (int)mask, cs.x, -cs.y, gb);
    const DT *diag = static_cast<const DT *>(a.diag);
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        const double cz = single_cost(diag, (uint32_t)lidx<L>(t, r) & mask);
        const double2 ps = v[0][r], la = v[1][r];
        gg = fma(cz, fma(la.x, ps.y, -(la.y * ps.x)), gg);
        double c, s;
        cos_sin(gam * cz, c, s);
        rot_phase<double>(v[0][r], c, -s);
        rot_phase<double>(v[1][r], c, -s);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Output o of the set (0: energy, 1 + 2k: d/d gamma_k, 2 + 2k: d/d beta_k, before the final scaling)
// goes to put(o, value) in thread 0; NS = 1: the energy alone, and the final state to psi
// unless it is NULL.
template <int NS, typename DT, typename W, typename Put>
__device__ __forceinline__ void single_eval(const Single &a, W *lds, double *s_red, double2 *s_cs, int t, double2 *psi,
                                            Put put)
{
    const int p = a.p;
    const uint32_t mask = (1u << a.n) - 1u;
    const double *x = a.x;
    if (t < p) {
        double sb, cb;
        sincos(x[2 * t + 1], &sb, &cb);
        s_cs[t] = make_double2(cb, sb);
    }
    __syncthreads();
    double2 v[NS][kRegs];
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[0][r] = make_double2(a.amp0, 0.0);
    int k = 0;
    for (; k + 1 < p; k += 2) {
        single_layer<2, NS, DT>(lds, v, a, mask, t, x[2 * k], s_cs[k]);
        single_layer<1, NS, DT>(lds, v, a, mask, t, x[2 * k + 2], s_cs[k + 1]);
    }
    if (k < p) single_layer<2, NS, DT>(lds, v, a, mask, t, x[2 * k], s_cs[k]);
    // the state is in layout 1 (p odd) or 2 (p even)
    const bool odd = p & 1;
    const DT *diag = static_cast<const DT *>(a.diag);
    int te = t;
    asm volatile("" : "+v"(te));
    double e = 0.0;
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        const uint32_t i = (uint32_t)(odd ? lidx<1>(te, r) : lidx<2>(te, r));
        const double cz = single_cost(diag, i & mask);
        e = fma(fma(v[0][r].x, v[0][r].x, v[0][r].y * v[0][r].y), cz, e);
        if constexpr (NS > 1) v[1][r] = make_double2(cz * v[0][r].x, cz * v[0][r].y);
        if (NS == 1 && psi && i <= mask) psi[i] = v[0][r];
        __builtin_amdgcn_sched_barrier(0);
    }
    e = passes::wg_sum(e, s_red, t);
    if (t == 0) put(0, e);
    if constexpr (NS > 1) {
        auto sums = [&](int kk, double gb, double gg) __attribute__((always_inline)) {
            gb = passes::wg_sum(gb, s_red, t);
            gg = passes::wg_sum(gg, s_red, t);
            if (t == 0) {
                put(2 + 2 * kk, gb);
                put(1 + 2 * kk, gg);
            }
        };
        double gb, gg;
        k = p - 1;
        if ((k & 1) == 0) {  // p odd: the top layer is even and goes alone
            single_back<2, DT>(lds, v, a, mask, t, x[2 * k], s_cs[k], gb, gg);
            sums(k, gb, gg);
            --k;
        }
        for (; k >= 1; k -= 2) {
            single_back<1, DT>(lds, v, a, mask, t, x[2 * k], s_cs[k], gb, gg);
            sums(k, gb, gg);
            single_back<2, DT>(lds, v, a, mask, t, x[2 * k - 2], s_cs[k - 1], gb, gg);
            sums(k - 1, gb, gg);
        }
    }
}

}  // namespace p128
}  // namespace qq
