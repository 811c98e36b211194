// qq_many.hip -- one persistent launch evaluating many problems of uneven n and p.
//
// The launch drains a queue of work items (problem, parameter set, pass, tile
// chunk).  A multi-pass problem (n > 12) runs the same complex64 pass bodies as
// the per-pass kernels, one chunk of tiles per item; its pass j + 1 may start
// on a state once every chunk of pass j on that state has completed.  A problem
// with n <= 12 is a single item: one workgroup runs the whole evaluation (all p
// layers, the energy and the adjoint sweep) on one register-resident tile.
// The complex128 launch (many128_kernel) does the same with the complex128
// bodies.
//
// Ordering and progress.  Tickets are handed out in increasing order from one
// atomic counter, and items are numbered so that every pass of a state comes
// after its earlier passes (the host orders them by the fraction of each
// problem's pass chain done), so every item an item waits for has a smaller
// ticket and is held by a workgroup that is already running.  Hence the queue drains with
// any number of resident workgroups.  Every wait is bounded in wall-clock time;
// a wait that runs out sets an error flag, after which every workgroup stops
// taking items and the launch ends (the host reports the error).
//
// Memory ordering.  Each XCD has its own L2.  In the complex64 launch everything
// that one item writes and another reads (amplitudes, partial sums, counters) is
// accessed with agent-scope relaxed atomic operations, which are performed beyond
// the XCD's L2.  So an item is published when each wave has waited for its own
// stores and the workgroup has met at a barrier: thread 0's counter increment needs
// no cache write-back, and a waiting workgroup no invalidate.  Measured against a
// release and an acquire per item (XCD-wide cache operations): 512 problems 18.9
// against 20.5 ms, 128 problems 4.75 against 6.0, 96 problems 1.45 against 1.75.
// The language's memory model gives relaxed operations no order across addresses; what orders them here is
// the hardware and the compiled code.  A wave's agent-scope stores and loads are performed at the memory
// side of the L2s (write-through stores, loads that bypass the caches above), s_waitcnt(0) returns only once
// the wave's stores are acknowledged there, and the workgroup barriers, which the compiler moves no memory
// access across, keep thread 0's increment behind every wave's wait and every wave's loads behind thread
// 0's poll.  A compiler or target that kept any of these accesses in a cache of the XCD, moved one across
// a barrier or the wait, or let the wait end before the acknowledgement would need the release and
// acquire that FENCED adds (drain_queue).  The bitwise tests over grids and batches would show it.
// The complex128 launch keeps ordinary 16-byte accesses with a release and an
// acquire per item (its amplitudes as two 8-byte atomics: 12.6 against 10.4 ms).
//
// Reductions.  Each item writes its workgroup's FP64 partial sums, one per unit of its tiles; the workgroup that
// completes the last item of a state sums the partials in a fixed order (finish_state).  The units are the
// problem's own unless the caller sets the item size, so results are reproducible run to run and the same in
// every batch.
#include "qq_passes128.h"

namespace qq {
namespace {

using namespace dev;
using namespace passes;

// Partial sums, at agent scope.
__device__ __forceinline__ void st_partial(double *p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_partial(const double *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- problems with n <= 12: the whole evaluation in one tile ----------------------------------
// The tile holds 2^(12-n) identical copies of the state (tile bits n..11 are
// spectators: the cost diagonal is read at z & (2^n - 1) and those bits are never
// mixed), so tile sums are 2^(12-n) times the state's sums.

template <int L, typename DT>
__device__ __forceinline__ double cz_tile(const DT *diag, uint32_t mask, int t, int r)
{
    return (double)diag[(uint32_t)lidx<L>(t, r) & mask];
}

// psi *= exp(-i gamma C) in layout L.
template <int L, typename DT>
__device__ __forceinline__ void single_phase(float2 (&v)[kRegs], const DT *diag, uint32_t mask, int t, double g2pi)
{
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        float c, s;
        phase_rev(g2pi, cz_tile<L>(diag, mask, t, r), c, s);
        rot_phase<float>(v[r], c, s);
        QQ_CHUNK_FENCE(r);
    }
}

// sum |psi|^2 C; with GRAD also lambda = C psi.  The state is in layout 1 when
// L1 is set and in layout 2 otherwise (a uniform select of the register's index).
template <typename DT, bool GRAD>
__device__ __forceinline__ double single_energy(float2 (&v)[2][kRegs], const DT *diag, uint32_t mask, int t, bool L1)
{
    double e = 0.0;
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        const uint32_t z = (uint32_t)(L1 ? lidx<1>(t, r) : lidx<2>(t, r)) & mask;
        const double cz = (double)diag[z];
        const float pz = fmaf(v[0][r].x, v[0][r].x, v[0][r].y * v[0][r].y);
        e = fma((double)pz, cz, e);
        if constexpr (GRAD) {
            const float cf = (float)cz;
            v[1][r] = make_float2(cf * v[0][r].x, cf * v[0][r].y);
        }
        QQ_CHUNK_FENCE(r);
    }
    return e;
}

// sum C Im(conj(lambda) psi) in layout L, then both states un-phased.
template <int L, typename DT>
__device__ __forceinline__ double single_ggamma(float2 (&v)[2][kRegs], const DT *diag, uint32_t mask, int t,
                                                double g2pi)
{
    double gg = 0.0;
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
        const double cz = cz_tile<L>(diag, mask, t, r);
        const float2 ps = v[0][r], la = v[1][r];
        gg = fma(cz, (double)fmaf(la.x, ps.y, -la.y * ps.x), gg);
        float c, s;
        phase_rev(g2pi, cz, c, s);
        rot_phase<float>(v[0][r], c, -s);
        rot_phase<float>(v[1][r], c, -s);
        QQ_CHUNK_FENCE(r);
    }
    return gg;
}

// The thread index made opaque: per-register diagonal addresses and LDS slots are
// then formed where they are used rather than hoisted out of the layer loops
// (where 16 addresses per layout would stay live throughout).
__device__ __forceinline__ int fresh_index(int t)
{
    asm volatile("" : "+v"(t));
    return t;
}

// Forward layer k of a single-tile evaluation: phase, then the mixer from layout
// L (2 for even k, 1 for odd k) to the other layout.
template <int L, typename DT>
__device__ __forceinline__ void single_layer(float2 *lds, float2 (&v)[2][kRegs], const DT *diag, uint32_t mask,
                                             int t, int active, double g2pi, const MixCoef &c)
{
    const int tk = fresh_index(t);
    single_phase<L>(v[0], diag, mask, tk, g2pi);
    double unused = 0.0;
    mix_op<false, false, L, 2, 1, false, false>(lds, v, tk, active, c, unused);
}

// Adjoint step of layer k: inverse mixer with the beta-derivative, from the layout
// the forward layer ended in (1 for even k, 2 for odd k) back to L; then the
// gamma-derivative and the un-phase in L.  The un-phase after layer 0 is not needed
// and is harmless.  Returns (d/d beta_k, d/d gamma_k) partials of this thread.
template <int L, typename DT>
__device__ __forceinline__ void single_back(float2 *lds, float2 (&v)[2][kRegs], const DT *diag, uint32_t mask, int t,
                                            int active, double g2pi, const MixCoef &c, double &gb, double &gg)
{
    const int tk = fresh_index(t);
    gb = 0.0;
    mix_op<false, false, 3 - L, 2, 3, true, false>(lds, v, tk, active, c, gb);
    gg = single_ggamma<L>(v, diag, mask, tk, g2pi);
}

// Whole evaluation of parameter set b of a problem with n <= 12.  Output o of the
// problem (0: energy, 1 + 2k: d/d gamma_k, 2 + 2k: d/d beta_k, before the final
// scaling) is written to accumulator slot o, chunk 0.  Layer k's mixer runs 2 -> 1
// for even k and 1 -> 2 for odd k; the layers are taken in pairs so that every
// layout is fixed at compile time (the mixers use general butterflies, which serve
// both coefficient forms and the partial masks of n < 12).
template <typename DT, bool GRAD>
__device__ void single_eval(const ManyInst &I, double *partial, float2 *lds, double *s_red, MixCoef *s_coef, int t,
                            int b)
{
    const DT *diag = static_cast<const DT *>(I.diag);
    const uint32_t mask = (uint32_t)I.dim_mask;
    const int n = I.n, p = I.p;
    const int active = (1 << n) - 1;
    const double *x = I.params + (size_t)b * 2 * p;
    double *out = partial + I.partial_off + b;  // slot o at out[o * B]
    const size_t ostride = (size_t)I.B;
    // mixer coefficients of every layer (forward, then inverse), one thread per layer
    if (t < p) {
        s_coef[t] = mix_coef(x[2 * t + 1], false, n);
        s_coef[QQ_MAX_P + t] = mix_coef(x[2 * t + 1], true, n);
    }
    __syncthreads();
    float2 v[2][kRegs];
#pragma unroll
    for (int r = 0; r < kRegs; ++r) v[0][r] = make_float2((float)I.amp0, 0.0f);

    int k = 0;
    for (; k + 1 < p; k += 2) {
        single_layer<2>(lds, v, diag, mask, t, active, x[2 * k] * QQ_INV_TWO_PI, s_coef[k]);
        single_layer<1>(lds, v, diag, mask, t, active, x[2 * k + 2] * QQ_INV_TWO_PI, s_coef[k + 1]);
    }
    if (k < p) single_layer<2>(lds, v, diag, mask, t, active, x[2 * k] * QQ_INV_TWO_PI, s_coef[k]);
    // after layer p - 1 the state is in layout 1 (p odd) or 2 (p even)
    const int te = fresh_index(t);
    const double e = wg_sum(single_energy<DT, GRAD>(v, diag, mask, te, (p & 1) != 0), s_red, te);
    if (te == 0) st_partial(out, e);
    if constexpr (GRAD) {
        auto put = [&](int kk, double gb, double gg) {
            gb = wg_sum(gb, s_red, t);
            gg = wg_sum(gg, s_red, t);
            if (t == 0) {
                st_partial(out + (size_t)(2 + 2 * kk) * ostride, gb);
                st_partial(out + (size_t)(1 + 2 * kk) * ostride, gg);
            }
        };
        k = p - 1;
        double gb, gg;
        if ((k & 1) == 0) {  // p odd: the top layer is even and goes alone
            single_back<2>(lds, v, diag, mask, t, active, x[2 * k] * QQ_INV_TWO_PI, s_coef[QQ_MAX_P + k], gb, gg);
            put(k, gb, gg);
            --k;
        }
        for (; k >= 1; k -= 2) {
            single_back<1>(lds, v, diag, mask, t, active, x[2 * k] * QQ_INV_TWO_PI, s_coef[QQ_MAX_P + k], gb, gg);
            put(k, gb, gg);
            single_back<2>(lds, v, diag, mask, t, active, x[2 * k - 2] * QQ_INV_TWO_PI, s_coef[QQ_MAX_P + k - 1], gb,
                           gg);
            put(k - 1, gb, gg);
        }
    }
}

// ---- multi-pass problems: one chunk of one pass ---------------------------------------------
// Layer of an item's second mixer (its first one's is the pass's own layer k; the first pass's is 0).
__device__ __forceinline__ int second_layer(int kind, int k)
{
    return kind == FK_TURN ? k + 1 : kind == FK_BTURN ? k - 1 : k;
}

// A wave's sum of one value per lane, in lane 63: rows of 16 by shifts inside the row, then across the rows
// (DPP moves; the same sum over six dependent LDS permutes took 0.25 us per unit of a launch that waits on one
// chain).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, true);
    return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double x)
{
    x = dpp_add<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8: lane 15 of each row holds its row's sum
    x = dpp_add<0x112, 0xf>(x);
    x = dpp_add<0x114, 0xf>(x);
    x = dpp_add<0x118, 0xf>(x);
    x = dpp_add<0x142, 0xa>(x);     // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
}

// The units of an item, in order: body(u0, acc) runs the unit's tiles from u0 on, and the workgroup's
// fixed-order sums of acc are the unit's partial sums.  A unit is the problem's own (ManyInst::unit_log2), so that
// a state's sums do not depend on how the launch splits it into items.  A body holds barriers, which
// order one unit's reads of s_red before the next one's writes.
template <typename Body>
__device__ __forceinline__ void run_units(const ManyInst &I, const ManyPass &P, double *partial, double (*s_red)[4], int t,
                                          int b, int chunk, Body body)
{
    const uint64_t t0 = (uint64_t)chunk * (uint64_t)I.tpc, t1 = min(I.tiles, t0 + (uint64_t)I.tpc);
    for (uint64_t u0 = t0; u0 < t1; u0 += 1ull << I.unit_log2) {
        double acc[3] = {0.0, 0.0, 0.0};
        body(u0, acc);
        if (P.nslots == 0) continue;
        const int lane = t & 63, wave = t >> 6;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            if (s >= P.nslots) break;
            const double x = wave_total(acc[s]);
            if (lane == 63) s_red[wave][s] = x;
        }
        __syncthreads();
        if (t < P.nslots)
            st_partial(partial + I.partial_off + ((size_t)(P.slot_base + t) * I.B + b) * I.nunits + (u0 >> I.unit_log2),
                       (s_red[0][t] + s_red[1][t]) + (s_red[2][t] + s_red[3][t]));
    }
}

template <int KIND, typename DT>
__device__ __forceinline__ void run_geom(int geom, const FastArgs &a, float2 *lds, double (&acc)[3], int t, int b,
                                         int g, const MixCoef *s_coef)
{
    MixCoef c1 = s_coef[0], c2{};
    c1.formB = __builtin_amdgcn_readfirstlane(c1.formB);
    if constexpr (kind_two<KIND>()) {
        c2 = s_coef[1];
        c2.formB = __builtin_amdgcn_readfirstlane(c2.formB);
    }
    const double g2pi = phase_gamma<KIND>(a.params + (size_t)b * 2 * a.p, a.k) * QQ_INV_TWO_PI;
    if (geom == 0) {
        run_forms<KIND, false, true, DT, false, false, true, false>(a, lds, acc, t, b, g, c1, c2, g2pi);
    } else if constexpr (KIND != FK_FIRST) {  // the persistent plans take the qubit-0..11 set first
        if (geom == 1) run_forms<KIND, true, true, DT, false, false, true, false>(a, lds, acc, t, b, g, c1, c2, g2pi);
        else run_forms<KIND, true, false, DT, false, false, true, false>(a, lds, acc, t, b, g, c1, c2, g2pi);
    }
}

template <typename DT>
__device__ __forceinline__ void run_chunk(const ManyInst &I, const ManyPass &P, double *partial, float2 *lds,
                                          double (*s_red)[4], MixCoef *s_coef, int t, int b, int chunk)
{
    FastArgs a;
    a.B = I.B;
    a.G = 1;  // consecutive tiles
    a.p = I.p;
    a.k = P.k;
    a.dim_mask = I.dim_mask;
    a.pos4 = P.pos4;
    a.pos8 = P.pos8;
    a.w1 = P.w1;
    a.w2 = P.w2;
    a.active = P.active;
    a.nact = P.nact;
    a.store_psi = P.store_psi;
    a.slot_base = 0;
    a.slot_stride = 0;
    a.amp0 = I.amp0;
    a.params = I.params;
    a.diag = I.diag;
    a.psi = static_cast<float2 *>(I.psi);
    a.lam = static_cast<float2 *>(I.lam);
    a.state_stride = I.dim_mask + 1;
    a.partial = nullptr;
    a.blocked = 0;
    a.part = nullptr;
    a.tables = nullptr;
    a.cq = I.regq + 16 * (P.kind == FK_FIRST ? P.pos8 : P.pos4);
    a.pcq = nullptr;  // the persistent launch takes no partitioned phases
    a.pcq_runs = 0;
    a.shift = I.shift;
    a.ctab = P.ctab;
    a.cthr = P.cthr;
    a.xtab = a.xthr = nullptr;  // no partitioned phases here
    a.pre = nullptr;
    a.ilv = 0;  // separate psi and lambda arrays
    // the item's coefficients, formed by one thread each
    if (t < 2) {
        const int k = P.kind == FK_FIRST ? 0 : t == 0 ? P.k : second_layer(P.kind, P.k);
        const bool inverse = P.kind >= FK_BMID || (t == 1 && P.kind == FK_LASTG);
        s_coef[t] = mix_coef(I.params[((size_t)b * I.p + k) * 2 + 1], inverse, P.nact);
    }
    __syncthreads();
    run_units(I, P, partial, s_red, t, b, chunk, [&](uint64_t u0, double (&acc)[3]) __attribute__((always_inline)) {
        a.tiles = u0 + (1ull << I.unit_log2);
        const int g = (int)u0, ti = fresh_index(t);
        switch (P.kind) {
        case FK_FIRST: run_geom<FK_FIRST, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        case FK_MID: run_geom<FK_MID, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        case FK_TURN: run_geom<FK_TURN, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        case FK_LAST: run_geom<FK_LAST, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        case FK_LASTG: run_geom<FK_LASTG, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        case FK_BMID: run_geom<FK_BMID, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        case FK_BTURN: run_geom<FK_BTURN, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        default: run_geom<FK_BLAST, DT>(P.geom, a, lds, acc, ti, b, g, s_coef); break;
        }
    });
}

// Final results of state b: fixed-order sums of its partials.  16 lanes take a slot's units side by side, the
// workgroup 16 slots at once; one thread per output then adds the slots mapped to it.  Bound by the latency of
// reads beyond the L2, four in flight per lane; it stands at the end of every chain (one thread per output and
// one read at a time: one problem of n = 22, p = 6, whole call 2.45 ms against 1.33).
__device__ void finish_state(const ManyArgs &A, const ManyInst &I, double *lds, int b, int t)
{
    double *tot = lds;                                     // [nslots]
    int *out = reinterpret_cast<int *>(lds + kMaxSlots);  // [nslots]
    const int lane = t & 15;
    for (int s = t >> 4; s < I.nslots; s += kThreads / 16) {
        const double *src = A.partial + I.partial_off + ((size_t)s * I.B + b) * I.nunits;
        double x = 0.0;
        for (int c = lane; c < I.nunits; c += 64) {
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = c + 16 * u < I.nunits ? ld_partial(src + c + 16 * u) : 0.0;
#pragma unroll
            for (int u = 0; u < 4; ++u) x += v[u];
        }
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
        if (lane == 0) {
            tot[s] = x;
            out[s] = A.slot_out[I.slot_off + s];
        }
    }
    __syncthreads();
    const int nout = A.grad ? 1 + 2 * I.p : 1;
    for (int o = t; o < nout; o += kThreads) {
        double sum = 0.0;
        for (int s = 0; s < I.nslots; ++s)
            if (out[s] == o) sum += tot[s];
        const double v = o == 0 ? sum * I.escale + I.shift : sum * (2.0 * I.escale);
        if (I.energy_out) {
            if (o == 0) I.energy_out[b] = v;
            else I.grad_out[(size_t)b * 2 * I.p + (o - 1)] = v;
        } else {
            I.out_ws[(size_t)b * (1 + 2 * I.p) + o] = v;
        }
    }
    __syncthreads();  // the next item's body writes lds
}

// FENCED: an agent-scope release and acquire per item (bodies with ordinary state accesses).
// The queue of a persistent launch: take tickets until every item is taken or an error is flagged;
// wait until the item's state has completed its earlier passes, run(I, pass, b, chunk), publish
// the item, and let the workgroup that completes a state's last item finish that state.  The item
// bodies are lambdas marked always_inline: called out of line, they spill registers across the call.
template <bool FENCED, typename Run>
__device__ __forceinline__ void drain_queue(const ManyArgs &A, uint32_t *s_msg, double *lds, int t, Run run)
{
    uint32_t *head = A.ctl, *err = A.ctl + kCtlStride, *cnt = A.ctl + 2 * kCtlStride;
    int seg0 = 0;  // a segment at or before the next ticket's (tickets only grow)

    for (;;) {
        if (t == 0) {
            s_msg[0] = __hip_atomic_fetch_add(head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_msg[1] = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        const uint32_t ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_msg[0]);
        const uint32_t failed = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_msg[1]);
        __syncthreads();
        if (ticket >= A.total || failed) break;

        // the segment holding this ticket, the last one with first <= ticket: 64 segments ahead per probe,
        // at a stride of 64 and then of 1 (a binary search took a dozen dependent loads per item)
        int lo = seg0;
        const int lane = t & 63;
        for (int stride = 64; stride >= 1; stride >>= 6) {
            for (;;) {
                const int at = lo + lane * stride;
                const bool before = at < A.nseg && A.seg[at].first <= ticket;
                const int k = __popcll(__ballot(before));  // the lanes before it are a prefix, lane 0 among them
                lo += (k - 1) * stride;
                if (k < 64) break;
            }
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        seg0 = lo;
        const ManySeg sg = A.seg[lo];
        const ManyInst &I = A.inst[sg.inst];
        const int b = (int)sg.b;
        const int chunk = (int)(ticket - sg.first);
        const uint32_t state = (uint32_t)I.state0 + sg.b;

        if (sg.pass > 0) {
            // wait until every chunk of the previous passes on this state has completed
            const uint32_t need = sg.pass * (uint32_t)I.nchunks;
            if (t == 0) {
                uint32_t ok = 1;
                const uint64_t start = wall_clock64();
                while (__hip_atomic_load(cnt + (size_t)state * kCtlStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
                    if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        ok = 0;
                        break;
                    }
                    if (wall_clock64() - start > A.spin_ticks) {
                        __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ok = 0;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
                if constexpr (FENCED) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                s_msg[1] = ok;
            }
            __syncthreads();
            const uint32_t ok = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_msg[1]);
            __syncthreads();
            if (!ok) break;
            // (the barriers keep every amplitude load behind the poll)
        }

        run(I, (int)sg.pass, b, chunk);

        // publish: every wave waits until its own stores have been performed (at agent scope), the
        // barrier orders them before thread 0's increment
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (t == 0) {
            if constexpr (FENCED) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const uint32_t done = __hip_atomic_fetch_add(cnt + (size_t)state * kCtlStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
            s_msg[0] = done == (uint32_t)(I.npasses * I.nchunks) ? 1u : 0u;
        }
        __syncthreads();
        const uint32_t last = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_msg[0]);
        __syncthreads();
        if (last) finish_state(A, I, lds, b, t);
    }
}

template <typename DT>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) many_kernel(const ManyArgs A)
{
    __shared__ float2 lds[kLdsSlots];
    __shared__ double s_red[kThreads / 64][4];
    __shared__ uint32_t s_msg[2];
    __shared__ MixCoef s_coef[2 * QQ_MAX_P];
    const int t = threadIdx.x;
    drain_queue<false>(A, s_msg, reinterpret_cast<double *>(lds), t, [&](const ManyInst &I, int pass, int b, int chunk) __attribute__((always_inline)) {
        const ManyPass &P = A.pass[I.pass_off + pass];
        // The thread index, opaque per item: keeps each body's index arithmetic
        // inside its own branch instead of hoisted out of the item loop (where
        // the values of every body would stay live at once).
        int ti = t;
        asm volatile("" : "+v"(ti));
        if (P.kind == FK_SINGLE) {
            if (A.grad) single_eval<DT, true>(I, A.partial, lds, s_red[0], s_coef, ti, b);
            else single_eval<DT, false>(I, A.partial, lds, s_red[0], s_coef, ti, b);
        } else {
            run_chunk<DT>(I, P, A.partial, lds, s_red, s_coef, ti, b, chunk);
        }
    });
}

// ---- complex128 states -------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ void run_geom128(int geom, const p128::Args &a, double2 *lds, double (&acc)[3], int t, int b,
                                            int g, const double2 *s_cs)
{
    const p128::Coef f = p128::coef_of<KIND>(s_cs[0], s_cs[1], a.params + (size_t)b * 2 * a.p, a.k);
    // one-state kinds transpose in two rounds of 8-byte words (registers bound this kernel, not LDS)
    using W = typename std::conditional<kind_states<KIND>() == 2, double2, double>::type;
    W *l = reinterpret_cast<W *>(lds);
    if (geom == 0) {
        p128::pass_body<KIND, false, true, false>(a, l, acc, t, b, g, f);
    } else if constexpr (KIND != FK_FIRST) {  // the persistent plans take the qubit-0..11 set first
        if (geom == 1) p128::pass_body<KIND, true, true, false>(a, l, acc, t, b, g, f);
        else p128::pass_body<KIND, true, false, false>(a, l, acc, t, b, g, f);
    }
}

__device__ __forceinline__ void run_chunk128(const ManyInst &I, const ManyPass &P, double *partial, double2 *lds,
                                             double (*s_red)[4], double2 *s_cs, int t, int b, int chunk)
{
    p128::Args a;
    a.B = I.B;
    a.G = 1;  // consecutive tiles
    a.p = I.p;
    a.k = P.k;
    a.pos4 = P.pos4;
    a.pos8 = P.pos8;
    a.w1 = P.w1;
    a.w2 = P.w2;
    a.active = P.active;
    a.store_psi = P.store_psi;
    a.slot_base = 0;
    a.slot_stride = 0;
    a.amp0 = I.amp0;
    a.params = I.params;
    a.psi = static_cast<double2 *>(I.psi);
    a.lam = static_cast<double2 *>(I.lam);
    a.state_stride = I.dim_mask + 1;
    a.partial = nullptr;
    a.blocked = 0;
    a.cq = I.regq + 16 * (P.kind == FK_FIRST ? P.pos8 : P.pos4);
    a.ctab = P.ctab;
    a.cthr = P.cthr;
    a.ltab = a.lthr = a.xtab = a.xthr = nullptr;  // no partitioned phases here
    a.pre = nullptr;
    if (t < 2) {
        const int k = P.kind == FK_FIRST ? 0 : t == 0 ? P.k : second_layer(P.kind, P.k);
        double sb, cb;
        sincos(I.params[((size_t)b * I.p + k) * 2 + 1], &sb, &cb);
        s_cs[t] = make_double2(cb, sb);
    }
    __syncthreads();
    run_units(I, P, partial, s_red, t, b, chunk, [&](uint64_t u0, double (&acc)[3]) __attribute__((always_inline)) {
        a.tiles = u0 + (1ull << I.unit_log2);
        const int g = (int)u0, ti = fresh_index(t);
        switch (P.kind) {
        case FK_FIRST: run_geom128<FK_FIRST>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        case FK_MID: run_geom128<FK_MID>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        case FK_TURN: run_geom128<FK_TURN>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        case FK_LAST: run_geom128<FK_LAST>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        case FK_LASTG: run_geom128<FK_LASTG>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        case FK_BMID: run_geom128<FK_BMID>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        case FK_BTURN: run_geom128<FK_BTURN>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        default: run_geom128<FK_BLAST>(P.geom, a, lds, acc, ti, b, g, s_cs); break;
        }
    });
}

// The specialised complex128 bodies behind the same queue, two workgroups per compute unit (the
// operation-list bodies took 488 registers, one workgroup per unit).
template <typename DT>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) many128_kernel(const ManyArgs A)
{
    __shared__ double2 lds[kLdsSlots];
    __shared__ double s_red[kThreads / 64][4];
    __shared__ uint32_t s_msg[2];
    __shared__ double2 s_cs[QQ_MAX_P];
    const int t = threadIdx.x;
    drain_queue<true>(A, s_msg, reinterpret_cast<double *>(lds), t, [&](const ManyInst &I, int pass, int b, int chunk) __attribute__((always_inline)) {
        const ManyPass &P = A.pass[I.pass_off + pass];
        int ti = t;
        asm volatile("" : "+v"(ti));  // each body forms its indexes itself
        if (P.kind == FK_SINGLE) {
            const p128::Single e = {I.n, I.p, I.amp0, I.params + (size_t)b * 2 * I.p, I.diag};
            double *out = A.partial + I.partial_off + b;  // slot o at out[o * B]
            auto put = [&](int o, double v) __attribute__((always_inline)) { st_partial(out + (size_t)o * I.B, v); };
            if (A.grad) p128::single_eval<2, DT>(e, lds, s_red[0], s_cs, ti, nullptr, put);
            else p128::single_eval<1, DT>(e, lds, s_red[0], s_cs, ti, nullptr, put);
        } else {
            run_chunk128(I, P, A.partial, lds, s_red, s_cs, ti, b, chunk);
        }
    });
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// As many workgroups as can be resident at once (every one of them then runs until the queue is
// drained), at most max_grid (> 0) and at most one per item.
template <typename K>
hipError_t launch_resident(K kernel, const ManyArgs &a, int max_grid, hipStream_t s, int *grid_out)
{
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kThreads, 0)) != hipSuccess) return e;
    long grid = (long)std::max(1, per_cu) * std::max(1, cus);
    if (max_grid > 0) grid = std::min<long>(grid, max_grid);
    grid = std::max(1L, std::min<long>(grid, (long)a.total));
    if (grid_out) *grid_out = (int)grid;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

template <typename DT>
hipError_t launch_many_t(const ManyArgs &a, bool c128, int max_grid, hipStream_t s, int *grid_out)
{
    return c128 ? launch_resident(many128_kernel<DT>, a, max_grid, s, grid_out)
                : launch_resident(many_kernel<DT>, a, max_grid, s, grid_out);
}

}  // namespace

hipError_t launch_many(const ManyArgs &a, bool c128, int diag_type, int max_grid, hipStream_t s, int *grid_out)
{
    switch (diag_type) {
    case DIAG_F64: return launch_many_t<double>(a, c128, max_grid, s, grid_out);
    case DIAG_I32: return launch_many_t<int32_t>(a, c128, max_grid, s, grid_out);
    default: return launch_many_t<int16_t>(a, c128, max_grid, s, grid_out);
    }
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>(1024, (n + 255) / 256);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(blocks), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

}  // namespace qq
