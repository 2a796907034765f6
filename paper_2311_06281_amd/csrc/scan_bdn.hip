// Sequence-contiguous path: a, b, out are [rows, n] with rows = B*D; time runs along the lanes.
//
// Three kernels.
//  * rows_wave: one wave per row for rows that fit 64*ITEMS elements.  Lane i owns ITEMS consecutive
//    steps, scans them serially, the 64 lane summaries are scanned with DPP, each lane derives the
//    state at its first step and emits its elements.  No barrier, no global scratch; LDS only as the
//    wave's private staging area for coalesced global accesses.
//  * rows_packed: short rows, several per wave; the wave scan is confined to the lanes of a row.
//  * tiles: rows longer than that are cut into tiles of up to NW*64*ITEMS elements, one workgroup per
//    tile: the same lane and wave scans, wave summaries chained through LDS, tile summaries chained
//    through global memory in a two-level tree (see below); folds happen in a fixed order, so results
//    are bit-reproducible.
// All three move rows of any length and position as 16-byte vectors (see Span).
//
// What is computed is Sec. 4's expression applied by parts (Sec. 1, footnote on associativity); the
// arithmetic is in heinsen_math.hpp.
#include "heinsen_internal.hpp"
#include "heinsen_math.hpp"
#include "heinsen_tickets.hpp"
#include "scan_rules.hpp"

#include <algorithm>

namespace hs {
namespace {

// ---- lane-level pieces shared by the kernels ----------------------------------------------------------

// Encodes and scans the lane's elements serially.  On return Av[k], Mv[k] and bit k of sw (and of sm)
// hold the per-element records (see stash); the summary of all ITEMS steps is returned.
template <int DOM, bool LOG_IN, bool LOG_OUT, int ITEMS>
__device__ __forceinline__ Seg lane_scan(float (&Av)[ITEMS], float (&Mv)[ITEMS], uint32_t &sw, uint32_t &sm)
{
    static_assert(ITEMS <= 32, "sign bits are kept in one word");
    sw = sm = 0u;
    Seg run;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) lane_step<DOM, LOG_IN, LOG_OUT>(k, run, Av[k], Mv[k], sw, sm);
    lane_close<DOM, LOG_IN, LOG_OUT>(run);
    return run;
}


template <int DOM, bool LOG_OUT>
constexpr bool complex_output()
{
    return DOM == kSigned && LOG_OUT;
}

// ---- complex output: inputs kept in LDS, the definition in float64 ---------------------------------------
//
// By way of lane_scan's records a complex output costs six transcendentals per element (four of them in the
// log-domain steps), which is what bound it, and every step rounds a logarithm; one of 64 is good to 3e-6 of
// the number, which shows wherever x_k nearly cancels.  Where a wave's numbers allow it, it evaluates x_k =
// a_k x_{k-1} + b_k itself, in float64 (a fused multiply-add of which costs what one of float32 does here),
// in two passes over the lane's inputs: from 0 for the lane's summary (P, Z), x_e = P x_s + Z, which is
// composed across the lanes as it is, then from the lane's start state for the outputs, one logarithm per
// element.  Log-domain steps cannot leave their range, these can, so a wave takes them only if
//     a = 0 or |a| in [2^-36, 2^16], b = 0 or |b| in [2^-60, 2^60] for every element,
//     the lanes' products P that are above 1 multiply to at most 2^600 over the wave,
//     every lane's start state is in [2^-360, 2^600] (or is the row's x_0 = 0).
// The at most 16 steps of a lane then multiply any number by 0 or by 2^-576 to 2^256, so no state inside it reaches
// 2^-1022 or 2^1023, and neither does a Z (at most 2^(600 + 256 + 60) times the number of steps).  A term that
// underflows between lanes is below 2^-1022, grows by 2^600 at most, and is less than 2^-60 of any start state.
//
// Between the passes the inputs stay in the wave's LDS region, where the outputs then take their place:
// quads of a and b alternate, [a0..3][b0..3][a4..7][b4..7]..., and a lane's ITEMS/2 quads are followed by an
// empty one, so four elements leave eight floats exactly where they came from, in the order of the output.
// Registers hold one step's values (64 where the records of 16 steps took 96), and both passes are short
// loops.  8192 rows of 3001 steps: 148 us as records on eight waves of eight steps, 73 as records on three
// waves of 16, 70.5 this way, with 1/40 to 1/1000 of the error (3.6e-8 of the result's norm).
struct Lin {
    double P, Z;
};
__device__ __forceinline__ Lin lin_combine(const Lin &g1, const Lin &g2) { return Lin{g1.P * g2.P, fma(g1.Z, g2.P, g2.Z)}; }

constexpr int kLinUp = 600;

typedef float f32x4 __attribute__((ext_vector_type(4)));
struct Quads {
    f32x4 a, b;
};

// The passes.  get(q) returns elements 4q .. 4q+3 of the lane, put(q, re, im) takes their outputs.

// Pass 1 in float64; `up` = the exponent of P where that is positive.  Returns whether the lane's inputs are
// in range.
template <int ITEMS, typename GET>
__device__ __forceinline__ bool lin_summary(GET &&get, Lin &g, int &up)
{
    static_assert(ITEMS <= 16, "the bounds are for 16 steps per lane");
    float ahi = 1.0f, bhi = 0.0f;
    uint32_t alo = 0xffffffffu, blo = 0xffffffffu; // of 2|v| - 1 as an integer, which puts 0 above everything else
    g = Lin{1.0, 0.0};
#pragma unroll 2
    for (int q = 0; q < ITEMS / 4; ++q) {
        const Quads v = get(q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            g = lin_combine(g, Lin{(double)v.a[i], (double)v.b[i]});
            ahi = fmaxf(ahi, fabsf(v.a[i]));
            bhi = fmaxf(bhi, fabsf(v.b[i]));
            const uint32_t y = (f2u(v.a[i]) << 1) - 1u, z = (f2u(v.b[i]) << 1) - 1u;
            alo = y < alo ? y : alo;
            blo = z < blo ? z : blo;
        }
    }
    up = __builtin_amdgcn_frexp_exp(g.P);
    up = up > 0 ? up : 0;
    return alo >= ((127u - 36u) << 24) - 1u && ahi <= 0x1p16f && bhi <= 0x1p60f && blo >= ((127u - 60u) << 24) - 1u;
}

// Pass 2 in float64.
template <int ITEMS, typename GET, typename PUT>
__device__ __forceinline__ void lin_emit(double x, GET &&get, PUT &&put)
{
#pragma unroll 2
    for (int q = 0; q < ITEMS / 4; ++q) {
        const Quads v = get(q);
        f32x4 re, im;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x = fma((double)v.a[i], x, (double)v.b[i]);
            const float m = (float)__builtin_amdgcn_frexp_mant(x);
            re[i] = (log2_hw(fabsf(m)) + (float)__builtin_amdgcn_frexp_exp(x)) * kLn2;
            im[i] = u2f((uint32_t)((int32_t)f2u(m) >> 31) & f2u(kPi));
        }
        put(q, re, im);
    }
}

// The same passes by log-domain steps.  Pass 1 leaves every element's record (A_k, M_k) where a and b were
// (keep(q, A, M)), with its signs in sw and sm (see stash), so that pass 2 costs one log-add-exp per element.
template <int ITEMS, typename GET, typename KEEP>
__device__ __forceinline__ Seg log_summary(GET &&get, KEEP &&keep, uint32_t &sw, uint32_t &sm)
{
    static_assert(ITEMS <= 32, "sign bits are kept in one word");
    Seg run = seg_identity<kSigned>();
    sw = sm = 0u;
#pragma unroll 1
    for (int q = 0; q < ITEMS / 4; ++q) {
        const Quads v = get(q);
        f32x4 A, M;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float la, lb;
            uint32_t sa, sb;
            encode<kSigned, false>(v.a[i], la, sa);
            encode<kSigned, false>(v.b[i], lb, sb);
            if (q == 0 && i == 0) run = Seg{la, lb, sa, sb};
            else seg_step<kSigned>(run, la, sa, lb, sb);
            A[i] = run.A;
            M[i] = run.M;
            sw |= (run.sA >> 31) << (4 * q + i);
            sm |= (run.sM >> 31) << (4 * q + i);
        }
        keep(q, A, M);
    }
    return run;
}
template <int ITEMS, typename GET, typename PUT>
__device__ __forceinline__ void log_emit(const State &st, uint32_t sw, uint32_t sm, GET &&get, PUT &&put)
{
    const uint32_t swx = fold_state_sign<kSigned>(sw, st);
#pragma unroll 1
    for (int q = 0; q < ITEMS / 4; ++q) {
        const Quads v = get(q); // the records
        f32x4 re, im;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float re_i, im_i;
            emit_clog(st, v.a[i], v.b[i], swx, sm, 4 * q + i, re_i, im_i);
            re[i] = re_i;
            im[i] = im_i;
        }
        put(q, re, im);
    }
}

// Start state of a lane: in range for lin_emit?  `exact_zero`: a zero is x_0 itself.
__device__ __forceinline__ bool lin_state_ok(double x, bool exact_zero)
{
    return (fabs(x) >= 0x1p-360 && fabs(x) <= 0x1p600) || (exact_zero && x == 0.0);
}

// x_0 as a state (subnormal float32 counts as 0).
__device__ __forceinline__ double lin_x0(float x0) { return fabsf(x0) < 0x1p-126f ? 0.0 : (double)x0; }

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_d(double oldv, double v)
{
    const unsigned long long o = (unsigned long long)__double_as_longlong(oldv), x = (unsigned long long)__double_as_longlong(v);
    const uint32_t hi = dpp_u<CTRL, ROW_MASK>((uint32_t)(o >> 32), (uint32_t)(x >> 32));
    const uint32_t lo = dpp_u<CTRL, ROW_MASK>((uint32_t)o, (uint32_t)x);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ Lin lin_dpp(const Lin &g)
{
    return Lin{dpp_d<CTRL, ROW_MASK>(1.0, g.P), dpp_d<CTRL, ROW_MASK>(0.0, g.Z)};
}
__device__ __forceinline__ Lin lin_wave_inclusive_scan(Lin g)
{
    g = lin_combine(lin_dpp<0x111, 0xf>(g), g); // the steps of wave_inclusive_scan
    g = lin_combine(lin_dpp<0x112, 0xf>(g), g);
    g = lin_combine(lin_dpp<0x114, 0xf>(g), g);
    g = lin_combine(lin_dpp<0x118, 0xf>(g), g);
    g = lin_combine(lin_dpp<0x142, 0xa>(g), g);
    g = lin_combine(lin_dpp<0x143, 0xc>(g), g);
    return g;
}
__device__ __forceinline__ int wave_sum(int v)
{
    v += (int)dpp_u<0x111, 0xf>(0u, (uint32_t)v);
    v += (int)dpp_u<0x112, 0xf>(0u, (uint32_t)v);
    v += (int)dpp_u<0x114, 0xf>(0u, (uint32_t)v);
    v += (int)dpp_u<0x118, 0xf>(0u, (uint32_t)v);
    v += (int)dpp_u<0x142, 0xa>(0u, (uint32_t)v);
    v += (int)dpp_u<0x143, 0xc>(0u, (uint32_t)v);
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ bool wave_all(bool ok) { return __builtin_amdgcn_ballot_w64(!ok) == 0ull; }

// ---- one wave per row -------------------------------------------------------------------------------

struct RowsParams {
    const void *a;
    const void *b;
    const float *x0;
    float *out;
    int64_t rows, n;
    int x0_stride;
    int phase; // elements from the last 16-byte boundary to the first element of a and b (VECIO)
    bool both; // ask for a and b together
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A wave moves a row between global memory and its lanes through a private LDS region so that global
// accesses are coalesced (consecutive lanes touch consecutive 16-byte vectors) while each lane ends up
// with NV consecutive vectors of the row ("blocked").  Vector c of the row lives at slot c + c/NV: one
// empty slot after every lane's NV slots keeps both access patterns free of bank conflicts.  LDS
// operations of one wave execute in order, so only the compiler has to be kept from reordering them.
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); __builtin_amdgcn_wave_barrier(); }

// Rows of any length and position move as 16-byte vectors: a wave works on a window that begins at a
// 16-byte boundary at or before its first element, and only [lo, hi) of the window's elements exist (both
// wave-uniform; nothing outside is read or written).  What surrounds them is filled with steps that leave
// the state unchanged, so a row that starts inside a vector is simply a row with up to VL - 1 such steps in
// front.  Whole vectors move as such; the elements of the one vector at either end that is not whole move
// one by one, all of them in one predicated instruction.  Rows of odd length went one element at a time
// before (64 x 1024 rows of bf16: 2041 steps 596 -> 189 us, 300 steps of 64 x 4000 rows 251 -> 114 us).
struct Span {
    int lo, hi;
    __device__ __forceinline__ bool cut(int vl) const { return ((lo | hi) % vl) != 0; } // some vector is not whole (wave-uniform)
};
__device__ __forceinline__ Span wave_span(int64_t lo, int64_t hi, int cap)
{
    Span sp;
    sp.lo = lo < 0 ? 0 : (lo > cap ? cap : (int)lo);
    sp.hi = hi < 0 ? 0 : (hi > cap ? cap : (int)hi);
    return sp;
}

// The elements of the window's two partial vectors, one per lane: lanes 0 .. VL-1 take the vector that
// `lo` cuts, the next VL lanes the one that `hi` cuts.  Returns whether the lane has one, and which.
template <int VL>
__device__ __forceinline__ bool edge_element(int lo, int hi, int lane, int &e)
{
    e = lane < VL ? ((lo + VL - 1) / VL - 1) * VL + lane : hi / VL * VL + lane - VL;
    return lane < 2 * VL && e >= lo && e < hi;
}
// Global (striped, coalesced) -> the wave's LDS region: window vector c to slot c + c/NV.
template <typename InT, int NV>
__device__ __forceinline__ void wave_stage_span(const InT *win, Span sp, u32x4 fill, u32x4 *lds, int lane)
{
    constexpr int VL = 16 / (int)sizeof(InT);
    const u32x4 *wv = reinterpret_cast<const u32x4 *>(win);
    const int c_lo = (sp.lo + VL - 1) / VL;
    const int whole = sp.hi / VL - c_lo;
    const uint32_t count = whole > 0 ? (uint32_t)whole : 0u;
    const bool cut = sp.cut(VL);
    u32x4 t[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = j * 64 + lane;
        // streamed once: keep it out of the caches' way
        t[j] = ((uint32_t)(c - c_lo) < count) ? __builtin_nontemporal_load(wv + c) : fill;
    }
    InT x = 0;
    int e = 0;
    bool have = false;
    if (cut) {
        have = edge_element<VL>(sp.lo, sp.hi, lane, e);
        if (have) x = win[e];
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = j * 64 + lane;
        lds[c + c / NV] = t[j];
    }
    if (cut) {
        wave_lds_order();
        if (have) reinterpret_cast<InT *>(lds + (e / VL + e / VL / NV))[e % VL] = x;
    }
    wave_lds_order();
}

// The same in two parts, for a and b to be in flight together.  (Where they are not, the parts cost a launch that fills
// the chip 5 to 10 % over the whole: 32768 rows of 200 steps 15.6 and 14.7 us.)
template <typename InT, int NV>
__device__ __forceinline__ void span_fetch(const InT *win, Span sp, u32x4 fill, int lane, u32x4 (&t)[NV], InT &x)
{
    constexpr int VL = 16 / (int)sizeof(InT);
    const u32x4 *wv = reinterpret_cast<const u32x4 *>(win);
    const int c_lo = (sp.lo + VL - 1) / VL;
    const int whole = sp.hi / VL - c_lo;
    const uint32_t count = whole > 0 ? (uint32_t)whole : 0u;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = j * 64 + lane;
        t[j] = ((uint32_t)(c - c_lo) < count) ? __builtin_nontemporal_load(wv + c) : fill;
    }
    x = 0;
    if (sp.cut(VL)) {
        int e;
        if (edge_element<VL>(sp.lo, sp.hi, lane, e)) x = win[e];
    }
}
template <typename InT, int NV>
__device__ __forceinline__ void span_stage(Span sp, const u32x4 (&t)[NV], InT x, u32x4 *lds, int lane)
{
    constexpr int VL = 16 / (int)sizeof(InT);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = j * 64 + lane;
        lds[c + c / NV] = t[j];
    }
    if (sp.cut(VL)) {
        wave_lds_order();
        int e;
        if (edge_element<VL>(sp.lo, sp.hi, lane, e)) reinterpret_cast<InT *>(lds + (e / VL + e / VL / NV))[e % VL] = x;
    }
    wave_lds_order();
}

// Global (striped, coalesced) -> lanes (blocked), a and b.  Elements of the window outside [lo, hi) become fa, fb.
// `both`: both are asked for before either is waited for.
template <typename InT, int NV>
__device__ __forceinline__ void wave_load_spans(const InT *wa, const InT *wb, Span sp, u32x4 fa, u32x4 fb, bool both, u32x4 *lds,
                                                int lane, u32x4 (&va)[NV], u32x4 (&vb)[NV])
{
    auto pick = [&](u32x4 (&v)[NV]) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = lds[lane * (NV + 1) + q];
        wave_lds_order();
    };
    if (!both) {
        wave_stage_span<InT, NV>(wa, sp, fa, lds, lane);
        pick(va);
        wave_stage_span<InT, NV>(wb, sp, fb, lds, lane);
        pick(vb);
        return;
    }
    u32x4 ta[NV], tb[NV];
    InT xa, xb;
    span_fetch<InT, NV>(wa, sp, fa, lane, ta, xa);
    span_fetch<InT, NV>(wb, sp, fb, lane, tb, xb);
    if (NV == 1 && !sp.cut(16 / (int)sizeof(InT))) { // one vector per lane is where it belongs
        va[0] = ta[0];
        vb[0] = tb[0];
        return;
    }
    span_stage<InT, NV>(sp, ta, xa, lds, lane);
    pick(va);
    span_stage<InT, NV>(sp, tb, xb, lds, lane);
    pick(vb);
}

// The wave's LDS region -> global (striped, coalesced): floats [lo, hi) of the window are written.  A lane
// owns NV consecutive vectors of the window.  In ROUNDS rounds 64 / ROUNDS lanes at a time have theirs in the
// region, so that it need not grow with the output and every store instruction still writes one whole run.
// (Staging a part of every lane's vectors per round instead writes runs of a lane's part, 64 bytes, which
// cut the memory's sectors where a row does not begin on one: 8192 rows of 3001 complex values 127 us, of
// 3000 83 us.)
template <int NV, int ROUNDS>
__device__ __forceinline__ void wave_unstage_span(float *win, int lo, int hi, u32x4 *lds, int lane, int round)
{
    constexpr int STAGED = 64 / ROUNDS * NV; // vectors in the region
    u32x4 *wv = reinterpret_cast<u32x4 *>(win);
    const int first = round * STAGED;
    const int c_lo = (lo + 3) / 4;
    const int whole = hi / 4 - c_lo;
    const uint32_t count = whole > 0 ? (uint32_t)whole : 0u;
    u32x4 t[NV / ROUNDS];
#pragma unroll
    for (int j = 0; j < NV / ROUNDS; ++j) {
        const int c = j * 64 + lane;
        t[j] = lds[c + c / NV];
    }
#pragma unroll
    for (int j = 0; j < NV / ROUNDS; ++j) {
        const int c = first + j * 64 + lane;
        if ((uint32_t)(c - c_lo) < count) __builtin_nontemporal_store(t[j], wv + c);
    }
    if (((lo | hi) % 4) != 0) { // wave-uniform
        int f;
        if (edge_element<4>(lo, hi, lane, f)) {
            const int c = f / 4 - first;
            if (ROUNDS == 1 || (uint32_t)c < (uint32_t)STAGED) win[f] = reinterpret_cast<const float *>(lds + c + c / NV)[f % 4];
        }
    }
    wave_lds_order();
}

// The same two moves one element at a time, for a, b and out that lie differently to the 16-byte
// boundaries: global accesses are still coalesced (consecutive lanes, consecutive elements), the region
// holds 32-bit slots, element c of the wave's span at slot c + c/ITEMS.  `left` elements of the row exist
// from the wave's first one on.
template <typename InT, int ITEMS>
__device__ __forceinline__ void wave_load_blocked_elems(const InT *row, int64_t left, float fill, uint32_t *lds, int lane,
                                                        float (&x)[ITEMS])
{
    float t[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane;
        t[j] = (c < left) ? widen(__builtin_nontemporal_load(row + c)) : fill;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane;
        lds[c + c / ITEMS] = f2u(t[j]);
    }
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) x[k] = u2f(lds[lane * (ITEMS + 1) + k]);
    wave_lds_order();
}

// Lanes (blocked) -> global, one float at a time; a lane owns ITEMS * PARTS consecutive floats of the
// span and round `part` moves floats part*ITEMS .. part*ITEMS + ITEMS - 1 of every lane.
template <int ITEMS, int PARTS>
__device__ __forceinline__ void wave_store_blocked_elems(float *row, int64_t left, uint32_t *lds, int lane, int part,
                                                         const float (&x)[ITEMS])
{
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) lds[lane * (ITEMS + 1) + k] = f2u(x[k]);
    wave_lds_order();
    float t[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane;
        t[j] = u2f(lds[c + c / ITEMS]);
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane;
        const int gi = (c / ITEMS) * (ITEMS * PARTS) + part * ITEMS + c % ITEMS;
        if (gi < left) __builtin_nontemporal_store(t[j], row + gi);
    }
    wave_lds_order();
}

template <typename InT, int NVI, int ITEMS>
__device__ __forceinline__ void unpack_inputs(const u32x4 (&v)[NVI], float (&x)[ITEMS])
{
    if (sizeof(InT) == 4) {
#pragma unroll
        for (int q = 0; q < NVI; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[q * 4 + i] = u2f(v[q][i]);
    } else {
#pragma unroll
        for (int q = 0; q < NVI; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[q * 8 + 2 * i] = u2f(v[q][i] << 16);
                x[q * 8 + 2 * i + 1] = u2f(v[q][i] & 0xffff0000u);
            }
    }
}


// Output of the lane's elements, vector path: emitted and written, coalesced, through the wave's LDS region.
// `win` points at the wave's window in the output, `sp` holds the window's elements that exist.  A complex
// output has twice the bytes of a real one and goes through the region in two rounds, 32 lanes at a time.
template <int DOM, bool LOG_OUT, int ITEMS>
__device__ __forceinline__ void wave_emit_span(float *win, Span sp, u32x4 *lds, int lane, const State &st, const float (&Av)[ITEMS],
                                               const float (&Mv)[ITEMS], uint32_t sw, uint32_t sm)
{
    constexpr int NVO = ITEMS / 4;
    const uint32_t swx = fold_state_sign<DOM>(sw, st);
    if constexpr (DOM == kSigned && LOG_OUT) {
        constexpr int NVC = ITEMS / 2;
        u32x4 vo[NVC];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            float re, im;
            emit_clog(st, Av[k], Mv[k], swx, sm, k, re, im);
            vo[k / 2][2 * (k % 2)] = f2u(re);
            vo[k / 2][2 * (k % 2) + 1] = f2u(im);
        }
#pragma unroll
        for (int round = 0; round < 2; ++round) {
            if ((lane >> 5) == round) {
#pragma unroll
                for (int q = 0; q < NVC; ++q) lds[(lane & 31) * (NVC + 1) + q] = vo[q];
            }
            wave_lds_order();
            wave_unstage_span<NVC, 2>(win, 2 * sp.lo, 2 * sp.hi, lds, lane, round);
        }
    } else {
        u32x4 vo[NVO];
#pragma unroll
        for (int q = 0; q < NVO; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                vo[q][i] = f2u(emit<DOM, LOG_OUT>(st, Av[q * 4 + i], Mv[q * 4 + i], swx, q * 4 + i));
#pragma unroll
        for (int q = 0; q < NVO; ++q) lds[lane * (NVO + 1) + q] = vo[q];
        wave_lds_order();
        wave_unstage_span<NVO, 1>(win, sp.lo, sp.hi, lds, lane, 0);
    }
}

// Element-wise counterpart of the vector emit: `orow` points at the wave's first output element, `left`
// elements of the row exist from there on.
template <int DOM, bool LOG_OUT, int ITEMS>
__device__ __forceinline__ void wave_emit_blocked_elems(float *orow, int64_t left, uint32_t *lds, int lane, const State &st,
                                                        const float (&Av)[ITEMS], const float (&Mv)[ITEMS], uint32_t sw,
                                                        uint32_t sm)
{
    constexpr bool SIGNED = DOM == kSigned;
    const uint32_t swx = fold_state_sign<DOM>(sw, st);
    left = left < 0 ? 0 : left;
    if constexpr (SIGNED && LOG_OUT) {
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            float o[ITEMS];
#pragma unroll
            for (int i = 0; i < ITEMS / 2; ++i) {
                const int k = part * (ITEMS / 2) + i;
                emit_clog(st, Av[k], Mv[k], swx, sm, k, o[2 * i], o[2 * i + 1]);
            }
            wave_store_blocked_elems<ITEMS, 2>(orow, 2 * left, lds, lane, part, o);
        }
    } else {
        float o[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) o[k] = emit<DOM, LOG_OUT>(st, Av[k], Mv[k], swx, k);
        wave_store_blocked_elems<ITEMS, 1>(orow, left, lds, lane, 0, o);
    }
}


// Complex output: a and b of the wave's window -> its region, in quads as described above.  Everything
// is asked for before anything is waited for.  Elements that do not exist become a = 1, b = 0.
template <int ITEMS>
constexpr int clog_slots()
{
    return 64 * (ITEMS / 2 + 1); // 16-byte slots per wave
}
template <int ITEMS>
__device__ __forceinline__ int clog_slot(int quad, int which) // quad of the window; which: 0 a, 1 b
{
    return quad / (ITEMS / 4) * (ITEMS / 2 + 1) + 2 * (quad % (ITEMS / 4)) + which;
}

template <typename InT, int ITEMS>
__device__ __forceinline__ void clog_stage_span(const InT *wa, const InT *wb, Span sp, u32x4 *lds, int lane)
{
    constexpr int VL = 16 / (int)sizeof(InT), NV = ITEMS / VL;
    const int c_lo = (sp.lo + VL - 1) / VL;
    const int whole = sp.hi / VL - c_lo;
    const uint32_t count = whole > 0 ? (uint32_t)whole : 0u;
    const bool cut = sp.cut(VL);
    const uint32_t one = sizeof(InT) == 4 ? 0x3f800000u : 0x3f803f80u;
    u32x4 ta[NV], tb[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = j * 64 + lane;
        ta[j] = u32x4{one, one, one, one};
        tb[j] = u32x4{0u, 0u, 0u, 0u};
        if ((uint32_t)(c - c_lo) < count) {
            ta[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(wa) + c);
            tb[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(wb) + c);
        }
    }
    float xa = 0.0f, xb = 0.0f;
    int e = 0;
    bool have = false;
    if (cut) {
        have = edge_element<VL>(sp.lo, sp.hi, lane, e);
        if (have) {
            xa = widen(wa[e]);
            xb = widen(wb[e]);
        }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c = j * 64 + lane;
        float fa[VL], fb[VL];
        u32x4 va[1] = {ta[j]}, vb[1] = {tb[j]};
        unpack_inputs<InT, 1, VL>(va, fa);
        unpack_inputs<InT, 1, VL>(vb, fb);
#pragma unroll
        for (int i = 0; i < VL / 4; ++i) {
            const int quad = c * (VL / 4) + i;
            lds[clog_slot<ITEMS>(quad, 0)] = u32x4{f2u(fa[4 * i]), f2u(fa[4 * i + 1]), f2u(fa[4 * i + 2]), f2u(fa[4 * i + 3])};
            lds[clog_slot<ITEMS>(quad, 1)] = u32x4{f2u(fb[4 * i]), f2u(fb[4 * i + 1]), f2u(fb[4 * i + 2]), f2u(fb[4 * i + 3])};
        }
    }
    if (cut) {
        wave_lds_order();
        if (have) {
            reinterpret_cast<float *>(lds + clog_slot<ITEMS>(e / 4, 0))[e % 4] = xa;
            reinterpret_cast<float *>(lds + clog_slot<ITEMS>(e / 4, 1))[e % 4] = xb;
        }
    }
    wave_lds_order();
}

// The same one element at a time; `left` elements exist from the wave's first one on.
template <typename InT, int ITEMS>
__device__ __forceinline__ void clog_stage_elems(const InT *wa, const InT *wb, int64_t left, u32x4 *lds, int lane)
{
    float ta[ITEMS], tb[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane;
        ta[j] = (c < left) ? widen(__builtin_nontemporal_load(wa + c)) : 1.0f;
        tb[j] = (c < left) ? widen(__builtin_nontemporal_load(wb + c)) : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane;
        reinterpret_cast<float *>(lds + clog_slot<ITEMS>(c / 4, 0))[c % 4] = ta[j];
        reinterpret_cast<float *>(lds + clog_slot<ITEMS>(c / 4, 1))[c % 4] = tb[j];
    }
    wave_lds_order();
}

// The region's outputs -> global, one complex number at a time.
template <int ITEMS>
__device__ __forceinline__ void clog_unstage_elems(float *orow, int64_t left, const u32x4 *lds, int lane)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int c = j * 64 + lane; // element c: half of output vector c / 2
        const float *v = reinterpret_cast<const float *>(lds + c / 2 + c / 2 / (ITEMS / 2)) + 2 * (c % 2);
        const f32x2 x = {v[0], v[1]};
        if (c < left) __builtin_nontemporal_store(x, reinterpret_cast<f32x2 *>(orow) + c);
    }
    wave_lds_order();
}

// A lane's quads when its elements are those of its own slots in the window.
template <int ITEMS>
struct OwnQuads {
    u32x4 *lds; // the lane's first slot
    __device__ __forceinline__ Quads operator()(int q) const
    {
        const u32x4 a = lds[2 * q], b = lds[2 * q + 1];
        return Quads{f32x4{u2f(a[0]), u2f(a[1]), u2f(a[2]), u2f(a[3])}, f32x4{u2f(b[0]), u2f(b[1]), u2f(b[2]), u2f(b[3])}};
    }
    __device__ __forceinline__ void keep(int q, f32x4 A, f32x4 M) const // in the place of a and b
    {
        lds[2 * q] = u32x4{f2u(A[0]), f2u(A[1]), f2u(A[2]), f2u(A[3])};
        lds[2 * q + 1] = u32x4{f2u(M[0]), f2u(M[1]), f2u(M[2]), f2u(M[3])};
    }
    __device__ __forceinline__ void operator()(int q, f32x4 re, f32x4 im) const
    {
        lds[2 * q] = u32x4{f2u(re[0]), f2u(im[0]), f2u(re[1]), f2u(im[1])};
        lds[2 * q + 1] = u32x4{f2u(re[2]), f2u(im[2]), f2u(re[3]), f2u(im[3])};
    }
};

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT, int ITEMS, bool VECIO>
__global__ __launch_bounds__(256, VECIO ? 4 : 1) void heinsen_scan_rows_wave(RowsParams p)
{
    constexpr bool SIGNED = DOM == kSigned;
    // 16-byte slots per wave: the output row (ITEMS/4 vectors per lane, the larger of the two) plus padding.
    // (Writing the output in two rounds through half the region, for twice the workgroups per CU, was
    // measured on bf16 rows of 2048: 908 us against 713 -- the rounds write 64-byte pieces.)
    constexpr bool CLOG = complex_output<DOM, LOG_OUT>();
    __shared__ u32x4 stage[4][CLOG ? clog_slots<ITEMS>() : 64 * (ITEMS / 4 + 1)];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row = (int64_t)blockIdx.x * 4 + w;
    if (row >= p.rows) return; // whole wave leaves together
    const InT *arow = reinterpret_cast<const InT *>(p.a) + row * p.n;
    const InT *brow = reinterpret_cast<const InT *>(p.b) + row * p.n;
    constexpr int OW = (SIGNED && LOG_OUT) ? 2 : 1; // floats per output element
    float *orow = p.out + OW * row * p.n;

    Span sp{0, 0};
    int h = 0; // elements of the window before the row
    if (VECIO) {
        h = (int)((row * p.n + p.phase) & (16 / (int)sizeof(InT) - 1));
        sp = Span{h, h + (int)p.n}; // the row fits the window
    }
    if constexpr (CLOG) {
        u32x4 *const region = stage[w];
        if (VECIO) clog_stage_span<InT, ITEMS>(arow - h, brow - h, sp, region, lane);
        else clog_stage_elems<InT, ITEMS>(arow, brow, p.n, region, lane);
        const OwnQuads<ITEMS> own{region + lane * (ITEMS / 2 + 1)};
        const float x0 = p.x0[p.x0_stride ? row : 0];
        bool done = false; // wave-uniform
        Lin g;
        int up;
        if (wave_all(lin_summary<ITEMS>(own, g, up)) && wave_sum(up) <= kLinUp) {
            g = lin_dpp<0x138, 0xf>(lin_wave_inclusive_scan(g)); // of the lanes before this one
            const double x = fma(g.P, lin_x0(x0), g.Z);
            done = wave_all(lin_state_ok(x, lane == 0));
            if (done) lin_emit<ITEMS>(x, own, own);
        }
        if (!done) {
            uint32_t sw, sm;
            auto keep = [&](int q, f32x4 A, f32x4 M) { own.keep(q, A, M); };
            const Seg excl = wave_shift_up<DOM>(wave_inclusive_scan<DOM>(log_summary<ITEMS>(own, keep, sw, sm)));
            State st;
            encode<DOM, LOG_IN>(x0, st.lx, st.s);
            log_emit<ITEMS>(seg_apply<DOM>(st, excl), sw, sm, own, own);
        }
        wave_lds_order();
        if (VECIO) wave_unstage_span<ITEMS / 2, 1>(orow - OW * h, OW * sp.lo, OW * sp.hi, region, lane, 0);
        else clog_unstage_elems<ITEMS>(orow, p.n, region, lane);
        return;
    }

    float Av[ITEMS], Mv[ITEMS];
    uint32_t sw, sm;
    if (VECIO) {
        constexpr int VL = 16 / (int)sizeof(InT);
        constexpr int NVI = ITEMS / VL;
        static_assert(ITEMS % VL == 0 && NVI >= 1 && NVI <= 8, "lane chunk must be 1..8 vectors");
        // a = 1, b = 0 (log domain: 0, -inf) for the steps around the row
        const uint32_t one = sizeof(InT) == 4 ? 0x3f800000u : 0x3f803f80u;
        const uint32_t ninf = sizeof(InT) == 4 ? 0xff800000u : 0xff80ff80u;
        const uint32_t fa = LOG_IN ? 0u : one, fb = LOG_IN ? ninf : 0u;
        u32x4 va[NVI], vb[NVI];
        wave_load_spans<InT, NVI>(arow - h, brow - h, sp, u32x4{fa, fa, fa, fa}, u32x4{fb, fb, fb, fb},
                                      p.both || NVI == 1, stage[w], lane, va, vb);
        unpack_inputs<InT, NVI, ITEMS>(va, Av);
        unpack_inputs<InT, NVI, ITEMS>(vb, Mv);
    } else {
        uint32_t *slots = reinterpret_cast<uint32_t *>(stage[w]);
        wave_load_blocked_elems<InT, ITEMS>(arow, p.n, LOG_IN ? 0.0f : 1.0f, slots, lane, Av);
        wave_load_blocked_elems<InT, ITEMS>(brow, p.n, LOG_IN ? -INFINITY : 0.0f, slots, lane, Mv);
    }
    Seg mine = lane_scan<DOM, LOG_IN, LOG_OUT, ITEMS>(Av, Mv, sw, sm);
    Seg excl = wave_shift_up<DOM>(wave_inclusive_scan<DOM>(mine));

    State st;
    encode<DOM, LOG_IN>(p.x0[p.x0_stride ? row : 0], st.lx, st.s);
    st = seg_apply<DOM>(st, excl);
    if (VECIO)
        wave_emit_span<DOM, LOG_OUT, ITEMS>(orow - OW * h, sp, stage[w], lane, st, Av, Mv, sw, sm);
    else
        wave_emit_blocked_elems<DOM, LOG_OUT, ITEMS>(orow, p.n, reinterpret_cast<uint32_t *>(stage[w]), lane, st, Av, Mv, sw, sm);
}

// ---- several short rows per wave ---------------------------------------------------------------------
//
// Rows shorter than a wave's 64 * ITEMS steps would leave most of its lanes idle.  Here a row takes `group`
// lanes, ITEMS steps per lane, and a wave takes 64 / group consecutive rows, which are one contiguous span of
// memory: it moves between memory and LDS coalesced, as 16-byte vectors (VECIO), whatever the length of the
// rows, and every lane picks up its own vectors.  A row's lanes start at the vector that holds its first
// element, so up to VL - 1 elements of the row before it come with them and are replaced by steps that
// change nothing; what follows the row's end in its last lane reaches no other lane and is not written.
// The wave scan is confined to the lanes of a row.  Bound by memory: 262144 rows of 100 steps 54 us (5.8
// TB/s), of 249 steps 130 us.  (With groups of a power of two lanes, eight steps each, and element-wise moves
// wherever a row did not fill them it was bound by 107 vector instructions per element: 69 and 157 us.)
struct PackedParams {
    const void *a;
    const void *b;
    const float *x0;
    float *out;
    int64_t rows, n;
    int x0_stride;
    int phase;         // as in RowsParams
    int group;         // lanes per row
    uint32_t inv_group; // ceil(2^16 / group): lane / group = lane * inv_group >> 16 for lanes below 64
    int rows_per_wave; // 64 / group
};

template <int CTRL, int MASK>
struct dpp_ctrl {
    static constexpr int ctrl = CTRL, mask = MASK;
};

// Inclusive scan inside groups of `group` adjacent lanes starting at lane 0, `pos` = the lane's place in its
// group: the six steps of the wave scan, a step taking effect only in lanes whose group reaches back that
// far.  Steps no lane needs are skipped (group is wave-uniform).
template <typename STEP>
__device__ __forceinline__ void packed_scan_steps(STEP &&step, int lane, int pos, int group)
{
    if (group > 1) step(dpp_ctrl<0x111, 0xf>{}, pos >= 1);
    if (group > 2) step(dpp_ctrl<0x112, 0xf>{}, pos >= 2);
    if (group > 4) step(dpp_ctrl<0x114, 0xf>{}, pos >= 4);
    if (group > 8) step(dpp_ctrl<0x118, 0xf>{}, pos >= 8);
    if (16 % group != 0) { // some group crosses a row of 16 lanes
        step(dpp_ctrl<0x142, 0xa>{}, pos > (lane & 15)); // row_bcast:15 into rows 1,3
        if (32 % group != 0) step(dpp_ctrl<0x143, 0xc>{}, pos > (lane & 31)); // row_bcast:31 into rows 2,3
    }
}
template <int DOM>
__device__ __forceinline__ Seg packed_inclusive_scan(Seg g, int lane, int pos, int group)
{
    packed_scan_steps([&](auto ctrl, bool ok) {
        const Seg c = seg_combine<DOM>(seg_dpp<decltype(ctrl)::ctrl, decltype(ctrl)::mask, DOM>(g), g);
        g.A = ok ? c.A : g.A;
        g.M = ok ? c.M : g.M;
        g.sA = ok ? c.sA : g.sA;
        g.sM = ok ? c.sM : g.sM;
    }, lane, pos, group);
    return g;
}
__device__ __forceinline__ Lin lin_packed_inclusive_scan(Lin g, int lane, int pos, int group)
{
    packed_scan_steps([&](auto ctrl, bool ok) {
        const Lin c = lin_combine(lin_dpp<decltype(ctrl)::ctrl, decltype(ctrl)::mask>(g), g);
        g.P = ok ? c.P : g.P;
        g.Z = ok ? c.Z : g.Z;
    }, lane, pos, group);
    return g;
}

__device__ __forceinline__ int packed_inclusive_sum(int v, int lane, int pos, int group)
{
    packed_scan_steps([&](auto ctrl, bool ok) {
        const int before = (int)dpp_u<decltype(ctrl)::ctrl, decltype(ctrl)::mask>(0u, (uint32_t)v);
        v += ok ? before : 0;
    }, lane, pos, group);
    return v;
}

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT, int ITEMS, bool VECIO>
__global__ __launch_bounds__(256, 4) void heinsen_scan_rows_packed(PackedParams p)
{
    constexpr bool CLOG = complex_output<DOM, LOG_OUT>();
    constexpr int OW = CLOG ? 2 : 1;     // floats per output element
    constexpr int NVO = ITEMS * OW / 4;  // output vectors per lane
    __shared__ u32x4 stage[4][64 * (NVO + 1)];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + w) * p.rows_per_wave; // first row of this wave
    if (row0 >= p.rows) return; // whole wave leaves together
    const int nrows = (p.rows - row0 < p.rows_per_wave) ? (int)(p.rows - row0) : p.rows_per_wave;
    const int n = (int)p.n;
    const int r = (int)((uint32_t)lane * p.inv_group >> 16); // this lane's row of the wave
    const int pos = lane - r * p.group;                      // and its place in the row
    const bool row_ok = r < nrows;
    const int start = pos * ITEMS; // first of the lane's steps, from the start of the row's window

    const InT *abase = reinterpret_cast<const InT *>(p.a) + row0 * p.n;
    const InT *bbase = reinterpret_cast<const InT *>(p.b) + row0 * p.n;
    float *obase = p.out + OW * row0 * p.n;
    const float id_a = LOG_IN ? 0.0f : 1.0f, id_b = LOG_IN ? -INFINITY : 0.0f;

    int h0 = 0, h = 0; // elements of the window before the wave's first row; of the row's window before the row
    int at = 0;        // the lane's first element in the window
    const int span = nrows * n;
    constexpr int VL = VECIO ? 16 / (int)sizeof(InT) : 1;
    h0 = VECIO ? (int)((row0 * p.n + p.phase) & (VL - 1)) : 0;
    h = (h0 + r * n) & ((CLOG ? 4 : VL) - 1);
    at = row_ok ? h0 + r * n - h + start : 0; // a multiple of VL (complex output: of four, whatever VL)
    const int end = row_ok ? h + n - start : 0; // the lane's elements from `end` on are not the row's
    const Span sp{h0, h0 + span};
    uint32_t *slots = reinterpret_cast<uint32_t *>(stage[w]);
    const float x0 = p.x0[(p.x0_stride && row_ok) ? row0 + r : 0];

    if constexpr (CLOG) {
        u32x4 *const region = stage[w];
        if (VECIO) clog_stage_span<InT, ITEMS>(abase - h0, bbase - h0, sp, region, lane);
        else clog_stage_elems<InT, ITEMS>(abase, bbase, span, region, lane);
        // Element k of the lane is element at + k of the window.  Outputs take the place of inputs, so a quad
        // that rows share may not be written before all of them have read it.  The rows it begins read it
        // in the first turn of a pass, before anything is written (a row's lanes start at the quad of its
        // first element), and write it after the last turn; the row that ends in it does both in one turn.
        auto get = [&](int q) -> Quads {
            Quads v;
            const u32x4 a = region[clog_slot<ITEMS>(at / 4 + q, 0)], b = region[clog_slot<ITEMS>(at / 4 + q, 1)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool mine = start + 4 * q + i >= h && 4 * q + i < end;
                v.a[i] = mine ? u2f(a[i]) : id_a;
                v.b[i] = mine ? u2f(b[i]) : id_b;
            }
            return v;
        };
        auto write_own = [&](int q, f32x4 re, f32x4 im) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 4 * q + i, e = at + k;
                if (start + k >= h && k < end) {
                    uint32_t *o = reinterpret_cast<uint32_t *>(region + clog_slot<ITEMS>(e / 4, e % 4 / 2)) + 2 * (e % 2);
                    o[0] = f2u(re[i]);
                    o[1] = f2u(im[i]);
                }
            }
        };
        const bool ragged = ((p.phase | n) & 3) != 0; // some rows begin or end inside a quad (wave-uniform)
        const bool late = pos == 0 && h != 0; // the lane's first quad is written last
        f32x4 late_re = {}, late_im = {};
        auto put = [&](int q, f32x4 re, f32x4 im) {
            if (!ragged) {
                if (4 * q < end) {
                    region[clog_slot<ITEMS>(at / 4 + q, 0)] = u32x4{f2u(re[0]), f2u(im[0]), f2u(re[1]), f2u(im[1])};
                    region[clog_slot<ITEMS>(at / 4 + q, 1)] = u32x4{f2u(re[2]), f2u(im[2]), f2u(re[3]), f2u(im[3])};
                }
            } else if (q == 0) {
                late_re = re;
                late_im = im;
                if (!late) write_own(0, re, im);
            } else {
                write_own(q, re, im);
            }
            wave_lds_order();
        };
        // Every row of the wave decides for itself, so that what becomes of a row does not depend on its
        // neighbours' numbers.
        Lin g;
        int up;
        bool ok = lin_summary<ITEMS>(get, g, up);
        if (!wave_all(up * p.group <= kLinUp)) up = packed_inclusive_sum(up, lane, pos, p.group); // of the whole row in its last lane
        g = lin_dpp<0x138, 0xf>(lin_packed_inclusive_scan(g, lane, pos, p.group));
        if (pos == 0) g = Lin{1.0, 0.0}; // first lane of a row
        const double x = fma(g.P, lin_x0(x0), g.Z);
        ok = (ok && up <= kLinUp && lin_state_ok(x, pos == 0)) || !row_ok;
        const uint64_t bad = __builtin_amdgcn_ballot_w64(!ok);
        if (bad == 0ull) {
            lin_emit<ITEMS>(x, get, put);
        } else {
            const bool by_steps = (bad & (~0ull >> (64 - p.group)) << (r * p.group)) != 0ull;
            uint32_t sw, sm;
            auto keep = [&](int q, f32x4 A, f32x4 M) { // rows that share a quad keep their own elements of it
                if (!by_steps) return;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (start + 4 * q + i >= h && 4 * q + i < end) {
                        reinterpret_cast<float *>(region + clog_slot<ITEMS>(at / 4 + q, 0))[i] = A[i];
                        reinterpret_cast<float *>(region + clog_slot<ITEMS>(at / 4 + q, 1))[i] = M[i];
                    }
                }
                wave_lds_order();
            };
            Seg excl = wave_shift_up<DOM>(packed_inclusive_scan<DOM>(log_summary<ITEMS>(get, keep, sw, sm), lane, pos, p.group));
            if (pos == 0) excl = seg_identity<DOM>();
            State st;
            encode<DOM, LOG_IN>(x0, st.lx, st.s);
            st = seg_apply<DOM>(st, excl);
            // The two kinds of rows take their second passes one after the other: the quad in which a row
            // begins may by then hold outputs of the row that ends in it.
            const Quads head = get(0);
            auto get_after = [&](int q) -> Quads { return q == 0 ? head : get(q); };
            if (by_steps) log_emit<ITEMS>(st, sw, sm, get_after, put);
            else lin_emit<ITEMS>(x, get_after, put);
        }
        if (late) write_own(0, late_re, late_im);
        wave_lds_order();
        if (VECIO) wave_unstage_span<NVO, 1>(obase - OW * h0, OW * h0, OW * (h0 + span), region, lane, 0);
        else clog_unstage_elems<ITEMS>(obase, span, region, lane);
        return;
    }

    float Av[ITEMS], Mv[ITEMS];
    uint32_t sw, sm;
    if (VECIO) {
        constexpr int NV = ITEMS / VL;
        const u32x4 fill{0u, 0u, 0u, 0u}; // never looked at
        u32x4 va[NV], vb[NV];
        auto pick = [&](u32x4 (&v)[NV]) {
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const int c = at / VL + q;
                v[q] = stage[w][c + c / NV];
            }
            wave_lds_order();
        };
        // Few rows wait for one load, not two; with 16 steps per lane the launch is large, and the registers are
        // worth more (32768 rows of 200 steps 14.7 us, with both in flight 15.9).
        if constexpr (ITEMS > 8) {
            wave_stage_span<InT, NV>(abase - h0, sp, fill, stage[w], lane);
            pick(va);
            wave_stage_span<InT, NV>(bbase - h0, sp, fill, stage[w], lane);
            pick(vb);
        } else {
            u32x4 ta[NV], tb[NV];
            InT xa, xb;
            span_fetch<InT, NV>(abase - h0, sp, fill, lane, ta, xa);
            span_fetch<InT, NV>(bbase - h0, sp, fill, lane, tb, xb);
            if (NV == 1 && n == p.group * ITEMS && !sp.cut(VL)) { // one vector per lane is where it belongs
                va[0] = ta[0];
                vb[0] = tb[0];
            } else {
                span_stage<InT, NV>(sp, ta, xa, stage[w], lane);
                pick(va);
                span_stage<InT, NV>(sp, tb, xb, stage[w], lane);
                pick(vb);
            }
        }
        unpack_inputs<InT, NV, ITEMS>(va, Av);
        unpack_inputs<InT, NV, ITEMS>(vb, Mv);
        if (((p.phase | n) & (VL - 1)) != 0) { // rows that start inside a vector
#pragma unroll
            for (int k = 0; k < VL - 1; ++k) {
                const bool before = start + k < h;
                Av[k] = before ? id_a : Av[k];
                Mv[k] = before ? id_b : Mv[k];
            }
        }
    } else {
        // one element at a time, element i of the span in slot i + i / ITEMS
        auto gather = [&](const InT *src, float (&x)[ITEMS]) {
            float t[ITEMS];
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const int c = j * 64 + lane;
                t[j] = (c < span) ? widen(__builtin_nontemporal_load(src + c)) : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const int c = j * 64 + lane;
                slots[c + c / ITEMS] = f2u(t[j]);
            }
            wave_lds_order();
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int c = at + k;
                x[k] = u2f(slots[c + c / ITEMS]);
            }
            wave_lds_order();
        };
        gather(abase, Av);
        gather(bbase, Mv);
    }
    Seg mine = lane_scan<DOM, LOG_IN, LOG_OUT, ITEMS>(Av, Mv, sw, sm);
    Seg excl = wave_shift_up<DOM>(packed_inclusive_scan<DOM>(mine, lane, pos, p.group));
    if (pos == 0) excl = seg_identity<DOM>(); // first lane of a row

    State st;
    encode<DOM, LOG_IN>(x0, st.lx, st.s);
    st = seg_apply<DOM>(st, excl);
    const uint32_t swx = fold_state_sign<DOM>(sw, st);
    if (VECIO) {
        // Every lane drops the vectors that hold elements of its row into the span's place.  Where one row
        // ends and the next begins inside a vector, the row that ends there writes it first, the next one
        // then puts its own elements in one by one.
        float o[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) o[k] = emit<DOM, LOG_OUT>(st, Av[k], Mv[k], swx, k);
        const int c0 = at / 4;
#pragma unroll
        for (int q = 0; q < NVO; ++q) {
            const int c = c0 + q;
            if (start + 4 * q >= h && 4 * q < end)
                stage[w][c + c / NVO] = u32x4{f2u(o[4 * q]), f2u(o[4 * q + 1]), f2u(o[4 * q + 2]), f2u(o[4 * q + 3])};
        }
        if (((p.phase | n) & 3) != 0) { // some rows begin inside a vector (wave-uniform)
            wave_lds_order();
#pragma unroll
            for (int k = 1; k < VL; ++k) {
                const int c = c0 + k / 4;
                if (k % 4 != 0 && pos == 0 && k >= h && k / 4 * 4 < h && k < end) slots[4 * (c + c / NVO) + k % 4] = f2u(o[k]);
            }
        }
        wave_lds_order();
        wave_unstage_span<NVO, 1>(obase - h0, h0, h0 + span, stage[w], lane, 0);
    } else {
        // the reverse move
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int c = at + k;
            if (k < end) slots[c + c / ITEMS] = f2u(emit<DOM, LOG_OUT>(st, Av[k], Mv[k], swx, k));
        }
        wave_lds_order();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int c = j * 64 + lane;
            if (c < span) __builtin_nontemporal_store(u2f(slots[c + c / ITEMS]), obase + c);
        }
    }
}

// ---- tiles with a chained carry ------------------------------------------------------------------------
//
// Tile index c inside a row is read in base 32: c = (s*32 + g)*32 + r.  Summaries are published at two
// levels -- a tile's own (level 1) and the 32 tiles of a group folded by its last tile (level 2) -- and
// the state at the start of every 1024-tile super-block s, in float64, by the last tile of the previous
// one.  A tile therefore reads at most 31 + 31 summaries and one state, all in one round of loads (one
// per lane of wave 0), and folds them in a fixed order: results do not depend on timing.  A level-2
// summary is published as soon as the level-1 summaries it is made of are in, so no tile waits for
// another tile's wait; only the super-block states form a chain, n / (1024 * tile) links long.

// records per summary slot: the two records of a summary (or state) get a 128-byte line of their own, so
// that the tiles polling for one summary do not queue with the accesses to its neighbours
constexpr uint32_t kRecStride = 16;
constexpr int kLdsTileWaves = 16; // most waves of a row whose inputs stay in LDS (inputs_in_lds)
constexpr int kTileWaves = 8;   // waves per workgroup (4 and 16 measured 12 % and 28 % slower on one row of 2^26)
constexpr int kTileItems = 32;  // elements per lane (rows of one tile may use 8 or 16: a shorter serial chain)
constexpr int kTile = kTileWaves * 64 * kTileItems;
// A launch of few tiles is bound by the latency of a tile, not by memory: up to this many tiles it takes
// tiles of half the size (16 elements per lane).  Measured on one row: 6.0 against 7.4 us for 2^16 steps,
// 9.5 against 10.1 us for 2^20 (128 half tiles), even at 2^21, slower beyond.
constexpr int64_t kHalfTilesUpTo = 128;

struct TileParams {
    const void *a;
    const void *b;
    const float *x0;
    float *out;
    int64_t rows, n;
    int x0_stride;
    int phase;             // as in RowsParams
    int waves;             // waves per workgroup (rows of one tile: as many as the row needs)
    uint32_t tpr;          // tiles per row
    uint32_t ntiles;       // rows * tpr
    rec_t *header;         // scratch header (ticket queue 0 hands out the tiles in row-major order)
    rec_t *recs;           // per row: level-1 and level-2 summaries (2 records each), states (2 records each)
    uint32_t off2, off4, row_stride; // record offsets of level 2 and of the states inside a row's block
    uint32_t spin_limit;
    uint32_t drop_tile;
    uint32_t pace_ns;      // between the starts of the first tiles (0: none)
    Timeline tl;
};

// 16-byte slots a wave of the tiles kernel needs to move its elements through LDS; the pad slot after the
// last lane is never used by the vector path, and leaving it out lets four workgroups share a CU
template <bool VECIO, int ITEMS, bool IN_LDS>
constexpr int tile_stage_slots()
{
    return IN_LDS ? clog_slots<ITEMS>() : 64 * (ITEMS / 4 + 1) - (VECIO ? 1 : 0);
}

// Complex output whose inputs stay in LDS between the passes: rows of one tile with up to 16 steps per lane.
// (Longer tiles would hold two workgroups per CU to the waves of one; theirs stay in registers, as records.)
template <int DOM, bool LOG_OUT, bool MULTI, int ITEMS>
constexpr bool inputs_in_lds()
{
    return complex_output<DOM, LOG_OUT>() && !MULTI && ITEMS <= 16;
}

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT, bool VECIO, bool MULTI, int ITEMS>
__device__ __forceinline__ void tiles_tile(const TileParams &p, const uint32_t tile, const uint32_t epoch, u32x4 *stage)
{
    constexpr bool SIGNED = DOM == kSigned;
    constexpr int NW = inputs_in_lds<DOM, LOG_OUT, MULTI, ITEMS>() ? kLdsTileWaves : kTileWaves;
    const int nw = MULTI ? NW : p.waves;
    const int kTile = nw * 64 * ITEMS; // elements per tile
    static_assert(!MULTI || ITEMS == kTileItems || ITEMS == kTileItems / 2, "rows of several tiles use the full or the half tile");
    __shared__ float lds_A[NW], lds_M[NW];
    __shared__ uint32_t lds_S[NW];
    __shared__ float lds_startL;
    __shared__ uint32_t lds_startS;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int64_t row = tile / p.tpr;
    const uint32_t c = tile % p.tpr;
    const InT *arow = reinterpret_cast<const InT *>(p.a) + row * p.n;
    const InT *brow = reinterpret_cast<const InT *>(p.b) + row * p.n;

    // ---- wave 0 asks for the carry records it needs before the tile's own loads (see scan_bnd.hip) ---
    const uint32_t r = c & 31u, g = (c >> 5) & 31u, sb = c >> 10;
    const bool more = c + 1 < p.tpr;
    rec_t *const rrow = p.recs + (size_t)row * p.row_stride;
    rec_t ra = 0, rm = 0;
    const rec_t *fp = nullptr;
    bool need = false;
    if (MULTI && w == 0) {
        // lanes 0-30: level 2 (earlier groups of the super-block), lane 31: the super-block state,
        // lanes 32-62: level 1 (earlier tiles of the group)
        const uint32_t sub = (uint32_t)lane & 31u;
        if (lane < 31 && sub < g) { need = true; fp = rrow + p.off2 + kRecStride * (size_t)(((c >> 10) << 5) + sub); }
        if (lane == 31 && sb > 0) { need = true; fp = rrow + p.off4 + kRecStride * (size_t)sb; }
        if (lane >= 32 && lane < 63 && sub < r) { need = true; fp = rrow + kRecStride * (size_t)(((c >> 5) << 5) + sub); }
    }
    bool got = !need; // this lane's records are in
    auto fetch_records = [&]() -> uint64_t {
        if (!got) {
            ra = rec_get(fp);
            rm = rec_get(fp + 1);
            got = rec_ok(ra, epoch) && rec_ok(rm, epoch);
        }
        return __builtin_amdgcn_ballot_w64(got);
    };
    uint64_t have = 0;
    if (MULTI && w == 0) have = fetch_records();

    // x_0 as well: a memory latency of its own where it is asked for when it is used.  (Rows of one tile ask then: without the
    // first wave's hand-over, which keeps the workgroups that share a compute unit in step, they gain and lose: 1024 rows of 16384
    // logarithms 41.1 and 38.4 us, but 512 signed ones 18.1 and 19.9, 800 rows of 10000 25.0 and 22.6, of 6000 12.4 and 13.6.)
    float x0 = MULTI ? p.x0[p.x0_stride ? row : 0] : 0.0f;

    // global <-> lane traffic of each wave goes through its own LDS region (coalesced both ways)
    u32x4 *const region = stage + w * tile_stage_slots<VECIO, ITEMS, inputs_in_lds<DOM, LOG_OUT, MULTI, ITEMS>()>();
    const int64_t wstart = (int64_t)c * kTile + (int64_t)w * (64 * ITEMS); // first element of this wave's window
    constexpr int OW = complex_output<DOM, LOG_OUT>() ? 2 : 1; // floats per output element
    float *orow = p.out + OW * row * p.n;
    Span sp{0, 0};
    int h = 0; // elements of the row's window before the row
    if (VECIO) {
        h = (int)((row * p.n + p.phase) & (16 / (int)sizeof(InT) - 1));
        sp = wave_span(h - wstart, h + p.n - wstart, 64 * ITEMS);
    }
    if constexpr (inputs_in_lds<DOM, LOG_OUT, MULTI, ITEMS>()) {
        // the tile is the row
        __shared__ double lds_P[NW], lds_Z[NW];
        __shared__ int lds_up[NW];  // above kLinUp: the wave's inputs are out of range
        __shared__ int lds_bad[NW]; // some state of the wave is
        if (VECIO) clog_stage_span<InT, ITEMS>(arow - h + wstart, brow - h + wstart, sp, region, lane);
        else clog_stage_elems<InT, ITEMS>(arow + wstart, brow + wstart, p.n - wstart, region, lane);
        const OwnQuads<ITEMS> own{region + lane * (ITEMS / 2 + 1)};
        x0 = p.x0[p.x0_stride ? row : 0];
        Lin g;
        int up;
        const bool in_range = wave_all(lin_summary<ITEMS>(own, g, up));
        up = in_range ? wave_sum(up) : kLinUp + 1;
        g = lin_wave_inclusive_scan(g);
        p.tl.mark(tile, 2);
        if (lane == 63) {
            lds_P[w] = g.P;
            lds_Z[w] = g.Z;
            lds_up[w] = up;
        }
        __syncthreads();
        p.tl.mark(tile, 3);
        p.tl.mark(tile, 4); // no records
        // the row's states at the waves up to this one and at its lanes
        double x = lin_x0(x0);
        bool ok = up <= kLinUp;
        for (int j = 0; j < w; ++j) {
            ok = ok && lds_up[j] <= kLinUp && lin_state_ok(x, j == 0);
            x = fma(lds_P[j], x, lds_Z[j]);
        }
        g = lin_dpp<0x138, 0xf>(g); // of the lanes before this one
        x = fma(g.P, x, g.Z);
        ok = wave_all(ok && lin_state_ok(x, threadIdx.x == 0));
        if (lane == 0) lds_bad[w] = ok ? 0 : 1;
        __syncthreads();
        int bad = 0;
        for (int j = 0; j < nw; ++j) bad |= lds_bad[j];
        p.tl.mark(tile, 5);
        if (bad == 0) {
            lin_emit<ITEMS>(x, own, own);
        } else {
            // one wave of the row is out of range: the whole row by log-domain steps
            uint32_t sw, sm;
            auto keep = [&](int q, f32x4 A, f32x4 M) { own.keep(q, A, M); };
            const Seg incl = wave_inclusive_scan<DOM>(log_summary<ITEMS>(own, keep, sw, sm));
            if (lane == 63) {
                lds_A[w] = incl.A;
                lds_M[w] = incl.M;
                lds_S[w] = (incl.sA >> 31) | ((incl.sM >> 31) << 1);
            }
            __syncthreads();
            Seg excl = wave_shift_up<DOM>(incl);
            Seg before = seg_identity<DOM>();
            for (int j = 0; j < w; ++j) {
                const Seg g2{lds_A[j], lds_M[j], lds_S[j] << 31, lds_S[j] << 30};
                before = j == 0 ? g2 : seg_combine<DOM>(before, g2);
            }
            State st;
            encode<DOM, LOG_IN>(x0, st.lx, st.s);
            log_emit<ITEMS>(seg_apply<DOM>(st, seg_combine<DOM>(before, excl)), sw, sm, own, own);
        }
        wave_lds_order();
        if (VECIO) wave_unstage_span<ITEMS / 2, 1>(orow + OW * (wstart - h), OW * sp.lo, OW * sp.hi, region, lane, 0);
        else clog_unstage_elems<ITEMS>(orow + OW * wstart, p.n - wstart, region, lane);
        p.tl.mark(tile, 6);
        return;
    }
    float Av[ITEMS], Mv[ITEMS];
    uint32_t sw, sm;
    if (VECIO) {
        constexpr int VL = 16 / (int)sizeof(InT);
        constexpr int NVI = ITEMS / VL;
        const uint32_t one = sizeof(InT) == 4 ? 0x3f800000u : 0x3f803f80u;
        const uint32_t ninf = sizeof(InT) == 4 ? 0xff800000u : 0xff80ff80u;
        const uint32_t fa = LOG_IN ? 0u : one, fb = LOG_IN ? ninf : 0u;
        u32x4 va[NVI], vb[NVI];
        wave_load_spans<InT, NVI>(arow - h + wstart, brow - h + wstart, sp, u32x4{fa, fa, fa, fa}, u32x4{fb, fb, fb, fb}, !MULTI,
                                  region, lane, va, vb);
        unpack_inputs<InT, NVI, ITEMS>(va, Av);
        unpack_inputs<InT, NVI, ITEMS>(vb, Mv);
    } else {
        uint32_t *slots = reinterpret_cast<uint32_t *>(region);
        wave_load_blocked_elems<InT, ITEMS>(arow + wstart, p.n - wstart, LOG_IN ? 0.0f : 1.0f, slots, lane, Av);
        wave_load_blocked_elems<InT, ITEMS>(brow + wstart, p.n - wstart, LOG_IN ? -INFINITY : 0.0f, slots, lane, Mv);
    }
    Seg mine = lane_scan<DOM, LOG_IN, LOG_OUT, ITEMS>(Av, Mv, sw, sm);
    Seg incl = wave_inclusive_scan<DOM>(mine);
    Seg lane_excl = wave_shift_up<DOM>(incl);
    p.tl.mark(tile, 2);
    if (lane == 63) {
        lds_A[w] = incl.A;
        lds_M[w] = incl.M;
        lds_S[w] = (incl.sA >> 31) | ((incl.sM >> 31) << 1);
    }
    __syncthreads();

    // summary of the waves before this one, and (wave 0) of the whole tile, in wave order
    Seg wave_excl = seg_identity<DOM>();
    Seg total = seg_identity<DOM>();
    auto summary = [&](int j) {
        return Seg{lds_A[j], lds_M[j], SIGNED ? (lds_S[j] << 31) : 0u, SIGNED ? (lds_S[j] << 30) : 0u};
    };
    auto fold = [&](int j) {
        total = j == 0 ? summary(0) : seg_combine<DOM>(total, summary(j));
        if (j + 1 == w) wave_excl = total;
    };
    if (MULTI || nw == NW) {
        static_assert(inputs_in_lds<DOM, LOG_OUT, MULTI, ITEMS>() || NW == 8, "eight lanes fold eight summaries");
        // Eight lanes side by side: three combinations one after the other instead of seven, which every wave that waits for this tile
        // waited for too.  One row of 300 steps to 2^26: 2^18 7.34 and 7.04 us, 2^20 9.36 and 9.08, 2^23 25.4 and 25.0, 2^26 148.6 and 147.4 (x_0 asked for early, above, included);
        // signed 100000 steps 7.8 and 7.3, 300 rows of 4096 6.7 and 6.3, bf16 logarithms 33 10^6 steps 72.0 and 69.7.
        // That takes the waves in pairs, and lanes without a partner an empty one.  In wave order, as a sequence is evaluated, where the
        // difference shows: a sum of logarithms that is +inf (one a_t = +inf) has no logarithm of zero added to it, and products,
        // which two waves may take out of float32 where all that came before them is zero, are formed from the first wave on.
        const Seg own = summary(lane & (NW - 1));
        const Seg part = eighth_inclusive_scan<DOM>(own);
        if (w > 0) wave_excl = seg_readlane<DOM>(part, w - 1);
        if (MULTI && w == 0) total = seg_readlane<DOM>(part, NW - 1);
        if (DOM == kLinear) { // all asked for at once
#pragma unroll
            for (int j = 0; j < NW; ++j) fold(j);
        } else if (__builtin_expect(!wave_all(own.A < INFINITY), 0)) {
#pragma unroll 1
            for (int j = 0; j < NW; ++j) fold(j);
        }
    } else { // rows of one tile: nobody needs the last wave's
        for (int j = 0; j + 1 < nw; ++j) fold(j);
    }

    const Seg before = MULTI && w == 0 ? lane_excl : seg_combine<DOM>(wave_excl, lane_excl); // the lane's part of the tile
    if (w == 0) {
        State64 st;
        {
            float lx;
            if (!MULTI) x0 = p.x0[p.x0_stride ? row : 0];
            encode<DOM, LOG_IN>(x0, lx, st.s);
            st.lx = (double)lx;
        }
        p.tl.mark(tile, 3);
        if (MULTI) {
            if (more && r < 31u && lane == 0 && tile != p.drop_tile)
                seg_put<DOM>(rrow + kRecStride * (size_t)c, rrow + kRecStride * (size_t)c + 1, total, epoch);
            // The last tile of a group owes the later groups the summary of its group; it needs level 1
            // only and is published as soon as that is in, whatever else is still on its way.
            const bool lead = more && r == 31u;
            bool pub2 = !lead;
            Seg f1 = seg_identity<DOM>(), f2 = seg_identity<DOM>(), a2 = seg_identity<DOM>();
            const uint64_t m1 = 0x7fffffff00000000ull, all = ~0ull;
            bool lost = false; // some record never came
            uint32_t polls = 0;
            for (;;) {
                if (!lost && have != all && ++polls > p.spin_limit) {
                    // give up: go on as if everything were in, with NaN as the state, which is also handed on
                    lost = true;
                    have = all;
                    if (lane == 0) note_wait_gave_up(p.header);
                }
                if ((!pub2 && (have & m1) == m1) || have == all) {
                    Seg part = (need && got && lane != 31) ? seg_from<DOM>(ra, rm) : seg_identity<DOM>();
                    if (lost) part.M = __builtin_nanf("");
                    part = half_inclusive_scan<DOM>(part);
                    f2 = seg_readlane<DOM>(part, 31);
                    f1 = seg_readlane<DOM>(part, 63);
                    if (!pub2) {
                        a2 = seg_combine<DOM>(f1, total); // this group of 32 tiles
                        if (g < 31u && lane == 0)
                            seg_put<DOM>(rrow + p.off2 + kRecStride * (size_t)(c >> 5), rrow + p.off2 + kRecStride * (size_t)(c >> 5) + 1, a2, epoch);
                        pub2 = true;
                    }
                }
                if (have == all) break;
                __builtin_amdgcn_s_sleep(2);
                have = fetch_records();
            }
            p.tl.mark(tile, 4);
            if (sb > 0) {
                // lane 31 holds the super-block state: payloads are the high and low word of the double,
                // the sign rides in the user bits of the first record
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)rec_payload(ra), 31);
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)rec_payload(rm), 31);
                const uint32_t sg = (uint32_t)__builtin_amdgcn_readlane((int)rec_bits(ra), 31);
                st.lx = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
                st.s = SIGNED ? (sg << 31) : 0u;
            }
            if (lost) st.lx = __builtin_nan("");
            const State64 st2 = seg_apply64<DOM>(st, f2); // state at the start of the group
            if (lead && g == 31u) {
                const State64 nx = seg_apply64<DOM>(st2, a2); // start of the next super-block
                const unsigned long long bits = (unsigned long long)__double_as_longlong(nx.lx);
                if (lane == 0) {
                    rec_put(rrow + p.off4 + kRecStride * (size_t)(sb + 1), (uint32_t)(bits >> 32), epoch, SIGNED ? (nx.s >> 31) : 0u);
                    rec_put(rrow + p.off4 + kRecStride * (size_t)(sb + 1) + 1, (uint32_t)bits, epoch, 0u);
                }
            }
            st = seg_apply64<DOM>(st2, f1);
        }
        if (lane == 0) {
            lds_startL = (float)st.lx;
            lds_startS = st.s;
        }
    }
    __syncthreads();

    p.tl.mark(tile, 5);
    State st;
    st.lx = lds_startL;
    st.s = lds_startS;
    st = seg_apply<DOM>(st, before);
    if (VECIO)
        wave_emit_span<DOM, LOG_OUT, ITEMS>(orow + OW * (wstart - h), sp, region, lane, st, Av, Mv, sw, sm);
    else
        wave_emit_blocked_elems<DOM, LOG_OUT, ITEMS>(orow + OW * wstart, p.n - wstart, reinterpret_cast<uint32_t *>(region), lane,
                                                     st, Av, Mv, sw, sm);
    p.tl.mark(tile, 6);
}

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT, bool VECIO, bool MULTI, int ITEMS>
__global__ __launch_bounds__((inputs_in_lds<DOM, LOG_OUT, MULTI, ITEMS>() ? kLdsTileWaves : kTileWaves) * 64) void heinsen_scan_tiles(TileParams p)
{
    __shared__ uint32_t s_tile, s_epoch, s_flag;
    // tiles of a chained row always have kTileWaves waves; rows of one tile as many as the row needs, and
    // only their regions are asked for at launch, so that more workgroups share a CU
    extern __shared__ u32x4 stage_of_waves[];
    __shared__ u32x4 stage_of_tile[MULTI ? kTileWaves * tile_stage_slots<VECIO, ITEMS, inputs_in_lds<DOM, LOG_OUT, MULTI, ITEMS>()>() : 1];
    u32x4 *const stage = MULTI ? stage_of_tile : stage_of_waves;
    const unsigned long long t_begin = p.tl.stamps != nullptr ? wall_clock64() : 0ull;
    uint32_t tile = blockIdx.x, epoch = 0u;
    if (MULTI) {
        // tickets: a tile only ever waits for tiles with smaller tickets, which are already running
        if (threadIdx.x == 0) {
            const Draw d = draw_ticket(p.header, 0, p.ntiles, 1);
            if (paced_kernel(VECIO, complex_output<DOM, LOG_OUT>()) && p.pace_ns != 0 && d.ticket < kPacedTiles) pace_start(d.ticket * p.pace_ns);
            s_tile = d.ticket;
            s_epoch = d.epoch;
        }
        __syncthreads();
        tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tile);
        epoch = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_epoch);
    }
    if (tile < p.ntiles) {
        p.tl.mark_at(tile, 0, t_begin);
        p.tl.mark(tile, 1);
        tiles_tile<DOM, LOG_IN, LOG_OUT, InT, VECIO, MULTI, ITEMS>(p, tile, epoch, stage);
        p.tl.mark(tile, 7);
    }
    if (MULTI) end_of_workgroup(p.header, epoch, &s_flag);
}

// ---- host side -------------------------------------------------------------------------------------------

constexpr int64_t kRowsWaveMax = 64 * 32; // longest row the one-wave kernel takes

struct BdnPlan {
    bool wave_kernel;
    int group;    // > 0: several rows per wave, this many lanes per row
    int items;    // wave kernels: elements per lane
    bool vecio;
    int phase;    // see RowsParams
    bool multi;
    int tile_items; // tiles kernel: elements per lane
    int waves;      // tiles kernel: waves per workgroup
    int64_t rows;
    uint32_t tpr, ntiles;
    uint32_t off2, off4, row_stride;
    size_t records;
};

// Rows of one tile: with at least this many rows the chip is full whatever a row's workgroup looks like, and
// the fewest, fullest waves win (a lane's serial steps cost far less than its share of the scans across
// lanes and waves): 8192 rows of 3001 steps, complex output, took 147 us on eight waves of eight steps; 700 rows of 2500
// float32 steps 7.8 us on eight, 6.9 on three of 16.  With fewer rows a call is bound by the latency of one row, which
// all eight waves share (256 rows 5.5 us on eight waves, 5.6 and 6.2 on fewer).
constexpr int64_t kManyRows = 512;

// Rows of up to 512 steps: do several share a wave, on how many lanes each and of how many steps?
//   Steps per lane: eight as long as the launch does not fill the chip twice over anyhow (about 3 * 2^20 elements),
// since a lane's steps are one after the other (100 steps: 16384 rows 5.9 us with eight, 6.3 with 16; 32768 8.5 and
// 8.3; 131072 30.4 and 29.4), and beyond that where they fill the lanes better by more than a quarter.
//   Rows of more than 256 steps have a wave of eight steps per lane to themselves unless three fit one of 16 (300 steps,
// 4096 rows: 5.2 us alone, 6.3 shared; 32768: 25 and 22), or two and the launch is large (400 steps, 16384 rows: 16.1 and
// 14.7; from about 450 steps on nothing is gained).  bf16, whose loads are half as many, shares later.
//   Up to 1024 rows, one wave per SIMD, every row has its own: fewer steps of the scan across lanes do not make up
// for the rearrangement (200 steps, 512 rows: 3.0 us alone, 3.3 shared, 3.9 with 16 steps).
bool shares_waves(const ScanCall &c, int64_t lead, bool clog, bool vecio, int &items, int &group)
{
    const int64_t rows = c.B * c.D, elements = rows * c.n, before = clog && !vecio ? 3 : lead; // a complex output works on quads in any case
    const int g16 = (int)ceil_div(c.n + before, 16), g8 = (int)ceil_div(c.n + before, 8);
    if (rows <= 1024 && (c.n >= 64 || rows == 1)) return false;
    if (c.n <= 256) {
        items = elements <= (3ll << 20) || 8 * (64 / g8) > 5 * (64 / g16) ? 8 : 16;
    } else {
        items = 16;
        if (!(64 / g16 >= 3 && elements > (2ll << 20)) && !(c.n <= 448 && elements > (3ll << 20)) && !(c.bf16 && elements > (9ll << 19))) return false;
    }
    group = items == 16 ? g16 : g8;
    return true;
}

BdnPlan make_plan(const ScanCall &c)
{
    BdnPlan pl = {};
    pl.rows = c.B * c.D;
    // The vector path needs a, b and out to lie alike relative to the 16-byte boundaries (the usual case: all
    // three start on one): then every row, whatever its length, has its vectors at the same elements in all.
    const int64_t es = c.bf16 ? 2 : 4, vl = 16 / es;
    const int64_t os = (c.is_signed && c.log_out) ? 8 : 4, ol = 16 / os;
    const int64_t at_a = (int64_t)(reinterpret_cast<uintptr_t>(c.a) % 16) / es, at_b = (int64_t)(reinterpret_cast<uintptr_t>(c.b) % 16) / es;
    const int64_t at_o = (int64_t)(reinterpret_cast<uintptr_t>(c.out) % 16) / os;
    pl.vecio = at_a == at_b && at_a % ol == at_o;
    // elements of a row's window that may lie before the row
    int64_t lead = (c.n % vl == 0 && at_a == 0) ? 0 : vl - 1;
    auto element_wise = [&]() {
        pl.vecio = false;
        lead = 0;
    };
    if (!pl.vecio) element_wise();
    // A float32 row that its lead would push to twice the steps per lane: element by element it is the faster one (1022
    // steps, 600 rows 4.9 and 5.3 us, 4096 rows 9.2 and 10.7; bf16, two bytes per load: 9.0 and 4.9).  A few complex
    // rows, whose moves are a small part of them, keep the vectors.
    const bool clog = c.is_signed && c.log_out;
    if (!c.bf16 && ((c.n <= 512 && c.n + lead > 512) || (c.n <= 1024 && c.n + lead > 1024)) && pl.rows >= (clog ? kManyRows : c.n > 512 ? 64 : 1))
        element_wise();
    // a complex output keeps at most 16 steps per lane (see inputs_in_lds)
    pl.wave_kernel = c.n + lead <= (clog ? kRowsWaveMax / 2 : kRowsWaveMax) && !(pl.rows < 64 && c.n > 512);
    if (pl.wave_kernel) {
        pl.phase = pl.vecio ? (int)at_a : 0;
        if (c.n + std::max<int64_t>(lead, clog ? 3 : 0) <= 512 && shares_waves(c, lead, clog, pl.vecio, pl.items, pl.group)) return pl;
        pl.items = c.n + lead > 1024 ? 32 : (c.n + lead > 512 ? 16 : 8);
        return pl;
    }
    // a row of one tile is bound by latency: spread it over all waves of the workgroup
    const int64_t wide = kTileWaves * 64; // lanes of a full workgroup
    if (c.n <= wide * kTileItems && c.n + lead > wide * kTileItems) element_wise(); // still one tile
    pl.waves = kTileWaves;
    pl.tile_items = c.n + lead <= wide * 8 ? 8 : (c.n + lead <= wide * 16 ? 16 : kTileItems);
    if (c.n <= kTile) {
        if (pl.rows >= kManyRows) {
            const int64_t w32 = ceil_div(c.n + lead, 64 * 32), w16 = ceil_div(c.n + lead, 64 * 16);
            // 16 steps where they fill their lanes better by an eighth, and while there are not two or three waves
            // per SIMD even so (4096 steps, logarithms, 512 rows: 8.3 -> 7.0 us)
            const bool finer = clog ? w16 <= kLdsTileWaves : (w16 <= kTileWaves && (8 * w16 < 7 * 2 * w32 || pl.rows * w32 <= 2400));
            // five waves and more share a CU no better than all eight (12000 steps, 2048 rows: 55 us, eight waves 53)
            if (finer || w32 <= 4 || pl.rows * w32 <= 4096) {
                pl.tile_items = finer ? 16 : 32;
                pl.waves = (int)(finer ? w16 : w32);
            }
        }
    } else {
        if (pl.rows * ceil_div(c.n, kTile / 2) <= kHalfTilesUpTo) pl.tile_items = kTileItems / 2;
        // a row whose lead would cost one more tile goes element by element: its scratch is what it was
        const int64_t tile = wide * pl.tile_items;
        if (ceil_div(c.n + lead, tile) != ceil_div(c.n, tile)) element_wise();
    }
    pl.phase = pl.vecio ? (int)at_a : 0;
    pl.tpr = (uint32_t)ceil_div(c.n + lead, (int64_t)pl.waves * 64 * pl.tile_items);
    pl.ntiles = (uint32_t)(pl.rows * pl.tpr);
    pl.multi = pl.tpr > 1;
    if (!pl.multi) return pl;
    const uint32_t n1 = pl.tpr, n2 = (pl.tpr + 31) / 32, n4 = (pl.tpr + 1023) / 1024 + 1;
    pl.off2 = kRecStride * n1;
    pl.off4 = pl.off2 + kRecStride * n2;
    pl.row_stride = pl.off4 + kRecStride * n4;
    pl.records = (size_t)pl.rows * pl.row_stride;
    return pl;
}

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT>
hipError_t launch_mode(const ScanCall &c, const BdnPlan &pl, const LaunchCtx &ctx)
{
    if (pl.wave_kernel && pl.group > 0) {
        PackedParams p;
        p.a = c.a;
        p.b = c.b;
        p.x0 = c.x0;
        p.out = c.out;
        p.rows = pl.rows;
        p.n = c.n;
        p.x0_stride = c.x0_scalar ? 0 : 1;
        p.phase = pl.phase;
        p.group = pl.group;
        p.inv_group = (65536u + (uint32_t)pl.group - 1u) / (uint32_t)pl.group;
        p.rows_per_wave = 64 / pl.group;
        const int64_t waves = ceil_div(pl.rows, p.rows_per_wave);
        dim3 grid((unsigned)ceil_div(waves, 4)), block(256);
#define HS_PACKED(ITEMS_, VEC_) \
    hipLaunchKernelGGL((heinsen_scan_rows_packed<DOM, LOG_IN, LOG_OUT, InT, ITEMS_, VEC_>), grid, block, 0, c.stream, p)
        if (pl.items == 16) {
            if (pl.vecio) HS_PACKED(16, true);
            else HS_PACKED(16, false);
        } else {
            if (pl.vecio) HS_PACKED(8, true);
            else HS_PACKED(8, false);
        }
#undef HS_PACKED
        return hipGetLastError();
    }
    if (pl.wave_kernel) {
        RowsParams p;
        p.a = c.a;
        p.b = c.b;
        p.x0 = c.x0;
        p.out = c.out;
        p.rows = pl.rows;
        p.n = c.n;
        p.x0_stride = c.x0_scalar ? 0 : 1;
        p.phase = pl.phase;
        // A launch of few waves waits for its loads once instead of twice (600 rows of 1021 steps 4.8 -> 4.5 us); one
        // that fills the chip does better with one array of a row after the other (4096 rows 8.8, together 9.3).
        p.both = pl.rows * c.n <= (3ll << 20);
        dim3 grid((unsigned)ceil_div(pl.rows, 4)), block(256);
#define HS_ROWS(ITEMS_, VEC_)                                                                            \
    hipLaunchKernelGGL((heinsen_scan_rows_wave<DOM, LOG_IN, LOG_OUT, InT, ITEMS_, VEC_>), grid, block, 0, \
                       c.stream, p)
        if (pl.items == 32) {
            if constexpr (!complex_output<DOM, LOG_OUT>()) {
                if (pl.vecio) HS_ROWS(32, true);
                else HS_ROWS(32, false);
            }
        } else if (pl.vecio) {
            if (pl.items == 16) HS_ROWS(16, true);
            else HS_ROWS(8, true);
        } else {
            if (pl.items == 16) HS_ROWS(16, false);
            else HS_ROWS(8, false);
        }
#undef HS_ROWS
        return hipGetLastError();
    }
    TileParams p;
    p.a = c.a;
    p.b = c.b;
    p.x0 = c.x0;
    p.out = c.out;
    p.rows = pl.rows;
    p.n = c.n;
    p.x0_stride = c.x0_scalar ? 0 : 1;
    p.phase = pl.phase;
    p.waves = pl.waves;
    p.pace_ns = pace_ns(pl.vecio, complex_output<DOM, LOG_OUT>(), c.bf16, pl.tpr, pl.ntiles);
    p.tpr = pl.tpr;
    p.ntiles = pl.ntiles;
    rec_t *records = pl.multi ? ctx.scratch : nullptr;
    if (pl.multi && records == nullptr) return hipErrorInvalidValue;
    p.header = records;
    p.recs = records ? records + kRecordBase : nullptr;
    p.spin_limit = ctx.spin_limit;
    p.drop_tile = ctx.drop_tile;
    p.tl.stamps = ctx.timeline;
    p.tl.tiles = ctx.timeline_tiles;
    p.off2 = pl.off2;
    p.off4 = pl.off4;
    p.row_stride = pl.row_stride;
    dim3 grid(pl.ntiles), block(pl.waves * 64);
#define HS_TILES(VEC_, MULTI_, ITEMS_)                                                                          \
    hipLaunchKernelGGL((heinsen_scan_tiles<DOM, LOG_IN, LOG_OUT, InT, VEC_, MULTI_, ITEMS_>), grid, block,      \
                       (MULTI_ ? 0 : pl.waves * tile_stage_slots<VEC_, ITEMS_, inputs_in_lds<DOM, LOG_OUT, MULTI_, ITEMS_>()>() * sizeof(u32x4)), c.stream, p)
    if (pl.multi && pl.tile_items == kTileItems / 2) {
        if (pl.vecio) HS_TILES(true, true, kTileItems / 2);
        else HS_TILES(false, true, kTileItems / 2);
    } else if (pl.multi) {
        if (pl.vecio) HS_TILES(true, true, kTileItems);
        else HS_TILES(false, true, kTileItems);
    } else if (pl.tile_items == 8) {
        if (pl.vecio) HS_TILES(true, false, 8);
        else HS_TILES(false, false, 8);
    } else if (pl.tile_items == 16) {
        if (pl.vecio) HS_TILES(true, false, 16);
        else HS_TILES(false, false, 16);
    } else {
        if (pl.vecio) HS_TILES(true, false, kTileItems);
        else HS_TILES(false, false, kTileItems);
    }
#undef HS_TILES
    return hipGetLastError();
}

hipError_t launch_dispatch(const ScanCall &c, const BdnPlan &pl, const LaunchCtx &ctx)
{
    HS_DISPATCH_MODE(c, launch_mode, c, pl, ctx);
}

} // namespace

ScratchNeed bdn_scratch(const ScanCall &c)
{
    BdnPlan pl = make_plan(c);
    return ScratchNeed{pl.records};
}

hipError_t bdn_launch(const ScanCall &c, const LaunchCtx &ctx)
{
    BdnPlan pl = make_plan(c);
    return launch_dispatch(c, pl, ctx);
}


const char *bdn_kernel_name(const ScanCall &c)
{
    const BdnPlan pl = make_plan(c);
    if (pl.wave_kernel) return pl.group > 0 ? "heinsen_scan_rows_packed" : "heinsen_scan_rows_wave";
    return "heinsen_scan_tiles";
}

void bdn_tile_shape(const ScanCall &c, int &rows, int64_t &steps)
{
    const BdnPlan pl = make_plan(c);
    if (pl.wave_kernel) {
        // one wave per row, or 64 / group rows per wave; workgroups of four waves
        rows = pl.group > 0 ? 4 * (64 / pl.group) : 4;
        steps = c.n;
    } else {
        rows = 1;
        steps = (int64_t)pl.waves * 64 * pl.tile_items;
    }
}

} // namespace hs
