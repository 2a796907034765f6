// Channel-contiguous path: a, b, out are [B, n, D]; lanes own channels, time runs down the rows.
//
// A workgroup of NW waves owns CH = 64*VEC adjacent channels for NW*T consecutive time steps ("tile").
// Wave w of the workgroup scans steps [w*T, (w+1)*T) of the tile serially in each lane (one lane = VEC
// adjacent channels, so a wave's loads and stores are contiguous runs of 256*VEC bytes), keeping the T
// per-element records in registers.  The wave summaries go to LDS, where the first CH threads of the
// workgroup -- one per channel -- turn them into exclusive prefixes; the same threads chain the tiles of
// their channel through global memory: tiles are grouped G at a time along the time axis, a tile folds
// the published summaries of the earlier tiles of its group (always in the same order, so results are
// bit-reproducible) onto the state at the start of the group, and the last tile of a group publishes the
// state at the start of the next.  Every element is read once and written once.
//
// Tiles are handed out by ticket queues, one per compute die: the channel columns are dealt to the
// queues in contiguous runs and a queue hands out its columns' tiles in time order, so a tile only ever
// waits for tiles that were started before it, the draws of the eight dies do not queue behind one
// another, and each die streams through a compact part of memory.
//
// Variations chosen on the host (make_plan): the tile shape; fewer waves per tile for short sequences, no
// tickets at all when a column is one short tile; with few columns, a second carry level whose records the
// waves of a tile share (TREE); where channels do not fill the lanes, columns of channels of several batch
// items (DENSE).
//
// What is computed is Sec. 4's expression applied by parts (Sec. 1, footnote on associativity); the
// arithmetic is in heinsen_math.hpp.
#include "heinsen_internal.hpp"
#include "heinsen_math.hpp"
#include "heinsen_tickets.hpp"
#include "scan_rules.hpp"

#include <algorithm>
#include <type_traits>

namespace hs {
namespace {

struct BndParams {
    const void *a;
    const void *b;
    const float *x0;
    float *out;       // float32 per element; (re, im) float32 pairs for a log output on a signed domain
    int64_t D, n;
    int x0_stride;    // 0: one x0 for all, 1: x0[b*D + d]
    int cols_per_b;   // ceil(D / CH)
    int ncols;        // B * cols_per_b; DENSE: ceil(B / items per column), D > 32: ceil(B * D / 64)
    int64_t places;   // DENSE: B * pad (TREE, RUNS: B * D),
    uint32_t pad;     //   lanes an item takes (RUNS: 16-byte slots from one item's run, or half of it, to the next in LDS, of
                      //   the inputs in the low half of the word, of the output in the high half),
    int lanes;        //   channels per column
    int nchunks;      // ceil(n / (NW*T))
    uint32_t ntiles;  // ncols * nchunks; tile id = chunk * ncols + col
    int nq;           // ticket queues in use (1 or 8); workgroup i draws from queue i mod nq
    int cols_per_q;   // columns dealt to each queue (the last queues may get fewer, or none)
    uint32_t draws_per_q; // workgroups per queue = grid size / nq
    rec_t *header;    // scratch header (ticket queues); null when the launch needs no carries
    rec_t *agg;       // [ntiles][2][CH]  tile summaries: plane 0 = {A | signs}, plane 1 = {M}
                      // (the last tile of a group has no use for its own.  TREE: A of its group's summary is
                      // there instead, float64 in two records, and behind the last group of a super-group the
                      // state at the start of the next one)
    rec_t *state;     // [ngroups][ncols][2][CH] state at the start of a group: float64 log2|x| in two records
                      // (high word | sign, low word).  TREE: M of the group's summary
    uint32_t spin_limit;
    uint32_t drop_tile;
    Timeline tl;
};

// MI355X: 256 MB of memory-side cache; an output up to three quarters of it is left to be cached
constexpr int64_t kLastLevelCacheBytes = 192ll << 20;

// How a kernel touches memory; every element is used once.  (A compile-time choice: written as a run-time
// branch the optimiser merges the two kinds of access into plain ones.)
//   kKeepOut: inputs past the caches, output left in them for whoever consumes it next;
//   kStream:  both past the caches: the output is larger than the last-level cache;
//   kShared:  rows that do not keep to 128-byte lines: neighbouring columns (and neighbouring steps, where an
//             item's channels are fewer than a line) read and write parts of the same lines, which stay in
//             the die's L2 for that.
//   kThrough: kKeepOut where waves write whole lines: written through the die's L2 at once instead of back at some
//             time later, and at the end of the launch what is left, up to 4 MB per die.  The output is in the memory-side
//             cache either way.
enum Mem { kKeepOut, kStream, kShared, kThrough };

template <int MEM, typename InT>
__device__ __forceinline__ float load_elem(const InT *p)
{
    return MEM == kShared ? widen(*p) : widen(__builtin_nontemporal_load(p));
}
template <int MEM>
__device__ __forceinline__ uint32_t load_bits(const uint16_t *p)
{
    return MEM == kShared ? *p : __builtin_nontemporal_load(p);
}
template <int MEM>
__device__ __forceinline__ void store_elem(float *p, float v)
{
    if (MEM == kStream)
        __builtin_nontemporal_store(v, p);
    else if (MEM == kThrough)
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *p = v;
}
template <int MEM>
__device__ __forceinline__ void store_pair(float *p, float re, float im)
{
    typedef float vec_t __attribute__((ext_vector_type(2)));
    const vec_t x = {re, im};
    if (MEM == kStream)
        __builtin_nontemporal_store(x, reinterpret_cast<vec_t *>(p));
    else if (MEM == kThrough)
        __hip_atomic_store(reinterpret_cast<rec_t *>(p), ((rec_t)f2u(im) << 32) | f2u(re), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *reinterpret_cast<vec_t *>(p) = x;
}

__device__ __forceinline__ uint32_t pack_signs(const Seg &g) { return (g.sA >> 31) | ((g.sM >> 31) << 1); }
__device__ __forceinline__ void unpack_signs(uint32_t s, Seg &g)
{
    g.sA = s << 31;
    g.sM = s << 30;
}

// Hand-over between the waves of a workgroup through LDS without a barrier: the producer writes its data,
// then the flag; the consumer polls the flag, then reads the data.  LDS operations of one wave are carried
// out in order, so only the compiler has to be kept from moving them.
// (Some flags are pointed to as what they are, words of LDS; through generic pointers they are flat accesses, each of which waits
// for all that the wave has in flight, its record and output stores included.  As words of LDS in tiles whose scan stands behind
// each way to load (EARLY: 4 x 500 x 100 10.4 and 9.4 us), in those of two carry levels, and for bf16 in runs (719 x 3461 x 9 49.0 and
// 48.3) and whole lines (2 x 9728 x 1088 40.8 and 40.4, 32 x 8000 x 192 80.6 and 80.0, 16 x 1024 x 576 19.4 and 19.5).
// The others are faster with the flat ones: bf16 that cuts lines 4 x 2816 x 1066 31.8 (as words of LDS 32.4), 2 x 1949 x 1170 15.6 (15.9),
// runs of float32 700 x 8102 x 2 41.0 (42.1), 852 x 1620 x 4 18.7 (19.0); wide tiles and shared lines come out even.)
typedef __attribute__((address_space(3))) volatile uint32_t lds_flag_t;
template <typename Flag>
__device__ __forceinline__ void lds_signal(Flag *flag)
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    *flag = 1u;
}
template <typename Flag>
__device__ __forceinline__ bool lds_ready(Flag *flag)
{
    if constexpr (!std::is_same_v<Flag, lds_flag_t>) return *flag != 0u; // no word of LDS
    const bool ready = __builtin_amdgcn_readfirstlane((int)*flag) != 0;
    asm volatile("" ::: "memory");
    return ready;
}
// `count` flags one behind the other, at most 64
__device__ __forceinline__ bool lds_ready_all(lds_flag_t *flags, int count)
{
    const int lane = threadIdx.x & 63;
    const bool ready = lane >= count || flags[lane] != 0;
    asm volatile("" ::: "memory");
    return __builtin_amdgcn_ballot_w64(!ready) == 0ull;
}
__device__ __forceinline__ void lds_await_all(lds_flag_t *flags, int count)
{
    while (!lds_ready_all(flags, count)) __builtin_amdgcn_s_sleep(1);
}
template <typename Flag>
__device__ __forceinline__ void lds_await(Flag *flag)
{
    while (!lds_ready(flag)) __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
}

// ---- items of fewer than 32 channels: whole runs of memory ------------------------------------------------
//
// T steps of an item of few channels are one contiguous run of memory, T * D elements, and a column's items are
// as many such runs.  Taken step by step a wave's accesses are pieces of D elements, and the pieces are what bounds it:
// out = a + b in them reaches 3.9 TB/s for 256 x 4096 x 19 and 1.4 for 900 x 4096 x 3.  Here they are the runs' 16-byte
// vectors, consecutive lanes consecutive vectors, which every wave deals out to its lanes through LDS of its own; what is
// left is the wait for predecessors and, below two rounds of tiles, ramp and drain.  Before and now, the stores of
// runs_in_lines included (five sets of buffers in turn): 256 x 4096 x 16 50.9 and 45.5 us, x 19 67.2 and 55.6, 512 x 4096 x 8
// 71.2 and 46.4, 900 x 4096 x 3 115.6 and 33.1, 64 x 16384 x 5 47.3 and 24.4, bf16 719 x 3461 x 9 107.0 and 49.2, 256 x 4096 x 16
// 45.1 and 34.0; with more than 192 MB of output 700 x 4099 x 19 166 and 148, 3000 x 4096 x 5 252 and 153.  The last steps of a
// sequence, fewer than a wave takes, still go one by one; where they are most of a short one's time it may be 3 % slower
// (8 x 156 x 10 without logarithms 6.4 and 6.6).  A run begins wherever its item does: the vectors are aligned
// as elements are, which global accesses of four words may be.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_at2 __attribute__((aligned(2)));
typedef u32x4 u32x4_at4 __attribute__((aligned(4)));
__device__ __forceinline__ u32x4 load_run(const float *p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4_at4 *>(p)); }
__device__ __forceinline__ u32x4 load_run(const uint16_t *p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4_at2 *>(p)); }
// Vector that begins at element `at` of the wave's output; kThrough is for outputs of up to kLastLevelCacheBytes.  (An atomic store,
// which is how single words are written through, has 64 bits at most.)
template <int MEM>
__device__ __forceinline__ void store_run(float *out, uint32_t at, u32x4 v)
{
    u32x4_at4 *p = reinterpret_cast<u32x4_at4 *>(out + at);
    if (MEM == kStream)
        __builtin_nontemporal_store(v, p);
    else if (MEM == kThrough)
        __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)kLastLevelCacheBytes, 0x00027000), (int)(4u * at), 0, 16); // sc1
    else
        *p = v;
}

// Slots of 16 bytes per wave: an item's run is T * D / 4 of them in float32, and up to 15 between items keep the lanes,
// which pick up step k of their channels all at once, on different banks (run_pitch); halves of runs have a slot more per item
// of two channels: without it their 32 items begin on four banks, and 355 x 5248 x 2 takes 34.7 us instead of 17.6, 256 x 32731
// x 2 80.8 instead of 63.1.  TREE, which needs much of the LDS itself and whose records leave fewer registers, deals the runs out in two
// halves.  (Pieces and runs: 20 x 4000 x 31 18.1 and 16.3 us, 24 x 3000 x 20 16.1 and 15.0, 2 x 1500000 x 30 382 and 354.)
constexpr int run_rounds(int G) { return G > 4 ? 2 : 1; }
constexpr int run_slots(int rounds) { return rounds == 1 ? 544 : 288; }

constexpr int kTreeBlock = 4; // TREE: summaries that one wave adds up for the others (see bnd_tile)
constexpr int kHalfTile = 8;  // TREE: waves of a tile that are folded in float32

// Which item and which vector of its run the wave's vector g is.
struct RunAt {
    uint32_t item, v;
};
__device__ __forceinline__ uint32_t run_inverse(uint32_t per_item) { return ((1u << 20) + per_item - 1u) / per_item; }
__device__ __forceinline__ RunAt run_at(uint32_t g, uint32_t per_item, uint32_t inv)
{
    const uint32_t item = (g * inv) >> 20; // g < 512, per_item of 4 to 256: exact
    return RunAt{item, g - item * per_item};
}
__device__ __forceinline__ void wave_lds_order()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// One tile.  The NW waves of the workgroup stand CG side by side along the channels and TS = NW / CG deep
// along time; a lane owns one channel for T steps.  G tiles per group along time.  SB: keep the scheduler
// from hoisting work across time steps (bounds register pressure).  DENSE: the lanes of a column are up to
// 64 adjacent channels of all B * D, whatever batch items they belong to (same tiles, carries and
// arithmetic; only the lane -> memory mapping differs: a wave's accesses are pieces of rows of one or more
// batch items).  TREE: launches of few columns, where the chain of group states would bound the launch (2 x
// 131072 x 96: 203 us, of which a tile waited 34 of its 43 us): the last tile of a group also publishes the
// summary of its group, and states are handed on only from one super-group of G groups to the next.  A
// tile then reads up to G - 1 tile summaries, G - 1 group summaries and one state; each of its waves fetches
// one of each level beside its own loads and passes it on through LDS, the last wave of every four adds up theirs, and
// the first wave folds the sums.  Whatever is folded beyond eight waves (256 steps) is folded in float64, as the chain of states is:
// beyond a tile, and the two halves of a tile of sixteen waves, whose summary is rounded to float32 once more then.  That is some
// 200 cycles each, which one after the other were half of what a tile waited.  Registers are full of the tile itself, so nothing
// of this stays in them: records are looked at as soon as they are there and go to LDS, and addresses in LDS are formed anew in
// every round of polling (kept, they pushed elements into scratch memory, whose loads wait for every store before them).  Before
// and now: 2 x 131072 x 96 72.6 and 66.1 us, 1 x 1048576 x 64 248 and 168, 12 x 4096 x 64 14.4 and 12.7, 3 x 1100 x 64 9.2 and 8.9.
//
// No wave waits for more than it needs.  The first wave along time of each 64-channel column fetches the
// carry records, forms the state at the start of the tile and hands it to the waves behind it through
// LDS; a later wave waits only for the summaries of the waves before it in its own column; the last wave
// along time publishes the tile's summary (and, closing a group, the state for the next group).  TREE: where some a_t is +inf or
// NaN, or a product leaves float32, it first waits for the state at the start of the tile (see carry_append64).  `flags`
// are words of LDS, as many as the kernel says, zero when the tile begins.
template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT, int T, int NW, int G, bool SB, bool DENSE, bool TREE, bool RUNS, int CG, int MEM>
__device__ __forceinline__ void bnd_tile(const BndParams &p, const uint32_t tile, const uint32_t epoch, lds_flag_t *flags)
{
    constexpr bool SIGNED = DOM == kSigned;
    constexpr int CH = 64 * CG;  // channels of the tile
    constexpr int TS = NW / CG;  // waves one after the other along time
    // Whether the scan stands behind each way to load.  One scan behind them all is one where the compiler, which cannot tell there
    // what is still on its way, has the first step wait for the last input (6 x 3072 x 768 36.9 and 36.1 us, 4 x 1000 x 1000 14.0
    // and 13.2).  Not for bf16 (8 x 8192 x 1536 151.0 and 152.1), whose loads are half as long, where lines are shared (8 x 8000 x
    // 1501, logarithms, 252.5 and 254.5), for the wide tiles (16 x 16384 x 2048 1039 and 1042) and for runs, which leave no registers.
    constexpr bool EARLY = sizeof(InT) == 4 && !RUNS && CG == 1 && MEM != kShared;
    constexpr bool TALL = TREE && TS > kHalfTile;
    constexpr int PT = TREE ? 1 : (G > 1 ? G - 1 : 1); // tile summaries a wave fetches
    static_assert(T <= 32, "one sign word per channel");
    static_assert(NW % CG == 0, "the waves form a CG x TS grid");
    static_assert(!DENSE || CG == 1, "dense columns are mapped one channel per lane");
    static_assert(!RUNS || (DENSE && NW > 1 && !(SIGNED && LOG_OUT)), "runs are of columns of whole items");
    static_assert(!TREE || (CG == 1 && G == TS && TS % kTreeBlock == 0), "every wave of a tile takes one summary of each level");
    static_assert(!TREE || TS == kHalfTile || TS == 2 * kHalfTile, "a tile is one half or two");
    __shared__ float lds_A[TS][CH];
    __shared__ float lds_M[TS][CH];
    __shared__ uint32_t lds_S[SIGNED ? TS : 1][CH];
    __shared__ double lds_startL[CH]; // float64: the wave that closes a group hands it on as it is
    __shared__ uint32_t lds_startS[CH];
    // TREE: every wave's tile summary and its group summary, and the sums of BL of them
    constexpr int BL = kTreeBlock, NBL = TREE ? G / BL : 1;
    __shared__ float lds_tileA[TREE ? G : 1][CH], lds_tileM[TREE ? G : 1][CH];
    __shared__ double lds_groupA[TREE ? G : 1][CH], lds_groupM[TREE ? G : 1][CH];
    __shared__ uint32_t lds_tileS[TREE ? G : 1][CH], lds_groupS[TREE ? G : 1][CH];
    __shared__ double lds_sumA[2][NBL][CH], lds_sumM[2][NBL][CH]; // of tiles, of groups
    __shared__ uint32_t lds_sumS[2][NBL][CH];
    // and, while the records are waited for, the wave's fold of the waves before it (registers are full)
    __shared__ float lds_preA[TREE ? TS : 1][CH], lds_preM[TREE ? TS : 1][CH];
    __shared__ uint32_t lds_preS[TREE ? TS : 1][CH];
    __shared__ double lds_superL[TREE ? CH : 1]; // state at the start of the super-group
    __shared__ uint32_t lds_superS[TREE ? CH : 1];
    __shared__ double lds_restA[TREE ? CH : 1], lds_restM[TREE ? CH : 1]; // everything between there and the tile
    __shared__ uint32_t lds_restS[TREE ? CH : 1];
    // the fold of the first half's waves
    __shared__ float lds_halfA[TALL ? CH : 1], lds_halfM[TALL ? CH : 1];
    __shared__ uint32_t lds_halfS[TALL ? CH : 1];

    constexpr int ROUNDS = run_rounds(G);
    __shared__ u32x4 lds_runs[RUNS ? NW : 1][RUNS ? run_slots(ROUNDS) : 1];

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); // wave-uniform, kept in an SGPR
    // The rows the workgroup reads and writes are runs of 256*CG contiguous bytes, requested by its CG
    // columns at about the same time, which is what the memory system wants to see.
    const int wc = w % CG, ts = w / CG;
    constexpr bool HALVES = sizeof(InT) == 2 && CG == 1 && NW == 8 && (RUNS || MEM == kThrough || MEM == kStream); // runs, whole lines
    using flag_t = std::conditional_t<EARLY || TREE || HALVES, lds_flag_t, volatile uint32_t>;
    flag_t *flag_run = (flag_t *)flags;              // [TS][CG]: the wave's summary is in LDS
    flag_t *flag_start = flag_run + TS * CG;  // [CG]: the column's start state is in LDS
    lds_flag_t *flag_part = flags + TS * CG + CG; // TREE: [2][TS]: the wave's summaries are in LDS,
    lds_flag_t *flag_sum = flag_part + 2 * G;     //   [2][NBL]: the sums of BL of them, [1]: the super-group's state, [1]: what lies between, [1]: the first half's fold

    const int chunk = (int)(tile / (uint32_t)p.ncols);
    const int col = (int)(tile % (uint32_t)p.ncols);
    const int bidx = col / p.cols_per_b;
    const int cg = col % p.cols_per_b;
    const int g = chunk / G;
    const int r = chunk % G;
    const bool more = chunk + 1 < p.nchunks;

    const int c = wc * 64 + lane; // the lane's channel inside the tile
    const int64_t t0 = (int64_t)chunk * (TS * T) + (int64_t)ts * T;
    uint32_t moff;   // the only per-lane part of every global address (elements): the addresses are a
                     // wave-uniform 64-bit base, advanced by scalar arithmetic, plus this 32-bit offset
    bool chan_ok;    // the lane has a channel
    int64_t ubase;   // wave-uniform part of the addresses
    int64_t x0_at;   // the channel's place in x0
    if constexpr (DENSE) {
        // An item takes `pad` of the column's lanes (see make_plan).
        constexpr bool CLOSE = TREE || RUNS; // the items of a column stand close together
        const uint32_t pad = CLOSE ? (uint32_t)p.D : p.pad;
        const uint32_t first = (uint32_t)col * (CLOSE ? (uint32_t)p.lanes : 64u), place = first + (uint32_t)lane;
        const uint32_t b0 = first / pad, bb = place / pad;   // batch items of the column's first lane and of this one
        const uint32_t at = place - bb * pad;                // the lane's channel in its item
        chan_ok = (CLOSE ? lane < p.lanes : at < (uint32_t)p.D) && place < p.places;
        moff = (bb - b0) * (uint32_t)(p.n * p.D) + at; // the host checks that this fits 31 bits
        ubase = ((int64_t)b0 * p.n + t0) * p.D;
        x0_at = CLOSE ? place : bb * (uint32_t)p.D + at;
    } else {
        const int64_t d0 = (int64_t)cg * CH + c;
        chan_ok = d0 < p.D;
        moff = (uint32_t)c;
        ubase = ((int64_t)bidx * p.n + t0) * p.D + (int64_t)cg * CH;
        x0_at = (int64_t)bidx * p.D + d0;
    }
    const InT *ap = reinterpret_cast<const InT *>(p.a) + ubase;
    const InT *bp = reinterpret_cast<const InT *>(p.b) + ubase;

    // ---- the first wave of a column asks for the carry records it will need before anything else is in
    //      flight: once the kernel is past its first round the earlier tiles of the group have usually
    //      published, and the records then arrive ahead of the tile's own loads at no cost in latency ---
    const bool first = ts == 0; // wave-uniform
    const bool fetches = TREE || first;
    struct Recs { // (what is not asked for is not set)
        rec_t A[PT], M[PT], Q[4] = {}, S = 0, S2 = 0;
    };
    Recs recs;
    const int q = TREE ? g / G : g;   // TREE: super-group, and the group's place in it
    const int gi = TREE ? g % G : 0;
    const bool has_state = first && q > 0;
    bool want_state = has_state, want_tile = TREE && ts < r, want_group = TREE && ts < gi; // TREE: still missing (wave-uniform)
    int cv = c; // TREE: renewed in every round of the loop below, so that no address that depends on it stays in a register
    auto issue_records = [&](Recs &R) {
        if (want_state) {
            const rec_t *sp = (TREE ? p.agg + ((size_t)(q * G * G - 1) * p.ncols + col) * (2 * CH)
                                    : p.state + ((size_t)q * p.ncols + col) * (2 * CH)) + cv;
            R.S = rec_get(sp);
            R.S2 = rec_get(sp + CH);
        }
        if constexpr (TREE) {
            if (want_tile) {
                const rec_t *tp = p.agg + ((size_t)(g * G + ts) * p.ncols + col) * (2 * CH) + cv;
                R.A[0] = rec_get(tp);
                R.M[0] = rec_get(tp + CH);
            }
            if (want_group) {
                const rec_t *gp = p.agg + ((size_t)((q * G + ts) * G + G - 1) * p.ncols + col) * (2 * CH) + cv;
                const rec_t *mp = p.state + ((size_t)(q * G + ts) * p.ncols + col) * (2 * CH) + cv;
                R.Q[0] = rec_get(gp);
                R.Q[1] = rec_get(gp + CH);
                R.Q[2] = rec_get(mp);
                R.Q[3] = rec_get(mp + CH);
            }
        } else {
#pragma unroll
            for (int j = 0; j < G - 1; ++j) {
                if (j < r) {
                    const rec_t *tp = p.agg + ((size_t)(g * G + j) * p.ncols + col) * (2 * CH) + cv;
                    R.A[j] = rec_get(tp);
                    R.M[j] = rec_get(tp + CH);
                }
            }
        }
    };
    auto tile_in = [&](const Recs &R, int j) -> bool { return rec_ok(R.A[j], epoch) && rec_ok(R.M[j], epoch); }; // of this lane
    auto group_in = [&](const Recs &R) -> bool {
        return rec_ok(R.Q[0], epoch) && rec_ok(R.Q[1], epoch) && rec_ok(R.Q[2], epoch) && rec_ok(R.Q[3], epoch);
    };
    auto state_in = [&](const Recs &R) -> bool { return !has_state || (rec_ok(R.S, epoch) && rec_ok(R.S2, epoch)); };
    auto records_in = [&](const Recs &R) -> bool { // one carry level: all of this lane's
        bool ok = true;
        if constexpr (!TREE) {
#pragma unroll
            for (int j = 0; j < G - 1; ++j)
                if (j < r) ok = ok && tile_in(R, j);
        }
        return ok && state_in(R);
    };
    auto wave_all = [](bool ok) -> bool { return __builtin_amdgcn_ballot_w64(!ok) == 0ull; };
    bool have_records = false;
    if (fetches) issue_records(recs);
    // TREE: what is in goes to LDS at once (and with `lost`, NaN for what never came): registers are full
    auto pass_on = [&](const Recs &R, bool lost) {
        if constexpr (TREE) {
            if (want_tile && (lost || wave_all(tile_in(R, 0)))) {
                want_tile = false;
                Seg part = seg_from<DOM>(R.A[0], R.M[0]);
                if (!tile_in(R, 0)) part.M = __builtin_nanf("");
                lds_tileA[ts][cv] = part.A;
                lds_tileM[ts][cv] = part.M;
                if (SIGNED) lds_tileS[ts][cv] = pack_signs(part);
                lds_signal(&flag_part[ts]);
            }
            if (want_group && (lost || wave_all(group_in(R)))) {
                want_group = false;
                const Seg64 part = seg64_from<DOM>(R.Q);
                lds_groupA[ts][cv] = part.A;
                lds_groupM[ts][cv] = group_in(R) ? part.M : __builtin_nan("");
                if (SIGNED) lds_groupS[ts][cv] = (part.sA >> 31) | ((part.sM >> 31) << 1);
                lds_signal(&flag_part[G + ts]);
            }
            if (want_state && (lost || wave_all(state_in(R)))) {
                want_state = false;
                const State64 x = state64_from(R.S, R.S2, SIGNED);
                lds_superL[cv] = state_in(R) ? x.lx : __builtin_nan("");
                lds_superS[cv] = x.s;
                lds_signal(&flag_sum[2 * NBL]);
            }
        }
    };

    // ---- load the lane's T inputs, encode and scan them serially; Av/Mv become the per-element records (see stash).  EARLY:
    //      every way to load has the scan behind it; otherwise it stands behind them all -----------------------------
    float Av[T], Mv[T];
    uint32_t sw = 0u, sm = 0u;
    Seg run;
    auto scan = [&]() {
#pragma unroll
        for (int k = 0; k < T; ++k) {
            lane_step<DOM, LOG_IN, LOG_OUT>(k, run, Av[k], Mv[k], sw, sm);
            if (SB) __builtin_amdgcn_sched_barrier(0);
        }
    };
    const float id_a = LOG_IN ? 0.0f : 1.0f; // a = 1, b = 0 leave the state unchanged
    const float id_b = LOG_IN ? -INFINITY : 0.0f;
    // RUNS: the part of the wave's LDS region that its lane reads and writes (elements from one step to the next: D)
    const bool whole = RUNS && t0 + T <= p.n; // wave-uniform: the last steps of a sequence go one by one
    const uint32_t D32 = (uint32_t)p.D, run_item = RUNS && chan_ok ? (uint32_t)lane / D32 : 0u;
    const uint32_t run_ch = RUNS && chan_ok ? (uint32_t)lane - run_item * D32 : 0u;
    uint32_t run_n = 0; // items of this column (wave-uniform)
    const uint32_t pitch_in = p.pad & 0xffffu, pitch_out = p.pad >> 16;
    if constexpr (RUNS) {
        const uint32_t first_place = (uint32_t)col * (uint32_t)p.lanes, left = (uint32_t)p.places - first_place;
        run_n = ((uint32_t)p.lanes < left ? (uint32_t)p.lanes : left) / D32;
    }
    if (RUNS && whole) {
        constexpr int VL = 16 / (int)sizeof(InT), NV = T / VL / ROUNDS, TR = T / ROUNDS;
        const uint32_t per = (uint32_t)(TR / VL) * D32, all = run_n * per, inv = run_inverse(per);
        const uint32_t to_next = (uint32_t)(p.n * p.D);
        auto ask = [&](const InT *from, u32x4(&t)[ROUNDS * NV]) { // lanes without a vector take the first
#pragma unroll
            for (int j = 0; j < ROUNDS * NV; ++j) {
                const uint32_t g = (uint32_t)(j % NV * 64 + lane);
                const RunAt r2 = run_at(g < all ? g : 0u, per, inv);
                t[j] = load_run(from + (r2.item * to_next + ((uint32_t)(j / NV) * per + r2.v) * VL));
            }
        };
        auto deal = [&](const u32x4(&t)[ROUNDS * NV], float(&x)[T]) {
            const InT *mine = reinterpret_cast<const InT *>(&lds_runs[w][run_item * pitch_in]) + run_ch;
#pragma unroll
            for (int h = 0; h < ROUNDS; ++h) {
#pragma unroll
                for (int j = 0; j < NV; ++j) {
                    const uint32_t g = (uint32_t)(j * 64 + lane);
                    const RunAt r2 = run_at(g, per, inv);
                    if (g < all) lds_runs[w][r2.item * pitch_in + r2.v] = t[h * NV + j];
                }
                wave_lds_order();
#pragma unroll
                for (int k = 0; k < TR; ++k) x[h * TR + k] = widen(mine[(uint32_t)k * D32]);
                wave_lds_order();
            }
        };
        u32x4 ta[ROUNDS * NV], tb[ROUNDS * NV];
        ask(ap, ta);
        if (ROUNDS == 1) ask(bp, tb); // both at once, where there are registers for it
        deal(ta, Av);
        if (ROUNDS > 1) ask(bp, tb);
        deal(tb, Mv);
    } else if ((EARLY || chan_ok) && t0 + T <= p.n) {
        const InT *arow = ap, *brow = bp; // wave-uniform row pointers
        const uint32_t off = !EARLY || chan_ok ? moff : 0u; // lanes without a channel take the first one's
#pragma unroll
        for (int k = 0; k < T; ++k) {
            Av[k] = load_elem<MEM, InT>(arow + off);
            Mv[k] = load_elem<MEM, InT>(brow + off);
            arow += p.D;
            brow += p.D;
        }
        if (EARLY) {
            pass_on(recs, false);
            scan();
        }
    } else if constexpr (sizeof(InT) == 2) {
        // As stored until all are asked for: widened inside the branches, every step would be waited for before the next
        // one is asked for, which is what bounds short and ragged calls (25 x 285 x 320 17.8 us so, 8.8 now; 52 x 183 x 13 10.6
        // and 7.7; 36 x 702 x 1184, logarithms, 78.5 and 57.7).
        uint32_t ra[T], rb[T]; // (1, 0 and -inf are exact in bf16)
#pragma unroll
        for (int k = 0; k < T; ++k) {
            ra[k] = f2u(id_a) >> 16;
            rb[k] = f2u(id_b) >> 16;
            if (chan_ok && t0 + k < p.n) {
                ra[k] = load_bits<MEM>(ap + (int64_t)k * p.D + moff);
                rb[k] = load_bits<MEM>(bp + (int64_t)k * p.D + moff);
            }
        }
#pragma unroll
        for (int k = 0; k < T; ++k) {
            asm("" : "+v"(ra[k]), "+v"(rb[k])); // keeps the shift out of the branches
            Av[k] = u2f(ra[k] << 16);
            Mv[k] = u2f(rb[k] << 16);
        }
    } else {
#pragma unroll
        for (int k = 0; k < T; ++k) {
            if (chan_ok && t0 + k < p.n) {
                Av[k] = load_elem<MEM, InT>(ap + (int64_t)k * p.D + moff);
                Mv[k] = load_elem<MEM, InT>(bp + (int64_t)k * p.D + moff);
            } else {
                Av[k] = id_a;
                Mv[k] = id_b;
            }
        }
        if (EARLY) {
            pass_on(recs, false);
#pragma unroll
            for (int k = 0; k < T; ++k) asm volatile("" : "+v"(Av[k]), "+v"(Mv[k])); // all are asked for before the first is used
            scan();
        }
    }
    if (!EARLY) {
        if (!TREE && first) have_records = wave_all(records_in(recs)); // first look: answered while the tile's loads were in flight
        pass_on(recs, false);
        scan();
    }
    lane_close<DOM, LOG_IN, LOG_OUT>(run);
    p.tl.mark(tile, 2);

    // ---- the waves behind this one in the column need its summary --------------------------------
    if (TS > 1 && (TREE || ts < TS - 1)) {
        lds_A[ts][c] = run.A;
        lds_M[ts][c] = run.M;
        if (SIGNED) lds_S[ts][c] = pack_signs(run);
        lds_signal(&flag_run[ts * CG + wc]);
    }
    p.tl.mark(tile, 3);
    if (EARLY && !TREE && first) have_records = wave_all(records_in(recs));

    // ---- a later wave: the fold of the waves before it in its column, in wave order (tall tiles: in its half); the last one along
    //      time closes the tile: its fold with its own summary is the tile's.  (TREE: one wave after the other as well.  From sums of
    //      four and a tall tile as one, the fold rounds more often: 2 x 131072 x 96, relative rms error over gates 7.51e-8 instead
    //      of 7.49e-8, with decays within 1e-2 of one 1.076e-7 and 1.068e-7; the time is the same, 66.2 and 66.1 us.) ----
    Seg pre = seg_identity<DOM>(), total = seg_identity<DOM>();
    const bool closing = TS > 1 && ts == TS - 1; // wave-uniform
    bool apart = false; // TREE: waves before this one have, in some channel, no summary for every state (see carry_append64),
    bool late = false;  // closing wave: nor has the tile
    auto mine = [&]() -> Seg { // TREE: read back, registers are full
        if constexpr (!TREE) return run;
        Seg h;
        h.A = lds_A[ts][c];
        h.M = lds_M[ts][c];
        h.sA = h.sM = 0u;
        if (SIGNED) unpack_signs(lds_S[ts][c], h);
        return h;
    };
    auto get_run = [&](int j) -> Seg {
        if (!TREE) lds_await(&flag_run[j * CG + wc]);
        Seg h;
        h.A = lds_A[j][c];
        h.M = lds_M[j][c];
        h.sA = h.sM = 0u;
        if (SIGNED) unpack_signs(lds_S[j][c], h);
        return h;
    };
    auto put_tile = [&]() { // closing wave
        if (r < G - 1 && tile != p.drop_tile) {
            rec_t *tp = p.agg + (size_t)tile * (2 * CH) + c;
            seg_put<DOM>(tp, tp + CH, total, epoch);
        }
    };
    auto keep_total = [&]() { // TREE: its slot among the waves' summaries is free
        lds_A[TS - 1][c] = total.A;
        lds_M[TS - 1][c] = total.M;
        if (SIGNED) lds_S[TS - 1][c] = pack_signs(total);
    };
    const bool second = TALL && ts >= kHalfTile; // wave-uniform: a wave of the second half
    auto get_half = [&]() -> Seg {
        Seg h{lds_halfA[TALL ? c : 0], lds_halfM[TALL ? c : 0], 0u, 0u};
        if (SIGNED) unpack_signs(lds_halfS[TALL ? c : 0], h);
        return h;
    };
    lds_flag_t *flag_half = &flag_sum[2 * NBL + 2];
    auto tile_of = [&](const Seg &half) -> Seg { // closing wave: the tile's summary, of its last half
        if constexpr (!TALL) return half;
        const Seg64 sum = seg_append64<DOM>(seg64(get_half()), half);
        return Seg{(float)sum.A, (float)sum.M, sum.sA, sum.sM};
    };
    if (!first) {
        if constexpr (TREE) {
            const int from = second ? kHalfTile : 0;
            lds_await_all(&flag_run[from], ts - from);
            if (ts > from) pre = get_run(from);
#pragma unroll 1
            for (int j = from + 1; j < ts; ++j) pre = seg_combine<DOM>(pre, get_run(j));
            if (TALL && ts == kHalfTile - 1) {
                const Seg half = seg_combine<DOM>(pre, mine());
                lds_halfA[c] = half.A;
                lds_halfM[c] = half.M;
                if (SIGNED) lds_halfS[c] = pack_signs(half);
                lds_signal(flag_half);
            }
        } else {
#pragma unroll
            for (int j = 0; j < TS - 1; ++j)
                if (j < ts) pre = (j == 0) ? get_run(j) : seg_combine<DOM>(pre, get_run(j));
        }
        if (closing && more) {
            const Seg half = seg_combine<DOM>(pre, mine());
            if (TALL) lds_await(flag_half);
            total = tile_of(half);
            late = TREE && !wave_all(seg_sums<DOM>(total.A));
            if (!late) put_tile();
        }
        if constexpr (TREE) {
            apart = !wave_all(seg_sums<DOM>(pre.A));
            lds_preA[ts][c] = pre.A;
            lds_preM[ts][c] = pre.M;
            if (SIGNED) lds_preS[ts][c] = pack_signs(pre);
            if (closing && !late) keep_total();
            asm volatile("" ::: "memory");
        }
    }
    auto get_total = [&]() -> Seg { // closing wave
        if constexpr (!TREE) return total;
        Seg g2;
        g2.A = lds_A[TS - 1][cv];
        g2.M = lds_M[TS - 1][cv];
        g2.sA = g2.sM = 0u;
        if (SIGNED) unpack_signs(lds_S[TS - 1][cv], g2);
        return g2;
    };

    auto get_pre = [&]() -> Seg {
        if constexpr (!TREE) return pre;
        Seg h{lds_preA[TREE ? ts : 0][c], lds_preM[TREE ? ts : 0][c], 0u, 0u};
        if (SIGNED) unpack_signs(lds_preS[TREE ? ts : 0][c], h);
        return h;
    };
    auto state_behind = [&](State64 x, int waves) -> State64 { // so many waves of the tile, one after the other
#pragma unroll 1
        for (int j = 0; j < waves; ++j) x = seg_apply64<DOM>(x, get_run(j));
        return x;
    };

    State st;                // state at the wave's first step
    State64 st64{0.0, 0u};   // the same in float64, along the chain of tiles
    auto state_from_x0 = [&]() {
        float x0v = LOG_IN ? 0.0f : 1.0f, lx;
        int64_t at = x0_at;
        if (TREE) { // formed here: registers are full
            int l = threadIdx.x & 63;
            asm volatile("" : "+v"(l));
            at = DENSE ? (int64_t)col * p.lanes + l : (int64_t)bidx * p.D + (int64_t)cg * CH + l;
        }
        if (chan_ok) x0v = p.x0[p.x0_stride ? at : 0];
        encode<DOM, LOG_IN>(x0v, lx, st64.s);
        st64.lx = (double)lx;
    };
    if constexpr (TREE) {
        // ---- every wave passes on its summaries as soon as they are in, and the last wave of a block of BL the sum of the
        //      block's: one after the other the 15 of a group are four microseconds of float64 in the way of every tile behind ---
        auto get_tile = [&](int j) -> Seg {
            Seg g2;
            g2.A = lds_tileA[j][cv];
            g2.M = lds_tileM[j][cv];
            g2.sA = g2.sM = 0u;
            if (SIGNED) unpack_signs(lds_tileS[j][cv], g2);
            return g2;
        };
        auto get64 = [&](const double (&A)[CH], const double (&M)[CH], const uint32_t (&S)[CH]) -> Seg64 {
            const uint32_t sg = SIGNED ? S[cv] : 0u;
            return Seg64{A[cv], M[cv], sg << 31, sg << 30};
        };
        auto put64 = [&](double (&A)[CH], double (&M)[CH], uint32_t (&S)[CH], const Seg64 &v) {
            A[cv] = v.A;
            M[cv] = v.M;
            if (SIGNED) S[cv] = (v.sA >> 31) | ((v.sM >> 31) << 1);
        };
        const int bl = ts / BL * BL;         // first of the wave's block
        const bool sums = ts % BL == BL - 1; // it adds up the block's summaries, if there are as many
        // Without logarithms only group by group: the products of a of two groups may leave float64, where those of one (eight
        // tiles, in float32 each) cannot.
        constexpr bool SUM_GROUPS = DOM != kLinear;
        const int gi_sums = SUM_GROUPS ? gi / BL : 0; // blocks of groups
        bool tile_sum = !(sums && bl + BL <= r), group_sum = !(sums && SUM_GROUPS && bl + BL <= gi);
        bool owes = closing && more && r == G - 1 && gi < G - 1; // the last tile of a group owes the later groups its sum
        auto put_group = [&]() {
            Seg64 sum = get64(lds_sumA[0][0], lds_sumM[0][0], lds_sumS[0][0]);
#pragma unroll 1
            for (int j = 1; j < NBL - 1; ++j) sum = carry_append64<DOM>(sum, get64(lds_sumA[0][j], lds_sumM[0][j], lds_sumS[0][j]));
#pragma unroll 1
            for (int j = G - BL; j < G - 1; ++j) sum = carry_append64<DOM>(sum, get_tile(j));
            seg64_put<DOM>(p.agg + (size_t)tile * (2 * CH) + cv, p.state + ((size_t)g * p.ncols + col) * (2 * CH) + cv, CH,
                           carry_append64<DOM>(sum, get_total()), epoch);
        };
        uint32_t polls = 0;
        for (;;) {
            asm volatile("" : "+v"(cv));
            if (want_tile || want_group || want_state) {
                Recs again;
                issue_records(again);
                if (++polls > p.spin_limit) note_wait_gave_up(p.header); // go on as if everything were in, with NaN for what is missing
                pass_on(again, polls > p.spin_limit);
            }
            if (!tile_sum && lds_ready_all(&flag_part[bl], BL)) {
                tile_sum = true;
                Seg64 sum = seg64(get_tile(bl));
#pragma unroll 1
                for (int j = bl + 1; j < bl + BL; ++j) sum = carry_append64<DOM>(sum, get_tile(j));
                put64(lds_sumA[0][bl / BL], lds_sumM[0][bl / BL], lds_sumS[0][bl / BL], sum);
                lds_signal(&flag_sum[bl / BL]);
            }
            if (!group_sum && lds_ready_all(&flag_part[G + bl], BL)) {
                group_sum = true;
                Seg64 sum = get64(lds_groupA[bl], lds_groupM[bl], lds_groupS[bl]);
#pragma unroll 1
                for (int j = bl + 1; j < bl + BL; ++j) sum = carry_append64<DOM>(sum, get64(lds_groupA[j], lds_groupM[j], lds_groupS[j]));
                put64(lds_sumA[1][bl / BL], lds_sumM[1][bl / BL], lds_sumS[1][bl / BL], sum);
                lds_signal(&flag_sum[NBL + bl / BL]);
            }
            if (owes && !late && lds_ready_all(flag_sum, NBL - 1) && lds_ready_all(&flag_part[G - BL], BL - 1)) {
                owes = false;
                put_group();
            }
            if (!want_tile && !want_group && !want_state && tile_sum && group_sum && (!owes || late)) break;
            __builtin_amdgcn_s_sleep(1);
        }
        p.tl.mark(tile, 4);
        // what lies between the super-group's start and the tile, in order: the sums of whole blocks, then what is behind them
        auto rest = [&](auto &&take) {
#pragma unroll 1
            for (int j = 0; j < gi_sums; ++j) {
                lds_await(&flag_sum[NBL + j]);
                take(get64(lds_sumA[1][j], lds_sumM[1][j], lds_sumS[1][j]));
            }
#pragma unroll 1
            for (int j = gi_sums * BL; j < gi; ++j) {
                lds_await(&flag_part[G + j]);
                take(get64(lds_groupA[j], lds_groupM[j], lds_groupS[j]));
            }
#pragma unroll 1
            for (int j = 0; j < r / BL; ++j) {
                lds_await(&flag_sum[j]);
                take(get64(lds_sumA[0][j], lds_sumM[0][j], lds_sumS[0][j]));
            }
#pragma unroll 1
            for (int j = r / BL * BL; j < r; ++j) {
                lds_await(&flag_part[j]);
                take(get_tile(j));
            }
        };
        lds_flag_t *flag_rest = &flag_sum[2 * NBL + 1];
        // Behind the first super-group the second wave adds it all up: a link of the chain of states is one step then, however late
        // the state (one column of 400000 steps 89.7 and 75.9 us, of 1048576 206 and 168).
        if (SUM_GROUPS && ts == 1 && q > 0) {
            Seg64 sum{0.0, -INFINITY, 0u, 0u};
            rest([&](const auto &part) { sum = carry_append64<DOM>(sum, part); });
            put64(lds_restA, lds_restM, lds_restS, sum);
            lds_signal(flag_rest);
        }
        if (first) {
            if (q == 0) state_from_x0();
            else st64 = State64{lds_superL[c], lds_superS[c]};
            if (SUM_GROUPS && q > 0) {
                lds_await(flag_rest);
                st64 = carry_apply64<DOM>(st64, get64(lds_restA, lds_restM, lds_restS));
            } else {
                rest([&](const auto &part) { st64 = carry_apply64<DOM>(st64, part); });
            }
            st.lx = (float)st64.lx;
            st.s = st64.s;
            lds_startL[c] = st64.lx;
            lds_startS[c] = st64.s;
            lds_signal(&flag_start[wc]);
        }
        if (late) {
            lds_await(&flag_start[wc]);
            const Seg sum = tile_of(seg_combine<DOM>(get_pre(), get_run(TS - 1))), end = seg_of_state(state_behind(State64{lds_startL[c], lds_startS[c]}, TS));
            const bool sums = seg_sums<DOM>(sum.A);
            total = Seg{sums ? sum.A : end.A, sums ? sum.M : end.M, sums ? sum.sA : end.sA, sums ? sum.sM : end.sM};
            keep_total();
            if (owes) {
                lds_await_all(flag_sum, NBL - 1);
                lds_await_all(&flag_part[G - BL], BL - 1);
                put_group();
            }
            put_tile();
        }
    } else if (first) {
        // ---- obtain the state at the start of the tile ------------------------------------------
        bool lost = false; // this lane's records never came
        if (!have_records) {
            issue_records(recs);
            uint32_t polls = 0;
            for (;;) {
                const bool ok = records_in(recs);
                if (wave_all(ok)) break;
                if (++polls > p.spin_limit) {
                    lost = !ok;
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
                issue_records(recs);
            }
        }
        p.tl.mark(tile, 4);
        if (g == 0) {
            state_from_x0();
        } else {
            st64 = state64_from(recs.S, recs.S2, SIGNED);
        }
        // fold the earlier tiles of the group in tile order
#pragma unroll
        for (int j = 0; j < G - 1; ++j) {
            if (j < r) st64 = seg_apply64<DOM>(st64, seg_from<DOM>(recs.A[TREE ? 0 : j], recs.M[TREE ? 0 : j]));
        }
        if (lost) {
            st64.lx = __builtin_nan("");
            note_wait_gave_up(p.header);
        }
        st.lx = (float)st64.lx;
        st.s = st64.s;
        if (TS > 1) {
            lds_startL[c] = st64.lx;
            lds_startS[c] = st64.s;
            lds_signal(&flag_start[wc]);
        } else {
            // a single wave along time closes the tile itself
            if (more && r < G - 1 && tile != p.drop_tile) {
                rec_t *tp = p.agg + (size_t)tile * (2 * CH) + c;
                seg_put<DOM>(tp, tp + CH, run, epoch);
            }
            if (more && r == G - 1) {
                rec_t *sp = p.state + ((size_t)(g + 1) * p.ncols + col) * (2 * CH) + c;
                state64_put(sp, sp + CH, seg_apply64<DOM>(st64, run), epoch, SIGNED);
            }
        }
    }
    if (!first) {
        lds_await(&flag_start[wc]);
        st64.lx = lds_startL[c];
        st64.s = lds_startS[c];
        st.lx = (float)st64.lx;
        st.s = st64.s;
        if (closing && more && r == G - 1 && (!TREE || gi == G - 1)) {
            // last tile of a group (TREE: of a super-group): the state after this tile starts the next one
            rec_t *sp = (TREE ? p.agg + (size_t)tile * (2 * CH) : p.state + ((size_t)(q + 1) * p.ncols + col) * (2 * CH)) + c;
            state64_put(sp, sp + CH, TREE ? carry_apply64<DOM>(st64, get_total()) : seg_apply64<DOM>(st64, get_total()), epoch, SIGNED);
        }
        if constexpr (TREE) {
            bool sums = true;
            if (second) {
                lds_await(flag_half);
                const Seg half = get_half();
                sums = seg_sums<DOM>(half.A);
                apart = apart || !wave_all(sums);
                const State64 mid = seg_apply64<DOM>(st64, half);
                st.lx = (float)mid.lx;
                st.s = mid.s;
            }
            pre = get_pre();
            if (!TALL || ts != kHalfTile) st = seg_apply<DOM>(st, pre);
            if (__builtin_expect(apart, 0)) {
                const State64 x = state_behind(st64, ts);
                sums = sums && seg_sums<DOM>(pre.A);
                st.lx = sums ? st.lx : (float)x.lx;
                st.s = sums ? st.s : x.s;
            }
        } else {
            st = seg_apply<DOM>(st, pre);
        }
    }

    p.tl.mark(tile, 5);
    // ---- every element ----------------------------------------------------------------------------
    constexpr int OW = (SIGNED && LOG_OUT) ? 2 : 1; // floats per output element
    float *op = p.out + OW * ubase;
    const bool full = chan_ok && t0 + T <= p.n;
    const uint32_t swx = fold_state_sign<DOM>(sw, st);
    auto emit_store = [&](int k, bool wanted) {
        if constexpr (SIGNED && LOG_OUT) {
            // complex output: (re, im) pairs, two floats per element
            float re, im;
            emit_clog(st, Av[k], Mv[k], swx, sm, k, re, im);
            if (wanted) store_pair<MEM>(op + 2 * ((int64_t)k * p.D + moff), re, im);
        } else {
            const float o = emit<DOM, LOG_OUT>(st, Av[k], Mv[k], swx, k);
            // the last steps of runs, in pieces of D: lines are put together in the L2
            if (wanted) store_elem<RUNS && MEM == kThrough ? kKeepOut : MEM>(op + (int64_t)k * p.D + moff, o);
        }
    };
    if (RUNS && whole) {
        constexpr int NV = T / 4 / ROUNDS, TR = T / ROUNDS;
        const uint32_t per = (uint32_t)(TR / 4) * D32, all = run_n * per, inv = run_inverse(per);
        const uint32_t to_next = (uint32_t)(p.n * p.D);
        float *mine = reinterpret_cast<float *>(&lds_runs[w][run_item * pitch_out]) + run_ch;
        __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0), as below
#pragma unroll
        for (int h = 0; h < ROUNDS; ++h) {
            if (chan_ok) {
#pragma unroll
                for (int k = 0; k < TR; ++k) mine[(uint32_t)k * D32] = emit<DOM, LOG_OUT>(st, Av[h * TR + k], Mv[h * TR + k], swx, h * TR + k);
            }
            wave_lds_order();
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const uint32_t g = (uint32_t)(j * 64 + lane);
                const RunAt r2 = run_at(g, per, inv);
                if (g < all) {
                    const u32x4 o = lds_runs[w][r2.item * pitch_out + r2.v];
                    store_run<MEM>(op, r2.item * to_next + ((uint32_t)h * per + r2.v) * 4, o);
                }
            }
            wave_lds_order();
        }
    } else if (full) {
        float *orow = op; // wave-uniform row pointer
#pragma unroll
        for (int k = 0; k < T; ++k) {
            if constexpr (SIGNED && LOG_OUT) {
                float re, im;
                emit_clog(st, Av[k], Mv[k], swx, sm, k, re, im);
                store_pair<MEM>(orow + 2 * (size_t)moff, re, im);
            } else {
                store_elem<MEM>(orow + moff, emit<DOM, LOG_OUT>(st, Av[k], Mv[k], swx, k));
            }
            orow += OW * p.D;
            if (SB) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // Every store below is a block of its own, and the compiler, which cannot tell there whether a record it did not
        // need is still on its way, would wait in each for all that is, the store before it included (1 x 3000 x
        // 512: 15.3 us, 13.7 with one wait here).
        __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0)
#pragma unroll
        for (int k = 0; k < T; ++k) {
            emit_store(k, chan_ok && t0 + k < p.n);
            if (SB) __builtin_amdgcn_sched_barrier(0);
        }
    }
    p.tl.mark(tile, 6);
}

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT, int T, int NW, int G, int MINW, bool SB, bool DENSE, bool TREE, bool RUNS, int CG, int MEM>
__global__ __launch_bounds__(NW * 64, MINW) void heinsen_scan_bnd(BndParams p)
{
    __shared__ uint32_t s_tile, s_epoch, s_flag;
    constexpr int NFLAGS = NW + CG + (TREE ? 2 * G + 2 * G / kTreeBlock + 3 : 0);
    __shared__ uint32_t s_flags[NFLAGS];
    const unsigned long long t_begin = p.tl.stamps != nullptr ? wall_clock64() : 0ull;
    uint32_t tile, epoch = 0u;
    if (threadIdx.x < NFLAGS) s_flags[threadIdx.x] = 0u;
    if (p.header == nullptr) {
        // A launch whose columns are one short tile long (at most 64 steps) has nothing to wait for and
        // comes without tickets: there the draw's round trip would be a large part of a tile's life.
        // Workgroups go to the eight compute dies in turn (workgroup i to die i mod 8): give every die a
        // contiguous eighth of the tiles, so that the tiles in flight form eight compact windows of memory
        // instead of a wide, ragged one.
        const uint32_t die = blockIdx.x & 7u, j = blockIdx.x >> 3;
        const uint32_t qn = p.ntiles >> 3, rem = p.ntiles & 7u;
        tile = die * qn + (die < rem ? die : rem) + j;
    } else {
        // Tiles are handed out in start order, so every tile a workgroup may wait for (same column,
        // earlier chunk => same queue, smaller ticket) belongs to a workgroup that is already running.
        if (threadIdx.x == 0) {
            const int qi = (int)(blockIdx.x % (uint32_t)p.nq);
            const Draw d = draw_ticket(p.header, qi, p.draws_per_q, p.nq);
            int cols = p.ncols - qi * p.cols_per_q; // columns of this queue
            cols = cols > p.cols_per_q ? p.cols_per_q : cols;
            uint32_t t = 0xffffffffu;
            if (cols > 0) {
                const uint32_t chunk = d.ticket / (uint32_t)cols, cq = d.ticket % (uint32_t)cols;
                if (chunk < (uint32_t)p.nchunks) t = chunk * (uint32_t)p.ncols + (uint32_t)(qi * p.cols_per_q) + cq;
            }
            s_tile = t;
            s_epoch = d.epoch;
        }
    }
    __syncthreads(); // the only barrier of a tile: ticket and cleared flags are in LDS
    if (p.header != nullptr) {
        tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_tile);
        epoch = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_epoch);
    }
    if (tile < p.ntiles) {
        p.tl.mark_at(tile, 0, t_begin);
        p.tl.mark(tile, 1);
        bnd_tile<DOM, LOG_IN, LOG_OUT, InT, T, NW, G, SB, DENSE, TREE, RUNS, CG, MEM>(p, tile, epoch, (lds_flag_t *)s_flags);
        p.tl.mark(tile, 7);
    }
    if (p.header != nullptr) end_of_workgroup(p.header, epoch, &s_flag);
}

// ---- a few steps of many channels ---------------------------------------------------------------------
//
// A model that generates one token after the other calls the scan with a handful of steps.  Such a call is
// bound by how fast the chip starts waves: as a tile of 32 steps with the others masked, one step of 64 x 4096
// channels took 4096 waves and 7.2 us for 4 MB (a first call 22.9 us from call to result, 19.7 now).  Here a thread takes VEC adjacent channels (16 bytes of
// float32 per access), asks for all of their steps at once and evaluates the definition (Sec. 3), x_t =
// a_t x_{t-1} + b_t, in float64, so that as in the log domain no state on the way leaves the range: eight
// float32 factors stay within 2^1024.  Subnormal float32 counts as 0, in and out.
struct StepsParams {
    const void *a;
    const void *b;
    const float *x0;
    float *out;
    uint32_t nchan, D; // B * D; the host checks that it fits
    int n;
    int x0_stride;
};
constexpr int kMaxSteps = 8;

__device__ __forceinline__ float flush_subnormal(float v) { return fabsf(v) < 0x1p-126f ? 0.0f : v; }

template <typename InT, int VEC>
__global__ __launch_bounds__(256) void heinsen_scan_steps(StepsParams p)
{
    typedef InT in_t __attribute__((ext_vector_type(VEC)));
    typedef float out_t __attribute__((ext_vector_type(VEC)));
    const uint32_t chan = (blockIdx.x * 256u + threadIdx.x) * (uint32_t)VEC;
    if (chan >= p.nchan) return;
    const uint32_t b = chan / p.D, d = chan - b * p.D; // VEC divides D: the channels are of one batch item
    const int64_t base = (int64_t)b * p.n * p.D + d;
    in_t av[kMaxSteps], bv[kMaxSteps];
#pragma unroll
    for (int t = 0; t < kMaxSteps; ++t) {
        if (t < p.n) { // wave-uniform
            const int64_t at = base + (int64_t)t * p.D;
            av[t] = __builtin_nontemporal_load(reinterpret_cast<const in_t *>(reinterpret_cast<const InT *>(p.a) + at));
            bv[t] = __builtin_nontemporal_load(reinterpret_cast<const in_t *>(reinterpret_cast<const InT *>(p.b) + at));
        }
    }
    double x[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) x[i] = (double)flush_subnormal(p.x0[p.x0_stride ? chan + i : 0]);
#pragma unroll
    for (int t = 0; t < kMaxSteps; ++t) {
        if (t < p.n) {
            out_t o;
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                x[i] = fma((double)flush_subnormal(widen(av[t][i])), x[i], (double)flush_subnormal(widen(bv[t][i])));
                o[i] = flush_subnormal((float)x[i]);
            }
            *reinterpret_cast<out_t *>(p.out + base + (int64_t)t * p.D) = o;
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------

struct BndPlan {
    int cg, T, NW, G, CH;
    bool ticketless;
    bool dense;          // columns of adjacent channels of all B * D (see bnd_tile),
    int lanes;           // this many
    int pad;             // lanes an item takes: D, or the power of two at or above it
    bool runs;           // whole runs of memory (D < 32, see bnd_tile)
    int pitch_in, pitch_out;
    int cols_per_b, ncols, nchunks, ngroups;
    uint32_t ntiles;
    int nq, cols_per_q;
    uint32_t grid;
    bool tree;          // second carry level, the waves of a tile share the record loads
    size_t off_agg, off_state, records; // in records, relative to kRecordBase
};

// TREE, tiles of eight waves: tiles per group and groups per super-group, and the number of columns below which it is used.
// Without it a link of the chain of group states takes 1.2-1.4 us and a group of four tiles is 786 KB per
// column, 0.12 us of memory traffic: up to about 12 columns the chain is the slower of the two.  Measured with
// and without, summaries folded one by one: 3 columns of 131072 steps 75 and 176 us (tall tiles, which they take, 66), 1 of 400000
// 109 and 479 (in block sums 77), 16 of 131072 283 and 279, 32 of 32768 147 and 144 (the record loads).
constexpr int kTreeGroup = 8;
constexpr int kTreeBelow = 16;
// Tall tiles (see tall_tiles): sixteen waves one after the other along time, and as many tiles per group and groups per
// super-group.
constexpr int kTallWaves = 16;

// Workgroups of eight waves that the chip holds at a time.
constexpr int kPlaces = 512;

// Channels that do not fill 64 lanes per batch item (D > 32): columns of 64 channels of whatever items?  Where
// that saves a sixteenth of the columns, and
//   - D is a multiple of 16: pieces of rows begin on 64 bytes (2 x 131072 x 96: three columns instead of four); or
//   - the sequence is one tile, with logarithms, or with an eighth of the columns saved (3226 x 20 x 65: 13.7 us,
//     with columns of their own 18.1; 139 x 100 x 301, a twentieth saved: 14.5 and 13.8); or
//   - the tiles take fewer rounds of the chip, with logarithms (215 x 300 x 65 complex: 25 and 41), or, where memory is
//     what bounds them, from three rounds on and with a fifth of the columns saved (860 x 300 x 65: 50 and 68 us).
// Otherwise fewer tiles only mean fewer loads in flight (63 x 2000 x 33: 24.9 us, 18.9 with columns of their own).
bool columns_across_items(const ScanCall &c, int64_t own, int64_t shared, int64_t steps, int waves)
{
    if (shared + shared / 16 >= own) return false;
    if (c.D % 16 == 0) return true;
    const bool logs = c.log_in || c.log_out;
    if (c.n <= 128) return logs || 8 * shared <= 7 * own;
    const int64_t chunks = ceil_div(c.n, steps), places = waves > 8 ? kPlaces / 2 : kPlaces;
    return ceil_div(shared * chunks, places) < ceil_div(own * chunks, places) && (logs || (own * chunks > 2 * places && 5 * shared <= 4 * own));
}

// RUNS: distance, in 16-byte slots, from one item's run to the next in LDS, for D channels per item whose runs are
// `vectors` slots.  The lanes pick up words 4 * i * pitch + d of items i and channels d at once (bf16: half-words): the
// pitch is the smallest of those that put fewest of them on one of the 64 banks.
constexpr int run_pitch(int D, bool halves, int vectors, int slots)
{
    const int items = 64 / D, words = halves ? (D + 1) / 2 : D;
    int best = vectors, fewest = 1 << 30;
    for (int pitch = vectors; pitch < vectors + 16 && items * pitch <= slots; ++pitch) {
        int on[64] = {}, most = 0;
        for (int i = 0; i < items; ++i)
            for (int d = 0; d < words; ++d) {
                const int n = ++on[(4 * i * pitch + d) % 64];
                most = n > most ? n : most;
            }
        if (most < fewest) {
            fewest = most;
            best = pitch;
        }
    }
    return best;
}
struct RunPitches {
    int of[2][2][33] = {}; // [float32, bf16][whole runs, halves of them][D]
    constexpr RunPitches()
    {
        for (int D = 2; D <= 32; ++D)
            for (int h = 0; h < 2; ++h) {
                const int slots = run_slots(1 + h);
                of[0][h][D] = run_pitch(D, false, 8 * D >> h, slots);
                of[1][h][D] = run_pitch(D, true, 4 * D >> h, slots);
            }
    }
};
constexpr RunPitches kRunPitches;

BndPlan make_plan(const ScanCall &c, bool allow_wide = true, bool want_tree = false)
{
    BndPlan pl = {};
    // Default tile: 64 channels x 256 steps (8 waves one after the other along time, 32 steps each;
    // <= 128 VGPRs, two workgroups per CU).  With many wide rows the tile is 128 channels x 128 steps
    // instead (two waves side by side): the rows a workgroup touches are then 512 contiguous bytes, which
    // the memory system serves about 4 % faster, at the price of twice as many tiles along time.
    pl.cg = 1;
    pl.T = 32;
    pl.NW = 8;
    pl.G = 4;
    const bool complex_out = c.is_signed && c.log_out;
    if (complex_out) {
        // complex output: the signed log-domain emit needs more registers per element; 16 steps per wave
        // and 16 waves keep the tile the same and the kernel free of spills
        pl.T = 16;
        pl.NW = 16;
    } else if (c.n <= 128) {
        // short sequences: no more waves than have steps to work on
        pl.NW = c.n <= 32 ? 1 : (c.n <= 64 ? 2 : 4);

    } else if (allow_wide && c.D % 128 == 0 && c.B * (c.D / 128) >= 2 * kMinColsPerQueueWide && c.n >= 1024) {
        pl.cg = 2;
    }
    pl.CH = 64 * pl.cg;
    pl.cols_per_b = (int)ceil_div(c.D, pl.CH);
    pl.ncols = (int)(c.B * pl.cols_per_b);

    // Channels that do not fill their columns.  Up to 32 per batch item: a column takes as many whole items as lanes
    // of the next power of two fit.  (Items cut by the ends of columns read the lines at the cut twice: 256 x 4096 x 19
    // 85 us, whole items 76.)  Each begins on such a lane: without lanes between them 419 x 2000 x 5 takes 41 us
    // instead of 36.  Two carry levels, where few tiles are waited for rather than memory, go without them.  More
    // channels: see columns_across_items.  A lane's offset from its column's base -- it may lie some items further on
    // -- has to fit 31 bits.
    pl.lanes = 64;
    pl.pad = 64;
    int64_t pad = c.D;
    if (pl.cg == 1) {
        if (c.D <= 32)
            for (pad = 2; pad < c.D;) pad *= 2;
        const int64_t items = c.D <= 32 ? 64 / pad : 1, cols = ceil_div(c.B * pad, 64), further = c.D <= 32 ? items - 1 : (c.D + 62) / c.D;
        pl.dense = (c.D <= 32 ? cols < pl.ncols : columns_across_items(c, pl.ncols, cols, (int64_t)pl.NW * pl.T, pl.NW)) && c.B * pad < ((int64_t)1 << 31) &&
                   further * c.n * c.D + c.D < ((int64_t)1 << 31);
        if (pl.dense) {
            if (c.D <= 32) pl.lanes = (int)(items * c.D);
            pl.ncols = (int)cols;
        }
    }
    // Fewer than 32 channels move as whole runs.  (The pieces of 32 are lines or halves of lines as they are: 24 x 16384 x
    // 32 40.5 us, as runs 43.)  An item's place in a column need not begin anywhere in particular then, and a column
    // may take as many items as lanes hold instead of as many of the next power of two.  That pays where it saves a
    // quarter of the columns of a launch that does not fit the chip: 719 x 3461 x 9 bf16 58 and 49 us, 544 x 1294 x 19 41.2
    // and 36.9; a launch that fits waits less in shorter columns (300 x 700 x 20 16.6 and 17.4), and from four rounds of
    // tiles on float32 is bound by memory either way (256 x 4096 x 19 55.8 and 55.5).
    pl.runs = c.D < 32 && pl.cg == 1 && pl.NW == 8 && pl.T == 32;
    if (pl.runs) {
        for (pad = 2; pad < c.D;) pad *= 2;
        int64_t items = std::min(64 / pad, c.B);
        const int64_t own = ceil_div(c.B, items), close = ceil_div(c.B, 64 / c.D), tiles = own * ceil_div(c.n, (int64_t)pl.NW * pl.T);
        if (4 * close <= 3 * own && tiles > kPlaces && (c.bf16 || tiles < 4 * kPlaces)) items = 64 / c.D;
        pl.runs = items * c.n * c.D < ((int64_t)1 << 31) && ceil_div(c.B, items) * items * c.D < ((int64_t)1 << 31);
        if (pl.runs) {
            pl.dense = true;
            pl.lanes = (int)(items * c.D);
            pl.ncols = (int)ceil_div(c.B, items);
        }
    }
    const bool tiles8 = pl.cg == 1 && pl.NW == 8 && pl.T == 32 && c.n > 4 * pl.NW * pl.T;
    pl.tree = tiles8 && (pl.ncols < kTreeBelow || want_tree);
    if (pl.tree) pl.G = kTreeGroup;
    if (tiles8 && !c.linear && tall_tiles(pl.ncols, ceil_div(c.n, (int64_t)pl.NW * pl.T), c.D, pl.runs, c.bf16, kQueues)) {
        pl.tree = true;
        pl.NW = pl.G = kTallWaves;
    }
    if (pl.dense) pl.pad = (int)(pl.tree || pl.runs ? c.D : pad);
    if (pl.runs) {
        pl.pitch_out = kRunPitches.of[0][run_rounds(pl.G) - 1][c.D];
        pl.pitch_in = kRunPitches.of[c.bf16][run_rounds(pl.G) - 1][c.D];
    }
    pl.nchunks = (int)ceil_div(c.n, (int64_t)(pl.NW / pl.cg) * pl.T);
    pl.ngroups = (int)ceil_div(pl.nchunks, pl.G);
    pl.ntiles = (uint32_t)pl.ncols * (uint32_t)pl.nchunks;
    pl.off_agg = 0;
    pl.off_state = (size_t)pl.ntiles * 2 * pl.CH;
    pl.records = pl.off_state + (size_t)pl.ngroups * pl.ncols * 2 * pl.CH;
    pl.ticketless = pl.nchunks == 1 && c.n <= 64; // short single-tile columns: no records, no tickets
    // A queue's workgroups that find no tile behind their ticket (uneven deal) end at once.
    pl.nq = ticket_queues(kQueues, pl.ncols, pl.cg > 1);
    // Eight queues of fewer than 16 columns are for lines that columns share and for short sequences.  Long ones
    // wait for their predecessors less in four (80 columns of 16384 steps: 169 and 174 us), and an uneven deal may be
    // what makes a launch that fits the chip take a second round on one die (100 columns of 1100 steps, bf16: 18.3 and
    // 21.9 us).
    if (pl.cg == 1 && pl.nq == kQueues && pl.ncols < 2 * kMinColsPerQueue * kQueues && c.D * (c.bf16 ? 2 : 4) % 128 == 0 &&
        (c.n >= 4096 || (pl.ntiles <= (uint32_t)kPlaces && ceil_div(pl.ncols, kQueues) * pl.nchunks > kPlaces / kQueues)))
        pl.nq /= 2;
    pl.cols_per_q = (int)ceil_div(pl.ncols, pl.nq);
    pl.grid = pl.ntiles;
    if (pl.ticketless) {
        pl.records = 0;
    } else {
        pl.grid = (uint32_t)pl.nq * (uint32_t)pl.cols_per_q * (uint32_t)pl.nchunks;
    }
    // A caller with a fixed scratch buffer may have to do without the wide tiles, which take twice the records,
    // and with the second carry level, whose groups are longer.
    if (c.scratch_budget != 0 && kRecordBase + pl.records > c.scratch_budget) {
        if (pl.cg > 1) return make_plan(c, false);
        if (!want_tree && pl.ncols < 64) {
            const BndPlan t = make_plan(c, false, true);
            if (t.tree) return t;
        }
    }
    return pl;
}

template <int DOM, bool LOG_IN, bool LOG_OUT, typename InT>
hipError_t launch_mode(const ScanCall &c, const BndPlan &pl, const LaunchCtx &ctx)
{
    constexpr bool SIGNED = DOM == kSigned;
    rec_t *records = pl.ticketless ? nullptr : ctx.scratch;
    BndParams p;
    p.a = c.a;
    p.b = c.b;
    p.x0 = c.x0;
    p.out = c.out;
    p.D = c.D;
    p.n = c.n;
    p.x0_stride = c.x0_scalar ? 0 : 1;
    // see Mem.  kShared where it wins however the caller goes through its buffers.  float32, more than 32 channels: in
    // place of kStream only, since kKeepOut finds lines of the last calls' outputs in the memory-side cache as long as
    // few sets of buffers take turns (8 x 3001 x 1111, 320 MB a call: kKeepOut 70 us over two sets, 76 over three, 78
    // over five, kShared 78, 79, 78; 8 x 8000 x 1501, 1.2 GB: kStream 658, kShared 490).  bf16, whose pieces of 64 channels
    // are one line long and touch two: from the size of that cache on (16 x 8192 x 301, 316 MB: kKeepOut 84 us over one
    // set, 97 over two, 109 over five, kShared 77, 83, 84).  Items narrower than half a column, whose lines successive
    // steps of one wave share as well: likewise (256 x 4096 x 19, 239 MB: 75 over one set and over five, kShared 53 and 69).
    const int64_t elements = c.B * c.D * c.n;
    const int64_t out_bytes = elements * ((SIGNED && LOG_OUT) ? 8 : 4);
    const bool large_out = out_bytes > kLastLevelCacheBytes;
    const int64_t bytes = out_bytes + 2 * elements * (int64_t)sizeof(InT);
    const bool shares_lines = c.D * (int64_t)sizeof(InT) % 128 != 0 &&
                              (c.D <= 32 ? bytes > kLastLevelCacheBytes : (c.bf16 ? bytes > kLastLevelCacheBytes * 3 / 2 : large_out));
    // Lines that a wave writes whole gain nothing from waiting in the L2: written through, 8 x 4096 x 1024 takes 77.8 us
    // instead of 79.1, 32 x 1024 x 1024 76.1 and 80.2, 16 x 1024 x 256 12.0 and 13.9, runs (256 x 4096 x 16) 45.3 and 47.9,
    // and a kernel that reads the output next is no slower (out = a + b in these pieces and a pass over out, 8 x 4096
    // x 1024: 96 us, 99.6 with ordinary stores, 102 past the caches).  Lines that columns share do (6 x 3001 x 770: 48.7
    // and 45.4, 9 x 20000 x 48 39.1 and 38.4).  (Runs: see runs_in_lines.)
    const bool on_line = reinterpret_cast<uintptr_t>(c.out) % 128 == 0;
    const bool whole_lines = pl.runs ? runs_in_lines(on_line, c.B, c.n * c.D, bytes) : on_line && c.D % 32 == 0;
    const bool through = whole_lines && !waits_behind_stores(pl.NW, pl.ncols, pl.nchunks, pl.tree, c.linear, pl.runs);
    const int mem = shares_lines && !pl.runs ? kShared : (large_out ? kStream : (through ? kThrough : kKeepOut));
    p.cols_per_b = pl.cols_per_b;
    p.pad = pl.runs ? (uint32_t)(pl.pitch_in | pl.pitch_out << 16) : (uint32_t)pl.pad;
    p.places = c.B * pl.pad;
    p.lanes = pl.lanes;
    p.ncols = pl.ncols;
    p.nchunks = pl.nchunks;
    p.ntiles = pl.ntiles;
    p.nq = pl.nq;
    p.cols_per_q = pl.cols_per_q;
    p.draws_per_q = pl.grid / (uint32_t)pl.nq;
    p.header = records; // null when the launch needs no carries
    p.agg = records ? records + kRecordBase + pl.off_agg : nullptr;
    p.state = records ? records + kRecordBase + pl.off_state : nullptr;
    p.spin_limit = ctx.spin_limit;
    p.drop_tile = ctx.drop_tile;
    p.tl.stamps = ctx.timeline;
    p.tl.tiles = ctx.timeline_tiles;
    if (!pl.ticketless && records == nullptr) return hipErrorInvalidValue;
    // The plan's shape and the kernel's must be the same one: a wave that is not there would be waited for.
#define HS_BND(T_, NW_, G_, DENSE_, TREE_, RUNS_, CG_, MEM_)                                                              \
    do {                                                                                                           \
        if (pl.T != T_ || pl.NW != NW_ || pl.G != G_ || pl.cg != CG_ || pl.tree != TREE_ || pl.dense != DENSE_ || pl.runs != RUNS_) \
            return hipErrorInvalidValue;                                                                           \
        hipLaunchKernelGGL((heinsen_scan_bnd<DOM, LOG_IN, LOG_OUT, InT, T_, NW_, G_, 4, true, DENSE_, TREE_, RUNS_, CG_, MEM_>), \
                           dim3(pl.grid), dim3(NW_ * 64), 0, c.stream, p);                                         \
    } while (0)
#define HS_BND_SHORT(NW_, DENSE_)                                             \
    do {                                                                      \
        if (mem == kThrough) HS_BND(32, NW_, 4, DENSE_, false, false, 1, kThrough); \
        else HS_BND(32, NW_, 4, DENSE_, false, false, 1, kKeepOut);           \
    } while (0)
#define HS_BND_MEM(T_, NW_, G_, DENSE_, TREE_)                                \
    do {                                                                      \
        if (mem == kShared) HS_BND(T_, NW_, G_, DENSE_, TREE_, false, 1, kShared);      \
        else if (mem == kThrough) HS_BND(T_, NW_, G_, DENSE_, TREE_, false, 1, kThrough);      \
        else if (mem == kStream) HS_BND(T_, NW_, G_, DENSE_, TREE_, false, 1, kStream); \
        else HS_BND(T_, NW_, G_, DENSE_, TREE_, false, 1, kKeepOut);                    \
    } while (0)
#define HS_BND_RUNS(T_, NW_, G_, TREE_)                                       \
    do {                                                                      \
        if constexpr (T_ == 32) {                                             \
            if (mem == kStream) HS_BND(T_, NW_, G_, true, TREE_, true, 1, kStream); \
            else if (mem == kThrough) HS_BND(T_, NW_, G_, true, TREE_, true, 1, kThrough); \
            else HS_BND(T_, NW_, G_, true, TREE_, true, 1, kKeepOut);         \
        }                                                                     \
    } while (0)
#define HS_BND_ANY(T_, NW_, G_, TREE_)                     \
    do {                                                   \
        if (pl.runs) HS_BND_RUNS(T_, NW_, G_, TREE_);         \
        else if (pl.dense) HS_BND_MEM(T_, NW_, G_, true, TREE_); \
        else HS_BND_MEM(T_, NW_, G_, false, TREE_);           \
    } while (0)
    if constexpr (SIGNED && LOG_OUT) {
        HS_BND_ANY(16, 16, 4, false);
    } else if (pl.cg == 2) {
        if (mem == kStream) HS_BND(32, 8, 4, false, false, false, 2, kStream);
        else if (mem == kThrough) HS_BND(32, 8, 4, false, false, false, 2, kThrough);
        else HS_BND(32, 8, 4, false, false, false, 2, kKeepOut);
    } else if (pl.tree && pl.NW == kTallWaves) {
        if constexpr (DOM != kLinear) HS_BND_ANY(32, kTallWaves, kTallWaves, true);
        else return hipErrorInvalidValue;
    } else if (pl.tree) {
        HS_BND_ANY(32, 8, kTreeGroup, true);
    } else if (pl.NW == 8) {
        HS_BND_ANY(32, 8, 4, false);
    } else if (pl.dense) { // short sequences
        if (pl.NW == 1) HS_BND_SHORT(1, true);
        else if (pl.NW == 2) HS_BND_SHORT(2, true);
        else HS_BND_SHORT(4, true);
    } else {
        if (pl.NW == 1) HS_BND_SHORT(1, false);
        else if (pl.NW == 2) HS_BND_SHORT(2, false);
        else HS_BND_SHORT(4, false);
    }
#undef HS_BND_ANY
#undef HS_BND_RUNS
#undef HS_BND_SHORT
#undef HS_BND_MEM
#undef HS_BND
    return hipGetLastError();
}

// Plain numbers in and out, at most kMaxSteps of them per channel.  (Logarithms keep to the log domain.)  Large
// calls of a few channels for more than four steps are left to the tiles, which read such pieces of lines in fewer
// instructions (2796202 x 8 x 3 bf16: 410 us here, 364 as tiles; 43690 x 8 x 3 5.1 and 7.8).
bool is_steps(const ScanCall &c)
{
    return !c.linear && !c.log_in && !c.log_out && c.n <= kMaxSteps && (c.n <= 4 || c.D >= 8 || c.B * c.D * c.n < (1ll << 25)) && c.B * c.D < ((int64_t)1 << 31);
}

template <typename InT>
hipError_t launch_steps(const ScanCall &c)
{
    const StepsParams p{c.a, c.b, c.x0, c.out, (uint32_t)(c.B * c.D), (uint32_t)c.D, (int)c.n, c.x0_scalar ? 0 : 1};
    auto on = [](const void *ptr, size_t bytes) { return reinterpret_cast<uintptr_t>(ptr) % bytes == 0; };
    const bool vec = c.D % 4 == 0 && on(c.a, 4 * sizeof(InT)) && on(c.b, 4 * sizeof(InT)) && on(c.out, 16);
    const dim3 grid((unsigned)ceil_div(c.B * c.D, vec ? 1024 : 256)), block(256);
    if (vec) hipLaunchKernelGGL((heinsen_scan_steps<InT, 4>), grid, block, 0, c.stream, p);
    else hipLaunchKernelGGL((heinsen_scan_steps<InT, 1>), grid, block, 0, c.stream, p);
    return hipGetLastError();
}

hipError_t launch_dispatch(const ScanCall &c, const BndPlan &pl, const LaunchCtx &ctx)
{
    HS_DISPATCH_MODE(c, launch_mode, c, pl, ctx);
}

} // namespace

ScratchNeed bnd_scratch(const ScanCall &c)
{
    if (is_steps(c)) return ScratchNeed{0};
    BndPlan pl = make_plan(c);
    return ScratchNeed{pl.records};
}

hipError_t bnd_launch(const ScanCall &c, const LaunchCtx &ctx)
{
    if (is_steps(c)) return c.bf16 ? launch_steps<uint16_t>(c) : launch_steps<float>(c);
    BndPlan pl = make_plan(c);
    return launch_dispatch(c, pl, ctx);
}

const char *bnd_kernel_name(const ScanCall &c) { return is_steps(c) ? "heinsen_scan_steps" : "heinsen_scan_bnd"; }

void bnd_tile_shape(const ScanCall &c, int &channels, int64_t &steps)
{
    if (is_steps(c)) {
        channels = c.D % 4 == 0 ? 1024 : 256;
        steps = c.n;
        return;
    }
    const BndPlan pl = make_plan(c);
    channels = pl.dense && pl.lanes > c.D ? pl.lanes : pl.CH; // (an item alone in its column has it to itself)
    steps = (int64_t)(pl.NW / pl.cg) * pl.T;
}

} // namespace hs
