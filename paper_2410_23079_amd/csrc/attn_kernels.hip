// Decode attention over the retained BUZZ cache (eq. 3 / eq. 5 of the paper) as ONE kernel per step:
// the append of eq. 2, the split-softmax attention, the merge of the splits and the accumulated-score
// update ("A" of Alg. 2) all happen inside attn_split.
//
//  - One block per (key-range split, unit).  Two streaming variants: on the vector ALU a wave reads
//    64 x 16 B per load instruction = RPW consecutive cache rows, LPR = 64 / RPW lanes per row (every
//    load is one contiguous 1 KB burst), q.k is a two-element-dot chain per lane plus an LPR-lane DPP
//    reduction, softmax runs online per lane group and p.V accumulates in registers; with several
//    query heads per kv head on a 16-bit cache both contractions run on the matrix cores instead.
//  - The scaled logit of every row is written to a scratch array.  A row's probability needs the
//    maximum and sum over ALL splits, which only exist once the step is over, so the score update of
//    step t is applied by step t+1 while it streams the same rows anyway (one lane per row, coalesced):
//    score += sum_g exp2(logit_t - M_t[g]) / L_t[g].  flush_scores applies a pending update to every row
//    right away (before an export, or an eviction that moves old rows); the usual eviction applies it only to
//    the rows it ranks and leaves the rest pending.
//  - The block that finishes last for a unit (atomic ticket, nobody waits) merges the split partials
//    into the attention output and publishes (M, 1/L) for the next step's score update.
#include <stddef.h>
#include <algorithm>
#include <type_traits>

#include "buzz_internal.h"

namespace buzz {
namespace {

struct bf16_t { uint16_t x; };
struct fp16_t { uint16_t x; };

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Build-time tuning knobs (defaults are the measured best; a sweep overrides them with -D).
// 16-byte loads of K (and of V) per lane and tile.  Group size 1 keeps two tiles in flight; small tiles win
// there because the waves claim them dynamically (finer balance): 2 loads when the cache streams from HBM
// (4: -2%, 1: -9%, too little in flight), 1 load when it is served by the last-level cache (+3.5% over 2).
#ifndef BUZZ_U_G1
#define BUZZ_U_G1 2
#endif
#ifndef BUZZ_U_G1_CACHED
#define BUZZ_U_G1_CACHED 1
#endif
#ifndef BUZZ_U_G2
#define BUZZ_U_G2 4
#endif
#ifndef BUZZ_U_G4
#define BUZZ_U_G4 4
#endif
#ifndef BUZZ_U_G8
#define BUZZ_U_G8 2
#endif
#ifndef BUZZ_MIN_BLOCKS
#define BUZZ_MIN_BLOCKS 1  // second argument of __launch_bounds__
#endif

// Optional in-kernel time stamps (a tuning aid, compiled out unless BUZZ_TRACE is defined): slot s of
// block b holds the wall clock (100 MHz) at which the block passed point s of the last launch.
#if defined(BUZZ_TRACE) && BUZZ_TU == 2
__device__ unsigned long long g_trace[kMaxBlocks * 16];
#define BUZZ_STAMP(slot) do { g_trace[(size_t)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 16 + (slot)] = wall_clock64(); } while (0)
#define BUZZ_STAMP_VALUE(slot, v) do { g_trace[(size_t)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 16 + (slot)] = (v); } while (0)
#else
#define BUZZ_STAMP(slot) do { } while (0)
#define BUZZ_STAMP_VALUE(slot, v) do { } while (0)
#endif

template <typename T> struct Elem;
// cvt: 16 bytes -> VEC floats.  dot: sum over the 16 bytes of q * k in fp32 (16-bit types use the
// two-element dot instruction on the raw words: exact products, fp32 accumulation, no conversion).
template <> struct Elem<float> {
    [[maybe_unused]] static constexpr int VEC = 4;
    static __device__ inline void cvt(const u32x4& r, float* f) {
        f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
        f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
    }
    static __device__ inline float dot(const u32x4& q, const u32x4& k) {
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) d = fmaf(__uint_as_float(q[i]), __uint_as_float(k[i]), d);
        return d;
    }
};
template <> struct Elem<bf16_t> {
    [[maybe_unused]] static constexpr int VEC = 8;
    static __device__ inline void cvt(const u32x4& r, float* f) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(r[i] << 16);
            f[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
        }
    }
    static __device__ inline float dot(const u32x4& q, const u32x4& k) {
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, (unsigned int)q[i]),
                                                __builtin_bit_cast(bf16x2_t, (unsigned int)k[i]), d, false);
        return d;
    }
};
template <> struct Elem<fp16_t> {
    [[maybe_unused]] static constexpr int VEC = 8;
    static __device__ inline void cvt(const u32x4& r, float* f) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const half2_t h = __builtin_bit_cast(half2_t, (unsigned int)r[i]);
            f[2 * i] = (float)h.x;
            f[2 * i + 1] = (float)h.y;
        }
    }
    static __device__ inline float dot(const u32x4& q, const u32x4& k) {
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            d = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, (unsigned int)q[i]),
                                       __builtin_bit_cast(half2_t, (unsigned int)k[i]), d, false);
        return d;
    }
};

// NT: streaming hint for data that will not be re-read before it would be evicted anyway
template <bool NT> __device__ inline u32x4 load16(const char* p) {
    if constexpr (NT) return __builtin_nontemporal_load((const u32x4*)p);
    else return *(const u32x4*)p;
}

template <int CTRL> __device__ inline float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// The two values that lanes l and l ^ 16 (32) hold, in both of them: `a` the one of the lane with that bit clear.
struct LanePair { float a, b; };
template <int BIT> __device__ inline LanePair lane_pair(float v)
{
    static_assert(BIT == 16 || BIT == 32, "rows of 16 lanes or halves of a wave");
    const unsigned x = __builtin_bit_cast(unsigned, v);
    if constexpr (BIT == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return {__uint_as_float(r[0]), __uint_as_float(r[1])};
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return {__uint_as_float(r[0]), __uint_as_float(r[1])};
    }
}
template <int BIT> __device__ inline float pair_sum(float v) { const LanePair p = lane_pair<BIT>(v); return p.a + p.b; }
template <int BIT> __device__ inline float pair_max(float v) { const LanePair p = lane_pair<BIT>(v); return fmaxf(p.a, p.b); }

// Sum over the LPR consecutive lanes that share a cache row; every lane of the group gets the total.  VIA_LDS: rows of 16 lanes
// exchange through LDS, which paces the loop (see launch_split_t).
template <int LPR, bool VIA_LDS> __device__ inline float row_sum(float v) {
    v += dpp_move<0xB1>(v);                 // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);                 // quad_perm [2,3,0,1]
    if constexpr (LPR >= 8) v += dpp_move<0x141>(v);  // row_half_mirror
    if constexpr (LPR >= 16) v += dpp_move<0x140>(v); // row_mirror
    if constexpr (LPR >= 32) v = VIA_LDS ? v + __shfl_xor(v, 16) : pair_sum<16>(v);
    if constexpr (LPR >= 64) v = VIA_LDS ? v + __shfl_xor(v, 32) : pair_sum<32>(v);
    return v;
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// How split partials travel between the blocks of one launch (finish_split).
//
// Device-wide form (blocks of a unit possibly on different dies, each die with its own L2).  A block writes
// its partial with relaxed device-scope atomic stores (`sc1`: written through the die's L2 to the memory
// side), every wave waits with s_waitcnt vmcnt(0) for its own stores, the block synchronises, one thread takes
// a ticket (relaxed atomic add), and the block that draws the last ticket reads every partial with relaxed
// device-scope atomic loads (`sc1`: not served from a die's private copy).  Why the merging block cannot see a
// stale partial: this is the compiler's own release / acquire sequence for device scope on this target with
// the two cache-wide operations taken out, and neither is needed here.
//   * Release side.  The documented release sequence is "write back the L2 (buffer_wbl2 sc1), then
//     s_waitcnt vmcnt(0), then the releasing atomic".  vmcnt counts a store until the level that the store's
//     scope names has acknowledged it; that is what makes the wait the completion point of the sequence, and
//     for an sc1 store the acknowledgement comes from the memory side.  The write-back exists for data written
//     earlier with weaker scope that may still sit dirty in the L2; every byte of a partial is written with an
//     sc1 store, so there is nothing to write back.  (A device-scope fence here costs a full L2 write-back per
//     block: 2.5-30x on the whole kernel.)  The wait is per wave, so every wave executes it before the block
//     barrier, and only after the barrier does thread 0 take the ticket: the ticket is ordered after the
//     acknowledgement of every store of the block.  Without the explicit wait the compiler is free to let the
//     relaxed stores drain later, and the ticket then overtook a partial about once in 10^5 launches.
//   * Acquire side.  The documented acquire sequence is "the acquiring atomic, then invalidate L1 and the
//     non-local L2 lines (buffer_inv sc1)", so that LATER ORDINARY loads cannot hit stale copies.  The merging
//     block reads the partials with sc1 atomic loads, which are coherent at device scope by themselves, so no
//     invalidate is needed.  They cannot start early: the ticket's value goes through LDS and a block barrier
//     to every thread, the loads are control-dependent on it (`last`), and a workgroup-scope acquire fence
//     sits between the barrier and the loads, across which the compiler may not move atomic accesses.
//   * The ticket itself is one atomic counter per unit; read-modify-write atomics execute at the point of
//     coherence of their address whatever cache holds a copy.  The merging block resets it for the next launch.
// Nobody waits for anybody: a block that is not last simply ends.
//
// Die-local form (LOCAL = true).  When all blocks of a unit run on ONE die (the host arranges that by block
// number where the shape allows, see make_ctx), the same handshake runs one level lower: workgroup-scope
// atomic stores and loads (`sc0`: through the compute unit's L1, served by the die's L2, which all its compute
// units share), the same wait, the same ticket.  The hardware argument is the same with "the die's L2" in
// place of "the memory side".  It lies outside the language memory model, which knows no scope between one
// workgroup and the device, so it is guarded twice: the host enables it only on a GPU where a probe launch
// has shown that block numbers equal mod 8 share a die, and every block compares the die it actually runs on
// with the probe's record and flags a difference in the ticket, which turns the unit's output into NaN.
// BUZZ_FLAG_DEVICE_MERGE selects the device-wide form everywhere.
template <bool LOCAL> constexpr int merge_scope() { return LOCAL ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT; }
template <bool LOCAL> __device__ inline void publish(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, merge_scope<LOCAL>()); }
template <bool LOCAL> __device__ inline float acquire(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, merge_scope<LOCAL>()); }

// Where a block works: logical rows [j0, j1) of one unit.  The range is cut into at most three physically
// contiguous runs of stored rows (linear region, ring before the wrap, ring after the wrap) and the row being appended.
struct SplitCtx {
    int split, unit;
    int home;            // die-local merge: launch-order block number mod 8, which decides the die
    int j0, j1, jl1, wrap;
    size_t ubase;
};

// The arguments, in scalar registers from the start.  Left to itself the compiler fetches each where it is first used: a
// dozen fetches one after the other in front of the stream and half as many in the tail, each a wait, the first on each of
// four cache lines a wait for memory.  Asked for at once they are one wait (what is fetched again later finds its line).
// (256 steps of 8 units of 110 rows of one fp32 head of 64: 1396 -> 1288 us, half of that from request_fresh_row; 256 steps of
// 256 units of 1240 rows of one fp16 head of 128 5453 -> 5288; 64 steps of 8 units of 1540 rows, 4 bf16 heads of 128, 478 -> 470.)
__device__ inline void hold_arguments(const AttnArgs& a)
{
    asm volatile("" :: "s"(a.q), "s"(a.k_new), "s"(a.v_new), "s"(a.K), "s"(a.V), "s"(a.score), "s"(a.logit), "s"(a.logit_prev),
                 "s"(a.part_ml), "s"(a.part_o), "s"(a.stat), "s"(a.stat_prev), "s"(a.ticket), "s"(a.out),
                 "s"(__builtin_bit_cast(i32x4, a.map)), "s"(a.n), "s"(a.cap),
                 "s"(a.rows_per_split), "s"(a.n_splits), "s"(a.s_cap), "s"(a.pending), "s"(a.fixed_tiles), "s"(a.xcd_local),
                 "s"(a.die_map), "s"(a.scale_log2), "s"(a.units_per_die), "s"(a.new_phys));
}

__device__ inline SplitCtx make_ctx(const AttnArgs& a)
{
    SplitCtx x;
    x.split = blockIdx.x; x.unit = blockIdx.y;
    x.home = 0;
    if (a.xcd_local) {
        // The hardware deals the blocks of a grid to the dies (XCDs) round-robin in launch order: block b runs
        // on die b mod 8.  The grid is (8, n_splits, units / 8), x first in launch order, so the n_splits blocks of a
        // unit share b mod 8 = blockIdx.x (units is a multiple of 8 here) and die d gets units d * units/8 ...
        x.home = blockIdx.x;
        x.split = blockIdx.y;
        x.unit = blockIdx.x * a.units_per_die + blockIdx.z;
    }
    x.j0 = x.split * a.rows_per_split;
    x.j1 = min(a.n, x.j0 + a.rows_per_split);
    x.jl1 = min(x.j1, a.n - 1);                           // rows already stored in the arena end here
    x.wrap = a.map.front + a.map.ring_cap - a.map.ring_head;   // first logical row after the ring wraps
    x.ubase = (size_t)x.unit * a.cap;
    return x;
}

// The tiles of a split: WROWS consecutive rows each, numbered across its (up to three) stored runs from each run's
// first row on; the row being appended, which comes from the caller's buffer, is a tile of its own at the end.
// ANCHOR: the tiles of a run sit on a grid of multiples of WROWS physical rows (`lead` rows before its first row are
// masked), so that a tile's rows are one aligned piece of the arena.
// A block's waves do not own fixed tiles: apart from the first one each (two with two buffers), a wave claims its next tile
// from a counter in LDS.  (With fixed round-robin tiles the waves launched first -- which the memory pipeline serves first
// -- ended 15% earlier than the others, and the block waited for the slowest.)
// run: first logical and physical row, length and masked rows (both from the anchor on); first row of the tile in it
struct Tile { int lo, phys, cnt, lead, base; bool fresh; };

template <int WROWS, bool ANCHOR>
struct TileMap {
    int lo0, lo1, lo2, ph0, ph1, ph2, c0, c1, c2, ld0, ld1, ld2, f1, f2, f3, n_tiles, n;
    __device__ inline TileMap(const AttnArgs& a, const SplitCtx& x)
    {
        n = a.n;
        lo0 = x.j0; ph0 = lo0; c0 = min(x.jl1, a.map.front) - lo0;
        lo1 = max(x.j0, a.map.front); ph1 = a.map.ring_base + a.map.ring_head + (lo1 - a.map.front); c1 = min(x.jl1, x.wrap) - lo1;
        lo2 = max(x.j0, x.wrap); ph2 = a.map.ring_base + (lo2 - x.wrap); c2 = x.jl1 - lo2;
        if constexpr (ANCHOR) {
            ld0 = ld1 = ld2 = 0;
            static_assert((WROWS & (WROWS - 1)) == 0, "tiles anchor at multiples of WROWS");
            if (c0 > 0) c0 += ld0 = ph0 & (WROWS - 1);
            if (c1 > 0) c1 += ld1 = ph1 & (WROWS - 1);
            if (c2 > 0) c2 += ld2 = ph2 & (WROWS - 1);
        }
        f1 = (max(c0, 0) + WROWS - 1) / WROWS;
        f2 = f1 + (max(c1, 0) + WROWS - 1) / WROWS;
        f3 = f2 + (max(c2, 0) + WROWS - 1) / WROWS;
        n_tiles = f3 + (x.j1 == a.n && x.j0 < a.n ? 1 : 0);
    }
    __device__ inline int total() const { return n_tiles; }
    __device__ inline Tile locate(int t) const
    {
        // (sums of "difference or 0" rather than nested selects between members: the latter turn into
        // an indexed read of the structure and push it into private memory)
        const bool r1 = t >= f1, r2 = t >= f2;
        Tile k;
        k.fresh = t >= f3;
        k.lo = lo0 + (r1 ? lo1 - lo0 : 0) + (r2 ? lo2 - lo1 : 0);
        k.phys = ph0 + (r1 ? ph1 - ph0 : 0) + (r2 ? ph2 - ph1 : 0);
        k.cnt = c0 + (r1 ? c1 - c0 : 0) + (r2 ? c2 - c1 : 0);
        if constexpr (ANCHOR) k.lead = ld0 + (r1 ? ld1 - ld0 : 0) + (r2 ? ld2 - ld1 : 0); else k.lead = 0;
        k.base = (t - (r1 ? f1 : 0) - (r2 ? f2 - f1 : 0)) * WROWS;
        if (k.fresh) { k.lo = n - 1; k.cnt = 1; k.base = 0; }
        if (ANCHOR && k.fresh) k.lead = 0;
        return k;
    }
};

// A tile of a short split (one to three tiles for each wave of the block): WROWS logical rows, wherever they are stored.  Short
// steps are bound by latency and by the instructions in front of the first load and behind the last.  All of the split's
// rows are requested at once, at their own 32-bit offsets from the unit's first row, so there are no runs to cut tiles at (the
// linear region's end, the ring's wrap and the new row each began another tile, and often a second round of loads for the
// whole block), no tiles to claim, and no barrier before the stream.  256 steps of 8 units of 110 rows, one fp32 head of
// 64: 1233 -> 970 us; 64 steps of 8 units of 1540 rows in 13 splits, 4 bf16 heads of 128, 470 -> 449; 48 of 8 of 1060 in 9, 4 fp32
// heads of 64, 384 -> 356; per step, 8 units of 600 rows in 5 splits, one bf16 head of 128, 6.5 -> 5.0 us.
template <int WROWS>
struct ShortTile {
    int j0, cnt, base;
    __device__ inline ShortTile(const SplitCtx& x, int t) : j0(x.j0), cnt(x.j1 - x.j0), base(t * WROWS) {}
    __device__ inline bool exists() const { return base < cnt; }
    __device__ inline bool last(const SplitCtx& x, int n) const { return x.j1 == n && base + WROWS >= cnt; }   // has the new row
    // its logical row i, or the split's last
    __device__ inline int row(int i) const { return j0 + min(base + i, cnt - 1); }
    __device__ inline Tile tile() const { Tile k; k.lo = j0; k.phys = 0; k.cnt = cnt; k.lead = 0; k.base = base; k.fresh = false; return k; }
};

__device__ inline int claim_tile(int* counter)
{
    int t = 0;
    if ((threadIdx.x & 63) == 0) t = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return __builtin_amdgcn_readfirstlane(t);
}

// The tile a wave takes after tile `last`: claimed from the block's counter, or -- when the caller asked
// for results that do not depend on timing -- the next one of a fixed round-robin over `nw` waves.
__device__ inline int next_tile(const AttnArgs& a, int* counter, int last, int nw)
{
    return a.fixed_tiles ? last + nw : claim_tile(counter);
}

// A barrier that orders LDS only: loads from memory that are in flight stay in flight across it.
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A wave's way through the tiles.  TWO: two tile buffers, the next tile's loads are issued before the current tile is
// consumed.  (The compiler waits for both at once, because the next tile may not exist.  With the loads
// issued unconditionally, and the loop shaped so that it waits for the older half only, the stream was no faster -- 52
// us of 62 on one sequence of 23.6k rows by 32 heads, 7.4 TB/s either way -- and waves with one tile paid for loads of
// tiles that do not exist: 8 units of 1500 rows, 4 heads each, 10.1 instead of 8.0 us per step.)
// TILE_FIRST: the first tile's loads go before the side requests.  The step starts earlier, but the stream gets thinner: the compiler
// knows of two loads behind the first tile for certain (row 0 of the side phase), and the wait that this allows before a tile
// is consumed stands in the loop, where it lets two loads of the next tile stay in flight and waits for the others.  Nothing is lost
// where a tile is two loads (K and V of cached rows of up to 256 bytes: 256 units of 1450 28.8 us per step, 29.1 with the
// side requests first).  Where it is four, the loop waits twice as often for half as much; first / behind:
//   cached, 8-wave blocks     144 units of 1711 bf16 rows of 256 48.9 / 42.5, 144 of 1769 fp32 rows of 128 47.6 / 41.3; half a percent
//                             for the side requests over 2100 random steps, at most 4% against
//   streaming, 4-wave blocks  272 units of 2872 bf16 rows of 128 86.5 / 74.7, 400 of 1953 66.1 / 63.9; but where 1.6 to 4 blocks on a
//                             compute unit crowd the memory the thinner stream is the faster one: 480 of 1627 62.4 / 63.8, 560 of
//                             1395 69.0 / 72.8, 600 of 2929 150.5 / 157.9, 900 of 868 66.9 / 68.7; 1100 of 710 71.9 / 71.1
//   cached, 4-wave blocks     the same: 300 units of 874 bf16 rows of 256 55.0 / 50.0, 560 of 375 35.7 / 37.8, 1100 units +3%
//   streaming, 8-wave blocks  behind: 200 of 2630 44.9 / 41.7, 96 of 4663 rows of 256 77.0 / 70.4
// Rows of 1024 bytes (eight loads): first, 272 units of 799 79.3 / 90.8, 8-wave blocks 0 to 1.5%, but in 4-wave blocks from 1.6 of
// them on a compute unit on behind: 560 units +3%.  (The first tile consumed in front of the loop, so that no wait in it depends on what
// follows that tile: 272 units 78.3, 512 of 3900 155.8, first 154.2.)  With one buffer they come behind, too: hoisted, the loop
// copies its registers, 64 steps of 32 units of 7800 rows, 4 heads, 1550 -> 1576 us.
template <bool TWO, bool TILE_FIRST, typename Buf, typename Load, typename Requests, typename Compute>
__device__ inline void stream_tiles(const AttnArgs& a, int* counter, int wave, int nw, int total, Load load, Requests requests, Compute compute)
{
    int t = wave;
    if constexpr (TWO) {
        Buf first, second;
        int tn = t + nw;
        if (TILE_FIRST && t < total) load(first, t);
        requests();
        lds_barrier();                                    // the counter is set
        if (!TILE_FIRST && t < total) load(first, t);
        while (t < total) {
            if (tn < total) load(second, tn);
            int t2 = next_tile(a, counter, tn, nw);
            compute(first, t);
            t = tn; tn = t2;
            if (t >= total) break;
            if (tn < total) load(first, tn);
            t2 = next_tile(a, counter, tn, nw);
            compute(second, t);
            t = tn; tn = t2;
        }
    } else {
        requests();
        lds_barrier();                                    // the counter is set
        while (t < total) {
            Buf buf;
            load(buf, t);
            const int tn = next_tile(a, counter, t, nw);
            compute(buf, t);
            t = tn;
        }
    }
}

// The side phase: per row of the split, this step's logits out, and the score with the previous step's probability
// added (one step late, because a probability needs the maximum and sum over all splits).  A thread takes the rows
// tid, tid + NTHR, ...: every access of a wave is one contiguous piece whatever the row's place in the arena is.
// The first SR rows of a thread are requested when the kernel starts and consumed after the streaming loop, so that
// their latency is never exposed; longer splits take further rounds of SR rows.
template <int G> constexpr int side_rows() { return G == 1 ? 8 : (G <= 4 ? 4 : 2); }

template <int G, int SR> struct SideRows {
    float M[G], iL[G];                                    // the previous step's softmax statistics of the unit
    float sc[SR], lp[SR][G];                              // old scores and the previous step's logits
    u32x4 fresh;                                          // one of the new row's pieces (K's, then V's), last split only
};

// eq. 2: the caller's new row joins the cache.  Its pieces are requested when the kernel starts and stored in the
// side phase (stores between the streaming loop's loads would make the compiler wait for more than it needs).
template <int ROWB>
__device__ inline bool fresh_piece(const AttnArgs& a, const SplitCtx& x) { return x.j1 == a.n && x.j0 < a.n && (int)threadIdx.x < 2 * (ROWB / 16); }
template <int ROWB, int G, int SR>
__device__ inline void request_fresh_row(const AttnArgs& a, const SplitCtx& x, SideRows<G, SR>& p)
{
    constexpr int P = ROWB / 16;
    const int i = threadIdx.x;
    // (the arguments as values: selected in place, the compiler fetched them with a load per lane and waited for everything
    // requested so far, in front of the stream)
    const char* k = (const char*)a.k_new + (size_t)x.unit * ROWB;
    const char* v = (const char*)a.v_new + (size_t)x.unit * ROWB - ROWB;
    if (fresh_piece<ROWB>(a, x)) p.fresh = *(const u32x4*)((i < P ? k : v) + i * 16);
}
template <int ROWB, int G, int SR>
__device__ inline void store_fresh_row(const AttnArgs& a, const SplitCtx& x, const SideRows<G, SR>& p)
{
    constexpr int P = ROWB / 16;
    const int i = threadIdx.x;
    if (fresh_piece<ROWB>(a, x)) {
        *(u32x4*)((char*)(i < P ? a.K : a.V) + (x.ubase + a.new_phys) * ROWB + (i < P ? i : i - P) * 16) = p.fresh;
        if (i == 0) a.pos[x.ubase + a.new_phys] = a.new_pos;
    }
}

// element i of an array that starts at a wave-uniform address: a scalar base and a 32-bit offset per lane
__device__ inline float* lane_element(const float* base, unsigned i) { return (float*)((char*)base + i * 4u); }

template <int G, int NTHR, int SR>
__device__ inline void request_side_rows(const AttnArgs& a, const SplitCtx& x, int first, SideRows<G, SR>& p)
{
    const float* score_u = a.score + x.ubase;
    const float* logit_prev_u = a.logit_prev + x.ubase * G;
    auto request = [&](int i, int j) {
        const unsigned ph = a.map.phys(j);
        p.sc[i] = *lane_element(score_u, ph);
#pragma unroll
        for (int g = 0; g < G; ++g) p.lp[i][g] = *lane_element(logit_prev_u + (size_t)g * a.cap, ph);
    };
    // One head: straight-line requests (lanes past the range ask for its last row; nothing is used where nothing is
    // pending).  With several heads the loads that a lane does not need cost more than the branches around them
    // (8 units x 110 rows of one head: 1394 us per session against 1467 with the branches; 8 units of 4 heads: 517
    // against 508 us per 64 steps).
    if (G > 1 && !a.pending) return;
#pragma unroll
    for (int i = 0; i < SR; ++i) {
        if (x.j0 + first + i * NTHR >= x.jl1 && (G > 1 || i > 0)) break;
        const int j = x.j0 + first + (int)threadIdx.x + i * NTHR;
        if constexpr (G == 1) request(i, max(min(j, x.jl1 - 1), 0));
        else if (j < x.jl1) request(i, j);
    }
}

template <int G, int SR>
__device__ inline void request_prev_stat(const AttnArgs& a, int unit, SideRows<G, SR>& p)
{
    // Through the constant address space: no launch writes what it reads here, and scalar registers hold it.  (In vector
    // registers it costs wide groups a resident block: 256 units of 3800 rows, 6 fp16 heads of 64, 53 -> 71 us.)
    const auto* prev = (const __attribute__((address_space(4))) float*)(a.stat_prev + (size_t)unit * G * 2);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        p.M[g] = prev[2 * g];                                   // (read but not used where nothing is pending)
        p.iL[g] = prev[2 * g + 1];
    }
}

template <int G, int NTHR, int SR>
__device__ inline void store_side_rows(const AttnArgs& a, const SplitCtx& x, int first, const SideRows<G, SR>& p, const float* stage)
{
    float* score_u = a.score + x.ubase;
    float* logit_u = a.logit + x.ubase * G;               // [G][cap] for this unit, written by this step
#pragma unroll
    for (int i = 0; i < SR; ++i) {
        if (x.j0 + first + i * NTHR >= x.j1) break;
        const int r = first + (int)threadIdx.x + i * NTHR, j = x.j0 + r;
        if (j < x.j1) {
            const unsigned ph = a.map.phys(j);
#pragma unroll
            for (int g = 0; g < G; ++g) *lane_element(logit_u + (size_t)g * a.cap, ph) = stage[g * a.rows_per_split + r];
            float sc = p.sc[i];
#pragma unroll
            for (int g = 0; g < G; ++g) sc = add_probability(sc, p.lp[i][g], p.M[g], p.iL[g]);
            const bool fresh = j == a.n - 1;              // the appended row starts from score 0
            if (fresh || a.pending) *lane_element(score_u, ph) = fresh ? 0.f : sc;
        }
    }
}

// The running results of a block's waves in LDS; acc is written 16 bytes at a time.
template <int G, int D, int NW> struct WaveResults {
    alignas(16) float acc[NW][G][D];                      // unnormalised output
    float2 ml[G][NW];                                     // (max, sum)
    int ticket, next_tile;
};

__device__ inline float lane_value(float v, int lane)     // of a wave-uniform lane
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Maximum and sum over the wave, in every lane: 16 lanes by DPP, the four rows through scalar registers.
__device__ inline float wave_max(float v)
{
    v = fmaxf(v, dpp_move<0xB1>(v));
    v = fmaxf(v, dpp_move<0x4E>(v));
    v = fmaxf(v, dpp_move<0x141>(v));
    v = fmaxf(v, dpp_move<0x140>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ inline float wave_sum(float v)
{
    v = row_sum<16, false>(v);
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// The last block of a unit merges the partials of its S splits, 64 output elements (of one head) per wave and group:
// lane s fetches the (max, sum) pair of split s and turns it into that split's weight, every lane fetches its element
// of the splits' outputs, up to four groups and 8 (16) splits at a time in one round of loads without a branch in
// between, and the weights reach the lanes as scalars: one exponential per wave and split instead of one per
// element, half the loads of a pair per element, one round trip for up to 16 splits.  Groups of one head that a wave
// has anyway share their weights.  What counts here is the number of instructions the waves have to issue between the
// ticket and the output: with a branch-free burst of pairs and elements per thread, and two rounds of it, a step of 8
// units, 12 splits, 4 heads of 128 took 9.3 us, with weights for each group 8.0, now 7.3.  (Spreading the splits over
// all waves of the block and their sums through LDS: 8.2.)  128 units, 2 splits, 7 heads of 256: 29.3, 32.8 and 27.8 us.
// More than four groups at a time cost the streaming kernels a resident block (300 units, 8 heads of 128: 28 -> 42 us).
template <int G, int D, int NM>
__device__ inline void merge_splits(const AttnArgs& a, int unit, int wave, bool poisoned, float* outp)
{
    constexpr int NG = G * D / 64, NMW = NM / 64;         // groups of 64 elements, merging waves
    constexpr int PER = (NG + NMW - 1) / NMW;             // groups per wave
    constexpr int HG = PER >= D / 64 ? D / 64 : PER >= 2 && D >= 128 ? 2 : 1;   // groups of one head that stay together ...
    constexpr int NH = NG / HG, PERH = (NH + NMW - 1) / NMW;
    constexpr int HB = PERH * HG <= 4 ? PERH : 4 / HG;    // ... and how many such chunks a wave takes at a time
    constexpr int GB = HB * HG, CH = GB <= 2 && NMW > 2 ? 16 : 8;
    static_assert(NG % HG == 0 && (D / 64) % HG == 0, "a chunk lies inside one head");
    const int S = a.n_splits, lane = threadIdx.x & 63;
    const unsigned long long* ml = (const unsigned long long*)(a.part_ml + (size_t)unit * a.s_cap * G * 2);
    const float* po = a.part_o + (size_t)unit * a.s_cap * G * D;
#pragma unroll 1
    for (int c0 = wave; c0 < NH; c0 += NMW * HB) {
        float M[HB], L[HB], o[GB];
#pragma unroll
        for (int h = 0; h < HB; ++h) { M[h] = -INFINITY; L[h] = 0.f; }
#pragma unroll
        for (int b = 0; b < GB; ++b) o[b] = 0.f;
        auto chunk = [&](int h) { return min(c0 + h * NMW, NH - 1); };
        // 16 (8) splits per round; the running maximum moves from round to round
#pragma unroll 1
        for (int s0 = 0; s0 < S; s0 += CH) {
            unsigned long long pair[HB];
            float xr[GB][CH];
            auto request = [&](auto local) {
                constexpr bool LOCAL = decltype(local)::value;
#pragma unroll
                for (int h = 0; h < HB; ++h)
                    pair[h] = __hip_atomic_load(ml + min(s0 + (lane & (CH - 1)), S - 1) * G + chunk(h) * HG * 64 / D, __ATOMIC_RELAXED, merge_scope<LOCAL>());
#pragma unroll
                for (int half = 0; half < CH; half += 8) {
                    if (half > 0 && s0 + half >= S) break;
#pragma unroll
                    for (int b = 0; b < GB; ++b) {
#pragma unroll
                        for (int e = half; e < half + 8; ++e) xr[b][e] = acquire<LOCAL>(po + (size_t)min(s0 + e, S - 1) * (G * D) + (chunk(b / HG) * HG + b % HG) * 64 + lane);
                    }
                }
            };
            if (a.xcd_local) request(std::true_type{}); else request(std::false_type{});
            const bool have = lane < CH && s0 + lane < S;
            float w[HB];
#pragma unroll
            for (int h = 0; h < HB; ++h) {
                const float m = have ? __uint_as_float((unsigned)pair[h]) : -INFINITY;
                const float mx = fmaxf(M[h], wave_max(m));   // finite: the appended row is always present
                const float keep = fast_exp2(M[h] - mx);     // 0 in the first round
                w[h] = fast_exp2(m - mx);
                L[h] = fmaf(L[h], keep, wave_sum(have ? w[h] * __uint_as_float((unsigned)(pair[h] >> 32)) : 0.f));
#pragma unroll
                for (int b = h * HG; b < (h + 1) * HG; ++b) o[b] *= keep;
                M[h] = mx;
            }
#pragma unroll
            for (int half = 0; half < CH; half += 8) {
                if (half > 0 && s0 + half >= S) break;
#pragma unroll
                for (int b = 0; b < GB; ++b) {
#pragma unroll
                    for (int e = half; e < half + 8; ++e) o[b] = fmaf(lane_value(w[b / HG], e), s0 + e < S ? xr[b][e] : 0.f, o[b]);
                }
            }
        }
#pragma unroll
        for (int h = 0; h < HB; ++h) {
            const int c = c0 + h * NMW;
            if (c >= NH) continue;
#pragma unroll
            for (int b = 0; b < HG; ++b) outp[(c * HG + b) * 64 + lane] = poisoned ? __builtin_nanf("") : o[h * HG + b] / L[h];
            if (c * HG * 64 % D == 0 && lane == 0) {
                a.stat[((size_t)unit * G + c * HG * 64 / D) * 2] = M[h];
                a.stat[((size_t)unit * G + c * HG * 64 / D) * 2 + 1] = 1.0f / L[h];
            }
        }
    }
}

// Everything a block does once its waves have put their (max, sum, unnormalised output) into LDS:
//   1. merge the waves; the only split of a unit writes the result, else publish the split's partial;
//   2. wait for the published stores, synchronise, take the ticket;
//   3. in the block that drew the last ticket the upper half of the waves (all of them for a wide output) merges the
//      splits and writes the output;
//   4. side phase: this step's logits leave LDS, the previous step's score update is applied.  (The read
//      stream of the block is over by then.  Doing the score update at the start of the block instead, under the
//      latency of the first K/V loads, was measured 8% slower: its writes then compete with the ramping stream.
//      Between 1 and 2 it delays the tickets: 8 units, 12 splits: 8.4 instead of 8.0 us per step.)
template <int G, int D, int NW, int ROWB, bool ONE_ROUND, int SR>
__device__ inline void finish_split(const AttnArgs& a, const SplitCtx& x, SideRows<G, SR>& side, const float* stage, WaveResults<G, D, NW>& sm)
{
    constexpr int NTHR = NW * 64;                         // threads per block
    const int tid = threadIdx.x, unit = x.unit;
    const int S = a.n_splits;
    // the NW results in LDS -> emit(element, head, column, max, sum, output)
    auto merge_waves = [&](auto emit) {
        for (int i = tid; i < G * D; i += NTHR) {
            const int g = i / D, d = i - g * D;
            float2 ml[NW];
            float av[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) { ml[w] = sm.ml[g][w]; av[w] = sm.acc[w][g][d]; }
            float M = ml[0].x;
#pragma unroll
            for (int w = 1; w < NW; ++w) M = fmaxf(M, ml[w].x);
            const float mref = (M == -INFINITY) ? 0.f : M;
            float o = 0.f, L = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float wgt = fast_exp2(ml[w].x - mref);
                o = fmaf(wgt, av[w], o);
                L = fmaf(wgt, ml[w].y, L);
            }
            emit(i, g, d, M, L, o);
        }
    };
    float* outp = a.out + (size_t)unit * G * D;           // heads of a unit are consecutive: unit * G = b * Hq + kvh * G
    auto write = [&](int i, int g, int d, float M, float L, float o) {
        outp[i] = o / L;
        if (d == 0) {
            a.stat[((size_t)unit * G + g) * 2] = M;
            a.stat[((size_t)unit * G + g) * 2 + 1] = 1.0f / L;
        }
    };
    lds_barrier();
    if (S == 1) {
        merge_waves(write);
        if (tid == 0) BUZZ_STAMP(2);
    } else {
        const size_t pbase = ((size_t)unit * a.s_cap + x.split) * G;
        float* part_o = a.part_o + pbase * D;
        float* part_ml = a.part_ml + pbase * 2;
        if (a.xcd_local)
            merge_waves([&](int i, int g, int d, float M, float L, float o) {
                publish<true>(part_o + i, o);
                if (d == 0) { publish<true>(part_ml + 2 * g, M); publish<true>(part_ml + 2 * g + 1, L); }
            });
        else
            merge_waves([&](int i, int g, int d, float M, float L, float o) {
                publish<false>(part_o + i, o);
                if (d == 0) { publish<false>(part_ml + 2 * g, M); publish<false>(part_ml + 2 * g + 1, L); }
            });
        if (tid == 0) BUZZ_STAMP(2);

        // Ticket: the block that arrives last for this unit sees every split's partial.  Every wave first
        // waits until its own published stores have been acknowledged (vmcnt(0)), then the block synchronises,
        // then one thread takes the ticket: the ticket can never overtake a partial (the argument is written out
        // above merge_scope).  No cache maintenance is involved.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0), expcnt / lgkmcnt untouched
        __syncthreads();
        if (tid == 0) {
            // A die-local merge is only right if this block really runs where its number says: the host has
            // recorded which die served block numbers 0..7 (die_map, 4 bits each); a block that finds itself
            // elsewhere says so in the ticket's upper half, and the merging block sees every earlier arrival's.
            int add = 1, before;
            if (a.xcd_local) {
                if ((__builtin_amdgcn_s_getreg((31 << 11) | 20) & 7u) != ((a.die_map >> (4 * x.home)) & 15u)) add += 0x10000;   // XCC_ID
                before = __hip_atomic_fetch_add(a.ticket + unit, add, __ATOMIC_RELAXED, merge_scope<true>());
            } else {
                before = __hip_atomic_fetch_add(a.ticket + unit, add, __ATOMIC_RELAXED, merge_scope<false>());
            }
            sm.ticket = before + (add & 0x10000);
        }
        __syncthreads();
        if (tid == 0) BUZZ_STAMP(4);
        const int arrival = __builtin_amdgcn_readfirstlane(sm.ticket);
        if ((arrival & 0xffff) == S - 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            // merging threads: the lower half starts its side phase, unless the block has only 4 waves for a wide output, or a
            // short split's side phase and more groups of outputs than waves (2 units, 32 splits of 125 rows, 8 heads of 128: 10.1
            // us per step, 9.25 so; with 4 heads 8 units, 13 splits, half of them: 6.82, all 6.91)
            constexpr int NM = G * D >= kWideBlockMaxGD || (ONE_ROUND && G * D / 64 > NW) ? NTHR : NTHR / 2;
            if (tid >= NTHR - NM) {
                // A die-local merge with a block on an unexpected die may have missed partials: its output is NaN
                // rather than plausible numbers.
                merge_splits<G, D, NM>(a, unit, __builtin_amdgcn_readfirstlane((tid - (NTHR - NM)) >> 6), (arrival >> 16) != 0, outp);
                if (tid == NTHR - NM) {                   // ready for the next step
                    if (a.xcd_local) __hip_atomic_store(a.ticket + unit, 0, __ATOMIC_RELAXED, merge_scope<true>());
                    else __hip_atomic_store(a.ticket + unit, 0, __ATOMIC_RELAXED, merge_scope<false>());
                }
                if (tid == NTHR - NM) BUZZ_STAMP(5);
            }
        }
    }
    store_fresh_row<ROWB>(a, x, side);
    store_side_rows<G, NTHR>(a, x, 0, side, stage);
    if constexpr (!ONE_ROUND) {
#pragma unroll 1
        for (int first = SR * NTHR; x.j0 + first < x.j1; first += SR * NTHR) {
            request_side_rows<G, NTHR>(a, x, first, side);
            store_side_rows<G, NTHR>(a, x, first, side, stage);
        }
    }
    if (tid == 0) BUZZ_STAMP(3);
}

// Vector-ALU streaming kernel (any dtype; the choice for one query head per kv head).
template <typename T, int D, int G, int U, bool NT, int NW, int SHORT, bool TILE_FIRST, bool VIA_LDS>
__global__ __launch_bounds__(NW * 64, BUZZ_MIN_BLOCKS) void attn_split_kernel(const AttnArgs a)
{
    using E = Elem<T>;
    constexpr int VEC = E::VEC;
    constexpr int LPR = D / VEC;          // lanes per cache row
    constexpr int RPW = 64 / LPR;         // rows per wave-wide load
    constexpr int ROWB = D * (int)sizeof(T);
    constexpr int WROWS = RPW * U;        // rows one wave consumes per trip
    static_assert(LPR >= 8 && LPR <= 64, "row must span 8..64 lanes");

    extern __shared__ float stage[];                      // [G][rows_per_split] logits of this split's rows
    __shared__ WaveResults<G, D, NW> sm;
    static_assert(alignof(decltype(sm)) >= 16 && offsetof(decltype(sm), acc) % 16 == 0 && D % 4 == 0, "16-byte stores into acc");

    hold_arguments(a);
    const SplitCtx x = make_ctx(a);
    const int unit = x.unit, j0 = x.j0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // tile numbers and addresses stay in scalar registers
    const int c = lane % LPR, rs = lane / LPR;
    if (tid == 0) { BUZZ_STAMP(0); BUZZ_STAMP_VALUE(6, __builtin_amdgcn_s_getreg((31 << 11) | 4)); BUZZ_STAMP_VALUE(7, __builtin_amdgcn_s_getreg((31 << 11) | 20)); }
    constexpr bool TWO = G == 1;
    if (!SHORT && tid == 0) sm.next_tile = TWO ? 2 * NW : NW;       // the waves' first tiles are not claimed

    u32x4 qr[G];                                          // this lane's 16 bytes of every query head, raw
    {
        const char* qb = (const char*)a.q + (size_t)unit * G * ROWB + c * 16;
#pragma unroll
        for (int g = 0; g < G; ++g) qr[g] = *(const u32x4*)(qb + (size_t)g * ROWB);
    }

    const size_t ubase = x.ubase;
    char* Kb = (char*)a.K + ubase * ROWB;                 // wave-uniform bases; lanes add 32-bit offsets
    char* Vb = (char*)a.V + ubase * ROWB;
    const unsigned lane_off = c * 16;

    float m[G], l[G], acc[G][VEC];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[g][v] = 0.f;
    }

    // The streaming phase only reads: logits are staged in LDS, and all per-row side traffic (this step's logits out,
    // the previous step's logits and the old score in, the new score out) happens in one dense phase at the end of
    // the block.  Writes that trickle into a saturated read stream were measured to cost ~5% of the kernel per 1% of
    // extra bytes.
    struct Buf { u32x4 k[U], v[U]; };
    const TileMap<WROWS, false> tiles(a, x);
    auto load_t = [&](u32x4 (&kr)[U], u32x4 (&vr)[U], int t) {
        const Tile k = tiles.locate(t);
        const char* kp = k.fresh ? (const char*)a.k_new + (size_t)unit * ROWB : Kb + (size_t)k.phys * ROWB;
        const char* vp = k.fresh ? (const char*)a.v_new + (size_t)unit * ROWB : Vb + (size_t)k.phys * ROWB;
#pragma unroll
        for (int u = 0; u < U; ++u) {      // lanes past the run's end re-read its last row
            const unsigned off = (unsigned)min(k.base + u * RPW + rs, k.cnt - 1) * ROWB + lane_off;
            kr[u] = load16<NT>(kp + off);
            vr[u] = load16<NT>(vp + off);
        }
    };

    auto compute_t = [&](const u32x4 (&kr)[U], const u32x4 (&vr)[U], const Tile& k) {
        const int stg = k.lo - j0 + k.base;               // staging index (row relative to the split's first row)
        float s[G][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = k.base + u * RPW + rs < k.cnt;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float d = row_sum<LPR, VIA_LDS>(E::dot(qr[g], kr[u])) * a.scale_log2;
                s[g][u] = ok ? d : -INFINITY;
                if (c == 0 && ok) stage[g * a.rows_per_split + stg + u * RPW + rs] = d;
            }
        }
        // online softmax: s becomes the unnormalised probability relative to the running maximum
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float tmax = s[g][0];
#pragma unroll
            for (int u = 1; u < U; ++u) tmax = fmaxf(tmax, s[g][u]);
            const float mn = fmaxf(m[g], tmax);
            const float mref = (mn == -INFINITY) ? 0.f : mn;
            const float alpha = fast_exp2(m[g] - mref);
            m[g] = mn;
            float psum = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s[g][u] = fast_exp2(s[g][u] - mref);
                psum += s[g][u];
            }
            l[g] = fmaf(l[g], alpha, psum);
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[g][v] *= alpha;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float vf[VEC];
            E::cvt(vr[u], vf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[g][v] = fmaf(s[g][u], vf[v], acc[g][v]);
            }
        }
    };

    SideRows<G, SHORT ? (SHORT * WROWS + 63) / 64 : side_rows<G>()> side;
    auto requests = [&] {
        request_side_rows<G, NW * 64>(a, x, 0, side);
        request_prev_stat(a, unit, side);
        request_fresh_row<ROWB>(a, x, side);
    };
    if constexpr (SHORT) {
        const char* kn = (const char*)a.k_new + (size_t)unit * ROWB;
        const char* vn = (const char*)a.v_new + (size_t)unit * ROWB;
        Buf b[SHORT];
#pragma unroll
        for (int i = 0; i < SHORT; ++i) {
            const ShortTile<WROWS> own(x, wave + i * NW);
            if (!own.exists()) break;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned off = (unsigned)a.map.phys(own.row(u * RPW + rs)) * ROWB + lane_off;
                b[i].k[u] = load16<NT>(Kb + off);
                b[i].v[u] = load16<NT>(Vb + off);
            }
            if (own.last(x, a.n)) {                       // the new row is still the caller's
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (own.row(u * RPW + rs) == a.n - 1) {
                        b[i].k[u] = load16<NT>(kn + lane_off);
                        b[i].v[u] = load16<NT>(vn + lane_off);
                    }
                }
            }
        }
        requests();
#pragma unroll
        for (int i = 0; i < SHORT; ++i) {
            const ShortTile<WROWS> own(x, wave + i * NW);
            if (own.exists()) compute_t(b[i].k, b[i].v, own.tile());
        }
    } else {
        stream_tiles<TWO, TILE_FIRST, Buf>(a, &sm.next_tile, wave, NW, tiles.total(), [&](Buf& b, int t) { load_t(b.k, b.v, t); }, requests, [&](Buf& b, int t) { compute_t(b.k, b.v, tiles.locate(t)); });
    }

    if (lane == 0) BUZZ_STAMP(8 + (wave & 7));

    // merge the RPW lane groups of this wave (same columns, different rows)
    auto merge_groups = [&](auto bit) {
        constexpr int BIT = decltype(bit)::value;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const LanePair mp = lane_pair<BIT>(m[g]), lp = lane_pair<BIT>(l[g]);
            const float mn = fmaxf(mp.a, mp.b);
            const float mref = (mn == -INFINITY) ? 0.f : mn;
            const float wa = fast_exp2(mp.a - mref), wb = fast_exp2(mp.b - mref);
            l[g] = lp.a * wa + lp.b * wb;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const LanePair ap = lane_pair<BIT>(acc[g][v]);
                acc[g][v] = ap.a * wa + ap.b * wb;
            }
            m[g] = mn;
        }
    };
    if constexpr (LPR <= 8) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float mo = dpp_move<0x128>(m[g]), lo = dpp_move<0x128>(l[g]);   // row_ror 8: the row's other half
            const float mn = fmaxf(m[g], mo);
            const float mref = (mn == -INFINITY) ? 0.f : mn;
            const float wa = fast_exp2(m[g] - mref), wb = fast_exp2(mo - mref);
            l[g] = l[g] * wa + lo * wb;
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[g][v] = acc[g][v] * wa + dpp_move<0x128>(acc[g][v]) * wb;
            m[g] = mn;
        }
    }
    if constexpr (LPR <= 16) merge_groups(std::integral_constant<int, 16>{});
    if constexpr (LPR <= 32) merge_groups(std::integral_constant<int, 32>{});

    // this wave's result into LDS
    if (rs == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int v = 0; v < VEC; v += 4)
                *(f32x4*)&sm.acc[wave][g][c * VEC + v] = f32x4{acc[g][v], acc[g][v + 1], acc[g][v + 2], acc[g][v + 3]};
        }
        if (c == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) sm.ml[g][wave] = make_float2(m[g], l[g]);
        }
    }
    finish_split<G, D, NW, ROWB, SHORT != 0>(a, x, side, stage, sm);
}

// ---------------------------------------------------------------------------------------------------
// Matrix-core streaming kernel for grouped queries (G >= 2 query heads per kv head, 16-bit cache).
// With several heads per cache row, q.K^T and p.V are small dense contractions; on the vector ALU they
// cost ~100 instructions per row pair and the kernel stops being bandwidth-bound.  Here a wave works
// on tiles of 16 cache rows with 16x16 MFMA tiles whose 16 "head" slots hold the G real heads:
//
//   S[row][head]  = K[16 rows x D] . Q^T[D x 16]       v_mfma_f32_16x16x32, D/32 instructions
//   O[head][d]   += P[16 x 16 rows] . V[16 rows x d]   v_mfma_f32_16x16x16, 8 column groups x (hi + lo)
//
// Lane l = (j = l % 16, q = l / 16).
//  * K operand: lane (j, q) holds row j of the tile, 16-byte chunks 4p + q, p = 0 .. D/32-1 (one load
//    instruction fetches 64 contiguous bytes of each of 16 rows).  The contraction index may be permuted
//    freely as long as Q uses the same permutation: lane (j, q) of the Q operand holds head j, the same
//    chunks (for j >= G those of the last head again; their products are not used).
//  * S comes out with lane (j, q) holding head j, rows 4q .. 4q+3: exactly the layout the P operand of
//    the second contraction needs, so softmax results go straight back into the matrix core.
//    P is split into a 16-bit head and a 16-bit remainder (two MFMAs) to keep ~16 bits of it.
//  * V operand: lane (j, q) needs rows 4q .. 4q+3 of one column.  It loads the 16-byte chunk j of those
//    four rows (each load instruction: four whole, contiguous rows) and transposes the 4 x 8 block in
//    registers, which yields the operands of 8 column groups; column group m of lane j is column 8j + m.
//  * O comes out with lane (j, q) holding heads 4q .. 4q+3 of its 8 columns.
template <typename T> struct Mma;
template <> struct Mma<bf16_t> {
    static __device__ inline f32x4 qk(const u32x4& k, const u32x4& q, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, k), __builtin_bit_cast(bf16x8_t, q), c, 0, 0, 0);
    }
    static __device__ inline f32x4 pv(const u32x2& p, const u32x2& v, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, p), __builtin_bit_cast(s16x4_t, v), c, 0, 0, 0);
    }
    static __device__ inline void split(float p, unsigned& hi, unsigned& lo) {   // p ~= hi + lo, both bf16
        const __bf16 h = (__bf16)p;
        hi = __builtin_bit_cast(unsigned short, h);
        lo = __builtin_bit_cast(unsigned short, (__bf16)(p - (float)h));
    }
};
template <> struct Mma<fp16_t> {
    static __device__ inline f32x4 qk(const u32x4& k, const u32x4& q, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, k), __builtin_bit_cast(f16x8_t, q), c, 0, 0, 0);
    }
    static __device__ inline f32x4 pv(const u32x2& p, const u32x2& v, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4_t, p), __builtin_bit_cast(f16x4_t, v), c, 0, 0, 0);
    }
    static __device__ inline void split(float p, unsigned& hi, unsigned& lo) {
        const _Float16 h = (_Float16)p;
        hi = __builtin_bit_cast(unsigned short, h);
        lo = __builtin_bit_cast(unsigned short, (_Float16)(p - (float)h));
    }
};

template <typename T, int D, int G, bool NT, int NW, bool ANCHOR, int SHORT>
__global__ __launch_bounds__(NW * 64) void attn_split_mfma_kernel(const AttnArgs a)
{
    constexpr int ROWB = D * 2;
    constexpr int NCH = D / 8;                            // 16-byte chunks per row
    constexpr int QP = NCH / 4;                           // K / Q chunks per lane
    constexpr int VS = (NCH + 15) / 16;                   // sets of 16 column chunks
    constexpr int WROWS = 16;
    static_assert(G >= 2 && G <= 16 && NCH % 4 == 0, "grouped queries, head_dim multiple of 32");

    extern __shared__ float stage[];                      // [G][rows_per_split] logits of this split's rows
    __shared__ WaveResults<G, D, NW> sm;
    static_assert(alignof(decltype(sm)) >= 16 && offsetof(decltype(sm), acc) % 16 == 0 && D % 4 == 0, "16-byte stores into acc");

    hold_arguments(a);
    const SplitCtx x = make_ctx(a);
    const int unit = x.unit, j0 = x.j0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // tile numbers and addresses stay in scalar registers
    const int j = lane & 15, q = lane >> 4;
    if (tid == 0) { BUZZ_STAMP(0); BUZZ_STAMP_VALUE(6, __builtin_amdgcn_s_getreg((31 << 11) | 4)); BUZZ_STAMP_VALUE(7, __builtin_amdgcn_s_getreg((31 << 11) | 20)); }
    if (!SHORT && tid == 0) sm.next_tile = NW;            // tiles 0 .. NW-1 are the waves' first tiles

    u32x4 qb[QP];                                         // Q operand: head j (slots without one repeat the last), chunks 4p + q
#pragma unroll
    for (int p = 0; p < QP; ++p) {
        qb[p] = *(const u32x4*)((const char*)a.q + (size_t)unit * G * ROWB + (unsigned)(min(j, G - 1) * ROWB + (4 * p + q) * 16));
    }

    char* Kb = (char*)a.K + x.ubase * ROWB;
    char* Vb = (char*)a.V + x.ubase * ROWB;

    float m_run = -INFINITY, l_run = 0.f;                 // head j (replicated over q; l_run is this lane's share)
    f32x4 O[VS][8];                                       // heads 4q .. 4q+3 of columns 8 (16 t + j) + m
#pragma unroll
    for (int t = 0; t < VS; ++t) {
#pragma unroll
        for (int mcol = 0; mcol < 8; ++mcol) O[t][mcol] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    struct Buf { u32x4 k[QP], v[VS][4]; };
    const TileMap<WROWS, ANCHOR> tiles(a, x);
    // row i of a tile, counted from its run's first row; outside the run its nearest row again
    auto row = [&](const Tile& k, int i) { return (unsigned)(ANCHOR ? min(max(k.base + i, k.lead), k.cnt - 1) - k.lead : min(k.base + i, k.cnt - 1)); };
    auto load_t = [&](u32x4 (&kk)[QP], u32x4 (&vv)[VS][4], int t) {
        const Tile k = tiles.locate(t);
        const char* kp = k.fresh ? (const char*)a.k_new + (size_t)unit * ROWB : Kb + (size_t)k.phys * ROWB;
        const char* vp = k.fresh ? (const char*)a.v_new + (size_t)unit * ROWB : Vb + (size_t)k.phys * ROWB;
        const unsigned krow = row(k, j) * ROWB;
#pragma unroll
        for (int p = 0; p < QP; ++p) kk[p] = load16<NT>(kp + (unsigned)(krow + (4 * p + q) * 16));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned vrow = row(k, 4 * q + e) * ROWB;
#pragma unroll
            for (int t2 = 0; t2 < VS; ++t2) vv[t2][e] = load16<NT>(vp + (unsigned)(vrow + ((16 * t2 + j) % NCH) * 16));
            // The two halves of a 512-byte row one behind the other: left to itself the compiler loads all rows' first halves,
            // then the second (per step, 36 units of 5900 bf16 rows, 8 heads 43.0 us, 41.4 so; 240 of 985, 6 heads 44.6 / 42.6).
            if constexpr (VS > 1) __builtin_amdgcn_sched_barrier(0x38F);   // everything but accesses to memory may cross
        }
    };

    auto compute_t = [&](const u32x4 (&kk)[QP], const u32x4 (&vv)[VS][4], const Tile& k) {
        const int stg = k.lo - j0 + k.base - k.lead;      // staging index (row relative to the split's first row)
        f32x4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < QP; ++p) sacc = Mma<T>::qk(kk[p], qb[p], sacc);
        float s[4];
        float tmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool ok = k.base + 4 * q + v < k.cnt && (!ANCHOR || k.base + 4 * q + v >= k.lead);
            const float d = sacc[v] * a.scale_log2;
            s[v] = ok ? d : -INFINITY;
            if (ok && j < G) stage[j * a.rows_per_split + stg + 4 * q + v] = d;
            tmax = fmaxf(tmax, s[v]);
        }
        tmax = pair_max<32>(pair_max<16>(tmax));
        const float mn = fmaxf(m_run, tmax);
        const float mref = (mn == -INFINITY) ? 0.f : mn;
        const float alpha = fast_exp2(m_run - mref);
        m_run = mn;
        unsigned hi[4], lo[4];
        float psum = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float pr = fast_exp2(s[v] - mref);
            Mma<T>::split(pr, hi[v], lo[v]);
            psum += pr;
        }
        l_run = fmaf(l_run, alpha, psum);
        const u32x2 p_hi = {hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
        const u32x2 p_lo = {lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
        if (__any(alpha != 1.0f)) {                       // a running maximum moved: rescale the outputs
            float av[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) av[v] = __shfl(alpha, (4 * q + v) & 15);   // head 4q+v lives in lane 4q+v
#pragma unroll
            for (int t = 0; t < VS; ++t) {
#pragma unroll
                for (int mcol = 0; mcol < 8; ++mcol) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) O[t][mcol][v] *= av[v];
                }
            }
        }
#pragma unroll
        for (int t = 0; t < VS; ++t) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {                 // dword w of the chunk = columns 2w and 2w+1
                const unsigned r0 = vv[t][0][w], r1 = vv[t][1][w], r2 = vv[t][2][w], r3 = vv[t][3][w];
                const u32x2 even = {(r0 & 0xffffu) | (r1 << 16), (r2 & 0xffffu) | (r3 << 16)};
                const u32x2 odd = {(r0 >> 16) | (r1 & 0xffff0000u), (r2 >> 16) | (r3 & 0xffff0000u)};
                O[t][2 * w] = Mma<T>::pv(p_hi, even, O[t][2 * w]);
                O[t][2 * w] = Mma<T>::pv(p_lo, even, O[t][2 * w]);
                O[t][2 * w + 1] = Mma<T>::pv(p_hi, odd, O[t][2 * w + 1]);
                O[t][2 * w + 1] = Mma<T>::pv(p_lo, odd, O[t][2 * w + 1]);
            }
        }
    };

    SideRows<G, SHORT ? 1 : side_rows<G>()> side;
    auto requests = [&] {
        request_prev_stat(a, unit, side);
        request_side_rows<G, NW * 64>(a, x, 0, side);
        request_fresh_row<ROWB>(a, x, side);
    };
    if constexpr (SHORT) {
        const char* kn = (const char*)a.k_new + (size_t)unit * ROWB;
        const char* vn = (const char*)a.v_new + (size_t)unit * ROWB;
        Buf b[SHORT];
#pragma unroll
        for (int i = 0; i < SHORT; ++i) {
            const ShortTile<WROWS> own(x, wave + i * NW);
            if (!own.exists()) break;
            const unsigned koff = (unsigned)a.map.phys(own.row(j)) * ROWB + q * 16;
#pragma unroll
            for (int p = 0; p < QP; ++p) b[i].k[p] = load16<NT>(Kb + (unsigned)(koff + p * 64));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned voff = (unsigned)a.map.phys(own.row(4 * q + e)) * ROWB;
#pragma unroll
                for (int t2 = 0; t2 < VS; ++t2) b[i].v[t2][e] = load16<NT>(Vb + (unsigned)(voff + ((16 * t2 + j) % NCH) * 16));
            }
            if (own.last(x, a.n)) {                       // the new row is still the caller's
                if (own.row(j) == a.n - 1) {
#pragma unroll
                    for (int p = 0; p < QP; ++p) b[i].k[p] = load16<NT>(kn + (unsigned)(q * 16 + p * 64));
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (own.row(4 * q + e) == a.n - 1) {
#pragma unroll
                        for (int t2 = 0; t2 < VS; ++t2) b[i].v[t2][e] = load16<NT>(vn + (unsigned)((16 * t2 + j) % NCH * 16));
                    }
                }
            }
        }
        requests();
#pragma unroll
        for (int i = 0; i < SHORT; ++i) {
            const ShortTile<WROWS> own(x, wave + i * NW);
            if (own.exists()) compute_t(b[i].k, b[i].v, own.tile());
        }
    } else {
        stream_tiles<false, false, Buf>(a, &sm.next_tile, wave, NW, tiles.total(), [&](Buf& b, int t) { load_t(b.k, b.v, t); }, requests, [&](Buf& b, int t) { compute_t(b.k, b.v, tiles.locate(t)); });
    }

    if (lane == 0) BUZZ_STAMP(8 + (wave & 7));
    // this wave's result into LDS
    const float l_tot = pair_sum<32>(pair_sum<16>(l_run));
    if (q == 0 && j < G) sm.ml[j][wave] = make_float2(m_run, l_tot);
#pragma unroll
    for (int t2 = 0; t2 < VS; ++t2) {
        if (16 * t2 + j < NCH) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (4 * q + v < G) {
                    float* dst = &sm.acc[wave][4 * q + v][8 * (16 * t2 + j)];
                    *(f32x4*)dst = f32x4{O[t2][0][v], O[t2][1][v], O[t2][2][v], O[t2][3][v]};
                    *(f32x4*)(dst + 4) = f32x4{O[t2][4][v], O[t2][5][v], O[t2][6][v], O[t2][7][v]};
                }
            }
        }
    }
    finish_split<G, D, NW, ROWB, SHORT != 0>(a, x, side, stage, sm);
}

constexpr int kScoreRowsPerBlock = 2048;

// Applies the pending score update of the last decode step to every retained row right away.
template <int G>
__global__ __launch_bounds__(256) void flush_scores_kernel(const AttnArgs a)
{
    const int chunk = blockIdx.x, unit = blockIdx.y, tid = threadIdx.x;
    float M[G], iL[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        M[g] = a.stat_prev[((size_t)unit * G + g) * 2];
        iL[g] = a.stat_prev[((size_t)unit * G + g) * 2 + 1];
    }
    const size_t ubase = (size_t)unit * a.cap;
    const float* logit_u = a.logit_prev + ubase * G;
    const int jbeg = chunk * kScoreRowsPerBlock;
    const int jend = min(a.n, jbeg + kScoreRowsPerBlock);
    for (int j = jbeg + tid; j < jend; j += 256) {
        const int ph = a.map.phys(j);
        float sc = a.score[ubase + ph];
#pragma unroll
        for (int g = 0; g < G; ++g) sc = add_probability(sc, logit_u[(size_t)g * a.cap + ph], M[g], iL[g]);
        a.score[ubase + ph] = sc;
    }
}

template <int G, bool NT> constexpr int unroll_for()
{
    return G == 1 ? (NT ? BUZZ_U_G1 : BUZZ_U_G1_CACHED) : (G == 2 ? BUZZ_U_G2 : (G <= 4 ? BUZZ_U_G4 : BUZZ_U_G8));
}

// Launches a decode kernel so that its blocks come out even.  Of `fit` blocks that a compute unit holds at a time, two
// rounds may leave the second one nearly empty, while one block less at a time takes as many rounds of equal work (what
// bounds the blocks is memory, which fewer of them saturate as well).  Then more LDS is asked for than is used, so that
// fewer fit.  1024 blocks (512 units, 2 splits of 2500 rows, 2 heads of 128): 3 at a time 268 us, 2 at a time 226; 1000
// units of 1000 rows: 108 and 95; 1000 units of 800 rows, 5 heads: 92 and 85.  From three rounds on the blocks' ends
// spread by themselves (2000 units of 300 rows: 65 us, 69 with fewer), and short blocks hide each other's starts and
// ends (1024 units of 200 rows: 20.9 us, 22.0 with fewer).  On the vector ALU up to 4 heads: 1280 units of 700 fp32 rows,
// 4 heads of 128: 185 and 172 us; 512 units of 1200, 8 heads of 64, which are not bound by memory: 92, 98 with fewer.
constexpr int kEvenRows = 512;                             // rows per split from which it counts
constexpr int kLdsPerUnit = 160 * 1024;                    // bytes of LDS of a compute unit

template <void (*kernel)(AttnArgs)>
void launch_even(const dim3& grid, const dim3& block, size_t lds, hipStream_t st, Timing tm, const AttnArgs& a)
{
    struct Footprint { int fit = 0; int64_t lds = 0; };    // resident blocks by registers, bytes of static LDS
    static const Footprint own = [&] {
        Footprint f;
        hipFuncAttributes attr{};
        int fit = 0;
        if (hipFuncGetAttributes(&attr, (const void*)kernel) == hipSuccess &&
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, (const void*)kernel, (int)block.x, 0) == hipSuccess) {
            f.fit = fit;
            f.lds = (int64_t)attr.sharedSizeBytes;
        }
        return f;
    }();
    const int64_t blocks = (int64_t)grid.x * grid.y * grid.z, per = (blocks + a.compute_units - 1) / a.compute_units;
    const int64_t fit = std::min<int64_t>(own.fit, kLdsPerUnit / (own.lds + (int64_t)lds + 1));
    auto share = [&](int64_t at_a_time) { return (per + at_a_time - 1) / at_a_time * at_a_time; };   // of blocks, empty places included
    if (a.rows_per_split >= kEvenRows && fit > 2 && per > fit && per <= 2 * fit) {
        int64_t best = fit;
        for (int64_t n = fit - 1; n >= 2; --n)
            if (share(n) < share(best)) best = n;
        const int64_t need = kLdsPerUnit / (best + 1) + 1;   // one block more does not fit
        if (best < fit && need <= 65536) lds = std::max<int64_t>((int64_t)lds, need - own.lds);
    }
    BUZZ_LAUNCH(kernel, grid, block, lds, st, tm, a);
}

// Streaming matrix-core kernels anchor their tiles where rows are 256 bytes or more and a split is long enough for the
// partial tile at each end not to count.  Tiles of 4 KB that straddle two aligned ones were up to 3% slower: 512 units of
// 2000 rows, 2 heads of 128: 86.8 us anchored, 88.1 not; 32 units of 20000 rows, 4 heads: 76.0 and 78.2.  With 350 rows per
// split the partial tiles and the masks cost 1%, with rows of 128 bytes 3%, from the last-level cache up to 8%.
constexpr int kAnchorRows = 1024;

template <typename T, int D, int G>
hipError_t launch_split_t(const AttnArgs& a, int units, hipStream_t st, Timing tm)
{
    const dim3 grid = a.xcd_local ? dim3(8, a.n_splits, units / 8) : dim3(a.n_splits, units), block(a.waves * 64);
    const size_t lds = (size_t)G * a.rows_per_split * sizeof(float);   // logit staging
    constexpr bool MATRIX = G >= 2 && !std::is_same<T, float>::value;   // grouped queries on a 16-bit cache: matrix cores
    constexpr int ROWB = D * (int)sizeof(T), TILE = short_tile_rows(MATRIX, G, ROWB);
    const int at_once = short_rows(MATRIX, G, D, ROWB, a.waves, step_bytes(units, a.n, ROWB), a.cap, a.streaming);
    auto is_short = [&](int tiles) { return a.rows_per_split <= at_once && a.rows_per_split <= tiles * TILE * a.waves; };
    if constexpr (MATRIX) {
        auto launch = [&](auto nt, auto nw, auto anchor) {
            launch_even<attn_split_mfma_kernel<T, D, G, decltype(nt)::value, decltype(nw)::value, decltype(anchor)::value, 0>>(grid, block, lds, st, tm, a);
        };
        auto flavour = [&](auto nw) {
            constexpr int NW = decltype(nw)::value;
            if (is_short(1)) { BUZZ_LAUNCH((attn_split_mfma_kernel<T, D, G, false, NW, false, 1>), grid, block, lds, st, tm, a); return; }
            if (!a.streaming) { launch(std::false_type{}, nw, std::false_type{}); return; }
            if constexpr (D >= 128) {
                if (a.rows_per_split >= kAnchorRows) { launch(std::true_type{}, nw, std::true_type{}); return; }
            }
            launch(std::true_type{}, nw, std::false_type{});
        };
        if (a.waves == 8) flavour(std::integral_constant<int, 8>{});
        else flavour(std::integral_constant<int, 4>{});
        return hipGetLastError();
    } else {
        constexpr int RPW = 64 / (D / Elem<T>::VEC);
        // a trip covers at least 4 rows
        constexpr int US = unroll_for<G, true>() * RPW >= 4 ? unroll_for<G, true>() : 4 / RPW;     // streaming loads
        constexpr int UC = unroll_for<G, false>() * RPW >= 4 ? unroll_for<G, false>() : 4 / RPW;   // cached loads
        constexpr int UH = TILE / RPW;                    // short splits
        const int64_t blocks = (int64_t)grid.x * grid.y * grid.z;
        auto launch_as = [&](auto nt, auto nw, auto u, auto tile_first, auto via_lds) {
            constexpr auto kernel = attn_split_kernel<T, D, G, decltype(u)::value, decltype(nt)::value, decltype(nw)::value, 0, decltype(tile_first)::value, decltype(via_lds)::value>;
            if constexpr (G <= 4) launch_even<kernel>(grid, block, lds, st, tm, a);
            else BUZZ_LAUNCH(kernel, grid, block, lds, st, tm, a);   // the vector ALU bounds these
        };
        auto launch = [&](auto nt, auto nw, auto u, auto tile_first) {
            // Of 2 to 2.5 blocks per compute unit, those that are three on one end last, the more the less time a block's loop takes beside
            // its loads.  Where memory and arithmetic are about even the lanes' exchange through LDS evens them: 516 to 600 units of
            // 3 fp32 heads of 256 take 3 to 10% less time so (520 of 319 rows 72.8 -> 62.8 us), of 4 of 128 2 to 5% (560 of 809 94.3 ->
            // 86.7); 512 units 5 and 3% more, 700 1%, 4 heads of 256 on 560 units 6%; 3 of 128 1% either way, 2 heads 1 to 3% more;
            // splits of less than 64 KB of K 1% more.
            if constexpr (decltype(nw)::value == 4 && (G == 3 || G == 4) && G * D >= 512 && G * D < 1024) {
                if (blocks > 2 * a.compute_units && 2 * blocks <= 5 * a.compute_units && a.rows_per_split * ROWB >= 65536) { launch_as(nt, nw, u, tile_first, std::true_type{}); return; }
            }
            launch_as(nt, nw, u, tile_first, std::false_type{});
        };
        auto flavour = [&](auto nw) {
            constexpr int NW = decltype(nw)::value;
            constexpr int TILES = short_tiles(MATRIX, G, ROWB, NW);
            // whether the first tile's loads go before the side requests: figures on both sides of each line at stream_tiles
            auto stream = [&](auto nt, auto u) {
                constexpr bool NT = decltype(nt)::value, TWO_LOADS = decltype(u)::value == 1, WIDEST = RPW == 1;
                if constexpr (G > 1) launch(nt, nw, u, std::false_type{});
                else if constexpr (TWO_LOADS) launch(nt, nw, u, std::true_type{});
                else if constexpr (NW == 8) launch(nt, nw, u, std::bool_constant<WIDEST && !NT>{});
                else {
                    const bool crowd = 5 * blocks >= 8 * a.compute_units;
                    if (WIDEST ? !crowd : crowd && blocks <= 4 * a.compute_units) launch(nt, nw, u, std::true_type{});
                    else launch(nt, nw, u, std::false_type{});
                }
            };
            if (a.streaming) stream(std::true_type{}, std::integral_constant<int, US>{});
            else if (is_short(1)) BUZZ_LAUNCH((attn_split_kernel<T, D, G, UH, false, NW, 1, false, false>), grid, block, lds, st, tm, a);
            else if (TILES >= 2 && is_short(2)) BUZZ_LAUNCH((attn_split_kernel<T, D, G, UH, false, NW, (TILES >= 2 ? 2 : 1), false, false>), grid, block, lds, st, tm, a);
            else if (TILES >= 3 && is_short(3)) BUZZ_LAUNCH((attn_split_kernel<T, D, G, UH, false, NW, TILES, false, false>), grid, block, lds, st, tm, a);
            else stream(std::false_type{}, std::integral_constant<int, UC>{});
        };
        if (a.waves == 8) flavour(std::integral_constant<int, 8>{});
        else flavour(std::integral_constant<int, 4>{});
        return hipGetLastError();
    }
}

template <typename T, int D>
hipError_t launch_split_g(int G, const AttnArgs& a, int units, hipStream_t st, Timing tm)
{
    switch (G) {
        case 1: return launch_split_t<T, D, 1>(a, units, st, tm);
        case 2: return launch_split_t<T, D, 2>(a, units, st, tm);
        case 3: return launch_split_t<T, D, 3>(a, units, st, tm);
        case 4: return launch_split_t<T, D, 4>(a, units, st, tm);
        case 5: return launch_split_t<T, D, 5>(a, units, st, tm);
        case 6: return launch_split_t<T, D, 6>(a, units, st, tm);
        case 7: return launch_split_t<T, D, 7>(a, units, st, tm);
        case 8: return launch_split_t<T, D, 8>(a, units, st, tm);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_split_d(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm)
{
    switch (D) {
        case 64: return launch_split_g<T, 64>(G, a, units, st, tm);
        case 128: return launch_split_g<T, 128>(G, a, units, st, tm);
        case 256: return launch_split_g<T, 256>(G, a, units, st, tm);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// This file is compiled four times (BUZZ_TU = 0, 1, 2: the streaming kernels of one dtype each;
// BUZZ_TU = 3: everything that does not depend on the dtype), so that the build runs in parallel.
#ifndef BUZZ_TU
#error "compile with -DBUZZ_TU=0..3 (see build.py)"
#endif
#if BUZZ_TU == 0
hipError_t launch_attn_split_fp32(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm) { return launch_split_d<float>(D, G, a, units, st, tm); }
#elif BUZZ_TU == 1
hipError_t launch_attn_split_fp16(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm) { return launch_split_d<fp16_t>(D, G, a, units, st, tm); }
#elif BUZZ_TU == 2
#ifdef BUZZ_TRACE
}  // namespace buzz
extern "C" int buzz_debug_trace_read(void* host, size_t bytes)
{
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(buzz::g_trace), bytes, 0, hipMemcpyDeviceToHost);
}
namespace buzz {
#endif
hipError_t launch_attn_split_bf16(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm) { return launch_split_d<bf16_t>(D, G, a, units, st, tm); }
#else
hipError_t launch_attn_split_fp32(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm);
hipError_t launch_attn_split_fp16(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm);
hipError_t launch_attn_split_bf16(int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm);

bool attn_supported(int dtype, int D, int G)
{
    if (dtype != BUZZ_FP32 && dtype != BUZZ_FP16 && dtype != BUZZ_BF16) return false;
    if (D != 64 && D != 128 && D != 256) return false;
    return G >= 1 && G <= 8;
}

int attn_tile_rows(int dtype, int D, int G)
{
    const int vec = dtype == BUZZ_FP32 ? 4 : 8;
    const int rpw = 64 / (D / vec);
    if (G >= 2 && dtype != BUZZ_FP32) return 16;          // matrix-core kernel: 16-row tiles
    int u = G == 1 ? BUZZ_U_G1_CACHED : (G == 2 ? BUZZ_U_G2 : (G <= 4 ? BUZZ_U_G4 : BUZZ_U_G8));
    if (u * rpw < 4) u = 4 / rpw;
    return rpw * u;                                       // rows of one wave-wide trip
}

hipError_t launch_attn_split(int dtype, int D, int G, const AttnArgs& a, int units, hipStream_t st, Timing tm)
{
    switch (dtype) {
        case BUZZ_FP32: return launch_attn_split_fp32(D, G, a, units, st, tm);
        case BUZZ_FP16: return launch_attn_split_fp16(D, G, a, units, st, tm);
        case BUZZ_BF16: return launch_attn_split_bf16(D, G, a, units, st, tm);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_flush_scores(int G, const AttnArgs& a, int units, hipStream_t st, Timing tm)
{
    if (a.n <= 0) return hipSuccess;
    dim3 grid((a.n + kScoreRowsPerBlock - 1) / kScoreRowsPerBlock, units), block(256);
    switch (G) {
        case 1: BUZZ_LAUNCH((flush_scores_kernel<1>), grid, block, 0, st, tm, a); break;
        case 2: BUZZ_LAUNCH((flush_scores_kernel<2>), grid, block, 0, st, tm, a); break;
        case 3: BUZZ_LAUNCH((flush_scores_kernel<3>), grid, block, 0, st, tm, a); break;
        case 4: BUZZ_LAUNCH((flush_scores_kernel<4>), grid, block, 0, st, tm, a); break;
        case 5: BUZZ_LAUNCH((flush_scores_kernel<5>), grid, block, 0, st, tm, a); break;
        case 6: BUZZ_LAUNCH((flush_scores_kernel<6>), grid, block, 0, st, tm, a); break;
        case 7: BUZZ_LAUNCH((flush_scores_kernel<7>), grid, block, 0, st, tm, a); break;
        case 8: BUZZ_LAUNCH((flush_scores_kernel<8>), grid, block, 0, st, tm, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
#endif  // BUZZ_TU

}  // namespace buzz
