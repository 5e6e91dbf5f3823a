// BeeHive eviction kernels (Sec. 3.3; the eviction branch of Alg. 1, Alg. 2):
//   segment_topk : one wavefront per (segment, unit) ranks the segment's accumulated scores and
//                  emits the top min(keep, len) rows in index order (ties -> lowest index, NaN lowest),
//                  one block per (segment, unit) where segments are long;
//   place_sampled: the same and the placement of a prompt in one launch;
//   gather_rows  : packs K, V, score and position of selected rows into their destination
//                  (survivors behind the old region, sink / window at prefill, export in cache order).
// Every segment yields min(keep, len) rows, so a survivor's destination is
// segment * keep + (rank among the segment's survivors): a wave-level prefix sum over the keep mask.
#include "buzz_internal.h"

namespace buzz {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSelWaves = 4;

// A wave's slice of the LDS, in floats: the ranking reads four scores at a time.
__host__ __device__ inline int wave_slice(int floats) { return (floats + 3) & ~3; }

// Ranks the len scores that a wave has put into its LDS slice (16-byte aligned; up to three more
// floats are read behind them and not used) and calls emit(rank among the survivors, offset) for its `take` >= 1 best: score descending, ties to
// the lowest offset, survivors numbered in offset order.  (A rank may be given out twice; the last one counts.)  A row
// survives if fewer than `take` rows are larger: one comparison and one addition per pair of rows, which is what bounds
// the kernel.  That count keeps too many rows only where equal scores straddle the boundary.  The last survivor's score
// is then the one that the most rows are larger than among the kept, its equals share the places that the larger rows
// leave, and a pass that only compares with that score numbers them: a tie costs one step per 64 rows.
// 448 segments of 64 in each of 32 units: 12.7 us with the tie-breaker in every comparison, 9 us now.  One segment of 1000
// rows in each of 32 units, evicted in place: 175 us with distinct scores and with equal ones, for which ties took 2.8 times
// as long when they were a second pass of comparisons.  (Where a launch of its own selects, a block takes such segments.)
template <typename Emit>
__device__ inline void rank_segment(const float* sc, int len, int take, int lane, Emit emit)
{
    const unsigned long long below = (1ull << lane) - 1ull;
    const int rows = __builtin_amdgcn_readfirstlane(len);
    auto larger_than = [&](float v) {              // rows of the segment
        int n = 0;
        auto count = [&](const float4& x) { n += x.x > v; n += x.y > v; n += x.z > v; n += x.w > v; };
        int i = 0;
#pragma unroll 1
        for (; i + 16 <= rows; i += 16) {        // four reads in flight: a wave is often alone on its SIMD
            float4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = *(const float4*)(sc + i + 4 * u);
#pragma unroll
            for (int u = 0; u < 4; ++u) count(x[u]);
        }
#pragma unroll 1
        for (; i + 4 <= rows; i += 4) count(*(const float4*)(sc + i));
        if (i < rows) {
            const float4 x = *(const float4*)(sc + i);
            n += x.x > v;
            if (i + 1 < rows) n += x.y > v;
            if (i + 2 < rows) n += x.z > v;
        }
        return n;
    };
    auto wave_max = [](int v) {
        for (int off = 32; off; off >>= 1) v = max(v, __shfl_xor(v, off));
        return v;
    };
    if (rows <= 64) {
        const int larger = larger_than(lane < len ? sc[lane] : 0.f);
        bool kp = lane < len && larger < take;
        unsigned long long mask = __ballot(kp);
        if (__popcll(mask) != take) {              // equal scores across the boundary: the first of them fill it
            const int top = wave_max(kp ? larger : -1);
            const unsigned long long ties = __ballot(kp && larger == top);
            kp = kp && (larger < top || __popcll(ties & below) < take - top);
            mask = __ballot(kp);
        }
        if (kp) emit(__popcll(mask & below), lane);
        return;
    }
    int kept = 0, most = -1;                       // of the rows that this lane would keep, the one with most larger rows:
    float last = 0.f;                              // ... how many, and its score
#pragma unroll 1
    for (int e0 = 0; e0 < rows; e0 += 64) {
        const int e = e0 + lane;
        const float v = e < len ? sc[e] : 0.f;
        const int larger = larger_than(v);
        const bool kp = e < len && larger < take;
        const unsigned long long mask = __ballot(kp);
        const int r = kept + __popcll(mask & below);
        if (kp && r < take) emit(r, e);
        if (kp && larger > most) { most = larger; last = v; }
        kept += __popcll(mask);
    }
    if (kept == take) return;
    // equal scores across the boundary: every survivor again
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int top = wave_max(most);
    const float bound = __shfl(last, __ffsll(__ballot(most == top)) - 1);
    const int room = take - top;                   // rows that equal the bound and survive
    int equal = 0;
    kept = 0;
#pragma unroll 1
    for (int e0 = 0; e0 < rows; e0 += 64) {
        const int e = e0 + lane;
        const float v = e < len ? sc[e] : -INFINITY;
        const unsigned long long ties = __ballot(e < len && v == bound);
        const bool kp = e < len && (v > bound || (v == bound && equal + __popcll(ties & below) < room));
        const unsigned long long mask = __ballot(kp);
        if (kp) emit(kept + __popcll(mask & below), e);
        kept += __popcll(mask);
        equal += __popcll(ties);
    }
}

__global__ __launch_bounds__(256) void segment_topk_kernel(const SelectArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // [kSelWaves][wave_slice(segment)]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seg = blockIdx.x * kSelWaves + wave, unit = blockIdx.y;
    const int n_seg = (a.new_count + a.segment - 1) / a.segment;
    const bool active = seg < n_seg;
    const int start = seg * a.segment;
    const int len = active ? min(a.segment, a.new_count - start) : 0;
    const int take = min(a.keep, len);
    float* sc = lds + wave * wave_slice(a.segment);
    const float* base = a.score + (size_t)unit * a.unit_stride;
    int* out = a.sel + (size_t)unit * a.sel_stride + seg * a.keep;
    if (a.ignore_scores) {                         // all equal: the lowest indices win
        for (int e = lane; e < take; e += 64) out[e] = a.lo + start + e;
        return;
    }
    if (!active) return;                           // no block-wide barrier below: a wave only reads what it wrote
    for (int e = lane; e < len; e += 64) {
        const int row = a.lo + start + e;
        float v = base[a.map.ring_cap ? a.map.phys(row) : row];
        if (v != v) v = -INFINITY;                 // NaN ranks below everything
        sc[e] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    rank_segment(sc, len, take, lane, [&](int r, int e) { out[r] = a.lo + start + e; });
}

// Long segments, the single segment of the H2O-style variant among them, which spans every row between sink and window:
// one block per (segment, unit) finds the `take` largest scores by a radix select on the order-preserving integer image of
// the scores -- up to three passes of a histogram in LDS, most significant digit first, each narrowing the candidates to
// one bin -- which ends with the digits of the last survivor's key and the number of rows with these digits that still
// fit.  Every row above survives and the first of the equal ones do (ties go to the lowest index).  Same result as the wave
// kernel, whose work grows with the square of the length.
// A wave takes a contiguous run of the rows, 64 at a time, so that rows are numbered by ballots and two counts per wave,
// without a barrier per 1024 rows.  Up to 32 of a wave's rounds stay in registers (segments of 32768 rows; 21688 rows in 16
// units, prefill and export: 66.7 us so, 81 read again in each pass); longer segments are read again, 16 rounds in flight.
// Digits of 11 bits keep the exponent and two more bits in the first: a prompt's scores then spread over a few dozen bins,
// where one byte puts nearly all of them into four, on whose counters the lanes of a wave queue.  (32 units of 4000 rows in
// one segment, prefill: 20.5 us with scores of three values, 26 with equal ones.)
constexpr int kTopkBlock = 1024, kTopkWaves = kTopkBlock / 64, kTopkBins = 2048;

__device__ inline unsigned score_key(float v)      // larger score <=> larger key; NaN ranks with -inf; -0 == +0
{
    if (v != v) v = -INFINITY;
    const unsigned b = __float_as_uint(v + 0.0f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

template <int ROUNDS, bool HELD>
__global__ __launch_bounds__(kTopkBlock) void segment_topk_block_kernel(const SelectArgs a)
{
    __shared__ int hist[kTopkBins];
    __shared__ int wave_sum[kTopkWaves], wave_equal[kTopkWaves];
    __shared__ unsigned sh_prefix;
    __shared__ int sh_remaining, sh_all;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), seg = blockIdx.x, unit = blockIdx.y;
    const unsigned long long below = (1ull << lane) - 1ull;
    const long long start = (long long)seg * a.segment;
    const int len = (int)min((long long)a.segment, (long long)a.new_count - start);
    const int take = min(a.keep, len);
    if (take <= 0) return;
    const float* base = a.score + (size_t)unit * a.unit_stride;
    const int run = ((len + kTopkWaves - 1) / kTopkWaves + 63) & ~63, first = wave * run, last = min(len, first + run);   // this wave's rows
    auto key_of = [&](int e) {
        const int row = a.lo + (int)start + min(e, len - 1);
        return a.ignore_scores ? 0x80000000u : score_key(base[a.map.ring_cap ? a.map.phys(row) : row]);
    };
    unsigned held[ROUNDS];
    auto load = [&](int e0) {
#pragma unroll
        for (int i = 0; i < ROUNDS; ++i) held[i] = key_of(e0 + 64 * i + lane);
    };
    if (HELD) load(first);
    // f(key, row) for this wave's rows, in order
    auto for_rows = [&](auto f) {
#pragma unroll 1
        for (int e0 = first; e0 < last; e0 += 64 * ROUNDS) {
            if (!HELD) load(e0);
#pragma unroll
            for (int i = 0; i < ROUNDS; ++i) {
                if (e0 + 64 * i >= last) break;
                f(held[i], e0 + 64 * i + lane);
            }
        }
    };
    // after the pass for a digit, `prefix` holds the digits so far of the last survivor's key and `remaining` how many
    // rows are still to be taken among those that share them
    unsigned prefix = 0, mask = 0;
    int remaining = take;
#pragma unroll 1
    for (int shift = 21; shift >= -1; shift -= 11) {        // bits 31..21, 20..10, 9..0
        const int at = max(shift, 0);
        const unsigned digit = shift < 0 ? 1023u : 2047u;
        for (int i = tid; i < kTopkBins; i += kTopkBlock) hist[i] = 0;
        __syncthreads();
        for_rows([&](unsigned k, int e) { if (e < last && (k & mask) == prefix) atomicAdd(&hist[(k >> at) & digit], 1); });
        __syncthreads();
        // the bin where the count from the largest digit down reaches `remaining`: a suffix sum, two bins per thread
        const int low = hist[2 * tid], high = hist[2 * tid + 1];
        int upto = low + high;                             // this lane's bins and those above, in the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_down(upto, off);
            if (lane + off < 64) upto += v;
        }
        if (lane == 0) wave_sum[wave] = upto;
        __syncthreads();
        for (int w = wave + 1; w < kTopkWaves; ++w) upto += wave_sum[w];
        const int above = upto - low - high;
        if (above < remaining && remaining <= upto) {
            const bool in_high = above + high >= remaining;
            sh_prefix = prefix | ((unsigned)(2 * tid + (in_high ? 1 : 0)) << at);
            sh_remaining = remaining - above - (in_high ? 0 : high);
            sh_all = sh_remaining == (in_high ? high : low);
        }
        __syncthreads();
        prefix = sh_prefix; remaining = sh_remaining;
        mask |= digit << at;
        if (sh_all) break;                                 // every row of the bin survives
    }
    // rows with larger digits and the first `remaining` with equal ones
    int n_larger = 0, n_equal = 0;
    for_rows([&](unsigned k, int e) {
        n_larger += __popcll(__ballot(e < last && (k & mask) > prefix));
        n_equal += __popcll(__ballot(e < last && (k & mask) == prefix));
    });
    __syncthreads();                                       // wave_sum is read above
    if (lane == 0) { wave_sum[wave] = n_larger; wave_equal[wave] = n_equal; }
    __syncthreads();
    int equal = 0, kept = 0;                               // before this wave's run
    for (int w = 0; w < wave; ++w) {
        kept += wave_sum[w] + min(max(remaining - equal, 0), wave_equal[w]);
        equal += wave_equal[w];
    }
    int* out = a.sel + (size_t)unit * a.sel_stride + (size_t)seg * a.keep;
    for_rows([&](unsigned k, int e) {
        const unsigned long long ties = __ballot(e < last && (k & mask) == prefix);
        const bool keeps = e < last && ((k & mask) > prefix || ((k & mask) == prefix && equal + __popcll(ties & below) < remaining));
        const unsigned long long kept_here = __ballot(keeps);
        if (keeps) out[kept + __popcll(kept_here & below)] = a.lo + (int)start + e;
        kept += __popcll(kept_here);
        equal += __popcll(ties);
    });
}

// Eviction of the new rows in one launch, for caches whose old rows stay in place.  A wave ranks one segment
// as above and then moves the segment's survivors itself (their destination depends on nothing but the
// segment number and the rank).  A score update that the last decode step left pending is applied on the fly
// to the rows of the segment -- nothing else needs it now: every other retained row keeps its physical place,
// and the next decode step applies the update there as it would have without an eviction.  A survivor arrives
// with its updated score, and its entry in that step's logit buffer is set to -inf so that the next step
// adds exactly 0 for it.
// Bound by latency: a chain of round trips to memory.  All of a row's logits are requested with its score, the statistics
// once per wave, and the survivors' scores are those that were ranked.  (With a loop over the heads each logit waited for
// the one before it, once to rank and again to move: 8 units, 32 rows, 8 heads of 128, 4.6 us per eviction, now 3.0; 32
// units of 64 rows, 4 heads, 6.4 and 4.2; 8 of 16 rows, one head of 64, 3.3 and 3.0.)
template <int G>
__global__ __launch_bounds__(256) void evict_new_rows_kernel(const EvictArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // [kSelWaves][wave_slice(segment + keep)]: scores, then kept offsets
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seg = blockIdx.x * kSelWaves + wave, unit = blockIdx.y;
    const int n_seg = (a.new_count + a.segment - 1) / a.segment;
    if (seg >= n_seg) return;                      // no block-wide barrier below: a wave only reads what it wrote
    const int start = seg * a.segment;
    const int len = min(a.segment, a.new_count - start);
    const int take = min(a.keep, len);
    float* sc = lds + wave * wave_slice(a.segment + a.keep);
    int* kept = (int*)sc + a.segment;
    const size_t ubase = (size_t)unit * a.cap;
    const float* logit_u = a.logit_prev + ubase * G;
    float stat[2 * G];
#pragma unroll
    for (int i = 0; i < 2 * G; ++i) stat[i] = a.stat_prev[(size_t)unit * 2 * G + i];   // (read but not used where nothing is pending)
    auto current_score = [&](int ph) {             // the row's score with the pending update applied
        float v = a.score[ubase + ph];
        if (a.logit_prev) {
            float logit[G];
#pragma unroll
            for (int g = 0; g < G; ++g) logit[g] = logit_u[(size_t)g * a.cap + ph];
#pragma unroll
            for (int g = 0; g < G; ++g) v = add_probability(v, logit[g], stat[2 * g], stat[2 * g + 1]);
        }
        return v;
    };
    if (a.ignore_scores) {                         // all equal: the lowest indices win
        for (int r = lane; r < take; r += 64) kept[r] = r;
    } else {
        for (int e = lane; e < len; e += 64) {
            float v = current_score(a.map.phys(a.lo + start + e));
            if (v != v) v = -INFINITY;             // NaN ranks below everything
            sc[e] = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        rank_segment(sc, len, take, lane, [&](int r, int e) { kept[r] = e; });
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // move the survivors: 16 bytes per lane, 64 / lpr rows per pass
    const int lpr = a.row_bytes >> 4;              // lanes per row (at most 64)
    const int c = lane % lpr, rr = lane / lpr, rows_per_pass = 64 / lpr;
    for (int r = rr; r < take; r += rows_per_pass) {
        const int sp = a.map.phys(a.lo + start + kept[r]);
        const int dp = a.dst_start + seg * a.keep + r;
        const size_t so = (ubase + sp) * a.row_bytes + c * 16, dof = (ubase + dp) * a.row_bytes + c * 16;
        const uint4 k = *(const uint4*)((const char*)a.K + so), v = *(const uint4*)((const char*)a.V + so);
        *(uint4*)((char*)a.K + dof) = k;
        *(uint4*)((char*)a.V + dof) = v;
    }
    for (int r = lane; r < take; r += 64) {
        const int sp = a.map.phys(a.lo + start + kept[r]), dp = a.dst_start + seg * a.keep + r;
        // the score that was ranked; what ranks lowest may have been NaN
        float v = a.ignore_scores ? -INFINITY : sc[kept[r]];
        if (v == -INFINITY) v = current_score(sp);
        a.score[ubase + dp] = v;
        a.pos[ubase + dp] = a.pos[ubase + sp];
        if (a.logit_prev) {
#pragma unroll
            for (int g = 0; g < G; ++g) a.logit_prev[ubase * G + (size_t)g * a.cap + dp] = -INFINITY;
        }
    }
}

// Row copies: bound by memory traffic, or by latency where there are few rows.  A thread moves ONE 16-byte piece of K
// and one of V, both requested before either is stored; rows are spread over as many blocks as that takes.  That is the
// shape in which a copy is fastest on this chip (1 GB device to device: one piece per thread 6.2 TB/s, four 5.7,
// eight 4.2); with 64 rows per block and four dependent load-store rounds per thread this kernel moved 5.0 TB/s.
// Rows are loaded past the last-level cache (256 MB), and stored past it (non-temporal) unless they come in from a caller: a
// prompt or an import of 10 MB or more that it holds is stored normally and stays there for what comes next, if the caller has
// not set BUZZ_FLAG_STREAMING.  Other rows each time: a prompt of which 126 MB are kept, placed and exported, 93.5 us with
// non-temporal stores into the cache, 81.9 so, 87 if the export loads normally as well; 126 MB imported, 64 steps, exported
// 1558, 1552 and 1567; 1 GB 10833 us with non-temporal accesses only, 10906 with normal stores into the cache: what they leave
// behind is written back under the decode steps.  So are the rows that evictions move: with normal accesses there, 8 caches
// of 74 MB in turn, an eviction (31 MB through the staging rows) and 3 steps each, 796 us instead of 765, 8 of 235 MB 1770
// instead of 1638; one cache alone, 128 MB moved, the eviction 111 instead of 118 us and no difference with 8 steps after it.
// The block's first threads carry the rows' scores and positions, one row each.
__device__ inline u32x4 load_piece(const char* p) { return __builtin_nontemporal_load((const u32x4*)p); }
template <bool NTD> __device__ inline void store_piece(char* p, const u32x4& v)
{
    if constexpr (NTD) __builtin_nontemporal_store(v, (u32x4*)p);
    else *(u32x4*)p = v;
}

// The copy of rows row_of(i0), row_of(i0 + 1), ... by one block, as many as it has threads for; row_of(i) >= n_rows: none.
template <bool NTD, typename RowOf>
__device__ inline void copy_rows(const GatherArgs& a, int lpr_log2, int unit, int i0, RowOf row_of)
{
    const int tid = threadIdx.x, rows = 256 >> lpr_log2;   // rows per block, 1 << lpr_log2 pieces each
    const size_t sbase = (size_t)unit * a.src_unit_rows, dbase = (size_t)unit * a.dst_unit_rows;
    auto source = [&](int r) {
        if (a.sel && r >= a.sel_lo && r < a.sel_hi)
            return a.sel[(size_t)unit * a.sel_stride + (size_t)(r - a.sel_lo) * a.sel_step];
        return a.src_start + r * a.src_step + (r >= a.sel_hi ? a.tail_shift : 0);
    };
    auto place = [&](int r) { return a.dst_map.ring_cap ? a.dst_map.phys(a.dst_start + r) : a.dst_start + r; };
    const int r = row_of(i0 + (tid >> lpr_log2));
    if (r < a.n_rows) {
        const int src = source(r), sp = a.src_map.ring_cap ? a.src_map.phys(src) : src;
        const int c = (tid & ((1 << lpr_log2) - 1)) * 16;
        const size_t so = (sbase + sp) * a.row_bytes + c, dof = (dbase + place(r)) * a.row_bytes + c;
        u32x4 k, v;
        if (a.dstK) k = load_piece((const char*)a.srcK + so);
        if (a.dstV) v = load_piece((const char*)a.srcV + so);
        if (a.dstK) store_piece<NTD>((char*)a.dstK + dof, k);
        if (a.dstV) store_piece<NTD>((char*)a.dstV + dof, v);
    }
    if (tid >= rows) return;
    const int rs = row_of(i0 + tid);
    if (rs < a.n_rows) {
        const int src = source(rs), sp = a.src_map.ring_cap ? a.src_map.phys(src) : src;
        const size_t d = dbase + place(rs);
        if (a.dstScore) {
            float v = a.srcScore ? a.srcScore[sbase + sp] : 0.f;
            if (a.logit_prev)
                for (int g = 0; g < a.G; ++g)
                    v = add_probability(v, a.logit_prev[(sbase * a.G) + (size_t)g * a.src_unit_rows + sp],
                                        a.stat_prev[((size_t)unit * a.G + g) * 2], a.stat_prev[((size_t)unit * a.G + g) * 2 + 1]);
            a.dstScore[d] = v;
        }
        if (a.dstPos) a.dstPos[d] = a.srcPos ? a.srcPos[sbase + sp] : src;
    }
}

template <bool NTD>
__global__ __launch_bounds__(256) void gather_rows_kernel(const GatherArgs a, const int lpr_log2)
{
    copy_rows<NTD>(a, lpr_log2, blockIdx.y, blockIdx.x * (256 >> lpr_log2), [](int i) { return i; });
    // (last: in front, the arguments behind its branch are fetched after it, 0.2 of 3.6 us for 4 MB)
    if (a.ticket && blockIdx.x == 0 && threadIdx.x == 0) a.ticket[blockIdx.y] = 0;
}

// Placement of a sampled prompt in one launch: the first `seg_blocks` blocks of a unit give a wave to each segment, which
// ranks it and moves its survivors, as many pieces per lane in flight as four passes have; the others copy sink and window
// rows meanwhile.  Bound by memory traffic; a launch of its own for the ranking left the memory idle while it
// ran and read its list back (32 units of 32768 rows, 64 per segment, 8 kept, a window of 4096: prefill and export 87.9 us, 82.5 so).
template <bool NTD>
__global__ __launch_bounds__(256) void place_sampled_kernel(const SelectArgs a, const GatherArgs g, const int lpr_log2, const int seg_blocks)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // [kSelWaves][wave_slice(scores + keep)]: scores, if any, then kept offsets
    const int unit = blockIdx.y;
    if ((int)blockIdx.x >= seg_blocks) {
        const int sampled = g.sel_hi - g.sel_lo;
        copy_rows<NTD>(g, lpr_log2, unit, (blockIdx.x - seg_blocks) * (256 >> lpr_log2), [&](int i) { return i < g.sel_lo ? i : i + sampled; });
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, seg = blockIdx.x * kSelWaves + wave;
    const int n_seg = (a.new_count + a.segment - 1) / a.segment;
    if (seg >= n_seg) return;                      // no block-wide barrier below: a wave only reads what it wrote
    const int start = seg * a.segment, len = min(a.segment, a.new_count - start), take = min(a.keep, len);
    const int scores = a.ignore_scores ? 0 : a.segment;
    float* sc = lds + wave * wave_slice(scores + a.keep);
    int* kept = (int*)sc + scores;
    const float* base = a.score + (size_t)unit * a.unit_stride + a.lo + start;
    if (a.ignore_scores) {                         // all equal: the lowest indices win
        for (int r = lane; r < take; r += 64) kept[r] = r;
    } else {
        for (int e = lane; e < len; e += 64) {
            const float v = base[e];
            sc[e] = v != v ? -INFINITY : v;        // NaN ranks below everything
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        rank_segment(sc, len, take, lane, [&](int r, int e) { kept[r] = e; });
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    constexpr int U = 4;
    const int rows = 64 >> lpr_log2, rr = lane >> lpr_log2, c = (lane & ((1 << lpr_log2) - 1)) * 16;   // rows per pass, this lane's
    const size_t from = ((size_t)unit * g.src_unit_rows + a.lo + start) * g.row_bytes + c;
    const size_t to_row = (size_t)unit * g.dst_unit_rows + g.sel_lo + (size_t)seg * a.keep, to = to_row * g.row_bytes + c;
    for (int r0 = rr; r0 < take; r0 += U * rows) {
        u32x4 k[U], v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u * rows >= take) break;
            const size_t at = from + (size_t)kept[r0 + u * rows] * g.row_bytes;
            k[u] = load_piece((const char*)g.srcK + at);
            v[u] = load_piece((const char*)g.srcV + at);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u * rows >= take) break;
            const size_t at = to + (size_t)(r0 + u * rows) * g.row_bytes;
            store_piece<NTD>((char*)g.dstK + at, k[u]);
            store_piece<NTD>((char*)g.dstV + at, v[u]);
        }
    }
    for (int r = lane; r < take; r += 64) {
        g.dstScore[to_row + r] = g.srcScore ? base[kept[r]] : 0.f;
        g.dstPos[to_row + r] = a.lo + start + kept[r];
    }
    if (g.ticket && seg == 0 && lane == 0) g.ticket[unit] = 0;
}

__global__ __launch_bounds__(256) void clear_f32_kernel(float* dst, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = 0.f;
}

__global__ __launch_bounds__(256) void plain_copy_kernel(uint4* dst, const uint4* src, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

}  // namespace

hipError_t launch_plain_copy(void* dst, const void* src, size_t bytes, hipStream_t st)
{
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(plain_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (uint4*)dst, (const uint4*)src, n16);
    return hipGetLastError();
}

hipError_t launch_evict_new_rows(const EvictArgs& a, int units, hipStream_t st, Timing tm)
{
    const int n_seg = (a.new_count + a.segment - 1) / a.segment;
    if (n_seg <= 0 || a.keep <= 0) return hipSuccess;
    if (a.row_bytes > 1024 || (a.row_bytes & 15) || 64 % (a.row_bytes >> 4)) return hipErrorInvalidValue;
    const dim3 grid((n_seg + kSelWaves - 1) / kSelWaves, units);
    const size_t lds = (size_t)kSelWaves * wave_slice(a.segment + a.keep) * sizeof(float);
    switch (a.G) {
        case 1: BUZZ_LAUNCH((evict_new_rows_kernel<1>), grid, dim3(256), lds, st, tm, a); break;
        case 2: BUZZ_LAUNCH((evict_new_rows_kernel<2>), grid, dim3(256), lds, st, tm, a); break;
        case 3: BUZZ_LAUNCH((evict_new_rows_kernel<3>), grid, dim3(256), lds, st, tm, a); break;
        case 4: BUZZ_LAUNCH((evict_new_rows_kernel<4>), grid, dim3(256), lds, st, tm, a); break;
        case 5: BUZZ_LAUNCH((evict_new_rows_kernel<5>), grid, dim3(256), lds, st, tm, a); break;
        case 6: BUZZ_LAUNCH((evict_new_rows_kernel<6>), grid, dim3(256), lds, st, tm, a); break;
        case 7: BUZZ_LAUNCH((evict_new_rows_kernel<7>), grid, dim3(256), lds, st, tm, a); break;
        case 8: BUZZ_LAUNCH((evict_new_rows_kernel<8>), grid, dim3(256), lds, st, tm, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Whether a block per segment selects faster than a wave per segment.  The latter takes 1.35e-4 us times the square of the
// length, however few there are, and as many times longer as there are more than 2700 waves (two to three per SIMD share
// it); a block 3 us, and 0.008 us per block where there are many.  Prefill and export of heads of 64, an eighth kept, wave /
// block: 16 segments of 256 rows 17.0 / 11.7 us, of 800 rows 108 / 12.6; 1024 of 256 24.3 / 25.5, of 320 30.1 / 25.2; 2048 of
// 320 38.4 / 44.0, of 400 54.7 / 47.8; 4096 of 360 76.6 / 83.5, of 450 110 / 92.4; 8192 of 400 160 / 162, of 450 191 / 171;
// 16384 of 360 249 / 299.  Below 256 rows a block gains a microsecond at most (16 segments of 192 12.3 / 11.6 us).
// Without scores to compare (interval sampling, a prompt that has none) a wave writes its segment's first rows, whatever
// the length: the block would search keys that are all equal, every lane on one counter (prefill, wave / block: 4 units,
// one segment of 1000 rows 5.9 / 12.7 us; 32 units, 4000 rows 8.5 / 24.5; 32 units of 32768 rows in segments of 512 27 / 64).
static bool block_selects(const SelectArgs& a, int n_seg, int units)
{
    const int segment = a.segment;
    if (a.ignore_scores) return false;
    const double length = segment, count = (double)n_seg * units, crowd = count > 2700.0 ? count / 2700.0 : 1.0;
    return segment > kMaxWaveSegment || (segment >= 256 && 3.0 + 0.008 * count < 1.35e-4 * length * length * crowd);
}

hipError_t launch_segment_topk(SelectArgs a, int units, hipStream_t st, Timing tm)
{
    const int n_seg = (a.new_count + a.segment - 1) / a.segment;
    if (n_seg <= 0) return hipSuccess;
    if (n_seg == 1) a.segment = a.new_count;       // no longer than what there is
    if (block_selects(a, n_seg, units)) {
        if ((int64_t)n_seg * kTopkBlock > UINT32_MAX) return hipErrorInvalidValue;
        const dim3 grid(n_seg, units), block(kTopkBlock);
        constexpr int per_round = kTopkBlock;          // rows
        if (a.segment <= 4 * per_round) BUZZ_LAUNCH((segment_topk_block_kernel<4, true>), grid, block, 0, st, tm, a);
        else if (a.segment <= 16 * per_round) BUZZ_LAUNCH((segment_topk_block_kernel<16, true>), grid, block, 0, st, tm, a);
        else if (a.segment <= 32 * per_round) BUZZ_LAUNCH((segment_topk_block_kernel<32, true>), grid, block, 0, st, tm, a);
        else BUZZ_LAUNCH((segment_topk_block_kernel<16, false>), grid, block, 0, st, tm, a);
        return hipGetLastError();
    }
    dim3 grid((n_seg + kSelWaves - 1) / kSelWaves, units), block(256);
    const size_t lds = a.ignore_scores ? 0 : (size_t)kSelWaves * wave_slice(a.segment) * sizeof(float);
    BUZZ_LAUNCH(segment_topk_kernel, grid, block, lds, st, tm, a);
    return hipGetLastError();
}

// 16-byte pieces per row: a power of two, at most 64; its logarithm, or -1
static int pieces_log2(int row_bytes)
{
    int lpr_log2 = 0;
    while ((16 << lpr_log2) < row_bytes) ++lpr_log2;
    return (16 << lpr_log2) == row_bytes && lpr_log2 <= 6 ? lpr_log2 : -1;
}

// Selection and placement of a sampled prompt, in one launch or two.  One takes that every survivor is kept (no thinning).
// It saves a launch, and where segments are many the time that the ranking would leave the memory idle; two spread the copy
// over all blocks, however unevenly segments and survivors are spread.  The line encloses shapes where one launch was never
// the slower of the two, of 256 measured (4 to 128 units of 2048 to 32768 rows of 128 to 512 bytes, 1 of 5 to 32 of 128 kept):
// at least 4096 segments of 32 to 256 pieces, two rows or more (prefill and export, two / one: 32 units of 32768 rows of 256
// bytes, 8 of 64 kept, 87.9 / 82.5 us; 128 of 4096, 2 of 16 kept, 52.8 / 45.4), and at most 512 segments of up to 128 pieces
// (8 units of 4096 rows of 256 bytes, 8 of 64 kept, 10.6 / 9.8).  Outside it goes either way and two launches stay: 8 units of
// 4096 rows, 4 of 32 kept, 10.3 / 8.3; 32 of 8192, 8 of 64, 27.9 / 24.6; but, of 128 bytes, 4 of 32768, 1 of 5, 16.4 / 20.0,
// 32 of 8192, 12 of 100, 19.2 / 21.1.
hipError_t launch_place_sampled(SelectArgs a, const GatherArgs& g, int units, hipStream_t st)
{
    const int n_seg = (a.new_count + a.segment - 1) / a.segment, lpr_log2 = pieces_log2(g.row_bytes);
    if (n_seg == 1) a.segment = a.new_count;
    if (lpr_log2 < 0) return hipErrorInvalidValue;
    const int64_t pieces = (int64_t)a.keep << lpr_log2, waves = (int64_t)n_seg * units;
    const int64_t lds = ((int64_t)(a.ignore_scores ? 0 : a.segment) + a.keep + 3) / 4 * 4 * kSelWaves * (int64_t)sizeof(float);
    const bool one = waves >= 4096 ? pieces >= 32 && pieces <= 256 && a.keep >= 2 : waves <= 512 && pieces <= 128;
    if (g.sel_step != 1 || block_selects(a, n_seg, units) || !one || lds > 65536) {
        if (hipError_t e = launch_segment_topk(a, units, st)) return e;
        return launch_gather_rows(g, units, st);
    }
    const int seg_blocks = (n_seg + kSelWaves - 1) / kSelWaves, rows = 256 >> lpr_log2;
    const int others = g.n_rows - (g.sel_hi - g.sel_lo);
    const dim3 grid(seg_blocks + (others + rows - 1) / rows, units);
    if (g.stream_dst) hipLaunchKernelGGL(place_sampled_kernel<true>, grid, dim3(256), (size_t)lds, st, a, g, lpr_log2, seg_blocks);
    else hipLaunchKernelGGL(place_sampled_kernel<false>, grid, dim3(256), (size_t)lds, st, a, g, lpr_log2, seg_blocks);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const GatherArgs& a, int units, hipStream_t st, Timing tm)
{
    if (a.n_rows <= 0 && !a.ticket) return hipSuccess;
    const int lpr_log2 = pieces_log2(a.row_bytes);
    if (lpr_log2 < 0) return hipErrorInvalidValue;
    const int rows = 256 >> lpr_log2;
    dim3 grid(a.n_rows > 0 ? (a.n_rows + rows - 1) / rows : 1, units), block(256);
    if (a.stream_dst) BUZZ_LAUNCH(gather_rows_kernel<true>, grid, block, 0, st, tm, a, lpr_log2);
    else BUZZ_LAUNCH(gather_rows_kernel<false>, grid, block, 0, st, tm, a, lpr_log2);
    return hipGetLastError();
}

hipError_t launch_clear_f32(float* dst, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(clear_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, dst, n);
    return hipGetLastError();
}

}  // namespace buzz
