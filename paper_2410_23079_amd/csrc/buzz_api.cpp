// Host side of the BUZZ decode library: C ABI, validation, workspace layout and the integer
// bookkeeping of Alg. 1 (sizes of sink / old / new / window regions).  Every size is a function of
// the configuration and the call history, so nothing is ever read back from the device.
#include <math.h>
#include <new>
#include <vector>

#include "buzz_internal.h"

using namespace buzz;

// Scratch of buzz_decode_step_static: the arrival counters and the per-split partial results of the split
// softmax, for callers that must not allocate.  One copy per GPU, held until the process ends; every call
// on a GPU shares it.  In host code this name is only a handle for hipGetSymbolAddress: the device address
// is looked up once per device and kept in g_static_scratch[].
constexpr size_t kStaticTicketBytes = 65536 * sizeof(int32_t);          // one counter per unit (units <= 65535)
constexpr size_t kStaticPartialBytes = (size_t)8 << 20;                 // (max, sum) pairs and partial outputs
constexpr size_t kStaticScratchBytes = kStaticTicketBytes + kStaticPartialBytes;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
void* g_static_scratch[kMaxDevices];   // device address of `scratch` on each GPU, nullptr until first use there

// Device address of this GPU's copy of the static scratch array (looked up once per device).
int static_scratch_ptr(char** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BUZZ_EHIP;
    if (!g_static_scratch[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return BUZZ_EHIP;
        g_static_scratch[dev] = p;
    }
    *out = (char*)g_static_scratch[dev];
    return BUZZ_OK;
}

// Which die (XCD) a block runs on, for every block of a small grid: the evidence for placing a unit's
// splits on one die by block number (see die_local_ok).
__global__ void die_probe_kernel(int32_t* out)
{
    if (threadIdx.x == 0)
        out[(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = (int32_t)(__builtin_amdgcn_s_getreg((31 << 11) | 20) & 7u);   // XCC_ID
}

int g_die_local[kMaxDevices];          // per GPU: 0 not probed yet, 1 blocks b and b + 8 share a die, 2 they do not
uint32_t g_die_map[kMaxDevices];       // per GPU: the die of block numbers 0..7, 4 bits each

// The die-local merge of the decode kernel relies on the hardware dealing the blocks of a grid to the dies
// round-robin in launch order (block b on die b mod 8), so that blocks whose numbers agree mod 8 share a die
// and its L2.  This checks that property once per GPU and process on two grid shapes, with one synchronisation
// of `st`; where it does not hold the decode step merges through device memory as it does for other shapes.
// Called from the prefill (never from a decode step, which must not synchronise).
int probe_die_placement(hipStream_t st)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BUZZ_EHIP;
    if (g_die_local[dev]) return BUZZ_OK;
    char* sp = nullptr;
    if (int rc = static_scratch_ptr(&sp)) return rc;
    int32_t* buf = (int32_t*)(sp + kStaticTicketBytes);                  // the partials area of the static scratch
    constexpr int kA = 8 * 64, kB = 3 * 40;
    int32_t host[kA + kB];
    hipLaunchKernelGGL(die_probe_kernel, dim3(8, 16, 4), dim3(64), 0, st, buf);   // the decode kernel's shape
    hipLaunchKernelGGL(die_probe_kernel, dim3(3, 40), dim3(64), 0, st, buf + kA);
    if (hipGetLastError() != hipSuccess) return BUZZ_EHIP;
    if (hipMemcpyAsync(host, buf, sizeof(host), hipMemcpyDeviceToHost, st) != hipSuccess) return BUZZ_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess) return BUZZ_EHIP;
    bool ok = true;
    for (int b = 8; b < kA; ++b) ok &= host[b] == host[b & 7];
    for (int b = 8; b < kB; ++b) ok &= host[kA + b] == host[kA + (b & 7)];
    uint32_t map = 0;
    for (int b = 0; b < 8; ++b) map |= (uint32_t)(host[b] & 7) << (4 * b);
    g_die_map[dev] = map;
    g_die_local[dev] = ok ? 1 : 2;
    return BUZZ_OK;
}

// Whether this GPU passed the placement probe; *map = the die of block numbers 0..7.
bool die_local_ok(uint32_t* map)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices || g_die_local[dev] != 1) return false;
    *map = g_die_map[dev];
    return true;
}

constexpr uint32_t kMagic = 0xB0220C4Eu;

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Layout {
    size_t K, V, score, pos, logit[2], stat[2], ticket, part_ml, part_o, sel, stK, stV, stScore, stPos, pscore, obs_stats, obs_partial, total;
    int32_t cap, old_cap, ring_cap, ring_base, s_cap, sel_stride, st_rows;
    int32_t units, G, elem, row_bytes, old_stride, keep;
    size_t obs_stats_cap, obs_partial_cap;   // elements ((max, sum) pairs, column sums) of the two scoring arrays
};

int make_layout(const buzz_config_t* c, Layout* L)
{
    if (!c) return BUZZ_EINVAL;
    if (c->batch < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->head_dim < 1) return BUZZ_EINVAL;
    if (c->n_q_heads % c->n_kv_heads) return BUZZ_EINVAL;
    if (c->kv_dtype < BUZZ_FP32 || c->kv_dtype > BUZZ_BF16) return BUZZ_EINVAL;
    if (c->sink < 0 || c->window < 0 || c->segment < 1 || c->keep < 0 || c->evict_every < 1) return BUZZ_EINVAL;
    if (c->old_stride < 0 || c->max_context < 1 || c->capacity < 0 || c->reserved != 0) return BUZZ_EINVAL;
    if (c->flags & ~(uint32_t)(BUZZ_FLAG_AUTO_EVICT | BUZZ_FLAG_DRY_RUN | BUZZ_FLAG_STREAMING | BUZZ_FLAG_CACHED |
                              BUZZ_FLAG_LOG_N | BUZZ_FLAG_THRESHOLD_TOTAL | BUZZ_FLAG_DETERMINISTIC |
                              BUZZ_FLAG_INTERVAL_NEW | BUZZ_FLAG_DEVICE_MERGE | BUZZ_FLAG_GLOBAL_TOPK))
        return BUZZ_EINVAL;
    if ((c->flags & BUZZ_FLAG_STREAMING) && (c->flags & BUZZ_FLAG_CACHED)) return BUZZ_EINVAL;
    if ((c->flags & BUZZ_FLAG_GLOBAL_TOPK) && (c->flags & (BUZZ_FLAG_THRESHOLD_TOTAL | BUZZ_FLAG_INTERVAL_NEW))) return BUZZ_EINVAL;
    if (!(c->softmax_scale >= 0.f) || isinf(c->softmax_scale)) return BUZZ_EINVAL;
    const int G = c->n_q_heads / c->n_kv_heads;
    if (!attn_supported(c->kv_dtype, c->head_dim, G)) return BUZZ_EUNSUPPORTED;
    if (c->segment > (1 << 28)) return BUZZ_EUNSUPPORTED;
    const int64_t units = (int64_t)c->batch * c->n_kv_heads;
    if (units > 65535) return BUZZ_EUNSUPPORTED;
    if (c->max_context > (1 << 28)) return BUZZ_EUNSUPPORTED;

    const int64_t k = c->sink, w = c->window, s = c->segment, T = c->evict_every;
    const bool global = c->flags & BUZZ_FLAG_GLOBAL_TOPK;       // one segment over everything between sink and window
    const int64_t keep = (global || c->keep < c->segment) ? c->keep : c->segment;   // a segment cannot yield more rows than it has
    const int64_t M = c->max_context > k + w ? c->max_context - k - w : 0;   // tokens that can ever be "new"
    int64_t old_cap;
    if (global) {
        old_cap = keep < M ? keep : M;                          // the survivors of the one segment
        if (c->capacity > 0 && c->capacity < k + old_cap + w + T) return BUZZ_EINVAL;
    } else if (c->capacity > 0) {
        old_cap = c->capacity - k - w - T;
        if (old_cap < 0) return BUZZ_EINVAL;
    } else if (c->flags & BUZZ_FLAG_THRESHOLD_TOTAL) {
        old_cap = keep == 0 ? 0 : T;                            // old + new never exceed T
    } else {
        const int64_t bound = keep * (ceil_div(M, s) + ceil_div(M, T) + 1);
        old_cap = keep == 0 ? 0 : (bound < M ? bound : M);
    }
    const int64_t ring = w + T;
    const int64_t cap = (int64_t)align_up((size_t)(k + old_cap + ring), 64);
    if (cap > (1 << 28)) return BUZZ_EUNSUPPORTED;

    L->units = (int32_t)units;
    L->G = G;
    L->elem = c->kv_dtype == BUZZ_FP32 ? 4 : 2;
    L->row_bytes = c->head_dim * L->elem;
    L->old_stride = c->old_stride > 0 ? c->old_stride : (c->segment + 1) / 2;
    L->keep = (int32_t)keep;
    L->cap = (int32_t)cap;
    L->old_cap = (int32_t)old_cap;
    L->ring_cap = (int32_t)ring;
    L->ring_base = (int32_t)(cap - ring);
    int64_t s_cap = kMaxBlocks / units;
    if (s_cap < 1) s_cap = 1;
    if (s_cap > kMaxSplits) s_cap = kMaxSplits;
    const int64_t s_need = ceil_div(cap * G, kStageFloats - 260 * G) + 1;   // a split's logits must fit the LDS staging
    if (s_need > kMaxSplits) return BUZZ_EUNSUPPORTED;
    if (s_cap < s_need) s_cap = s_need;
    L->s_cap = (int32_t)s_cap;
    const int64_t sel_bound = keep * (ceil_div(M, s) + 1);
    L->sel_stride = (int32_t)(keep == 0 ? 1 : (sel_bound < M ? sel_bound : (M > 0 ? M : 1)));
    L->st_rows = L->old_stride > 1 ? (int32_t)ceil_div(old_cap, L->old_stride) + 1 : 0;
    if (global) {                                               // survivors pass through the staging rows
        L->sel_stride = (int32_t)(old_cap > 0 ? old_cap : 1);
        L->st_rows = (int32_t)old_cap;
    }

    size_t off = 0;
    auto take = [&](size_t bytes) { size_t at = off; off = align_up(off + bytes, 256); return at; };
    const size_t rows = (size_t)units * cap;
    L->K = take(rows * L->row_bytes);
    L->V = take(rows * L->row_bytes);
    L->score = take(rows * 4);
    L->pos = take(rows * 4);
    L->ticket = take((size_t)units * 4);
    const size_t shared = off;                                  // scratch of the decode steps ...
    L->logit[0] = take(rows * G * 4);
    L->logit[1] = take(rows * G * 4);
    L->stat[0] = take((size_t)units * G * 2 * 4);
    L->stat[1] = take((size_t)units * G * 2 * 4);
    L->part_ml = take((size_t)units * s_cap * G * 2 * 4);
    L->part_o = take((size_t)units * s_cap * G * c->head_dim * 4);
    const size_t decode_end = off;
    off = shared;                                               // ... shares its place with that of the prompt scoring: a
    {                                                           // prefill leaves no score update pending, and a step
                                                                // writes its partial results before they are read
        // the queries' statistics and the column sums of scoring steps that are cut into parts
        size_t mma = (size_t)c->batch * c->n_q_heads * (c->max_context < kObsPassRows ? c->max_context : kObsPassRows);
        const size_t sums = (size_t)units * c->max_context * kObsItemParts;
        const size_t cut = mma * kObsKeyParts < kObsPartElems ? mma * kObsKeyParts : kObsPartElems;
        L->obs_stats_cap = mma = mma < cut ? cut : mma;         // (uncut, every query leaves one pair)
        L->obs_stats = take(mma * 2 * 4);
        L->obs_partial_cap = sums < kObsPartElems ? sums : kObsPartElems;
        L->obs_partial = take(L->obs_partial_cap * 4);
    }
    if (off < decode_end) off = decode_end;
    L->sel = take((size_t)units * L->sel_stride * 4);
    const size_t strows = (size_t)units * L->st_rows;
    L->stK = take(strows * L->row_bytes);
    L->stV = take(strows * L->row_bytes);
    L->stScore = take(strows * 4);
    L->stPos = take(strows * 4);
    L->pscore = take((size_t)units * c->max_context * 4);
    L->total = off;
    return BUZZ_OK;
}

}  // namespace

// What auto_splits prices a step with (us): a row of a split, a split, and what a split saves at least.
struct SplitModel { double row_us, split_us, whole_us; };

struct buzz_cache {
    uint32_t magic;
    buzz_config_t cfg;
    Layout L;
    char* ws;
    float scale;
    bool dry;
    // state (Alg. 1): n = sink_filled + n_old + tail
    bool ready;
    int64_t sink_filled, n_old, tail, head, tokens_seen;
    int32_t user_splits;
    SplitModel split_model;
    int64_t die_map_override;   // >= 0: use this instead of the placement probe's record (failure-handling tests)
    // the score update of the last decode step is applied lazily (by the next step or by a flush)
    bool pending;
    int last_buf;   // logit / stat buffer the last decode step wrote
    // benchmark profiling: event pairs per kernel class (0 attn, 1 epilogue, 2 eviction)
    bool prof;
    std::vector<hipEvent_t> ev[3];
    double prof_row_bytes;
    int64_t prof_evictions;

    int64_t n() const { return sink_filled + n_old + tail; }
    int64_t new_count() const
    {
        const int64_t v = n() - cfg.sink - n_old - cfg.window;
        return v > 0 ? v : 0;
    }
    int64_t trigger_count() const                               // what is compared with T
    {
        return (cfg.flags & BUZZ_FLAG_THRESHOLD_TOTAL) ? n_old + new_count() : new_count();
    }
    double log_n_factor(int64_t n_ctx) const                    // Sec. 3.5: log_512(n) for a query that sees n tokens
    {
        return (cfg.flags & BUZZ_FLAG_LOG_N) ? log((double)n_ctx) / log(512.0) : 1.0;
    }
    RingMap map() const
    {
        RingMap m;
        m.front = (int32_t)(sink_filled + n_old);
        m.ring_base = L.ring_base;
        m.ring_head = (int32_t)head;
        m.ring_cap = L.ring_cap;
        return m;
    }
    template <typename T> T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
};

namespace {

inline bool alive(const buzz_cache_t* c) { return c && c->magic == kMagic; }

// compute units of the current device (queried once, at the first launch)
int compute_units()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            cus = v;
        else
            cus = kDefaultCUs;
    }
    return cus;
}

constexpr size_t kMaxProfEvents = 1 << 15;

// a fresh event pair for one launch of kernel class `cls` while profiling is on, else an empty Timing
inline Timing prof_pair(buzz_cache_t* c, int cls)
{
    Timing tm;
    if (!c->prof || c->ev[cls].size() >= kMaxProfEvents) return tm;
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return tm;
    if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return tm; }
    c->ev[cls].push_back(a);
    c->ev[cls].push_back(b);
    tm.begin = a; tm.end = b;
    return tm;
}

void prof_clear(buzz_cache_t* c)
{
    for (auto& v : c->ev) {
        for (hipEvent_t e : v) (void)hipEventDestroy(e);
        v.clear();
    }
    c->prof_row_bytes = 0.0;
    c->prof_evictions = 0;
}
inline int hip_rc(hipError_t e) { return e == hipSuccess ? BUZZ_OK : BUZZ_EHIP; }

// Whether n rows per unit that go into the cache go past the last-level cache: it does not hold them, or the caller has said
// that nothing survives in it until they are read.  What is left there otherwise is written back under the decode steps: 8
// layers of 62 MB imported, then 4 steps of each, 700 us with normal stores and 683 so, of 93 MB 994 and 957.  A few rows go
// past it too: what reading them from there saves is less than their launch waits at its end for the caches of the dies.
// Imported, 4 steps, exported, normal stores / past it: 4 MB 36.3 / 35.5 us, 6 MB 41.5 / 40.8, 17 MB 53.4 / 54.9, 32 MB 66.5 / 72.2.
bool streams_into_cache(const buzz_cache_t* c, int64_t n)
{
    const double bytes = (double)c->L.units * (double)n * 2.0 * c->L.row_bytes;
    return (c->cfg.flags & BUZZ_FLAG_STREAMING) || bytes > kLastLevelCacheBytes || bytes < 1.0e7;
}

GatherArgs cache_gather_base(const buzz_cache_t* c)
{
    GatherArgs g{};
    g.srcK = c->at<char>(c->L.K); g.srcV = c->at<char>(c->L.V);
    g.srcScore = c->at<float>(c->L.score); g.srcPos = c->at<int32_t>(c->L.pos);
    g.src_unit_rows = c->L.cap;
    g.src_step = 1;
    g.dstK = c->at<char>(c->L.K); g.dstV = c->at<char>(c->L.V);
    g.dstScore = c->at<float>(c->L.score); g.dstPos = c->at<int32_t>(c->L.pos);
    g.dst_unit_rows = c->L.cap;
    g.row_bytes = c->L.row_bytes;
    g.stream_dst = 1;
    return g;
}

// Sizes an eviction (the eviction branch of Alg. 1) would leave behind on a cache of n rows, n_old of them old:
// old2 interval-sampled old rows, new2 segment survivors out of newc new rows.  False when nothing would be
// evicted (Remark 1: no more than sink + window rows).
struct EvictSizes { int64_t newc, old2, new2; };
bool evict_sizes(const buzz_cache_t* c, int64_t n, int64_t n_old, EvictSizes* z)
{
    const int64_t k = c->cfg.sink, w = c->cfg.window, s = c->cfg.segment, keep = c->L.keep;
    if (n <= k + w) return false;
    const int64_t newc = n - k - n_old - w > 0 ? n - k - n_old - w : 0;
    z->newc = newc;
    if (c->cfg.flags & BUZZ_FLAG_GLOBAL_TOPK) {                // old and new rows are one segment
        z->old2 = 0;
        z->new2 = keep < n - k - w ? keep : n - k - w;
        return true;
    }
    z->old2 = ceil_div(n_old, c->L.old_stride);                // interval sampling keeps offsets 0, s^, 2 s^, ...
    z->new2 = keep * (newc / s) + (newc % s < keep ? newc % s : keep);   // every segment yields min(keep, len)
    return true;
}

// Whether an eviction with these sizes stays inside what the workspace layout set aside: the old region
// (which ends where the ring begins), the list of selected rows, the staging rows.  The old-region bound is
// the caller-visible capacity; the others hold by construction of the layout and are checked all the same,
// before anything is enqueued: a launch must never be given a row the workspace does not have.
bool evict_uses_one_launch(const buzz_cache_t* c, int64_t n_old, const EvictSizes& z)
{
    return !(c->cfg.flags & BUZZ_FLAG_GLOBAL_TOPK) && z.old2 == n_old &&
           ((int64_t)c->cfg.segment + c->L.keep) * (int64_t)(4 * sizeof(float)) <= 65536;   // four waves' slices
}
bool evict_fits(const buzz_cache_t* c, int64_t n_old, const EvictSizes& z)
{
    const Layout& L = c->L;
    if (z.old2 + z.new2 > L.old_cap) return false;
    if (c->cfg.sink + z.old2 + z.new2 > L.ring_base) return false;
    if (c->cfg.flags & BUZZ_FLAG_GLOBAL_TOPK) return z.new2 <= L.st_rows && z.new2 <= L.sel_stride;
    if (evict_uses_one_launch(c, n_old, z)) return true;
    if (z.old2 < n_old && z.old2 > L.st_rows) return false;
    return z.new2 <= L.sel_stride;
}

// Applies the score update the last decode step left pending, so that the scores are current.
int flush_scores(buzz_cache_t* c, hipStream_t st)
{
    if (!c->pending || c->dry) { c->pending = false; return BUZZ_OK; }
    const Layout& L = c->L;
    AttnArgs a{};
    a.score = c->at<float>(L.score);
    a.logit_prev = c->at<float>(L.logit[c->last_buf]);
    a.stat_prev = c->at<float>(L.stat[c->last_buf]);
    a.map = c->map();
    a.n = (int32_t)c->n();
    a.cap = L.cap;
    if (hipError_t e = launch_flush_scores(L.G, a, L.units, st, prof_pair(c, 1))) return hip_rc(e);
    c->pending = false;
    return BUZZ_OK;
}

// The eviction branch of Alg. 1 on the current state.
int evict_impl(buzz_cache_t* c, hipStream_t st)
{
    const buzz_config_t& cfg = c->cfg;
    const Layout& L = c->L;
    const int64_t k = cfg.sink;
    EvictSizes z;
    if (!evict_sizes(c, c->n(), c->n_old, &z)) return BUZZ_OK; // Remark 1
    const int64_t newc = z.newc, sh = L.old_stride, old2 = z.old2, new2 = z.new2;
    if (!evict_fits(c, c->n_old, z)) return BUZZ_ECAPACITY;
    if (cfg.flags & BUZZ_FLAG_GLOBAL_TOPK) {
        // H2O-style: the top `keep` of ALL rows between sink and window survive.  Survivors may sit anywhere in
        // the old region or the ring and land where old rows are, so they travel through the staging rows.
        if (int rc = flush_scores(c, st)) return rc;
        if (!c->dry && new2 > 0) {
            if (c->prof) c->prof_evictions += 1;
            const int64_t mid = c->n() - k - cfg.window;
            SelectArgs sa{};
            sa.score = c->at<float>(L.score); sa.unit_stride = L.cap;
            sa.map = c->map(); sa.lo = (int32_t)k; sa.new_count = (int32_t)mid;
            sa.segment = (int32_t)mid;                          // one segment, whatever its length
            sa.keep = L.keep; sa.ignore_scores = 0;
            sa.sel = c->at<int32_t>(L.sel); sa.sel_stride = L.sel_stride;
            if (hipError_t e = launch_segment_topk(sa, L.units, st, prof_pair(c, 2))) return hip_rc(e);
            GatherArgs g = cache_gather_base(c);
            g.src_map = c->map();
            g.sel = c->at<int32_t>(L.sel); g.sel_stride = L.sel_stride; g.sel_step = 1; g.sel_hi = (int32_t)new2;
            g.dstK = c->at<char>(L.stK); g.dstV = c->at<char>(L.stV);
            g.dstScore = c->at<float>(L.stScore); g.dstPos = c->at<int32_t>(L.stPos);
            g.dst_unit_rows = L.st_rows; g.dst_start = 0; g.n_rows = (int32_t)new2;
            if (hipError_t e = launch_gather_rows(g, L.units, st, prof_pair(c, 2))) return hip_rc(e);
            GatherArgs b = cache_gather_base(c);
            b.srcK = c->at<char>(L.stK); b.srcV = c->at<char>(L.stV);
            b.srcScore = c->at<float>(L.stScore); b.srcPos = c->at<int32_t>(L.stPos);
            b.src_unit_rows = L.st_rows; b.src_start = 0; b.src_step = 1;
            b.dst_start = (int32_t)k; b.n_rows = (int32_t)new2;
            if (hipError_t e = launch_gather_rows(b, L.units, st, prof_pair(c, 2))) return hip_rc(e);
        }
        c->n_old = new2;
        c->head = (c->head + newc) % L.ring_cap;
        c->tail -= newc;
        return BUZZ_OK;
    }
    // Old rows that stay where they are (old stride 1) leave only the new rows to deal with, and one launch
    // does that: a score update still pending stays pending for every row that keeps its place.
    const bool in_place = evict_uses_one_launch(c, c->n_old, z);
    if (in_place) {
        if (!c->dry && new2 > 0) {
            if (c->prof) c->prof_evictions += 1;
            EvictArgs ea{};
            ea.K = c->at<char>(L.K); ea.V = c->at<char>(L.V);
            ea.score = c->at<float>(L.score); ea.pos = c->at<int32_t>(L.pos);
            ea.logit_prev = c->pending ? c->at<float>(L.logit[c->last_buf]) : nullptr;
            ea.stat_prev = c->at<float>(L.stat[c->last_buf]);
            ea.map = c->map(); ea.lo = ea.map.front; ea.new_count = (int32_t)newc;
            ea.segment = cfg.segment; ea.keep = L.keep;
            ea.ignore_scores = (cfg.flags & BUZZ_FLAG_INTERVAL_NEW) ? 1 : 0;
            ea.dst_start = (int32_t)(k + old2);
            ea.cap = L.cap; ea.row_bytes = L.row_bytes; ea.G = L.G;
            if (hipError_t e = launch_evict_new_rows(ea, L.units, st, prof_pair(c, 2))) return hip_rc(e);
        } else if (!c->dry && c->prof) {
            c->prof_evictions += 1;
        }
        c->n_old = old2 + new2;
        c->head = (c->head + newc) % L.ring_cap;
        c->tail -= newc;
        return BUZZ_OK;
    }
    if (int rc = flush_scores(c, st)) return rc;              // the selection reads the scores
    if (!c->dry) {
        if (c->prof) c->prof_evictions += 1;
        if (old2 < c->n_old) {                                 // thin the old region through the staging rows
            GatherArgs g = cache_gather_base(c);
            g.src_start = (int32_t)k; g.src_step = (int32_t)sh;
            g.dstK = c->at<char>(L.stK); g.dstV = c->at<char>(L.stV);
            g.dstScore = c->at<float>(L.stScore); g.dstPos = c->at<int32_t>(L.stPos);
            g.dst_unit_rows = L.st_rows; g.dst_start = 0; g.n_rows = (int32_t)old2;
            if (hipError_t e = launch_gather_rows(g, L.units, st, prof_pair(c, 2))) return hip_rc(e);
            GatherArgs b = cache_gather_base(c);
            b.srcK = c->at<char>(L.stK); b.srcV = c->at<char>(L.stV);
            b.srcScore = c->at<float>(L.stScore); b.srcPos = c->at<int32_t>(L.stPos);
            b.src_unit_rows = L.st_rows; b.src_start = 0; b.src_step = 1;
            b.dst_start = (int32_t)k; b.n_rows = (int32_t)old2;
            if (hipError_t e = launch_gather_rows(b, L.units, st, prof_pair(c, 2))) return hip_rc(e);
        }
        if (new2 > 0) {
            SelectArgs sa{};
            sa.score = c->at<float>(L.score); sa.unit_stride = L.cap;
            sa.map = c->map(); sa.lo = sa.map.front; sa.new_count = (int32_t)newc;
            sa.segment = cfg.segment; sa.keep = L.keep;
            sa.ignore_scores = (cfg.flags & BUZZ_FLAG_INTERVAL_NEW) ? 1 : 0;
            sa.sel = c->at<int32_t>(L.sel); sa.sel_stride = L.sel_stride;
            if (hipError_t e = launch_segment_topk(sa, L.units, st, prof_pair(c, 2))) return hip_rc(e);
            GatherArgs g = cache_gather_base(c);
            g.src_map = c->map();
            g.sel = c->at<int32_t>(L.sel); g.sel_stride = L.sel_stride; g.sel_step = 1; g.sel_hi = (int32_t)new2;
            g.dst_start = (int32_t)(k + old2); g.n_rows = (int32_t)new2;
            if (hipError_t e = launch_gather_rows(g, L.units, st, prof_pair(c, 2))) return hip_rc(e);
        }
    }
    c->n_old = old2 + new2;
    c->head = (c->head + newc) % L.ring_cap;
    c->tail -= newc;
    return BUZZ_OK;
}

}  // namespace

extern "C" {

int buzz_workspace_bytes(const buzz_config_t* cfg, size_t* bytes)
{
    if (!cfg || !bytes) return BUZZ_EINVAL;
    Layout L;
    if (int rc = make_layout(cfg, &L)) return rc;
    *bytes = L.total;
    return BUZZ_OK;
}

int buzz_cache_create(const buzz_config_t* cfg, void* dev_workspace, size_t bytes, buzz_cache_t** out)
{
    if (!cfg || !out) return BUZZ_EINVAL;
    Layout L;
    if (int rc = make_layout(cfg, &L)) return rc;
    const bool dry = cfg->flags & BUZZ_FLAG_DRY_RUN;
    if (!dry) {
        if (!dev_workspace || ((uintptr_t)dev_workspace & 255)) return BUZZ_EINVAL;
        if (bytes < L.total) return BUZZ_ECAPACITY;
    }
    buzz_cache_t* c = new (std::nothrow) buzz_cache_t();
    if (!c) return BUZZ_EINVAL;
    c->magic = kMagic;
    c->cfg = *cfg;
    c->L = L;
    c->ws = (char*)dev_workspace;
    c->scale = cfg->softmax_scale > 0.f ? cfg->softmax_scale : 1.0f / sqrtf((float)cfg->head_dim);
    c->dry = dry;
    c->ready = false;
    c->sink_filled = c->n_old = c->tail = c->head = c->tokens_seen = 0;
    c->user_splits = 0;
    const bool matrix = L.G >= 2 && cfg->kv_dtype != BUZZ_FP32, die_local = L.units % 8 == 0 && !(cfg->flags & BUZZ_FLAG_DEVICE_MERGE);
    c->split_model.row_us = (matrix ? 0.0078 : 0.009 * (1.0 + 0.237 * (L.G - 1))) * pow(L.row_bytes / 256.0, 0.63);
    c->split_model.split_us = (0.0366 + 0.006 * (L.units < 12 ? L.units : 12)) * (1.0 + 0.056 * (L.G - 1));
    c->split_model.whole_us = die_local ? 1.0 + 0.01 * (L.units < 52 ? L.units : 52) : 1.6;
    c->die_map_override = -1;
    c->pending = false;
    c->last_buf = 0;
    c->prof = false;
    c->prof_row_bytes = 0.0;
    c->prof_evictions = 0;
    *out = c;
    return BUZZ_OK;
}

int buzz_cache_destroy(buzz_cache_t* c)
{
    if (!c) return BUZZ_OK;
    if (!alive(c)) return BUZZ_EINVAL;
    prof_clear(c);
    c->magic = 0;
    delete c;
    return BUZZ_OK;
}

int buzz_cache_len(const buzz_cache_t* c, int64_t* n, int64_t* n_old, int64_t* new_count)
{
    if (!alive(c)) return BUZZ_EINVAL;
    if (n) *n = c->n();
    if (n_old) *n_old = c->n_old;
    if (new_count) *new_count = c->new_count();
    return BUZZ_OK;
}

int buzz_cache_set_splits(buzz_cache_t* c, int32_t n_splits)
{
    if (!alive(c) || n_splits < 0 || n_splits > c->L.s_cap) return BUZZ_EINVAL;
    c->user_splits = n_splits;
    return BUZZ_OK;
}

int buzz_cache_override_die_map(buzz_cache_t* c, int64_t die_map)
{
    if (!alive(c) || die_map > 0xffffffffll) return BUZZ_EINVAL;
    c->die_map_override = die_map < 0 ? -1 : die_map;
    return BUZZ_OK;
}

int buzz_prefill(buzz_cache_t* c, const void* kp, const void* vp, int64_t N, const void* q_obs, int64_t n_obs,
                 const float* init_score, void* hip_stream)
{
    if (!alive(c)) return BUZZ_EINVAL;
    if (N < 0 || n_obs < 0 || n_obs > N) return BUZZ_EINVAL;
    if (N > 0 && !c->dry && (!kp || !vp)) return BUZZ_EINVAL;
    if ((n_obs > 0) != (q_obs != nullptr) && !c->dry) return BUZZ_EINVAL;
    const buzz_config_t& cfg = c->cfg;
    const Layout& L = c->L;
    if (N > cfg.max_context) return BUZZ_ECAPACITY;
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t k = cfg.sink, w = cfg.window, s = cfg.segment, keep = L.keep, T = cfg.evict_every;
    const int64_t M = N - k - w;                                // prompt tokens between sink and window
    const bool sample = M >= T;
    int64_t survivors = 0, selected = 0, sel_step = 1;
    const bool global = cfg.flags & BUZZ_FLAG_GLOBAL_TOPK;
    if (sample && global) {
        survivors = selected = keep < M ? keep : M;             // H2O-style: one segment over the whole middle
    } else if (sample) {
        const int64_t last = M % s < keep ? M % s : keep;
        survivors = selected = keep * (M / s) + last;           // rows the selection lists; Remark 2 may thin them
        if (L.old_stride > 1 && (cfg.capacity > 0 || (cfg.flags & BUZZ_FLAG_THRESHOLD_TOTAL))) {   // Remark 2: sample until it fits
            while (survivors > L.old_cap) {
                const int64_t nxt = ceil_div(survivors, L.old_stride);
                if (nxt >= survivors) return BUZZ_ECAPACITY;
                survivors = nxt;
                sel_step *= L.old_stride;
            }
        }
        if (survivors > L.old_cap) return BUZZ_ECAPACITY;
    }
    const int64_t sink_rows = N < k ? N : k;
    const int64_t tail_rows = sample ? w : N - sink_rows;
    if (tail_rows > L.ring_cap) return BUZZ_ECAPACITY;
    // the layout's own regions: selected rows fit the selection list, survivors end before the ring begins
    if (selected > L.sel_stride || sink_rows + survivors > L.ring_base) return BUZZ_ECAPACITY;

    if (!c->dry) {
        if (int rc = probe_die_placement(st)) return rc;
        // prompt scores, one row of N per unit: what the scoring leaves, or the caller's (NULL: all zero)
        const float* ps = n_obs > 0 ? c->at<float>(L.pscore) : init_score;
        bool placed = false;
        if (n_obs > 0) {
            c->ready = c->pending = false;                      // from here on the scoring overwrites the logits of the last step
            const int max_q = kObsPassRows;                     // queries of one head per pass
            for (int64_t t0 = 0; t0 < n_obs; t0 += max_q) {
                ObsArgs oa{};
                oa.K = kp; oa.q_obs = q_obs; oa.score = c->at<float>(L.pscore); oa.stats = c->at<float>(L.obs_stats);
                oa.N = (int32_t)N; oa.n_obs = (int32_t)n_obs;
                oa.t_begin = (int32_t)t0; oa.t_count = (int32_t)((n_obs - t0) < max_q ? (n_obs - t0) : max_q);
                oa.Hq = cfg.n_q_heads; oa.Hkv = cfg.n_kv_heads;
                oa.scale_log2 = c->scale * 1.4426950408889634f;
                oa.log_n = (cfg.flags & BUZZ_FLAG_LOG_N) ? 1 : 0;
                oa.init = init_score; oa.first_pass = t0 == 0 ? 1 : 0;
                oa.partial = c->at<float>(L.obs_partial);
                oa.stats_cap = L.obs_stats_cap; oa.partial_cap = L.obs_partial_cap;
                oa.compute_units = compute_units();
                // A prompt that is kept whole may go to the cache with its last pass: the keys that the scoring reads are
                // stored while it computes, and so are the values.  Its launch says whether they were.
                if (survivors == 0 && tail_rows == N - sink_rows && t0 + max_q >= n_obs)
                    oa.place = PromptPlace{1, RingMap{(int32_t)sink_rows, L.ring_base, 0, L.ring_cap}, vp, c->at<char>(L.K), c->at<char>(L.V),
                                           c->at<float>(L.score), c->at<int32_t>(L.pos), c->at<int32_t>(L.ticket), L.cap};
                if (hipError_t e = launch_obs_scores(cfg.kv_dtype, cfg.head_dim, oa, L.units, &placed, st)) return hip_rc(e);
            }
        }
        // otherwise one launch places every row: sink, survivors behind it, the tail at the start of the ring
        GatherArgs g{};
        g.srcK = kp; g.srcV = vp; g.srcScore = ps;
        g.src_unit_rows = N; g.src_step = 1;
        g.dstK = c->at<char>(L.K); g.dstV = c->at<char>(L.V);
        g.dstScore = c->at<float>(L.score); g.dstPos = c->at<int32_t>(L.pos);
        g.dst_unit_rows = L.cap; g.row_bytes = L.row_bytes;
        g.dst_map = RingMap{(int32_t)(sink_rows + survivors), L.ring_base, 0, L.ring_cap};
        g.ticket = c->at<int32_t>(L.ticket);
        g.n_rows = (int32_t)(sink_rows + survivors + tail_rows);
        g.sel_lo = (int32_t)sink_rows; g.sel_hi = (int32_t)(sink_rows + survivors);
        g.tail_shift = (int32_t)(N - tail_rows - sink_rows - survivors);
        g.stream_dst = streams_into_cache(c, g.n_rows);
        if (survivors > 0) {
            SelectArgs sa{};
            sa.score = ps; sa.unit_stride = N;
            sa.map = RingMap{0, 0, 0, 0};
            sa.lo = (int32_t)k; sa.new_count = (int32_t)M;
            sa.segment = global ? (int32_t)M : cfg.segment;
            sa.keep = L.keep;
            sa.ignore_scores = ((cfg.flags & BUZZ_FLAG_INTERVAL_NEW) || !ps) ? 1 : 0;   // no scores: all equal
            sa.sel = c->at<int32_t>(L.sel); sa.sel_stride = L.sel_stride;
            g.sel = c->at<int32_t>(L.sel); g.sel_stride = L.sel_stride; g.sel_step = (int32_t)sel_step;
            if (hipError_t e = launch_place_sampled(sa, g, L.units, st)) return hip_rc(e);
        } else if (!placed) {
            if (hipError_t e = launch_gather_rows(g, L.units, st)) return hip_rc(e);
        }
    }
    c->pending = false;
    c->sink_filled = sink_rows;
    c->n_old = survivors;
    c->tail = tail_rows;
    c->head = 0;
    c->tokens_seen = N;
    c->ready = true;
    return BUZZ_OK;
}

}  // extern "C"

namespace {

// Whether a step of n rows reads K and V with the streaming hint.
bool reads_past_cache(const buzz_cache_t* c, int64_t n)
{
    if (c->cfg.flags & (BUZZ_FLAG_STREAMING | BUZZ_FLAG_CACHED)) return (c->cfg.flags & BUZZ_FLAG_STREAMING) != 0;
    return step_bytes(c->L.units, n, c->L.row_bytes) > kLastLevelCacheBytes;
}

// Key-range splits of a decode step, the automatic choice.  Few, long blocks amortise the per-block merge, and a block
// count that fills every compute unit the same number of times avoids a tail: at most one block per compute unit
// (floor(CUs / units) splits; with at least one unit per compute unit a unit is a single block and nothing is merged
// across blocks at all).  A short step takes fewer: a block needs row_us per row of its split, whose loads it waits for
// more than it streams (5 to 57 ns over the supported shapes), and the merge split_us per split, more where the partial
// results are larger or the units many (43 to 151 ns).  row_us n / S + split_us S is least at the root below; a cache whose
// rows take less than the publishing and merging does (whole_us) stays whole, up to 128 rows also one that a split does not
// save 1.6 us more, because both entry points split alike and the static scratch's counters cost a launch.  Over 2200 random such steps
// between 1.6 and 2.6 us a split takes 24% less time than the whole, 9% with the static scratch; of the latter 13% are slower, by up
// to 29% (2 splits, 96 units and more), though none slower than before short splits had a kernel of their own.  Beyond 8
// splits the merge goes by rounds of 8 and 16 loads: a root of more than 8 is rounded to 8, 16 or a larger multiple of 8.
// Around the root the time is flat to what the model leaves out (the tiles of a split over its waves), so splits of 128
// rows, one 16-row tile per wave, stay, whatever their number, unless the model gains 0.4 us: 8 units of 1512 rows of 4 bf16
// heads of 128 stay at 12, 6.8 us, 8 take 6.9.
// The constants are a fit to 1 to 64 units of 80 to 12000 rows, groups of 1 to 8, heads of 64 to 256, all types.  Against
// splits of at least 128 rows, on 220 random shapes of that range 4% less time on average, on 120 of 65 to 255 units 0.7%, on
// 67 of 12000 to 120000 rows 3%, none longer by more than 2% (whole_us ends to grow at 52 units: at 80 and 120 it left steps
// whole that took 3-4% longer so).  1 unit of 12000 rows, 4 heads of 128 in bf16, 13.0 us with 94 splits, 10.9 with 40; 3 of
// 175, 4 fp32 heads of 256, 14.2 with 2, 8.2 with 8; 100 of 154, 8 fp16 heads of 64, 7.7 with 2, 5.4 whole.
// One head, cached loads: a block requests 256 rows at once (128 of 1024 bytes; up to 384 of no more than 256 bytes, some 5%
// slower per row), which the model does not know.  A cache of no more, and no more than 55000 bytes of K per unit (214 rows of 256
// bytes), stays whole: 1900 such steps took 8% less time than with what the model gives (22% less to 17% more), from 224 rows on 10%
// more.  From 13 splits of 256 rows on these are taken where they are fewer than the model's: fewer publish less, 8 units of 4200
// bf16 rows of 128 in 17 splits 7.5 us, in 32 8.3; but a longer split waits longer for its rows, the more the wider they are, 2 units
// of 4053 fp32 rows of 128 in 16 splits 7.8 us, in 32 7.3.  So what the merge saves, split_us (S - fewest), must be 0.6 of what the model
// says that the rows cost, row_us n (1 / fewest - 1 / S), or more: 5100 random steps of 1 to 16 units that the rule changes take 6.4%
// less time, 2% of them over 2% more (with the line at 0.5 9%).  The count is never raised to such splits: 1 unit of 9000 bf16 rows of 64
// takes 7.1 us in the model's 32, 7.6 in 36.  Beyond 48 the model's count stays (1 unit of 16000 bf16 rows of 128: 56 splits of 286
// rows 9.8 us, 63 of 254 9.6).
int64_t rows_at_once(const buzz_cache_t* c, int64_t n)
{
    if (c->L.G > 1) return 0;
    // (also where the step is too large for two tiles of wide rows: 4 units of 9259 fp32 rows of 128 in 37 splits 11.6 us, in 64 13.6)
    const int most = short_rows(false, 1, c->cfg.head_dim, c->L.row_bytes, 8, 0.0, c->L.cap, reads_past_cache(c, n));
    return most < 256 ? most : 256;
}
int64_t auto_splits(const buzz_cache_t* c, int64_t n, int cus)
{
    const SplitModel& m = c->split_model;
    const int64_t units = c->L.units;
    if (units >= cus) return 1;
    const int64_t at_once = rows_at_once(c, n);
    if (n <= at_once && (double)n * c->L.row_bytes <= 55000.0) return 1;
    const double rows_us = m.row_us * (double)n;
    if (rows_us <= m.whole_us + (n <= 128 ? 1.6 : 0.0)) return 1;
    const int64_t most = cus / units, long_splits = ceil_div(n, 128) < most ? ceil_div(n, 128) : most;
    auto us = [&](int64_t s) { return rows_us / (double)s + m.split_us * (double)s; };
    int64_t S = (int64_t)(sqrt(rows_us / m.split_us) + 0.5);
    if (S < 2) S = 2;
    if (S > 8) S = S < 12 ? 8 : S < 22 ? 16 : (S + 4) / 8 * 8;
    if (S > most) S = most;
    if (long_splits > 1 && us(long_splits) - us(S) < 0.4) S = long_splits;
    const int64_t fewest = at_once > 0 ? ceil_div(n, at_once) : 0;   // splits whose rows are requested at once
    return fewest >= 13 && fewest <= 48 && fewest < S && m.split_us * (double)(fewest * S) >= 0.6 * rows_us ? fewest : S;
}

// One decode step.  static_scratch: the split-softmax scratch (arrival counters, per-split partials) is the
// library's static device array instead of the caller's workspace.
int decode_step_impl(buzz_cache_t* c, const void* q, const void* k_new, const void* v_new, float* out,
                     void* hip_stream, bool static_scratch)
{
    if (!alive(c)) return BUZZ_EINVAL;
    if (!c->dry && (!q || !k_new || !v_new || !out)) return BUZZ_EINVAL;
    if (!c->ready) return BUZZ_ESTATE;
    if (static_scratch && c->prof) return BUZZ_ESTATE;         // the profiling pass creates events per launch
    const buzz_config_t& cfg = c->cfg;
    const Layout& L = c->L;
    if (c->tokens_seen >= cfg.max_context) return BUZZ_ECAPACITY;
    hipStream_t st = (hipStream_t)hip_stream;

    const bool to_sink = c->sink_filled < cfg.sink && c->n_old == 0 && c->tail == 0;   // Remark 1: sink first
    if (!to_sink && c->tail >= L.ring_cap) return BUZZ_ECAPACITY;
    const int64_t new_phys = to_sink ? c->sink_filled : L.ring_base + (c->head + c->tail) % L.ring_cap;
    // state after the append of eq. 2
    const int64_t sink_filled = c->sink_filled + (to_sink ? 1 : 0);
    const int64_t tail = c->tail + (to_sink ? 0 : 1);
    const int64_t n = sink_filled + c->n_old + tail;
    // With automatic eviction the step ends with one when the threshold is reached: whether its survivors fit
    // is known now, before anything is enqueued or changed.
    bool evict_after = false;
    if (cfg.flags & BUZZ_FLAG_AUTO_EVICT) {
        EvictSizes z;
        if (evict_sizes(c, n, c->n_old, &z)) {
            const int64_t count = (cfg.flags & BUZZ_FLAG_THRESHOLD_TOTAL) ? c->n_old + z.newc : z.newc;
            evict_after = count >= cfg.evict_every;
            if (evict_after && !evict_fits(c, c->n_old, z)) return BUZZ_ECAPACITY;
        }
    }

    // the row being written must lie inside the sink or the ring, the rows stored linearly before the ring
    if (to_sink ? (new_phys < 0 || new_phys >= cfg.sink)
                : (new_phys < L.ring_base || new_phys >= (int64_t)L.ring_base + L.ring_cap || new_phys >= L.cap))
        return BUZZ_ECAPACITY;
    if (sink_filled + c->n_old > L.ring_base) return BUZZ_ECAPACITY;
    const int cus = compute_units();
    const int tile = attn_tile_rows(cfg.kv_dtype, cfg.head_dim, L.G);
    int64_t S = c->user_splits > 0 ? c->user_splits : auto_splits(c, n, cus);
    if (S < 1) S = 1;
    if (S > L.s_cap) S = L.s_cap;
    int64_t rps = ceil_div(ceil_div(n, S), tile) * tile;
    const int stage_cap = stage_floats(L.G, cfg.head_dim);
    while ((rps + 4) * L.G > stage_cap) {                      // LDS staging bound (+ alignment slack)
        S += 1;
        rps = ceil_div(ceil_div(n, S), tile) * tile;
    }
    const int64_t n_splits = ceil_div(n, rps);
    // the workspace holds s_cap partial results per unit (the static scratch has its own bound below)
    if (!static_scratch && n_splits > L.s_cap) return BUZZ_ECAPACITY;

    if (!c->dry) {
        AttnArgs a{};
        a.q = q; a.k_new = k_new; a.v_new = v_new;
        a.K = c->at<char>(L.K); a.V = c->at<char>(L.V);
        a.score = c->at<float>(L.score); a.pos = c->at<int32_t>(L.pos);
        const int cur = c->last_buf ^ 1;
        a.logit = c->at<float>(L.logit[cur]); a.logit_prev = c->at<float>(L.logit[c->last_buf]);
        a.stat = c->at<float>(L.stat[cur]); a.stat_prev = c->at<float>(L.stat[c->last_buf]);
        a.ticket = c->at<int32_t>(L.ticket);
        a.pending = c->pending ? 1 : 0;
        a.part_ml = c->at<float>(L.part_ml); a.part_o = c->at<float>(L.part_o);
        a.out = out;
        a.map = c->map();
        a.map.front = (int32_t)(sink_filled + c->n_old);
        a.n = (int32_t)n;
        a.new_phys = (int32_t)new_phys;
        a.new_pos = (int32_t)c->tokens_seen;
        a.cap = L.cap;
        a.compute_units = cus;
        a.s_cap = L.s_cap;
        a.scale_log2 = (float)(c->scale * 1.4426950408889634 * c->log_n_factor(c->tokens_seen + 1));
        a.streaming = reads_past_cache(c, n) ? 1 : 0;
        a.fixed_tiles = (cfg.flags & BUZZ_FLAG_DETERMINISTIC) ? 1 : 0;
        a.rows_per_split = (int32_t)rps;
        a.n_splits = (int32_t)n_splits;
        if (static_scratch && a.n_splits > 1) {
            // partials are laid out [units][n_splits] in the static array; the counters are cleared by a small
            // kernel (not a memset: the caller may be capturing a graph), whatever the last call left there
            const size_t ml_bytes = align_up((size_t)L.units * a.n_splits * L.G * 2 * sizeof(float), 256);
            const size_t o_bytes = (size_t)L.units * a.n_splits * L.G * cfg.head_dim * sizeof(float);
            if (ml_bytes + o_bytes > kStaticPartialBytes) return BUZZ_ECAPACITY;
            char* sp = nullptr;
            if (int rc = static_scratch_ptr(&sp)) return rc;
            a.ticket = (int32_t*)sp;
            a.part_ml = (float*)(sp + kStaticTicketBytes);
            a.part_o = (float*)(sp + kStaticTicketBytes + ml_bytes);
            a.s_cap = a.n_splits;
            if (hipError_t e = launch_clear_f32((float*)sp, L.units, st)) return hip_rc(e);
        }
        // about 8 waves per compute unit; 4-wave blocks also where 8 waves' partial outputs would not fit the LDS
        a.waves = ((int64_t)L.units * a.n_splits <= cus && L.G * cfg.head_dim < kWideBlockMaxGD) ? 8 : 4;
        // a unit's splits on one die, merged through that die's L2: possible when the units divide evenly over
        // the 8 dies
        a.xcd_local = (a.n_splits > 1 && L.units % 8 == 0 && !(cfg.flags & BUZZ_FLAG_DEVICE_MERGE) &&
                       die_local_ok(&a.die_map)) ? 1 : 0;
        a.units_per_die = L.units / 8;
        if (a.xcd_local && c->die_map_override >= 0) a.die_map = (uint32_t)c->die_map_override;
        if (hipError_t e = launch_attn_split(cfg.kv_dtype, cfg.head_dim, L.G, a, L.units, st,
                                             static_scratch ? Timing{} : prof_pair(c, 0)))
            return hip_rc(e);
        if (c->prof) c->prof_row_bytes += (double)L.units * (double)n * 2.0 * L.row_bytes;
        c->last_buf = cur;
    }
    c->pending = true;
    c->sink_filled = sink_filled;
    c->tail = tail;
    c->tokens_seen += 1;
    if (evict_after || ((cfg.flags & BUZZ_FLAG_AUTO_EVICT) && c->trigger_count() >= cfg.evict_every))
        return evict_impl(c, st);                              // cannot fail for capacity: checked above
    return BUZZ_OK;
}

}  // namespace

extern "C" {

int buzz_decode_step(buzz_cache_t* c, const void* q, const void* k_new, const void* v_new, float* out,
                     void* hip_stream)
{
    return decode_step_impl(c, q, k_new, v_new, out, hip_stream, false);
}

int buzz_decode_step_static(buzz_cache_t* c, const void* q, const void* k_new, const void* v_new, float* out,
                            void* hip_stream)
{
    return decode_step_impl(c, q, k_new, v_new, out, hip_stream, true);
}

int buzz_evict(buzz_cache_t* c, void* hip_stream)
{
    if (!alive(c)) return BUZZ_EINVAL;
    if (!c->ready) return BUZZ_ESTATE;
    return evict_impl(c, (hipStream_t)hip_stream);
}

int buzz_cache_export(buzz_cache_t* c, void* k, void* v, float* score, int32_t* pos, void* hip_stream)
{
    if (!alive(c)) return BUZZ_EINVAL;
    if (!c->ready) return BUZZ_ESTATE;
    if (c->dry) return BUZZ_OK;
    GatherArgs g = cache_gather_base(c);
    g.src_map = c->map();
    g.src_start = 0; g.src_step = 1;
    if (c->pending) {                                          // applied to the rows that leave; the cache keeps it pending
        g.logit_prev = c->at<float>(c->L.logit[c->last_buf]);
        g.stat_prev = c->at<float>(c->L.stat[c->last_buf]);
        g.G = c->L.G;
    }
    g.dstK = k; g.dstV = v; g.dstScore = score; g.dstPos = pos;
    g.dst_unit_rows = c->n(); g.dst_start = 0; g.n_rows = (int32_t)c->n();
    return hip_rc(launch_gather_rows(g, c->L.units, (hipStream_t)hip_stream));
}

int buzz_cache_import(buzz_cache_t* c, const void* k, const void* v, const float* score, const int32_t* pos,
                      int64_t n, int64_t n_old, int64_t tokens_seen, void* hip_stream)
{
    if (!alive(c) || n < 0 || n_old < 0 || n_old > n || tokens_seen < n) return BUZZ_EINVAL;
    if (!c->dry && n > 0 && (!k || !v || !score || !pos)) return BUZZ_EINVAL;
    const buzz_config_t& cfg = c->cfg;
    const Layout& L = c->L;
    if (tokens_seen > cfg.max_context || n_old > L.old_cap) return BUZZ_ECAPACITY;
    // Alg. 1 fills the sink first, and old rows only exist once the sink is full
    const int64_t sink_rows = n - n_old < cfg.sink ? n - n_old : cfg.sink;
    if (n_old > 0 && sink_rows < cfg.sink) return BUZZ_EINVAL;
    const int64_t tail_rows = n - sink_rows - n_old;
    if (tail_rows > L.ring_cap || sink_rows + n_old > L.ring_base) return BUZZ_ECAPACITY;
    if (!c->dry) {
        hipStream_t st = (hipStream_t)hip_stream;
        if (int rc = probe_die_placement(st)) return rc;
        GatherArgs g{};
        g.srcK = k; g.srcV = v; g.srcScore = score; g.srcPos = pos;
        g.src_unit_rows = n; g.src_step = 1; g.stream_dst = streams_into_cache(c, n);
        g.dstK = c->at<char>(L.K); g.dstV = c->at<char>(L.V);
        g.dstScore = c->at<float>(L.score); g.dstPos = c->at<int32_t>(L.pos);
        g.dst_unit_rows = L.cap; g.row_bytes = L.row_bytes;
        // sink and old rows: the linear region; buffered new rows and the window: the ring, from its base
        g.dst_map = RingMap{(int32_t)(sink_rows + n_old), L.ring_base, 0, L.ring_cap};
        g.ticket = c->at<int32_t>(L.ticket);
        g.n_rows = (int32_t)n;
        if (hipError_t e = launch_gather_rows(g, L.units, st)) return hip_rc(e);
    }
    c->pending = false;
    c->sink_filled = sink_rows;
    c->n_old = n_old;
    c->tail = tail_rows;
    c->head = 0;
    c->tokens_seen = tokens_seen;
    c->ready = true;
    return BUZZ_OK;
}

int buzz_cache_profile(buzz_cache_t* c, int enable)
{
    if (!alive(c)) return BUZZ_EINVAL;
    if (enable) prof_clear(c);
    c->prof = enable != 0 && !c->dry;
    return BUZZ_OK;
}

int buzz_cache_profile_read(buzz_cache_t* c, buzz_profile_t* out)
{
    if (!alive(c) || !out) return BUZZ_EINVAL;
    double ms[3] = {0, 0, 0};
    int64_t cnt[3] = {0, 0, 0};
    for (int cls = 0; cls < 3; ++cls) {
        const auto& v = c->ev[cls];
        for (size_t i = 0; i + 1 < v.size(); i += 2) {
            if (hipEventSynchronize(v[i + 1]) != hipSuccess) return BUZZ_EHIP;
            float t = 0.f;
            if (hipEventElapsedTime(&t, v[i], v[i + 1]) != hipSuccess) return BUZZ_EHIP;
            ms[cls] += t;
            cnt[cls] += 1;
        }
    }
    out->attn_launches = cnt[0]; out->epilogue_launches = cnt[1]; out->evictions = c->prof_evictions;
    out->attn_ms = ms[0]; out->epilogue_ms = ms[1]; out->evict_ms = ms[2];
    out->attn_row_bytes = c->prof_row_bytes;
    return BUZZ_OK;
}

int buzz_bench_copy(void* dst, const void* src, size_t bytes, void* hip_stream)
{
    if (!dst || !src || (bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15)) return BUZZ_EINVAL;
    return hip_rc(launch_plain_copy(dst, src, bytes, (hipStream_t)hip_stream));
}

int64_t buzz_suggest_threshold(int32_t segment, int32_t window)
{
    if (segment < 1 || window < 0) return 0;
    const double s = segment, w = window;
    const double t = (segment & 1) ? w * (s * s + 1.0) / (s + 1.0) : w * (s - 1.0);
    const int64_t r = (int64_t)floor(t + 0.5);
    return r < 1 ? 1 : r;
}

const char* buzz_strerror(int status)
{
    switch (status) {
        case BUZZ_OK: return "ok";
        case BUZZ_EINVAL: return "invalid argument or configuration";
        case BUZZ_ECAPACITY: return "cache or workspace capacity exceeded";
        case BUZZ_ESTATE: return "call not valid in the current state (prefill first)";
        case BUZZ_EHIP: return "HIP runtime error";
        case BUZZ_EUNSUPPORTED: return "shape, dtype or parameter not covered by the kernels";
    }
    return "unknown status";
}

}  // extern "C"
