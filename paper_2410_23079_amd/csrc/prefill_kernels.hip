// Prefill scoring: the accumulated score a prompt token starts with is the sum, over the observed
// prompt queries (the last n_obs positions) and the query heads of its kv head, of the causal
// attention probability it receives (eq. 3 applied to prompt queries; the score "A" of Alg. 2).
//
// Two steps per pass of up to kObsPassRows queries per head, both on the matrix cores (obs_mfma_kernel<.., 1> and
// <.., 2>): the first computes every query's softmax reference and sum over the keys it sees, the second forms the
// logits again and adds up every key's probabilities.
#include "buzz_internal.h"

#include <type_traits>

namespace buzz {
namespace {

// the prompt scores a pass of step 2 adds to: the caller's starting scores (or 0) before the first pass
__device__ inline float score_so_far(const ObsArgs& a, size_t i)
{
    return a.first_pass ? (a.init ? a.init[i] : 0.f) : a.score[i];
}

// the pass's result for a key: the prompt score so far, or, where the call places the prompt itself, the cache's row
__device__ inline void put_score(const ObsArgs& a, int unit, int key, float v)
{
    if (!a.place.on) { a.score[(size_t)unit * a.N + key] = v; return; }
    const size_t to = (size_t)unit * a.place.rows + a.place.map.phys(key);
    a.place.score[to] = v;
    a.place.pos[to] = key;
    if (key == 0) a.place.ticket[unit] = 0;
}

// ---------------------------------------------------------------------------------------------------
// One template serves both steps and all types.  A wave keeps 64 (fp32: 32) "stationary" vectors in registers as the
// B operand (column tiles of 16) and streams tiles of 16 "moving" vectors through the A
// operand; lane (j, q) = (lane % 16, lane / 16) holds, of vector j of a tile, the 16-byte pieces 4p + q
// (a permutation of the contraction index that both operands share), and receives the four products of
// moving vectors 4q .. 4q+3 with stationary vector j.  A 16-byte piece is one v_mfma_f32_16x16x32 of 16-bit elements
// or four v_mfma_f32_16x16x4 of fp32 ones (one per element, in full precision).
//   step 1 (row statistics): stationary = queries of one head, moving = the keys they may see;
//           every lane keeps a (reference, sum) of its query over its keys; merged over q at the end.
//   step 2 (column sums):    stationary = keys, moving = the queries that may see them, head after
//           head of the group; every lane adds exp2(s - reference_i) / sum_i of its key over its queries.
// The four waves of a block take adjacent groups of stationary vectors and share the moving rows: the
// block copies them, kChunk rows at a time, into one of two LDS buffers while it computes on the other
// (global loads of chunk c + 1 are issued before the tiles of chunk c and stored after them, one barrier
// per chunk).  A wave reading its tiles straight from memory, one tile ahead, spent more than half its
// time waiting for them.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes of packed 16-bit elements

template <int DT> __device__ inline f32x4 mma16(const u32x4& a, const u32x4& b, f32x4 c);
template <> __device__ inline f32x4 mma16<BUZZ_BF16>(const u32x4& a, const u32x4& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
template <> __device__ inline f32x4 mma16<BUZZ_FP16>(const u32x4& a, const u32x4& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

template <> __device__ inline f32x4 mma16<BUZZ_FP32>(const u32x4& a, const u32x4& b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, (unsigned)a[e]), __builtin_bit_cast(float, (unsigned)b[e]), c, 0, 0, 0);
    return c;
}

// Stationary vectors: 16-bit types take 64 per wave, so that an operand fetched from LDS feeds four column tiles and
// the vector work on them hides behind matrix instructions.  fp32 tiles are bound by the matrix pipe alone (16
// instructions of 32 cycles per 16 x 16 x 64 products); 32 vectors keep head_dim 256 in registers and give a
// small layer twice the blocks.
// (8 heads of 64, 2048 fp32 queries: scoring 3033 us with one vector-ALU thread per query or key and 256 queries per
// pass, 80 us here: 33-42 us per step against 14 us that its matrix instructions alone take with every SIMD busy.)
template <int DT> constexpr int col_tiles() { return DT == BUZZ_FP32 ? 2 : 4; }
template <int DT> constexpr int block_cols() { return 4 * 16 * col_tiles<DT>(); }   // per block of four waves

// Causal work is a triangle: the blocks of the last 256 queries (step 1) and of the first 256 keys (step 2)
// stream the whole prompt, the others proportionally less, and a layer with few heads has fewer blocks than the
// chip holds.  So a block streams at most `part_len` of its moving rows (in chunks; step 2: items of one chunk of
// one head), every group of stationary vectors is served by as many blocks as that takes, and all blocks but each
// group's last are equally long.  (The rule of the launch is at launch_obs_mfma_t.)
// How many parts the stationary queries of the block that holds query t (step 1) have: its latest query sees most.
__device__ inline int stat_parts(const ObsArgs& a, int t, int chunk_rows, int cols)
{
    const int block_end = min(t - (t - a.t_begin) % cols + cols, a.t_begin + a.t_count);
    const int chunks = (a.N - a.n_obs + block_end - 1) / chunk_rows + 1;
    return (chunks + a.key_part_len - 1) / a.key_part_len;
}

// Step 2: the chunks of queries, on the grid anchored at t_begin, that see the keys of the block starting at key
// j_block; *t_lo is the first one's first query.
__host__ __device__ inline int seeing_chunks(const ObsArgs& a, int j_block, int chunk_rows, int* t_lo)
{
    const int shift = a.N - a.n_obs, t_end = a.t_begin + a.t_count;
    const int t_first = j_block - shift > a.t_begin ? j_block - shift : a.t_begin;
    *t_lo = a.t_begin + (t_first - a.t_begin) / chunk_rows * chunk_rows;
    return *t_lo < t_end ? (t_end - *t_lo + chunk_rows - 1) / chunk_rows : 0;
}

// The keys that some query of the pass sees are the first visible_keys: the parts' column sums are laid out over these.
__host__ __device__ inline int visible_keys(const ObsArgs& a) { return a.N - a.n_obs + a.t_begin + a.t_count; }

// The moving rows of one chunk in LDS.  A row occupies its bytes plus 16: with that pitch the 16
// lanes that read the same piece of 16 different rows fall on 16 different groups of four banks.
template <int ROWB_>
struct MovingChunk {
    static constexpr int ROWB = ROWB_, PIECES = ROWB / 16, PITCH = ROWB + 16;
    static constexpr int ROWS = ROWB <= 256 ? 64 : 16384 / ROWB;      // two buffers stay within 64 KB of LDS
    static constexpr int PER_THREAD = ROWS * PIECES / 256;            // 16-byte pieces a thread copies per chunk
    static_assert(ROWS * PIECES % 256 == 0, "the block copies whole rounds of 256 pieces");
    // issue the loads of rows row0 .. row0 + ROWS - 1 (clamped to last_row) of the array at `base`; rows are
    // contiguous, so a chunk that lies inside the array is one block of memory and piece i sits 16 i bytes
    // into it: a uniform base plus a per-thread constant, no address arithmetic per load
    static __device__ inline void request(u32x4 (&r)[PER_THREAD], const char* base, int row0, int last_row)
    {
        if (row0 + ROWS - 1 <= last_row) {
            const char* chunk = base + (size_t)row0 * ROWB;
#pragma unroll
            for (int k = 0; k < PER_THREAD; ++k) r[k] = *(const u32x4*)(chunk + (threadIdx.x + 256 * k) * 16);
        } else {
#pragma unroll
            for (int k = 0; k < PER_THREAD; ++k) {
                const int piece = threadIdx.x + 256 * k, row = piece / PIECES, col = piece - row * PIECES;
                r[k] = *(const u32x4*)(base + (size_t)min(row0 + row, last_row) * ROWB + col * 16);
            }
        }
    }
    static __device__ inline void store(char* buf, const u32x4 (&r)[PER_THREAD])
    {
#pragma unroll
        for (int k = 0; k < PER_THREAD; ++k) {
            const int piece = threadIdx.x + 256 * k, row = piece / PIECES, col = piece - row * PIECES;
            *(u32x4*)(buf + row * PITCH + col * 16) = r[k];
        }
    }
    // The same pieces to their rows of the cache (the unit's rows start at `to`), past the last-level cache like the value
    // rows, whatever their size.  Stored normally the rows slow the scoring down where they are many, and speed up what
    // reads them next: prefill alone / with an export, non-temporal and normal, 8 MB of fp32 rows 71.6, 72.2 / 76.9, 77.7 us,
    // 31 MB (score of 4001 queries) 328, 328 / 346, 343, 128 MB 91.6, 87.6 / 138, 128, 200 MB 126, 134 / 196, 193, 512 MB 301, 313 / 475, 465.
    static __device__ inline void place(char* to, const RingMap& map, const u32x4 (&r)[PER_THREAD], int row0, int last_row)
    {
#pragma unroll
        for (int k = 0; k < PER_THREAD; ++k) {
            const int piece = threadIdx.x + 256 * k, row = row0 + piece / PIECES, col = piece % PIECES;
            if (row <= last_row) __builtin_nontemporal_store(r[k], (u32x4*)(to + (size_t)map.phys(row) * ROWB + col * 16));
        }
    }
    // A operand of tile `tile` (16 rows) of the chunk for this lane
    static __device__ inline void fetch(u32x4 (&f)[ROWB / 64], const char* buf, int tile, int j, int q)
    {
        const char* row = buf + (16 * tile + j) * PITCH + q * 16;
#pragma unroll
        for (int p = 0; p < ROWB / 64; ++p) f[p] = *(const u32x4*)(row + p * 64);
    }
};

// Value rows j_block .. j_block + ROWS - 1 of a unit on their way to the cache: N pieces per thread, up to BATCH of them in
// flight at once.  ALL: a whole batch from k0 on; else pieces k0 .. k1 - 1, at most a batch.
template <int ROWB, int ROWS>
struct ValueRows {
    static constexpr int PIECES = ROWB / 16, N = ROWS * PIECES / 256, BATCH = N < 16 ? N : 16;   // pieces per row, per thread, at a time
    static_assert(ROWS * PIECES % 256 == 0 && N % BATCH == 0 && (N + 1) / 2 <= BATCH, "whole rounds; half a block's pieces are a batch");
    u32x4 r[BATCH];
    template <bool ALL> __device__ inline void request(const ObsArgs& a, int unit, int j_block, int k0, int k1)
    {
        const char* from = (const char*)a.place.V_from + (size_t)unit * a.N * ROWB;
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            if (!ALL && k0 + k >= k1) break;
            const int piece = threadIdx.x + 256 * (k0 + k);
            r[k] = __builtin_nontemporal_load((const u32x4*)(from + (size_t)min(j_block + piece / PIECES, a.N - 1) * ROWB + piece % PIECES * 16));
        }
    }
    template <bool ALL> __device__ inline void store(const ObsArgs& a, int unit, int j_block, int k0, int k1) const
    {
        char* to = (char*)a.place.V + (size_t)unit * a.place.rows * ROWB;
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            if (!ALL && k0 + k >= k1) break;
            const int piece = threadIdx.x + 256 * (k0 + k), row = j_block + piece / PIECES;
            if (row < a.N) __builtin_nontemporal_store(r[k], (u32x4*)(to + (size_t)a.place.map.phys(row) * ROWB + piece % PIECES * 16));
        }
    }
};

template <int DT, int D, int STEP, bool LOGN>
__global__ __launch_bounds__(256) void obs_mfma_kernel(const ObsArgs a)
{
    // softmax scale (log2 units) of the query at prompt position `pos`; a template flag rather than a
    // run-time one: as a run-time select the logarithm would be evaluated for every row of every tile
    auto qscale = [&](int pos) {
        return LOGN ? a.scale_log2 * (logf((float)(pos + 1)) * (1.0f / 6.2383246250395077f)) : a.scale_log2;
    };
    constexpr int ROWB = D * (DT == BUZZ_FP32 ? 4 : 2);
    using MC = MovingChunk<ROWB>;
    constexpr int QP = ROWB / 64, CT = col_tiles<DT>(), COLS = 16 * CT, BLOCK_COLS = block_cols<DT>(), CH = MC::ROWS;
    constexpr bool AHEAD = ROWB <= 256;                    // a second operand buffer fits the register budget
    __shared__ __align__(16) char sm_rows[2][CH * MC::PITCH];
    __shared__ float2 sm_stat[2][CH];                      // step 2: (reference, 1 / sum) of the chunk's queries
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform values stay in scalar registers
    const int j = lane & 15, q = lane >> 4;
    const int G = a.Hq / a.Hkv;
    const int t_end = a.t_begin + a.t_count;               // queries [t_begin, t_end) of q_obs are scored by this pass
    const int shift = a.N - a.n_obs;                       // prompt position of query t is shift + t
    auto piece = [&](const char* row, int p) { return *(const u32x4*)(row + (4 * p + q) * 16); };
    u32x4 staged[MC::PER_THREAD];

    if constexpr (STEP == 1) {
        // the latest queries see the most keys: their blocks go first, for all heads, so that the launch
        // ends with the short blocks (the grid is linear, the head advances first, then the part, then the group).
        // Heads run over the units first: where these divide evenly over the 8 dies, a unit's heads share one, whose L2
        // then serves the keys (32 heads on 4 units each, 1535 queries: prefill and export 189 -> 183 us, 64 on 16: 355 -> 352).
        const int at = blockIdx.x % a.heads, slot = blockIdx.x / a.heads;
        const int unit = at % a.units, head = unit * G + at / a.units;   // b * Hkv + kvh, b * Hq + h
        const int part = slot % a.key_parts, group = slot / a.key_parts;
        const int t_block = a.t_begin + ((a.t_count - 1) / BLOCK_COLS - group) * BLOCK_COLS;
        const int t_base = t_block + wave * COLS;
        const bool active = t_base < t_end;                // a wave without queries still copies and synchronises
        const char* Qb = (const char*)a.q_obs + (size_t)head * a.n_obs * ROWB;
        const char* Kb = (const char*)a.K + (size_t)unit * a.N * ROWB;
        constexpr float kRefStart = -3.402823466e38f, kRefSlack = 1073741824.0f;   // lowest float, 2^30
        u32x4 qf[CT][QP];
        int pos[CT];
        float scale[CT], m[CT], l[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const int t = t_base + 16 * ct + j;
            pos[ct] = t < t_end ? shift + t : -1;          // -1: no key is visible, the column stays empty
            scale[ct] = qscale(max(pos[ct], 0));
            const char* row = Qb + (size_t)min(t, a.n_obs - 1) * ROWB;
#pragma unroll
            for (int p = 0; p < QP; ++p) qf[ct][p] = piece(row, p);
            m[ct] = kRefStart; l[ct] = 0.f;
        }
        const int k_last = shift + min(t_base + COLS, t_end) - 1;   // the wave's latest query sees keys 0 .. k_last
        const int k_free = shift + t_base;                 // keys up to here are visible to every query of the wave
        const int k_last_block = shift + min(t_block + BLOCK_COLS, t_end) - 1;
        const int n_chunks = k_last_block / CH + 1;
        const int c_begin = part * a.key_part_len, c_end = min(n_chunks, c_begin + a.key_part_len);   // this block's chunks
        if (c_begin >= c_end) return;                      // the group has fewer parts
        // Lazy reference: a lane sums exp2(s * scale - ref) against a reference that only moves when it has
        // to.  A chunk costs one fma, one exp2 and one add per element, straight-line code per tile
        // (independent chains of matrix instructions and the vector work on their results) with none
        // of the maximum bookkeeping, and one test at its end: if a sum of the wave has grown past kRefSlack
        // (or overflowed), the sums go back to their values before the chunk and the chunk is redone the
        // classic way, tile by tile: the reference rises to the running maximum and the sum so far is
        // rescaled.  The block's first chunk goes the classic way at once (the reference starts at the lowest
        // float, so trying it otherwise would only be thrown away); after it the test fails only when a logit
        // exceeds its lane's reference by about 30 (log2 units).  m[] holds the reference in scaled (log2) units.
        auto products = [&](const u32x4 (&kf)[QP], int ct) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < QP; ++p) acc = mma16<DT>(kf[p], qf[ct][p], acc);
            return acc;
        };
        // causal: key k0 + 4q + v against this lane's query.  An invisible key contributes 0 through a
        // select, not through a product of -inf: the log-n scale of the first prompt query is 0.
        auto tile_sum = [&](const f32x4& acc, int ct, int k0, auto masked_tag) {
            constexpr bool MASKED = decltype(masked_tag)::value;
            float e[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                e[v] = __builtin_amdgcn_exp2f(fmaf(acc[v], scale[ct], -m[ct]));
                if (MASKED && k0 + 4 * q + v > pos[ct]) e[v] = 0.f;
            }
            return (e[0] + e[1]) + (e[2] + e[3]);
        };
        auto add_tile = [&](const u32x4 (&kf)[QP], int k0, auto masked_tag) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) l[ct] += tile_sum(products(kf, ct), ct, k0, masked_tag);
        };
        auto add_tile_classic = [&](const u32x4 (&kf)[QP], int k0) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const f32x4 acc = products(kf, ct);
                float top = kRefStart;
#pragma unroll
                for (int v = 0; v < 4; ++v) top = fmaxf(top, k0 + 4 * q + v <= pos[ct] ? acc[v] * scale[ct] : kRefStart);
                // unchanged, and the factor exactly 1, where the tile brought nothing larger
                l[ct] *= __builtin_amdgcn_exp2f(fminf(m[ct] - top, 0.f));
                m[ct] = fmaxf(m[ct], top);
                l[ct] += tile_sum(acc, ct, k0, std::true_type{});
            }
        };
        // A prompt that is kept whole is placed by the scoring itself, which reads the keys anyway and is not bound by
        // memory: the blocks of the latest queries of a unit's first head stream every key of the unit once and store it
        // here, the blocks of step 2 carry the values (256 heads of 128, 256 queries, 4096 keys: 94 + 96 + 160 us
        // for the steps and a placement of their own, 120 + 165 so; prefill and export 505 -> 472 us).
        const bool places = a.place.on && at < a.units && group == 0;
        char* K_to = (char*)a.place.K + (size_t)unit * a.place.rows * ROWB;
        MC::request(staged, Kb, c_begin * CH, a.N - 1);
        MC::store(sm_rows[c_begin & 1], staged);
        if (places) MC::place(K_to, a.place.map, staged, c_begin * CH, a.N - 1);
        __syncthreads();
        for (int c = c_begin; c < c_end; ++c) {
            const bool more = c + 1 < c_end;
            if (more) MC::request(staged, Kb, (c + 1) * CH, a.N - 1);
            if (active) {
                float l_in[CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) l_in[ct] = l[ct];
                u32x4 kf[2][QP];
                bool classic = c == c_begin;
                if (!classic) {
                    // (rows up to 256 bytes) the operand of tile i + 1 leaves LDS while tile i is computed; reading
                    // past the wave's last tile stays inside the buffer and is never used
                    MC::fetch(kf[0], sm_rows[c & 1], 0, j, q);
#pragma unroll
                    for (int tile = 0; tile < CH / 16; ++tile) {
                        const int k0 = c * CH + 16 * tile;
                        if (AHEAD && tile + 1 < CH / 16) MC::fetch(kf[(tile + 1) & 1], sm_rows[c & 1], tile + 1, j, q);
                        if (!AHEAD && tile > 0) MC::fetch(kf[0], sm_rows[c & 1], tile, j, q);
                        if (k0 <= k_last) {
                            // wave-uniform: does a causal boundary or the end of the query list cross this tile?
                            if (k0 + 15 > k_free || t_base + COLS > t_end) add_tile(kf[AHEAD ? tile & 1 : 0], k0, std::true_type{});
                            else add_tile(kf[AHEAD ? tile & 1 : 0], k0, std::false_type{});
                        }
                    }
                    // the sums are nonnegative: their total passes the test only if each of them does; !(<=) also
                    // catches a sum that overflowed or is not a number
                    float total = l[0];
#pragma unroll
                    for (int ct = 1; ct < CT; ++ct) total += l[ct];
                    classic = __builtin_amdgcn_ballot_w64(!(total <= kRefSlack)) != 0;
                }
                if (__builtin_expect(classic, 0)) {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) l[ct] = l_in[ct];
#pragma unroll 1
                    for (int tile = 0; tile < CH / 16; ++tile) {
                        const int k0 = c * CH + 16 * tile;
                        if (k0 > k_last) break;
                        MC::fetch(kf[0], sm_rows[c & 1], tile, j, q);
                        add_tile_classic(kf[0], k0);
                    }
                }
            }
            if (more) {
                MC::store(sm_rows[(c + 1) & 1], staged);
                if (places) MC::place(K_to, a.place.map, staged, (c + 1) * CH, a.N - 1);
            }
            __syncthreads();
        }
        if (!active) return;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {                  // merge the four key subsets of a query
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const float mo = __shfl_xor(m[ct], off), lo = __shfl_xor(l[ct], off);
                const float ref = fmaxf(m[ct], mo);       // finite: every lane's reference is
                l[ct] = l[ct] * __builtin_amdgcn_exp2f(m[ct] - ref) + lo * __builtin_amdgcn_exp2f(mo - ref);
                m[ct] = ref;
            }
            const int t = t_base + 16 * ct + j;
            if (q == 0 && t < t_end) {                     // (a part without visible keys leaves (kRefStart, 0))
                float* st = a.stats + (((size_t)head * a.key_parts + part) * a.t_count + (t - a.t_begin)) * 2;
                st[0] = m[ct];                             // reference of the scaled logits (at most their maximum)
                st[1] = a.key_parts > 1 ? l[ct] : 1.0f / l[ct];
            }
        }
    } else {
        // the earliest keys are seen by the most queries: they go first (linear grid: unit, part, block of keys)
        const int unit = blockIdx.x % a.units, slot = blockIdx.x / a.units;
        const int part = slot % a.item_parts;
        const int b = unit / a.Hkv, kvh = unit - b * a.Hkv;
        const int j_block = slot / a.item_parts * BLOCK_COLS;
        // the block streams the queries from the first one that sees its first key, for every head of the group in
        // turn: item i = (head i / n_chunks, chunk i % n_chunks), and of these its own part
        int t_lo;
        const int n_chunks = seeing_chunks(a, j_block, CH, &t_lo);
        const int item0 = part * a.item_part_len, n_items = min(n_chunks * G, item0 + a.item_part_len);
        if (part > 0 && item0 >= n_items) return;          // fewer parts here (part 0 carries the scores over)
        const int j_base = j_block + wave * COLS;
        const bool active = j_base < a.N;
        // The parts of a cut step share the block's value rows: a launch of about four short blocks per compute unit ends with
        // whoever carries them alone (prefill and export, bf16, 2 heads on each of 4 units, D 256, 500 queries, 3000 keys: 48.8 us
        // with a copy of its own, 57.4 with all rows in part 0, 47.5 so; of 8 units, D 128, 256 queries, 2000 keys: 31.9, 33.2, 30.1).
        ValueRows<ROWB, BLOCK_COLS> values;
        const int parts_here = max(1, (n_chunks * G + a.item_part_len - 1) / a.item_part_len);
        const int piece0 = part * values.N / parts_here, piece1 = (part + 1) * values.N / parts_here;   // this part's share
        const bool places_all = a.place.on && parts_here == 1, places_some = a.place.on && parts_here > 1;
        if (places_all) {
#pragma unroll 1
            for (int k0 = values.BATCH; k0 < values.N; k0 += values.BATCH) {
                values.template request<true>(a, unit, j_block, k0, 0);
                values.template store<true>(a, unit, j_block, k0, 0);
            }
            values.template request<true>(a, unit, j_block, 0, 0);
        }
        if (places_some) values.template request<false>(a, unit, j_block, piece0, piece1);
        const char* Kb = (const char*)a.K + (size_t)unit * a.N * ROWB;
        u32x4 kf[CT][QP];
        float col[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            const char* row = Kb + (size_t)min(j_base + 16 * ct + j, a.N - 1) * ROWB;
#pragma unroll
            for (int p = 0; p < QP; ++p) kf[ct][p] = piece(row, p);
            col[ct] = 0.f;
        }
        const int head0 = b * a.Hq + kvh * G;
        float2 staged_stat = make_float2(0.f, 0.f);
        auto request = [&](int item) {
            const int g = item / n_chunks, t0 = t_lo + (item - g * n_chunks) * CH;
            MC::request(staged, (const char*)a.q_obs + (size_t)(head0 + g) * a.n_obs * ROWB, t0, a.n_obs - 1);
            if (threadIdx.x < CH)                          // the reference and 1 / sum of the chunk's queries
                staged_stat = *(const float2*)(a.stats + ((size_t)(head0 + g) * a.key_parts * a.t_count +
                                                          (min(t0 + (int)threadIdx.x, t_end - 1) - a.t_begin)) * 2);
        };
        auto store = [&](int buf) {
            MC::store(sm_rows[buf], staged);
            if (threadIdx.x < CH) sm_stat[buf][threadIdx.x] = staged_stat;
        };
        auto consume_as = [&](const u32x4 (&qf)[QP], const float2 (&st)[4], int t0, auto masked_tag) {
            constexpr bool MASKED = decltype(masked_tag)::value;
            float sc[4];
            int posq[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = t0 + 4 * q + v;
                posq[v] = (!MASKED || t < t_end) ? shift + t : -1;
                sc[v] = qscale(max(posq[v], 0));
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int p = 0; p < QP; ++p) acc = mma16<DT>(qf[p], kf[ct][p], acc);
                const int key = j_base + 16 * ct + j;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    // an invisible key takes nothing, not 0 times the query's 1 / sum, which may not be a number
                    const float e = __builtin_amdgcn_exp2f(fmaf(acc[v], sc[v], -st[v].x));
                    const float with = fmaf(e, st[v].y, col[ct]);
                    col[ct] = MASKED && key > posq[v] ? col[ct] : with;
                }
            }
        };
        if (places_all) values.template store<true>(a, unit, j_block, 0, 0);
        if (places_some) values.template store<false>(a, unit, j_block, piece0, piece1);
        if (item0 < n_items) {
            request(item0);
            store(item0 & 1);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): else the loop waits for the stationary rows, and with
                                                           // them for the rows it has just requested, in every tile
        __syncthreads();
        for (int item = item0; item < n_items; ++item) {
            const bool more = item + 1 < n_items;
            if (more) request(item + 1);
            if (active) {
                const int t_chunk = t_lo + (item % n_chunks) * CH;
                // the operand of tile i + 1 leaves LDS while tile i is computed; the statistics are read with
                // the tile itself, the products hide their latency
                u32x4 qf[2][QP];
                MC::fetch(qf[0], sm_rows[item & 1], 0, j, q);
#pragma unroll
                for (int tile = 0; tile < CH / 16; ++tile) {
                    const int t0 = t_chunk + 16 * tile;
                    if (AHEAD && tile + 1 < CH / 16) MC::fetch(qf[(tile + 1) & 1], sm_rows[item & 1], tile + 1, j, q);
                    if (!AHEAD && tile > 0) MC::fetch(qf[0], sm_rows[item & 1], tile, j, q);
                    // skipped: tiles past the last query, and tiles none of whose queries sees any key of the wave
                    if (t0 < t_end && shift + t0 + 15 >= j_base) {
                        float2 st[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) st[v] = sm_stat[item & 1][16 * tile + 4 * q + v];
                        // wave-uniform: unmasked if every query of the tile exists and sees every key of the wave
                        if (t0 + 16 > t_end || shift + t0 < j_base + COLS - 1) consume_as(qf[AHEAD ? tile & 1 : 0], st, t0, std::true_type{});
                        else consume_as(qf[AHEAD ? tile & 1 : 0], st, t0, std::false_type{});
                    }
                }
            }
            if (more) store((item + 1) & 1);
            __syncthreads();
        }
        if (!active) return;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            float c = col[ct] + __shfl_xor(col[ct], 16);
            c += __shfl_xor(c, 32);
            const int key = j_base + 16 * ct + j;
            if (a.item_parts == 1) {
                if (q == 0 && key < a.N) put_score(a, unit, key, score_so_far(a, (size_t)unit * a.N + key) + c);
            } else {
                const int keys = visible_keys(a);
                if (q == 0 && key < keys) a.partial[((size_t)part * a.units + unit) * keys + key] = c;
            }
        }
    }
}

// Merges the parts of a query's row statistics into its part 0: (reference, sum) of every part -> (reference,
// 1 / sum).  (Done by the blocks of step 2 as they stage a chunk, the arithmetic waits for loads that are
// otherwise in flight across a chunk's tiles: step 2 of 256 heads of 128, 256 queries, 4096 keys: 120 us with the merge inside, 98 us
// without, 5 us for this kernel.)
__global__ __launch_bounds__(256) void obs_merge_stats_kernel(const ObsArgs a, int chunk_rows, int cols)
{
    const int r = blockIdx.x * 256 + threadIdx.x, head = blockIdx.y;
    if (r >= a.t_count) return;
    float2* st = (float2*)a.stats + (size_t)head * a.key_parts * a.t_count + r;
    const int parts = stat_parts(a, a.t_begin + r, chunk_rows, cols);
    float2 got[kObsKeyParts];
#pragma unroll
    for (int k = 0; k < kObsKeyParts; ++k) got[k] = st[(size_t)min(k, parts - 1) * a.t_count];
    float ref = got[0].x;                                  // part 0 holds key 0: finite, sum > 0
#pragma unroll
    for (int k = 1; k < kObsKeyParts; ++k) ref = fmaxf(ref, got[k].x);
    float sum = got[0].y * __builtin_amdgcn_exp2f(got[0].x - ref);
#pragma unroll
    for (int k = 1; k < kObsKeyParts; ++k)
        if (k < parts) sum = fmaf(got[k].y, __builtin_amdgcn_exp2f(got[k].x - ref), sum);
    st[0] = make_float2(ref, 1.0f / sum);
}

// Adds the parts of a key block's column sums to the prompt scores, in part order (the same bits every time).
// Latency-bound, 5 us at 16 units of 4001 keys, against 290 us that the cut of step 2 saves there.
__global__ __launch_bounds__(256) void obs_sum_parts_kernel(const ObsArgs a, int chunk_rows, int cols)
{
    const int j = blockIdx.x * 256 + threadIdx.x, unit = blockIdx.y;
    if (j >= a.N) return;
    int t_lo;
    const int keys = visible_keys(a);
    const int items = j < keys ? seeing_chunks(a, j / cols * cols, chunk_rows, &t_lo) * (a.Hq / a.Hkv) : 0;
    const int parts = (items + a.item_part_len - 1) / a.item_part_len;
    const size_t at = (size_t)unit * a.N + j, sum = (size_t)unit * keys + j;
    float got[kObsItemParts];
#pragma unroll
    for (int p = 0; p < kObsItemParts; ++p) got[p] = p < parts ? a.partial[(size_t)p * a.units * keys + sum] : 0.f;
    float s = score_so_far(a, at);
#pragma unroll
    for (int p = 0; p < kObsItemParts; ++p) s += got[p];
    put_score(a, unit, j, s);
}

template <int DT, int D>
hipError_t launch_obs_mfma_t(ObsArgs a, int units, bool* placed, hipStream_t st, Timing tm)
{
    constexpr int CH = MovingChunk<D * (DT == BUZZ_FP32 ? 4 : 2)>::ROWS, COLS = block_cols<DT>();
    const int heads = units / a.Hkv * a.Hq, G = a.Hq / a.Hkv;
    a.heads = heads; a.units = units;
    const int q_blocks = (a.t_count + COLS - 1) / COLS;
    const int k_seen = (visible_keys(a) + COLS - 1) / COLS;            // blocks of keys with work
    // A step whose longest block is no more than its share of two blocks per compute unit stays whole: the long
    // blocks start first and have the SIMDs more and more to themselves, and parts would only repeat the blocks'
    // prologue (64 heads of 128, 4096 queries: 347 us whole, 385 us cut).  Below that it is cut for four blocks
    // per compute unit (64 heads of 128 on 16 units, 4001 queries: prefill and export 644 us whole, 342 cut).  Eight or
    // twelve blocks per unit gave 320 and 323 us there, but 146 instead of 131 us with heads of 256 and 385-390
    // instead of 378 for 256 heads with 256 queries, so four stays.
    auto split = [&](int64_t total, int longest, bool whole, int most, int* parts, int* len) {
        const int64_t cus = a.compute_units;
        int64_t l = whole && longest <= (total + 2 * cus - 1) / (2 * cus) ? longest : (total + 4 * cus - 1) / (4 * cus);
        if (l < (longest + most - 1) / most) l = (longest + most - 1) / most;
        *len = (int)(l < 1 ? 1 : l);
        *parts = longest > 0 ? (int)((longest + *len - 1) / *len) : 1;
    };
    int64_t total = 0;
    int longest = 0;
    for (int b = 0; b < q_blocks; ++b) {
        const int end = (b + 1) * COLS < a.t_count ? (b + 1) * COLS : a.t_count;
        const int chunks = (a.N - a.n_obs + a.t_begin + end - 1) / CH + 1;
        total += (int64_t)chunks * heads;
        longest = chunks;
    }
    int most = (int)(a.stats_cap / ((size_t)heads * a.t_count));       // what the statistics array holds
    // A few observed queries leave waves of a block without any.  Up to 1.5 waves with queries per SIMD, step 1 is cut all
    // the same, where a part is long enough to pay for the merge (5 us): the chunks' latencies are not hidden otherwise
    // (512 heads of 64, 16 bits, 128 queries, 4096 keys: 116 us whole, 84 + 5 cut; 576 heads of 128: 330 us of prefill
    // whole, 295 cut).  Rows of 128 need a wave per SIMD for that (512 heads, 64 queries: 188 us whole, 204 cut);
    // fp32 tiles and rows of 256 keep the matrix pipes busy (no difference, 2% slower).
    const int64_t waves = (int64_t)heads * ((a.t_count + COLS / 4 - 1) / (COLS / 4)), simds = 4 * (int64_t)a.compute_units;
    const bool idle = DT != BUZZ_FP32 && 2 * waves < 3 * simds && longest >= 24 && (D == 64 || (D == 128 && waves >= simds));
    split(total, longest, !idle, most < kObsKeyParts ? (most < 1 ? 1 : most) : kObsKeyParts, &a.key_parts, &a.key_part_len);
    total = 0;
    int t_lo;
    for (int b = 0; b < k_seen; ++b) total += (int64_t)seeing_chunks(a, b * COLS, CH, &t_lo) * G * units;
    longest = seeing_chunks(a, 0, CH, &t_lo) * G;
    most = (int)(a.partial_cap / ((size_t)units * visible_keys(a)));
    split(total, longest, true, most < kObsItemParts ? (most < 1 ? 1 : most) : kObsItemParts, &a.item_parts, &a.item_part_len);
    // Whether the steps place a prompt that is kept whole, or a copy of its own does.  They save its launch and its waits, if
    // enough blocks carry the rows: a block of step 2 has 32, 64 or 128 KB of values before its first tile, a block of step 1
    // stores all the chunks of its part.  With 32 KB they always do.  With more, whole (uncut) blocks have to be 8 (64 KB), or
    // half as many as compute units (128 KB): prefill and export, copy / steps, bf16 heads of 256, 16 queries, 48 blocks (16
    // units of 700 keys) 27.0 / 28.5 us, 96 (32 of 700) 36.3 / 37.4, 128 (16 of 2000) 43.8 / 42.8, 256 (32 of 2000) 67 / 63;
    // of 128, 3 blocks (1 unit of 700 keys) 18.4 / 18.5, 8 (8 of 200) 18.7 / 18.5, 16 (16 of 200) 19.3 / 19.0.  And step 1
    // must not be up to 32 blocks of 8 chunks or more each (1 unit of 12000 keys: heads of 128 39.3 / 40.6, of 256 51.4 / 55.9);
    // a larger one hides the stores (4 units of 10512 keys 47.6 / 45.7), however few of its blocks have some (64 heads of 128 on
    // 16 units, 4001 queries 351 / 340).
    if (a.place.on) {
        constexpr int value_bytes = COLS * D * (DT == BUZZ_FP32 ? 4 : 2);
        const int64_t blocks = (int64_t)units * ((a.N + COLS - 1) / COLS);
        const bool few = a.item_parts == 1 && blocks < (value_bytes > 65536 ? a.compute_units / 2 : 8);
        const bool long_parts = (int32_t)heads * q_blocks * a.key_parts <= 32 && a.key_part_len >= 8;
        if (value_bytes > 32768 && (few || long_parts)) a.place.on = 0;
    }
    *placed = a.place.on != 0;
    const int k_blocks = a.item_parts > 1 ? k_seen : (a.N + COLS - 1) / COLS;   // uncut blocks carry every score over
    const int64_t blocks1 = (int64_t)heads * q_blocks * a.key_parts, blocks2 = (int64_t)units * k_blocks * a.item_parts;
    if (blocks1 > INT32_MAX / 256 || blocks2 > INT32_MAX / 256) return hipErrorInvalidValue;   // (far beyond any GPU's memory)
    const dim3 g1((unsigned)blocks1), g2((unsigned)blocks2);
    if (a.log_n) BUZZ_LAUNCH((obs_mfma_kernel<DT, D, 1, true>), g1, dim3(256), 0, st, tm, a);
    else BUZZ_LAUNCH((obs_mfma_kernel<DT, D, 1, false>), g1, dim3(256), 0, st, tm, a);
    if (hipError_t e = hipGetLastError()) return e;
    if (a.key_parts > 1) {
        BUZZ_LAUNCH(obs_merge_stats_kernel, dim3((a.t_count + 255) / 256, heads), dim3(256), 0, st, tm, a, CH, COLS);
        if (hipError_t e = hipGetLastError()) return e;
    }
    if (a.log_n) BUZZ_LAUNCH((obs_mfma_kernel<DT, D, 2, true>), g2, dim3(256), 0, st, tm, a);
    else BUZZ_LAUNCH((obs_mfma_kernel<DT, D, 2, false>), g2, dim3(256), 0, st, tm, a);
    if (hipError_t e = hipGetLastError()) return e;
    if (a.item_parts > 1) {
        BUZZ_LAUNCH(obs_sum_parts_kernel, dim3((a.N + 255) / 256, units), dim3(256), 0, st, tm, a, CH, COLS);
        return hipGetLastError();
    }
    return hipSuccess;
}

template <int DT>
hipError_t launch_obs_mfma_d(int D, const ObsArgs& a, int units, bool* placed, hipStream_t st, Timing tm)
{
    switch (D) {
        case 64: return launch_obs_mfma_t<DT, 64>(a, units, placed, st, tm);
        case 128: return launch_obs_mfma_t<DT, 128>(a, units, placed, st, tm);
        case 256: return launch_obs_mfma_t<DT, 256>(a, units, placed, st, tm);
    }
    return hipErrorInvalidValue;
}

}  // namespace


hipError_t launch_obs_scores(int dtype, int D, const ObsArgs& a, int units, bool* placed, hipStream_t st, Timing tm)
{
    *placed = false;
    if (a.N <= 0 || a.t_count <= 0) return hipSuccess;
    switch (dtype) {
        case BUZZ_FP32: return launch_obs_mfma_d<BUZZ_FP32>(D, a, units, placed, st, tm);
        case BUZZ_FP16: return launch_obs_mfma_d<BUZZ_FP16>(D, a, units, placed, st, tm);
        case BUZZ_BF16: return launch_obs_mfma_d<BUZZ_BF16>(D, a, units, placed, st, tm);
    }
    return hipErrorInvalidValue;
}

}  // namespace buzz
