// The ledger: bookkeeping beyond the default decision rule.
//
//  * Persistence per indicator -- the other reading of Section 4.2's rule that
//    several indicators must deviate and keep deviating over successive evaluations:
//    every metric keeps its own k-of-W count per rank and per node, and the
//    multi-signal rule (primary among them, at least min_signals) is applied to
//    the metrics that are themselves sustained.
//  * The primary node score summed over the window as 16-bit integers, the key of
//    the ranking "by average score" (integer sums do not depend on the order of
//    addition, so the ring can be updated in any order).
//  * Recurrence: how many flag episodes of a node began within a horizon (a node
//    sent to triage three times within a week is terminally bad, Section 7).
//
// A batch (ledger_blocks_kernel) is counted in bit slices (gd_planes.h): the exceed bytes
// of four items are one word of 32 independent series, one per item and metric.  As in the
// window of the default rule, a wave takes 64 steps of 64 neighbouring words and leaves
// their sums as planes in LDS; the window that ends where a block of 64 steps begins is W /
// 64 whole blocks and the tail of one more.  Per block the words tell which items may come
// to satisfy the rule inside it (their counts at its start plus everything that enters).
// A few such words are walked one after another, one lane per step; where there are many --
// ranks that fall behind together, counts that hover about k -- every lane takes its own word
// through the 64 steps, still in bit slices (walk_all): 65 536 ranks x 512 steps, window 100, a
// third of the ranks coming and going 173 -> 59 us, all hovering about k 497 -> 163 (35 with
// nothing flagged).  A third kind of tile follows the default rule's
// own count of the nodes (the rule applied to each step's bytes before they are summed) and
// leaves one bit per (step, node) where an episode starts.  Every workgroup takes a stretch
// of blocks and loads the few before it once more (from the ring at the batch's start), so
// stretches are independent; the first flagged step is the minimum over them (an atomic max
// on 0xFFFFFFFF - step) and the last one stores the counts.
// Bound by the loads (rows of 256 bytes) and their addresses.  Before, a thread kept the
// eight counts of four ranks in 16-bit fields and took every step of a chunk of the
// window's length through a table in LDS: 65 536 ranks x 4 096 steps 257 -> 93 us, 25 840 x
// 142 60 -> 12 us.
// Short batches (ledger_steps_kernel): a thread per four ranks or per node brings the
// stored counts up to date, in time proportional to the steps, where the blocks need the
// whole window: up to 16 steps.
// ledger_finish_kernel, launched behind either: the rings take the batch's last steps, the
// score sums are brought up to date, and a lane per node walks the episode starts in step
// order.
#include "gd_grant.h"
#include "gd_internal.h"
#include "gd_lanes.h"
#include "gd_planes.h"

namespace {

constexpr int WAVE = 64;
constexpr int LED_NT = 256;
constexpr int LED_AHEAD = 8;     // steps whose bytes are fetched together
// Steps up to which counts are brought up to date one by one (whole update, 25 840 ranks x 8,
// window 93, and 65 536 x 8, window 256): 16 steps take 14 and 14 us that way, 32 take 22 and
// 22; blocks, which load the whole window, take 14 and 18 us for 33 steps, 16 and 22 for 64.
constexpr uint32_t SHORT_BATCH = 24;
constexpr uint32_t TILE = WAVE;  // words (of four items) of a workgroup's tile
constexpr int BLOCKS_NT = 1024;
constexpr uint32_t MAX_SLOTS = 2 * BLOCKS_NT / WAVE;      // blocks whose planes a workgroup holds
constexpr int MAX_STARTS = 8;
constexpr int FINISH_NT = 1024;
constexpr int FINISH_CHUNKS = 4 * FINISH_NT / WAVE;       // chunks of 64 steps looked through together

// bits 2j and 2j+1 of an exceed byte as the two 16-bit fields of a word
__device__ __forceinline__ uint32_t spread2(uint32_t b, int j) {
    const uint32_t v = (b >> (2 * j)) & 3u;
    return (v | (v << 15)) & 0x00010001u;
}

// bit m set iff the count of metric m has reached K (counts <= 1024 < 0x8000 - K)
__device__ __forceinline__ uint32_t sustained(const uint32_t (&c)[4], uint32_t K) {
    const uint32_t bias = (0x8000u - K) * 0x00010001u;
    uint32_t pm = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t t = c[j] + bias;
        pm |= ((t >> 15) & 1u) << (2 * j);
        pm |= ((t >> 31) & 1u) << (2 * j + 1);
    }
    return pm;
}

// the multi-signal rule on a byte of metric bits
__device__ __forceinline__ uint32_t combine(uint32_t bits, uint32_t primary, uint32_t min_signals) {
    return ((bits >> primary) & 1u) && (uint32_t)__popc(bits) >= min_signals ? 1u : 0u;
}

// The rule on biased counts (each 16-bit field holds count + 0x8000 - K, so its top
// bit says "sustained"; the primary metric's field is the low half of word 0):
// primary sustained and at least min_signals fields are.
__device__ __forceinline__ uint32_t rule_on_biased(const uint32_t (&c)[4], uint32_t min_signals) {
    uint32_t n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) n += (uint32_t)__popc(c[j] & 0x80008000u);
    return (c[0] & 0x8000u) && n >= min_signals ? 1u : 0u;
}

// Field f of the count words belongs to metric field_metric(f): the identity but for
// the primary metric and metric 0, which change places.
__device__ __forceinline__ uint32_t field_metric(uint32_t f, uint32_t primary) {
    return f == 0 ? primary : (f == primary ? 0u : f);
}

// Short batches.  IPT items per thread: ranks go four at a time (one 4-byte load per step), nodes
// singly, so that a wave's ballot is one word of the episode-start map.
// spread[b] (LDS) = the eight bits of byte b as eight 16-bit fields, spread[256 + b]
// the same words negated, so that one three-operand add per word takes a step.
template <bool NODE, int IPT>
__device__ __forceinline__ void count_items(const gd_ledger_args& a, uint32_t blk, const uint4* spread) {
    static_assert(IPT == 1 || IPT == 4, "count_items");
    static_assert(!NODE || IPT == 1, "count_items");
    const uint32_t n_items = NODE ? a.N : a.R;              // (R is a multiple of 8)
    const uint32_t item = (blk * LED_NT + threadIdx.x) * IPT;
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    if (item - lane * IPT >= n_items) return;               // whole wave out of range
    const bool live = item < n_items;
    const uint32_t i = live ? item : n_items - IPT;         // idle lanes repeat the last items, store nothing
    const uint8_t* mask = NODE ? a.node_mask : a.exceed_mask;
    const uint8_t* ring = a.led + (NODE ? a.lay.node_ring : a.lay.rank_ring);
    uint16_t* cnt = reinterpret_cast<uint16_t*>(a.led + (NODE ? a.lay.node_cnt : a.lay.rank_cnt));
    uint32_t* first = reinterpret_cast<uint32_t*>(a.led + (NODE ? a.lay.node_first : a.lay.rank_first));
    uint16_t* ccnt = reinterpret_cast<uint16_t*>(a.led + a.lay.node_ccnt);
    uint64_t* rise = a.rise;
    const uint32_t W = a.W, K = a.K, T = a.T;
    const uint32_t bias = (0x8000u - K) * 0x00010001u;      // counts <= 1024 and 1 <= K <= 1024: fields never wrap

    auto load = [&](const uint8_t* row) -> uint32_t {       // the IPT exceed bytes of this thread
        if (IPT == 4) return *reinterpret_cast<const uint32_t*>(row + i);
        return row[i];
    };
    // the exceed bytes of step s of the batch; s < 0 reaches back into the ring
    auto hist = [&](int64_t s) -> uint32_t {
        if (s >= 0) return load(mask + (size_t)s * n_items);
        const int64_t g = (int64_t)a.first_step + s;        // (below 2^31)
        return g >= 0 ? load(ring + (size_t)((uint32_t)g % W) * n_items) : 0u;
    };

    uint32_t c[IPT][4];                                     // biased counts
    uint32_t cc = 0;                                        // the default rule's count (nodes)
#pragma unroll
    for (int k = 0; k < IPT; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            c[k][j] = ((uint32_t)cnt[(size_t)field_metric(2 * j, a.primary) * n_items + i + k] |
                       ((uint32_t)cnt[(size_t)field_metric(2 * j + 1, a.primary) * n_items + i + k] << 16)) + bias;
    if (NODE) cc = ccnt[i];
    uint32_t best[IPT];                                     // 0xFFFFFFFF - first flagged step of the batch
#pragma unroll
    for (int k = 0; k < IPT; ++k) best[k] = 0;
    bool cflag = NODE && cc >= K;                           // the default rule's flag one step earlier

    for (uint32_t s = 0; s < T; s += LED_AHEAD) {
        uint32_t eb[LED_AHEAD], lb[LED_AHEAD];
#pragma unroll
        for (int q = 0; q < LED_AHEAD; ++q) {
            eb[q] = 0; lb[q] = 0;
            if (s + q < T) {
                eb[q] = load(mask + (size_t)(s + q) * n_items);
                lb[q] = hist((int64_t)(s + q) - W);
            }
        }
#pragma unroll
        for (int q = 0; q < LED_AHEAD; ++q) {
            if (s + q >= T) break;                          // uniform over the wave
            const uint32_t step_code = 0xFFFFFFFFu - (uint32_t)(a.first_step + s + q);
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint32_t e = (eb[q] >> (8 * k)) & 0xFFu, l = (lb[q] >> (8 * k)) & 0xFFu;
                const uint4 se = spread[e], nl = spread[256 + l];
                c[k][0] += se.x + nl.x; c[k][1] += se.y + nl.y;
                c[k][2] += se.z + nl.z; c[k][3] += se.w + nl.w;
                // the rule needs the primary metric sustained, which it rarely is: only then look further
                if ((c[k][0] & 0x8000u) && !best[k] && rule_on_biased(c[k], a.min_signals)) best[k] = step_code;
                if (NODE) cc = cc + combine(e, a.primary, a.min_signals) - combine(l, a.primary, a.min_signals);
            }
            if (NODE) {
                const bool now = cc >= K;
                const uint64_t rb = __ballot(live && now && !cflag);
                cflag = now;
                // one word per (64 nodes, step), the steps of a word side by side
                if (lane == 0) rise[(size_t)(item / 64) * T + (s + q)] = rb;
            }
        }
    }
    if (!live) return;
#pragma unroll
    for (int k = 0; k < IPT; ++k)
        if (best[k]) atomicMax(&first[i + k], best[k]);
#pragma unroll
    for (int k = 0; k < IPT; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = c[k][j] - bias;
            cnt[(size_t)field_metric(2 * j, a.primary) * n_items + i + k] = (uint16_t)(v & 0xFFFFu);
            cnt[(size_t)field_metric(2 * j + 1, a.primary) * n_items + i + k] = (uint16_t)(v >> 16);
        }
    if (NODE) ccnt[i] = (uint16_t)cc;
}

constexpr int RANK_IPT = 4;

// Blocks [0, rank_blocks) take ranks, the rest nodes.
__global__ __launch_bounds__(LED_NT) void ledger_steps_kernel(const gd_ledger_args a) {
    __shared__ uint4 spread[512];
    {
        const uint32_t b = threadIdx.x;                     // LED_NT == 256: one byte value per thread
        // bit 0 and the primary metric's bit change places: its field is the low half of word 0
        const uint32_t b0 = b & 1u, bp = (b >> a.primary) & 1u;
        const uint32_t v = (b & ~(1u | (1u << a.primary))) | bp | (b0 << a.primary);
        const uint4 f = make_uint4(spread2(v, 0), spread2(v, 1), spread2(v, 2), spread2(v, 3));
        spread[b] = f;
        spread[256 + b] = make_uint4(0u - f.x, 0u - f.y, 0u - f.z, 0u - f.w);
    }
    __syncthreads();
    const uint32_t rank_blocks = (a.R / RANK_IPT + LED_NT - 1) / LED_NT;
    if (blockIdx.x < rank_blocks) count_items<false, RANK_IPT>(a, blockIdx.x, spread);
    else count_items<true, 1>(a, blockIdx.x - rank_blocks, spread);
}

// the rule on the four bytes of a word: the answer is bit 0 of each byte
__device__ __forceinline__ uint32_t combine4(uint32_t E, uint32_t primary, uint32_t min_signals) {
    uint32_t pc = E - ((E >> 1) & 0x55555555u);
    pc = (pc & 0x33333333u) + ((pc >> 2) & 0x33333333u);
    pc = (pc + (pc >> 4)) & 0x0F0F0F0Fu;
    return ((E >> primary) & 0x01010101u) & ((pc + (0x80u - min_signals) * 0x01010101u) >> 7);
}

enum Tiles { RANK_METRICS, NODE_METRICS, NODE_RULE };

// Global pointers by type: a row's address that is put together from two halves would
// otherwise be loaded from as flat memory, through the LDS's counters and without a scalar
// base.
typedef const __attribute__((address_space(1))) uint8_t* gd_row;
struct __attribute__((packed)) gd_any_word { uint32_t v; };
__device__ __forceinline__ uint32_t word_at(gd_row p) {              // (any address)
    return reinterpret_cast<const __attribute__((address_space(1))) gd_any_word*>(p)->v;
}

// Where word w (items 4w .. 4w + 3) of a row of n bytes is loaded from: `at` bytes into the
// row less `back`, shifted down by `shift` bits.  Rows of ranks are whole words.  Rows of
// nodes have any length and address: the last word is loaded as the row's last four bytes,
// so that nothing beyond the row is read; of a row of fewer than four, as the four bytes
// that end with it -- and where that would reach back beyond the batch's first byte (`early`
// rows) as those that begin with it, which have to be moved up first.
struct WordPlace {
    uint32_t at, shift, back;
    __device__ __forceinline__ WordPlace(uint32_t w, uint32_t n, bool ranks) {
        back = ranks || n >= 4 ? 0u : 4u - n;
        at = ranks ? 4 * w : (n >= 4 ? min(4 * w, n - 4) : 0u);
        shift = ranks ? 0u : (n >= 4 ? 8 * (4 * w - at) : 8 * back);
    }
};

// Words of a block up to which candidates are walked one after another: a word costs about a
// microsecond that way (its loads), and a tenth for every item and metric; walk_all about seven
// in all.
constexpr int FEW_WORDS = 5;

// A block's candidates, all at once: a lane takes its word's 32 series from their counts at the
// block's start (c) through the 64 steps.  Per metric: the first step at which the rule holds
// for an item of `cand` goes to first_of.  Default rule: where a node's count comes to reach K
// its bit in this lane's step's word of `rise` is set.
template <Tiles KIND>
__device__ __forceinline__ void walk_all(const gd_ledger_args& a, const uint8_t* ring, const WordPlace& place,
                                         const uint32_t (&c)[GD_COUNT_PLANES], uint32_t cand, uint32_t before,
                                         uint32_t start, uint32_t w0, uint32_t wc, bool mine, uint32_t lane,
                                         uint32_t* first_of, uint64_t (&rise)[4]) {
    constexpr bool RANKS = KIND == RANK_METRICS, RULE = KIND == NODE_RULE;
    const uint8_t* mask = RANKS ? a.exceed_mask : a.node_mask;
    const uint32_t n_items = RANKS ? a.R : a.N, primary = a.primary, min_signals = a.min_signals;
    const int32_t first = (int32_t)a.first_step, W = (int32_t)a.W;
    uint32_t v[GD_COUNT_PLANES + 1], K = a.K;
    // (opaque: K's bits, a mask each, are otherwise worked out and spilled before every block)
    asm volatile("" : "+s"(K));
    gd_planes_bias(c, K, v);
    // lane j works out the rows of step j (nowhere: row 0 of the batch, dropped)
    const int32_t s = (int32_t)(start + lane), o = s - W;
    const bool ok = s < (int32_t)a.T, old = ok && first + o >= 0;
    auto is_early = [&](int32_t t) { return !RANKS && (uint64_t)(uint32_t)t * n_items < place.back; };
    const bool in_early = ok && is_early(s), out_early = old && o >= 0 && is_early(o);
    const uint8_t *enters = mask, *leaves = mask;
    if (ok) enters = mask + (size_t)(uint32_t)s * n_items - (in_early ? 0 : place.back);
    if (old && o >= 0) leaves = mask + (size_t)(uint32_t)o * n_items - (out_early ? 0 : place.back);
    if (old && o < 0) leaves = ring + (size_t)((uint32_t)(first + o) % (uint32_t)W) * n_items - place.back;
    const uint64_t in_valid = __ballot(ok), out_valid = __ballot(old);
    const uint64_t in_up = RANKS ? 0ull : __ballot(in_early), out_up = RANKS ? 0ull : __ballot(out_early);
    const uint32_t elo = (uint32_t)(uintptr_t)enters, ehi = (uint32_t)((uintptr_t)enters >> 32);
    const uint32_t llo = (uint32_t)(uintptr_t)leaves, lhi = (uint32_t)((uintptr_t)leaves >> 32);
    auto row_of = [&](uint32_t lo, uint32_t hi, int l) {
        return reinterpret_cast<gd_row>((uintptr_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, l) << 32 |
                                        (uint32_t)__builtin_amdgcn_readlane((int)lo, l));
    };
    auto load = [&](gd_row row) -> uint32_t {
        return RANKS ? reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(row)[wc] : word_at(row + place.at);
    };
    auto settle = [&](uint32_t x, bool up, bool on) -> uint32_t {       // (up, on: uniform)
        if (!RANKS) x = (up ? x << place.shift : x) >> place.shift;
        if (RULE) x = combine4(x, primary, min_signals);
        return on ? x : 0u;
    };
    uint32_t open = cand, prev = before, at[6] = {};
#pragma unroll 1
    for (int g = 0; g < 8; ++g) {
        uint32_t in[8], out[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            in[j] = load(row_of(elo, ehi, 8 * g + j));
            out[j] = load(row_of(llo, lhi, 8 * g + j));
        }
        const uint32_t was_open = open;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int l = 8 * g + j;
            gd_planes_step(v, settle(in[j], (in_up >> l) & 1ull, (in_valid >> l) & 1ull),
                           settle(out[j], (out_up >> l) & 1ull, (out_valid >> l) & 1ull));
            const uint32_t reach = v[GD_COUNT_PLANES];
            if (RULE) {
                const uint32_t starts = mine ? reach & ~prev & 0x01010101u : 0u;      // (past the last step nothing changes)
                prev = reach;
                if (__ballot(starts != 0) == 0) continue;
                // sixteen lanes' nodes make a word, the words of a step go to the step's lane
                const uint32_t nib = (starts | (starts >> 7) | (starts >> 14) | (starts >> 21)) & 0xFu;
                uint32_t lo = lane & 8u ? 0u : nib << (4 * (lane & 7u)), hi = lane & 8u ? nib << (4 * (lane & 7u)) : 0u;
                lo |= gd_lane_xor<1>(lo, lane); hi |= gd_lane_xor<1>(hi, lane);
                lo |= gd_lane_xor<2>(lo, lane); hi |= gd_lane_xor<2>(hi, lane);
                lo |= gd_lane_xor<4>(lo, lane); hi |= gd_lane_xor<4>(hi, lane);
                lo |= gd_lane_xor<8>(lo, lane); hi |= gd_lane_xor<8>(hi, lane);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint64_t word = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, 16 * q) << 32 |
                                          (uint32_t)__builtin_amdgcn_readlane((int)lo, 16 * q);
                    rise[q] = (int)lane == l ? word : rise[q];
                }
            } else {
                const uint32_t hit = combine4(reach, primary, min_signals) & open;
                open &= ~hit;
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    if ((j >> p) & 1) at[p] |= hit;
            }
        }
        if (!RULE) {
            const uint32_t hits = was_open & ~open;
#pragma unroll
            for (int p = 0; p < 3; ++p) at[3 + p] |= (g >> p) & 1 ? hits : 0u;
            if (__ballot(open != 0) == 0) break;
        }
    }
    if (RULE) return;
    for (uint32_t bits = cand & ~open; bits; bits &= bits - 1) {
        const uint32_t bit = (uint32_t)__builtin_ctz(bits), item = 4 * (w0 + lane) + bit / 8;
        uint32_t step = start;
#pragma unroll
        for (int p = 0; p < 6; ++p) step += ((at[p] >> bit) & 1u) << p;
        // (an item flagged earlier keeps its earlier step)
        if (item < n_items) atomicMax(&first_of[item], 0xFFFFFFFFu - ((uint32_t)first + step));
    }
}

// run: which stretch of `stretch` blocks of 64 steps; w0: the tile's first word.
template <Tiles KIND>
__device__ __forceinline__ void count_blocks(const gd_ledger_args& a, uint32_t w0, uint32_t run, uint32_t stretch, uint32_t* lds,
                                             uint32_t (&final_planes)[GD_COUNT_PLANES][TILE]) {
    constexpr bool RANKS = KIND == RANK_METRICS, RULE = KIND == NODE_RULE;
    const uint8_t* mask = RANKS ? a.exceed_mask : a.node_mask;
    const uint8_t* ring = a.led + (RANKS ? a.lay.rank_ring : a.lay.node_ring);
    uint32_t* first_of = reinterpret_cast<uint32_t*>(a.led + (RANKS ? a.lay.rank_first : a.lay.node_first));
    const uint32_t n_items = RANKS ? a.R : a.N, words = (n_items + 3) / 4;
    const uint32_t tid = threadIdx.x, nt = blockDim.x, lane = tid & (WAVE - 1);
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid / WAVE), waves = nt / WAVE;
    const uint32_t W = a.W, K = a.K, T = a.T, primary = a.primary, min_signals = a.min_signals;
    static_assert(SHORT_BATCH >= 8, "an early row has four bytes of the batch behind its first");
    const uint32_t q = W / 64, r = W % 64, hist = q + (r ? 1 : 0);     // whole blocks, steps of a tail, slots before a block
    const int32_t first = (int32_t)a.first_step;                       // (first + T below 2^31)
    const uint32_t s0 = run * stretch * 64;
    const uint32_t blocks = min((T - s0 + 63) / 64, stretch);
    const bool last = s0 + blocks * 64 >= T;
    const uint32_t last_start = s0 + (blocks - 1) * 64;                // (the batch's last block, where `last`)
    const uint32_t wc = min(w0 + lane, words - 1);                     // (lanes past the row repeat its last word, and store nothing)
    const bool mine = w0 + lane < words;
    // a slot's planes lie one behind another: of the whole block, then of its tail
    const uint32_t slot_words = (r ? 2 * GD_BLOCK_PLANES - 1 : GD_BLOCK_PLANES) * TILE;
    auto planes_of = [&](uint32_t slot) -> uint32_t* { return lds + slot * slot_words + lane; };
    const WordPlace place(wc, n_items, RANKS);
    // word w of step s of the batch; s < 0 reaches back into the ring
    auto word = [&](int32_t s, uint32_t w) -> uint32_t {
        const WordPlace p(w, n_items, RANKS);
        const uint8_t* row = s >= 0 ? mask + (size_t)(uint32_t)s * n_items : ring + (size_t)((uint32_t)(first + s) % W) * n_items;
        const bool early = !RANKS && s >= 0 && (uint64_t)(uint32_t)s * n_items < p.back;
        uint32_t v = word_at((gd_row)(row + p.at - (early ? 0 : p.back)));
        if (early) v <<= p.shift;
        v >>= p.shift;
        return RULE ? combine4(v, primary, min_signals) : v;
    };

    // Slots [0, hist): the blocks before the stretch; [hist, hist + blocks): its own; one more
    // for the steps that leave the window during the batch's last block.
    for (uint32_t slot = wv; slot < hist + blocks + (last ? 1 : 0); slot += waves) {
        const bool leaving = slot == hist + blocks;
        const int32_t start = leaving ? (int32_t)last_start - (int32_t)W : (int32_t)(s0 + slot * 64) - (int32_t)(hist * 64);
        const uint32_t n = leaving ? T - last_start : 64u;             // steps that count
        // Lane j works out where step j's row lies -- in the batch, before it in the ring, or
        // nowhere (row 0 of the batch is read then and dropped) -- and the rows' addresses are
        // read from the lanes one after another.
        const int32_t s = start + (int32_t)lane;
        const bool ok = lane < n && s < (int32_t)T && s >= -(int32_t)W && first + s >= 0;
        const bool early = !RANKS && ok && s >= 0 && (uint64_t)(uint32_t)s * n_items < place.back;
        const uint8_t* of_lane = mask;
        if (ok && s >= 0) of_lane = mask + (size_t)(uint32_t)s * n_items - (early ? 0 : place.back);
        if (ok && s < 0) of_lane = ring + (size_t)((uint32_t)(first + s) % W) * n_items - place.back;
        const uint64_t early_rows = RANKS ? 0ull : __ballot(early);
        const uint64_t valid = __ballot(ok), in_tail = r ? ~0ull << (64 - r) : 0;
        const uint32_t alo = (uint32_t)(uintptr_t)of_lane, ahi = (uint32_t)((uintptr_t)of_lane >> 32);
        uint32_t v[4][16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if ((valid >> (16 * g) & 0xFFFFull) == 0) continue;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)alo, 16 * g + j);
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)ahi, 16 * g + j);
                const gd_row row = reinterpret_cast<gd_row>((uintptr_t)hi << 32 | lo);
                if (RANKS) v[g][j] = reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(row)[wc];
                else v[g][j] = word_at(row + place.at);
            }
        }
        uint32_t all[GD_BLOCK_PLANES] = {}, end[GD_BLOCK_PLANES] = {};
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t on = (uint32_t)(valid >> (16 * g)) & 0xFFFFu, tail = (uint32_t)(in_tail >> (16 * g)) & on;
            if (on == 0) continue;
            if (!RANKS) {
                if (early_rows) {
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if ((early_rows >> (16 * g + j)) & 1ull) v[g][j] <<= place.shift;
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) v[g][j] >>= place.shift;
            }
            if (RULE) {
#pragma unroll
                for (int j = 0; j < 16; ++j) v[g][j] = combine4(v[g][j], primary, min_signals);
            }
            if (on != 0xFFFFu) {
#pragma unroll
                for (int j = 0; j < 16; ++j) v[g][j] &= (uint32_t)((int32_t)(on << (31 - j)) >> 31);
            }
            gd_add16(all, v[g]);
            if (tail) {
#pragma unroll
                for (int j = 0; j < 16; ++j) v[g][j] &= (uint32_t)((int32_t)(tail << (31 - j)) >> 31);
                gd_add16(end, v[g]);
            }
        }
        uint32_t* o = planes_of(slot);
#pragma unroll
        for (int p = 0; p < GD_BLOCK_PLANES; ++p) o[p * TILE] = all[p];
        if (r) {
#pragma unroll
            for (int p = 0; p < GD_BLOCK_PLANES - 1; ++p) o[(GD_BLOCK_PLANES + p) * TILE] = end[p];      // (at most 63)
        }
    }
    __syncthreads();

    for (uint32_t b = wv; b < blocks; b += waves) {
        // counts where the block begins, and those plus everything that enters during it
        const uint32_t slot = hist + b;
        uint32_t c[GD_COUNT_PLANES] = {}, u[GD_COUNT_PLANES], f[GD_BLOCK_PLANES];
        for (uint32_t back = 1; back <= q; ++back) {
#pragma unroll
            for (int p = 0; p < GD_BLOCK_PLANES; ++p) f[p] = planes_of(slot - back)[p * TILE];
            gd_planes_add(c, f);
        }
        if (r) {
            uint32_t e[GD_BLOCK_PLANES - 1];
#pragma unroll
            for (int p = 0; p < GD_BLOCK_PLANES - 1; ++p) e[p] = planes_of(slot - q - 1)[(GD_BLOCK_PLANES + p) * TILE];
            gd_planes_add(c, e);
        }
#pragma unroll
        for (int p = 0; p < GD_COUNT_PLANES; ++p) u[p] = c[p];
#pragma unroll
        for (int p = 0; p < GD_BLOCK_PLANES; ++p) f[p] = planes_of(slot)[p * TILE];
        gd_planes_add(u, f);
        // the count after the last step: what enters during the last block, less what leaves
        if (last && b == blocks - 1) {
            uint32_t fin[GD_COUNT_PLANES];
#pragma unroll
            for (int p = 0; p < GD_COUNT_PLANES; ++p) fin[p] = u[p];
#pragma unroll
            for (int p = 0; p < GD_BLOCK_PLANES; ++p) f[p] = planes_of(hist + blocks)[p * TILE];
            gd_planes_sub(fin, f);
#pragma unroll
            for (int p = 0; p < GD_COUNT_PLANES; ++p) final_planes[p][lane] = fin[p];
        }
        const uint32_t before = gd_planes_reach(c, K), most = gd_planes_reach(u, K);
        uint32_t cand;
        if (RULE) cand = most & ~gd_planes_reach(c, K + 64);           // (a flag that nothing can lower does not rise)
        else cand = combine4(most, primary, min_signals) & ~combine4(before, primary, min_signals);
        if (!mine) cand = 0;
        const int32_t start = (int32_t)(s0 + b * 64), s = start + (int32_t)lane;       // this lane's step in a walk
        const uint64_t upto = (2ull << lane) - 1;
        uint64_t rise[4] = {};                                         // this step's episode starts, 64 nodes a word
        uint64_t todo = __ballot(cand != 0);
        if (__builtin_expect(__popcll(todo) > FEW_WORDS, 0)) {
            walk_all<KIND>(a, ring, place, c, cand, before, (uint32_t)start, w0, wc, mine, lane, first_of, rise);
            todo = 0;
        }
        for (; todo; todo &= todo - 1) {
            const int src = __builtin_ctzll(todo);
            const uint32_t w = w0 + (uint32_t)src;
            uint32_t enters = 0, leaves = 0;
            if (s < (int32_t)T) {
                enters = word(s, w);
                if (first + s - (int32_t)W >= 0) leaves = word(s - (int32_t)W, w);
            }
            // the counts of the word's 32 series where the block begins, one in each lane ...
            uint32_t at_start = 0;
#pragma unroll
            for (int p = 0; p < GD_COUNT_PLANES; ++p)
                at_start |= (((uint32_t)__builtin_amdgcn_readlane((int)c[p], src) >> (lane & 31)) & 1u) << p;
            // ... and this lane's count of a series after its step
            auto count_of = [&](uint32_t bit) -> uint32_t {
                const uint64_t in = __ballot((enters >> bit) & 1u), out = __ballot((leaves >> bit) & 1u);
                return (uint32_t)__builtin_amdgcn_readlane((int)at_start, (int)bit) + (uint32_t)__popcll(in & upto) -
                       (uint32_t)__popcll(out & upto);
            };
            const uint32_t cands = (uint32_t)__builtin_amdgcn_readlane((int)cand, src);
            if (RULE) {
                const uint32_t flagged = (uint32_t)__builtin_amdgcn_readlane((int)before, src);
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    if (!((cands >> (8 * k)) & 1u)) continue;
                    const uint64_t on = __ballot(count_of(8 * k) >= K && s < (int32_t)T);
                    const uint64_t starts = on & ~((on << 1) | ((flagged >> (8 * k)) & 1u));
                    const uint64_t node = ((starts >> lane) & 1ull) << (4 * (src % 16) + k);
#pragma unroll
                    for (int g = 0; g < 4; ++g) rise[g] |= src / 16 == g ? node : 0ull;
                }
                continue;
            }
            // items flagged before this block are left alone, as are those beyond the last one
            const uint32_t item = 4 * w + (lane & 3);
            const uint32_t seen = item < n_items ? first_of[item] : 0xFFFFFFFFu;
            const uint32_t done = (uint32_t)__ballot(seen != 0 && 0xFFFFFFFFu - seen < (uint32_t)(first + start));
            const uint32_t may = (uint32_t)__builtin_amdgcn_readlane((int)most, src);      // series that may be sustained
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                if (!((cands >> (8 * k)) & 1u) || ((done >> k) & 1u) || 4 * w + k >= n_items) continue;
                const bool prim = count_of(8 * k + primary) >= K && s < (int32_t)T;
                if (__ballot(prim) == 0) continue;
                uint32_t n = 1;
                for (uint32_t bits = (may >> (8 * k)) & 0xFFu & ~(1u << primary); bits; bits &= bits - 1)
                    n += count_of(8 * k + (uint32_t)__builtin_ctz(bits)) >= K ? 1u : 0u;
                const uint64_t reach = __ballot(prim && n >= min_signals);
                if (reach && lane == 0)
                    atomicMax(&first_of[4 * w + k], 0xFFFFFFFFu - (uint32_t)(first + start + __builtin_ctzll(reach)));
            }
        }
        if (RULE) {
            // one word per (64 nodes, step), the steps of a word side by side
            const uint32_t NW = (n_items + 63) / 64;
#pragma unroll
            for (uint32_t g = 0; g < 4; ++g)
                if (w0 / 16 + g < NW && s < (int32_t)T) a.rise[(size_t)(w0 / 16 + g) * T + (uint32_t)s] = rise[g];
        }
    }
    if (!last) return;
    __syncthreads();
    uint16_t* cnt = reinterpret_cast<uint16_t*>(a.led + (RANKS ? a.lay.rank_cnt : (RULE ? a.lay.node_ccnt : a.lay.node_cnt)));
    for (uint32_t x = tid; x < TILE * 4 * (RULE ? 1u : 8u); x += nt) {
        const uint32_t at = x % (TILE * 4), m = x / (TILE * 4), item = 4 * w0 + at;
        if (item >= n_items) continue;
        uint32_t v = 0;
#pragma unroll
        for (int p = 0; p < GD_COUNT_PLANES; ++p) v |= ((final_planes[p][at / 4] >> (8 * (at % 4) + m)) & 1u) << p;
        cnt[(size_t)m * n_items + item] = (uint16_t)v;
    }
}

// A workgroup takes a tile (of ranks, of nodes, of nodes once more for the default rule) and a
// stretch: tiles along x and stretches along y where side_by_side, the other way round otherwise.
// Dynamic LDS: planes of every slot -- a block of the stretch or one of the few before it -- and word.
__global__ __launch_bounds__(BLOCKS_NT) void ledger_blocks_kernel(const gd_ledger_args a, uint32_t rank_tiles,
                                                                  uint32_t node_tiles, uint32_t stretch, bool side_by_side) {
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t final_planes[GD_COUNT_PLANES][TILE];
    const uint32_t y = side_by_side ? blockIdx.x : blockIdx.y, run = side_by_side ? blockIdx.y : blockIdx.x;
    if (y < rank_tiles) count_blocks<RANK_METRICS>(a, y * TILE, run, stretch, lds, final_planes);
    else if (y < rank_tiles + node_tiles) count_blocks<NODE_METRICS>(a, (y - rank_tiles) * TILE, run, stretch, lds, final_planes);
    else count_blocks<NODE_RULE>(a, (y - rank_tiles - node_tiles) * TILE, run, stretch, lds, final_planes);
}

__device__ __forceinline__ int32_t quantise(float z, float quant) {
    const float v = z * quant;
    float r = __builtin_rintf(v);                           // ties to even
    r = fminf(fmaxf(r, -32768.0f), 32767.0f);
    return v == v ? (int32_t)r : 0;                         // a NaN counts as 0
}

// Blocks [0, NW): 64 nodes, a lane each -- score ring and sum (every wave takes every
// waves-th step), then the episode starts in step order.  Blocks after them copy the batch's
// last min(T, W) exceed bytes into the rings, each a piece of a step's row: rank_pieces of
// 4 words per thread, then node_pieces of 8 bytes per thread.
__global__ __launch_bounds__(FINISH_NT) void ledger_finish_kernel(const gd_ledger_args a, uint32_t rank_pieces,
                                                                  uint32_t node_pieces) {
    __shared__ int32_t partial[FINISH_NT / WAVE][WAVE];
    __shared__ uint64_t found[FINISH_CHUNKS][WAVE], any[FINISH_CHUNKS];
    const uint32_t W = a.W, T = a.T, N = a.N, R = a.R, NW = (N + 63) / 64;
    const uint32_t keep = T < W ? T : W, nt = blockDim.x, tid = threadIdx.x;
    const uint32_t first = (uint32_t)a.first_step;          // (first + T below 2^31)
    if (blockIdx.x >= NW) {
        const uint32_t piece = (blockIdx.x - NW) % (rank_pieces + node_pieces);
        const uint32_t s = T - keep + (blockIdx.x - NW) / (rank_pieces + node_pieces), slot = (first + s) % W;
        if (piece < rank_pieces) {
            // (R is a multiple of 8 and both arrays are word-aligned)
            const uint32_t* from = reinterpret_cast<const uint32_t*>(a.exceed_mask + (size_t)s * R);
            uint32_t* to = reinterpret_cast<uint32_t*>(a.led + a.lay.rank_ring + (size_t)slot * R);
            uint32_t v[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) v[k] = from[min((piece * 4 + k) * nt + tid, R / 4 - 1)];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if ((piece * 4 + k) * nt + tid < R / 4) to[(piece * 4 + k) * nt + tid] = v[k];
        } else {
            const uint32_t at = (piece - rank_pieces) * 8 * nt + tid;
            const uint8_t* from = a.node_mask + (size_t)s * N;
            uint8_t* to = a.led + a.lay.node_ring + (size_t)slot * N;
            uint8_t v[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) v[k] = from[min(at + k * nt, N - 1)];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k)
                if (at + k * nt < N) to[at + k * nt] = v[k];
        }
        return;
    }
    const uint32_t lane = tid & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane(tid / WAVE), waves = nt / WAVE;
    const uint32_t n = blockIdx.x * WAVE + lane;
    const bool live = n < N;
    const uint32_t i = live ? n : N - 1;                    // (idle lanes repeat the last node, and store nothing)
    if (n == 0 && wv == 0) reinterpret_cast<uint64_t*>(a.led + a.lay.head)[0] = a.first_step + T;

    // score ring and sum
    int16_t* qring = reinterpret_cast<int16_t*>(a.led + a.lay.node_qring);
    int32_t* qsum = reinterpret_cast<int32_t*>(a.led + a.lay.node_qsum);
    int32_t sum = 0;
    for (uint32_t s = T - keep + wv; s < T; s += LED_AHEAD * waves) {
        float z[LED_AHEAD];
        int32_t old[LED_AHEAD];
#pragma unroll
        for (uint32_t q = 0; q < LED_AHEAD; ++q) {
            const uint32_t sq = min(s + q * waves, T - 1);
            z[q] = a.node_z[(size_t)sq * N + i];
            // (zero while the window is still filling; a batch of W steps or more starts afresh)
            old[q] = T < W ? (int32_t)qring[(size_t)((first + sq) % W) * N + i] : 0;
        }
#pragma unroll
        for (uint32_t q = 0; q < LED_AHEAD; ++q) {
            const uint32_t sq = s + q * waves;
            if (sq >= T) break;
            const int32_t v = quantise(z[q], a.quant);
            sum += v - old[q];
            if (live) qring[(size_t)((first + sq) % W) * N + i] = (int16_t)v;
        }
    }
    partial[wv][lane] = sum;
    __syncthreads();
    int32_t st[MAX_STARTS], tf = 0;
    int32_t* starts = reinterpret_cast<int32_t*>(a.led + a.lay.node_starts);
    int32_t* term = reinterpret_cast<int32_t*>(a.led + a.lay.node_term);
    if (wv == 0) {
        sum = T < W ? qsum[i] : 0;
        for (uint32_t q = 0; q < waves; ++q) sum += partial[q][lane];
        if (live) qsum[i] = sum;
#pragma unroll
        for (int j = 0; j < MAX_STARTS; ++j) st[j] = starts[(size_t)j * N + i];
        tf = term[i];
    }

    // Episode starts, in step order.  All waves look for words that hold one (a lane per
    // step, FINISH_CHUNKS chunks of 64 steps at a time); the first wave hands those round.
    const uint64_t* rise = a.rise + (size_t)blockIdx.x * T;
    bool changed = false;
    constexpr uint32_t PER = 4;                             // chunks that a wave fetches together
    const uint32_t at_once = PER * waves;                   // (at most FINISH_CHUNKS)
    for (uint32_t s = 0; s < T; s += at_once * WAVE) {
        uint64_t v[PER];
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t sq = s + (q * waves + wv) * WAVE + lane;
            v[q] = sq < T ? rise[sq] : 0ull;
        }
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint64_t some = __ballot(v[q] != 0);
            if (lane == 0) any[q * waves + wv] = some;
            if (some) found[q * waves + wv][lane] = v[q];
        }
        __syncthreads();
        if (wv == 0) {
            for (uint64_t chunks = __ballot(lane < at_once && any[lane < at_once ? lane : 0] != 0); chunks; chunks &= chunks - 1) {
                const uint32_t c = (uint32_t)__builtin_ctzll(chunks);
                const uint64_t mine = found[c][lane];
                for (uint64_t some = __ballot(mine != 0); some; some &= some - 1) {
                    const int j = __builtin_ctzll(some);
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, j);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), j);
                    const uint64_t w = ((uint64_t)hi << 32) | lo;
                    if (!((w >> lane) & 1ull)) continue;
                    const int64_t t = (int64_t)(a.first_step + s + c * WAVE + j);
#pragma unroll
                    for (int jj = MAX_STARTS - 1; jj > 0; --jj) st[jj] = st[jj - 1];
                    st[0] = (int32_t)t + 1;
                    changed = true;
                    // episodes that began inside (t - horizon, t], this one included
                    uint32_t inside = 0;
#pragma unroll
                    for (int jj = 0; jj < MAX_STARTS; ++jj)
                        inside += (st[jj] != 0 && (int64_t)(st[jj] - 1) + (int64_t)a.horizon > t) ? 1u : 0u;
                    if (inside >= a.limit && tf == 0) tf = (int32_t)t + 1;
                }
            }
        }
        __syncthreads();
    }
    if (wv == 0 && live && changed) {
#pragma unroll
        for (int j = 0; j < MAX_STARTS; ++j) starts[(size_t)j * N + i] = st[j];
        term[i] = tf;
    }
}

__global__ __launch_bounds__(LED_NT) void ledger_flags_kernel(const gd_ledger_flags_args a) {
    const uint32_t i = blockIdx.x * LED_NT + threadIdx.x;
    auto read_out = [&](const uint16_t* cnt, const uint32_t* first, uint32_t n_items, uint8_t* pmask,
                        uint8_t* pflag, int32_t* pfirst) {
        uint32_t c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            c[j] = (uint32_t)cnt[(size_t)(2 * j) * n_items + i] |
                   ((uint32_t)cnt[(size_t)(2 * j + 1) * n_items + i] << 16);
        const uint32_t pm = sustained(c, a.K);
        if (pmask) pmask[i] = (uint8_t)pm;
        if (pflag) pflag[i] = (uint8_t)combine(pm, a.primary, a.min_signals);
        if (pfirst) pfirst[i] = first[i] ? (int32_t)(0xFFFFFFFFu - first[i]) : -1;
    };
    if (i < a.R)
        read_out(reinterpret_cast<const uint16_t*>(a.led + a.lay.rank_cnt),
                 reinterpret_cast<const uint32_t*>(a.led + a.lay.rank_first), a.R, a.rank_pmask,
                 a.rank_pflag, a.rank_pfirst);
    if (i < a.N) {
        read_out(reinterpret_cast<const uint16_t*>(a.led + a.lay.node_cnt),
                 reinterpret_cast<const uint32_t*>(a.led + a.lay.node_first), a.N, a.node_pmask,
                 a.node_pflag, a.node_pfirst);
        if (a.node_score_sum)
            a.node_score_sum[i] = reinterpret_cast<const int32_t*>(a.led + a.lay.node_qsum)[i];
        const int32_t* starts = reinterpret_cast<const int32_t*>(a.led + a.lay.node_starts);
        const uint64_t next = reinterpret_cast<const uint64_t*>(a.led + a.lay.head)[0];
        if (a.node_episodes) {
            uint32_t inside = 0;
            if (next > 0) {
                const int64_t t = (int64_t)next - 1;        // the last step taken in
#pragma unroll
                for (int j = 0; j < MAX_STARTS; ++j) {
                    const int32_t st = starts[(size_t)j * a.N + i];
                    inside += (st != 0 && (int64_t)(st - 1) + (int64_t)a.horizon > t) ? 1u : 0u;
                }
            }
            a.node_episodes[i] = (uint8_t)min(inside, a.limit);
        }
        if (a.node_terminal_first)
            a.node_terminal_first[i] = reinterpret_cast<const int32_t*>(a.led + a.lay.node_term)[i] - 1;
    }
}

}  // namespace

hipError_t gd_launch_ledger(const gd_ledger_args& a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    if (a.limit < 1 || a.limit > (uint32_t)MAX_STARTS) return hipErrorInvalidValue;
    // The line moves up where the window's rows alone take long to load.  us by steps / by
    // blocks, window 1 024: 65 536 ranks, 25 steps 20 / 38, 32 23 / 38, 48 32 / 40, 56 36 / 41;
    // 49 152 ranks, 25 steps 19 / 25, 36 25 / 26; 32 768 ranks, 24 steps 19 / 22, 32 22 / 23.
    const uint64_t window_bytes = (uint64_t)a.W * a.R;
    const uint32_t by_step = SHORT_BATCH + (window_bytes > 1u << 25 ? (uint32_t)((window_bytes - (1u << 25)) >> 20) : 0u);
    if (a.T <= by_step) {
        const uint32_t item_blocks = (a.R / RANK_IPT + LED_NT - 1) / LED_NT + (a.N + LED_NT - 1) / LED_NT;
        hipLaunchKernelGGL(ledger_steps_kernel, dim3(item_blocks), dim3(LED_NT), 0, s, a);
    } else {
        const uint32_t rank_tiles = (a.R / 4 + TILE - 1) / TILE, node_tiles = ((a.N + 3) / 4 + TILE - 1) / TILE;
        const uint32_t tiles = rank_tiles + 2 * node_tiles;
        const uint32_t q = a.W / 64, r = a.W % 64, hist = q + (r ? 1 : 0), blocks = (a.T + 63) / 64;
        // Long stretches load less twice (hist blocks each), short ones fill the chip: two
        // blocks per wave of a 16-wave workgroup, less while there are not two workgroups per
        // CU to run side by side -- or as many as let two of eight waves share a CU by LDS, where
        // windows with a tail take twice the planes and there are few blocks to load twice.
        constexpr size_t slot_bytes = GD_BLOCK_PLANES * TILE * 4, tail_bytes = (GD_BLOCK_PLANES - 1) * TILE * 4;
        constexpr uint32_t TAIL_SLOTS = 22;
        static_assert(2 * (MAX_SLOTS * slot_bytes + 1024 + sizeof(uint32_t) * GD_COUNT_PLANES * TILE) <= 160 * 1024 &&
                      2 * (TAIL_SLOTS * (slot_bytes + tail_bytes) + 1024 + sizeof(uint32_t) * GD_COUNT_PLANES * TILE) <= 160 * 1024,
                      "two workgroups of eight waves share a CU's LDS");
        const bool tail_pairs = r && hist <= 4;
        uint32_t stretch = (tail_pairs ? TAIL_SLOTS : MAX_SLOTS) - 1 - hist;
        if (stretch > blocks) stretch = blocks;
        while (stretch > 4 && (uint64_t)((blocks + stretch - 1) / stretch) * tiles < 512) --stretch;
        const uint32_t stretches = (blocks + stretch - 1) / stretch, slots = hist + stretch + 1;
        if (stretches > 0x7FFFFFFFu / 1024 || tiles > 65535u) return hipErrorInvalidValue;
        // Sixteen waves (registers for as many a CU), or eight, two workgroups of which a CU holds: one
        // loads while the other counts.  An update, sixteen / eight: 65 536 ranks x 4 096 steps, window 64
        // 90.5 / 88, 100 100 / 85, 200 105 / 97.5, 256 102.4 / 94.0, 384 115 / 107, 512 123 / 115; 65 536 x
        // 2 000, window 20 63 / 51, 256 66 / 64; 16 384 x 10 000, 128 68 / 60, 100 72 / 70.5; 8 192 x 10 000,
        // 256 50.8 / 43.8; 32 768 x 4 096, 256 56 / 54.5.  Not where every wave has one block of sixteen or
        // less to load (65 536 x 512, 256 39.0 / 39.8), nor where few workgroups have long windows before them
        // (65 536 x 2 000, 512 77.7 / 83) or, with a tail, the many slots that these take leave room for
        // one workgroup (40 000 x 3 000, 300 69 / 75).
        const bool pairs = slots > (uint32_t)BLOCKS_NT / WAVE &&
                           (r ? tail_pairs : q <= 6 || (uint64_t)stretches * tiles >= 768);
        const uint32_t most_waves = (pairs ? BLOCKS_NT / 2 : BLOCKS_NT) / WAVE;
        const uint32_t nt = (slots < most_waves ? slots : most_waves) * WAVE;
        const size_t lds = (size_t)(r ? 2 * GD_BLOCK_PLANES - 1 : GD_BLOCK_PLANES) * slots * TILE * 4;
        constexpr size_t most = (size_t)(2 * GD_BLOCK_PLANES - 1) * MAX_SLOTS * TILE * 4;
        static_assert(most + sizeof(uint32_t) * GD_COUNT_PLANES * TILE <= 160 * 1024, "LDS budget of one CU");
        static std::atomic<uint64_t> granted{0};
        const hipError_t e = gd_grant_lds(granted, reinterpret_cast<const void*>(ledger_blocks_kernel), most);
        if (e != hipSuccess) return e;
        // Workgroups that start one behind another take neighbouring tiles of the same stretch, that is
        // neighbouring pieces of the same rows, where there are many of both.  An update, stretches of a tile
        // one behind another / tiles side by side, window 256: 65 536 ranks x 4 096 steps 102 / 103 us, x 2 000
        // 80 / 65, x 512 43 / 39; 32 768 x 4 096 69 / 56; 16 384 x 1 024 31.0 / 26.1 (320 workgroups), x 512
        // 21.3 / 21.7 (160), x 10 000 67.5 / 68.6; few tiles find less in the caches: 1 000 ranks (6 tiles) x
        // 10 000 21.4 / 22.9, window 1 024 45.6 / 48.0.
        const bool side_by_side = tiles >= 16 && (uint64_t)stretches * tiles > 256 && stretches <= 65535u;
        hipLaunchKernelGGL(ledger_blocks_kernel, side_by_side ? dim3(tiles, stretches) : dim3(stretches, tiles), dim3(nt),
                           lds, s, a, rank_tiles, node_tiles, stretch, side_by_side);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t NW = (a.N + 63) / 64, keep = a.T < a.W ? a.T : a.W;
    const uint32_t waves = keep < 8 * (FINISH_NT / WAVE) ? (keep + 7) / 8 : FINISH_NT / WAVE, nt = waves * WAVE;
    const uint32_t rank_pieces = (a.R / 4 + 4 * nt - 1) / (4 * nt), node_pieces = (a.N + 8 * nt - 1) / (8 * nt);
    hipLaunchKernelGGL(ledger_finish_kernel, dim3(NW + keep * (rank_pieces + node_pieces)), dim3(nt), 0, s, a,
                       rank_pieces, node_pieces);
    return hipGetLastError();
}

// Work spans for callers that may not allocate (code under graph capture, serving loops
// that forbid hipMalloc): one array per GPU, held from the first use until the process
// ends.  Host code never uses the array's name as an address: the device address is
// asked for once per device and kept.
constexpr size_t LEDGER_SCRATCH_BYTES = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[LEDGER_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
unsigned char* g_scratch_ptr[MAX_DEVICES];     // device address of `scratch` on each GPU, null = not asked yet
}  // namespace

size_t gd_ledger_static_bytes() { return LEDGER_SCRATCH_BYTES; }

hipError_t gd_launch_ledger_static(gd_ledger_args a, hipStream_t s, bool* fits) {
    *fits = true;
    if (a.T == 0) return hipSuccess;
    const size_t NW = ((size_t)a.N + 63) / 64;
    const size_t rise_bytes = ((size_t)a.T * NW * 8 + 255) & ~(size_t)255;
    // (counts_bytes: nothing is kept there any more, but the bound is the one that guard.h states,
    // and a batch that was refused stays refused)
    if (rise_bytes + a.lay.counts_bytes > LEDGER_SCRATCH_BYTES) { *fits = false; return hipSuccess; }
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
    }
    // The map does not have to start at zero: the counting kernel writes every (node word,
    // step) of it before the finishing kernel, behind it on the stream, reads them.
    a.rise = reinterpret_cast<uint64_t*>(g_scratch_ptr[dev]);
    return gd_launch_ledger(a, s);
}

hipError_t gd_launch_ledger_flags(const gd_ledger_flags_args& a, hipStream_t s) {
    const uint32_t blocks = (a.R + LED_NT - 1) / LED_NT;
    hipLaunchKernelGGL(ledger_flags_kernel, dim3(blocks), dim3(LED_NT), 0, s, a);
    return hipGetLastError();
}
