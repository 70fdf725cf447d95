// Sliding-window persistence (k anomalous evaluations among the last W: the
// requirement of Section 4.2 that a deviation persists over several evaluations
// in a row before a node is flagged) and the read-out of the current flags.
//
// State in HBM, per item (a rank or a node): a ring of the last W anomaly bits,
// stored as the scoring kernel's own bit words ring[step % W][item / 64]; a u16
// count of set bits inside the window; the first flagged step (+1, 0 = never).
//
// A batch (window_blocks_kernel) is counted in bit slices, 32 items per word (see
// gd_planes.h).  Steps are cut into blocks of 64.  A wave takes one block of 64
// neighbouring words (2 048 items): the rows' addresses are scalars, a lane's 64 loads
// are independent of each other and a row's 64 lanes read two whole cache lines.  It
// leaves the sum of the block, and of its last W % 64 steps, as planes in LDS.  The
// window that ends where a block begins is then W / 64 whole blocks and the tail of one
// more, a handful of bit-sliced additions.  An item can only reach k inside a block if
// its count at the block's start plus everything that enters does, and if it had not
// reached it already.  Where that test leaves a few words of a block, the wave walks them
// item by item, one lane per step (two ballots give an item's entering and leaving bits as
// 64-bit time vectors).  Where it leaves many -- ranks that fall behind together, counts that
// hover about k -- every lane takes its own word through the 64 steps, all items at once and
// still in bit slices (walk_all), which costs the same whatever the number of items: 65 536
// ranks x 1 024 steps, a third of them flagged at one step, 17 us, where the walk
// by item takes 396 (13 with nothing flagged).
//
// A workgroup takes a stretch of blocks and loads the W / 64 blocks before it once more.
// Stretches are as short as the window allows (four blocks at least): the loads are
// bound by the requests that one CU can have in flight, so they are spread over as many
// CUs as there are stretches (one workgroup per tile over all steps: 26.6 us where this
// takes 18).  Only the first stretch looks at the ring (the others begin W steps or
// more into the batch), so it also stores the ring's new words, behind its own last
// read; the last stretch stores the counts, which nobody reads.  The first flagged steps
// are kept by compare-and-swap (gathered in LDS first where there are many).
//
// Measured against the kernel of short batches: 65 536 ranks x 4 096 steps 52.5 -> 18 us
// (57 MB loaded in 9 of them), 16 384 x 10 000 117 -> 11.8 us, 1 024 x 2 000 29.4 -> 8.1 us.
//
// Short batches (window_short_kernel) start from the stored counts instead of the whole
// window: every 64 items have a wave that walks the batch in order, 64 steps at a time,
// transposing 64 x 64 bits across its lanes (one wave per SIMD at 65 536 ranks and fewer
// below, waiting for its loads and lane exchanges).
// One step per call (window_step_kernel) needs none of this: a thread per item.
#include "gd_grant.h"
#include "gd_internal.h"
#include "gd_lanes.h"
#include "gd_planes.h"

namespace {

constexpr int WAVE = 64;
constexpr int WIN_NT = 256;
constexpr uint32_t TILE = WAVE;          // 32-bit words of a workgroup's tile
constexpr uint32_t MIN_STRETCH = 4, MAX_STRETCH = 16;      // blocks of 64 steps
constexpr uint32_t MAX_HISTORY = 16;     // blocks that a window of 1 024 steps reaches back
constexpr int WIN_MAX_NT = 1024;
constexpr uint32_t SHORT_BATCH = 256;    // steps up to which a batch is walked in order, whatever the window
// Words of a block, and items of a word, up to which candidates are walked item by item: a
// word costs about a microsecond that way (its loads) and an item a tenth, walk_all about
// five in all.
constexpr int FEW_WORDS = 4, FEW_ITEMS = 8;
constexpr uint32_t FOUND_PITCH = TILE + 1;                 // (items in order and lanes side by side: no bank conflicts)

// Where one kind of item (ranks or nodes) lives.
struct WindowItems {
    const uint32_t* anom;    // [T][row]
    uint32_t* ring;          // [W][row]
    uint16_t* count;
    int32_t* first;
    uint32_t n, row;         // items; 32-bit words per step (even)
};

__device__ __forceinline__ WindowItems window_items(const gd_window_args& a, bool is_node) {
    WindowItems it;
    it.anom = reinterpret_cast<const uint32_t*>(is_node ? a.node_anom : a.rank_anom);
    it.ring = reinterpret_cast<uint32_t*>(a.state + (is_node ? a.lay.node_ring : a.lay.rank_ring));
    it.count = reinterpret_cast<uint16_t*>(a.state + (is_node ? a.lay.node_count : a.lay.rank_count));
    it.first = reinterpret_cast<int32_t*>(a.state + (is_node ? a.lay.node_first : a.lay.rank_first));
    it.n = is_node ? a.N : a.R;
    it.row = 2 * ((it.n + 63) / 64);
    return it;
}

// One step: blocks [0, rank_blocks) take ranks, the rest nodes.
__global__ __launch_bounds__(WIN_NT) void window_step_kernel(const gd_window_args a) {
    const uint32_t rank_blocks = (a.R + WIN_NT - 1) / WIN_NT;
    const bool is_node = blockIdx.x >= rank_blocks;
    const WindowItems it = window_items(a, is_node);
    const uint32_t item = (is_node ? blockIdx.x - rank_blocks : blockIdx.x) * WIN_NT + threadIdx.x;
    const uint32_t word = item / 32;
    if (word >= it.row) return;
    const uint32_t t = (uint32_t)a.first_step;                  // (below 2^31)
    uint32_t* slot = it.ring + (size_t)(t % a.W) * it.row + word;
    const uint32_t in = it.anom[word], out = t >= a.W ? *slot : 0u;
    if (item < it.n) {
        const uint32_t c = it.count[item] + ((in >> (item & 31)) & 1u) - ((out >> (item & 31)) & 1u);
        it.count[item] = (uint16_t)c;
        if (c >= a.K && it.first[item] == 0) it.first[item] = (int32_t)t + 1;
        if (is_node) reinterpret_cast<float*>(a.state + a.lay.node_z_last)[item] = a.node_z[item];
    }
    // (the word's 32 readers are lanes of one wave: all of them have read the slot)
    if ((item & 31) == 0) *slot = in;
}

// The first flagged step (+1, 0 = never) of an item becomes `step` unless it is an earlier one
// already, of an earlier batch or another block of this one.
__device__ __forceinline__ void lower_first(int32_t* to, int32_t step) {
    int32_t was = 0;
    while (was == 0 || was > step) {                                   // (ends: the stored step only ever falls)
        const int32_t now = atomicCAS(to, was, step);
        if (now == was) break;
        was = now;
    }
}

// The candidates `cand` of one block, all at once: a lane takes its word's 32 items from their
// counts at the block's start through the 64 steps and notes, in bit slices again, the step at
// which each reaches K first.  Those steps (of the batch) lower found[item's bit][lane].
__device__ __forceinline__ void walk_all(const WindowItems& it, const uint32_t (&c)[GD_COUNT_PLANES], uint32_t cand,
                                         uint32_t start, int32_t first, uint32_t T, uint32_t W, uint32_t K,
                                         uint32_t wc, uint32_t lane, uint32_t* found) {
    uint32_t v[GD_COUNT_PLANES + 1];
    // (opaque: K's bits, a mask each, are otherwise worked out and spilled before every block)
    asm volatile("" : "+s"(K));
    gd_planes_bias(c, K, v);
    // (lane j works out the rows of step j, as in the counting of the blocks)
    const uint32_t s = start + lane;
    const int32_t o = (int32_t)s - (int32_t)W;
    const bool ok = s < T, old = ok && (o >= 0 || first + o >= 0);
    const uint32_t* enters = it.anom + (ok ? (size_t)s * it.row : 0);
    const uint32_t* leaves = it.anom + (old && o >= 0 ? (size_t)(uint32_t)o * it.row : 0);
    if (old && o < 0) leaves = it.ring + (size_t)((uint32_t)(first + o) % W) * it.row;
    const uint64_t in_valid = __ballot(ok), out_valid = __ballot(old);
    const uint32_t elo = (uint32_t)(uintptr_t)enters, ehi = (uint32_t)((uintptr_t)enters >> 32);
    const uint32_t llo = (uint32_t)(uintptr_t)leaves, lhi = (uint32_t)((uintptr_t)leaves >> 32);
    uint32_t open = cand, at[6] = {};                // items not found yet; bit slices of the steps
#pragma unroll 1
    for (int g = 0; g < 8; ++g) {
        uint32_t in[8], out[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int l = 8 * g + j;
            const uint32_t e0 = (uint32_t)__builtin_amdgcn_readlane((int)elo, l), e1 = (uint32_t)__builtin_amdgcn_readlane((int)ehi, l);
            const uint32_t l0 = (uint32_t)__builtin_amdgcn_readlane((int)llo, l), l1 = (uint32_t)__builtin_amdgcn_readlane((int)lhi, l);
            in[j] = reinterpret_cast<const uint32_t*>((uintptr_t)e1 << 32 | e0)[wc];
            out[j] = reinterpret_cast<const uint32_t*>((uintptr_t)l1 << 32 | l0)[wc];
        }
        const uint32_t in_on = (uint32_t)(in_valid >> (8 * g)), out_on = (uint32_t)(out_valid >> (8 * g));
        const uint32_t before = open;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            gd_planes_step(v, in[j] & (uint32_t)((int32_t)(in_on << (31 - j)) >> 31),
                           out[j] & (uint32_t)((int32_t)(out_on << (31 - j)) >> 31));
            const uint32_t hit = v[GD_COUNT_PLANES] & open;      // (past the last step nothing changes any more)
            open &= ~hit;
#pragma unroll
            for (int p = 0; p < 3; ++p)
                if ((j >> p) & 1) at[p] |= hit;
        }
        const uint32_t hits = before & ~open;
#pragma unroll
        for (int p = 0; p < 3; ++p) at[3 + p] |= (g >> p) & 1 ? hits : 0u;
        if (__ballot(open != 0) == 0) break;
    }
    for (uint32_t bits = cand & ~open; bits; bits &= bits - 1) {
        const uint32_t bit = (uint32_t)__builtin_ctz(bits);
        uint32_t step = 0;
#pragma unroll
        for (int p = 0; p < 6; ++p) step |= ((at[p] >> bit) & 1u) << p;
        atomicMin(&found[bit * FOUND_PITCH + lane], start + step);
    }
}

// A short batch.  A thread owns one item and a wave one 64-item word of the rows, so every
// ring word is read and written by a single wave.  Lane l of a block of 64 steps fetches the
// word that enters at the block's step l and the word that leaves the window then; two bit
// transposes across the lanes make them the item's own time vectors, so that the count takes
// two popcounts a block, and only an item that may reach k inside the block walks its steps.
__global__ __launch_bounds__(WIN_NT) void window_short_kernel(const gd_window_args a) {
    const uint32_t rank_blocks = (a.R + WIN_NT - 1) / WIN_NT;
    const bool is_node = blockIdx.x >= rank_blocks;
    const WindowItems it = window_items(a, is_node);
    const uint32_t item = (is_node ? blockIdx.x - rank_blocks : blockIdx.x) * WIN_NT + threadIdx.x;
    const uint32_t lane = threadIdx.x & (WAVE - 1), words = it.row / 2, word = item / 64;
    if (word >= words) return;                                  // the whole wave
    const uint64_t* anom = reinterpret_cast<const uint64_t*>(it.anom);
    uint64_t* ring = reinterpret_cast<uint64_t*>(it.ring);
    const bool live = item < it.n;
    const uint32_t W = a.W, K = a.K, T = a.T, first = (uint32_t)a.first_step;      // (first + T below 2^31)

    // the entering and the leaving word of step s
    auto fetch = [&](uint32_t s, uint64_t* win, uint64_t* wout) {
        *win = 0; *wout = 0;
        if (s >= T) return;
        *win = anom[(size_t)s * words + word];
        if (s >= W) *wout = anom[(size_t)(s - W) * words + word];
        else if (first + s >= W) *wout = ring[(size_t)((first + s) % W) * words + word];
    };

    uint32_t c = live ? it.count[item] : 0;
    int32_t f = live ? it.first[item] : 0;
    constexpr uint32_t AHEAD = 4;                               // blocks fetched in advance
    uint64_t win[AHEAD], wout[AHEAD];
#pragma unroll
    for (uint32_t q = 0; q < AHEAD; ++q) fetch(q * WAVE + lane, &win[q], &wout[q]);
    for (uint32_t s0 = 0; s0 < T; s0 += AHEAD * WAVE) {
#pragma unroll
        for (uint32_t q = 0; q < AHEAD; ++q) {
            const uint32_t sq = s0 + q * WAVE;                  // uniform over the wave
            if (sq >= T) break;
            // bit j: does this item enter / leave as anomalous at step sq + j
            const uint64_t in = gd_transpose64(win[q], lane), out = gd_transpose64(wout[q], lane);
            fetch(sq + AHEAD * WAVE + lane, &win[q], &wout[q]);
            const uint32_t enters = (uint32_t)__popcll(in);
            if (f == 0 && c + enters >= K) {                    // the flag may first rise inside this block
                const uint32_t n = min((uint32_t)WAVE, T - sq);
                for (uint32_t j = 0; j < n; ++j) {
                    const uint64_t upto = (2ull << j) - 1;
                    if (c + __popcll(in & upto) - __popcll(out & upto) >= K) {
                        f = (int32_t)(first + sq + j) + 1;
                        break;
                    }
                }
            }
            c += enters - (uint32_t)__popcll(out);
        }
    }
    if (live) {
        it.count[item] = (uint16_t)c;
        it.first[item] = f;
        if (is_node) reinterpret_cast<float*>(a.state + a.lay.node_z_last)[item] = a.node_z[(size_t)(T - 1) * a.N + item];
    }
    // The batch's last min(T, W) words become the ring's newest slots: every ring word has
    // been read by now, and by this wave alone.
    const uint32_t keep = T < W ? T : W;
    for (uint32_t i = lane; i < keep; i += WAVE) {
        const uint32_t s = T - keep + i;
        ring[(size_t)((first + s) % W) * words + word] = anom[(size_t)s * words + word];
    }
}

// A batch.  blockIdx.y: tile of words (ranks first), blockIdx.x: stretch of `stretch`
// blocks (stretch * 64 >= W where there is more than one).  Dynamic LDS: planes of every
// slot -- a block of the stretch or one of the few before it -- and word.
__global__ __launch_bounds__(WIN_MAX_NT) void window_blocks_kernel(const gd_window_args a, uint32_t rank_tiles,
                                                                    uint32_t stretch) {
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t final_planes[GD_COUNT_PLANES][TILE];
    __shared__ __align__(16) uint32_t found[32 * FOUND_PITCH];       // first flagged step of the tile's items in this stretch
    __shared__ uint32_t walked;
    const bool is_node = blockIdx.y >= rank_tiles;
    const WindowItems it = window_items(a, is_node);
    const uint32_t w0 = (is_node ? blockIdx.y - rank_tiles : blockIdx.y) * TILE;
    const uint32_t tid = threadIdx.x, nt = blockDim.x, lane = tid & (WAVE - 1);
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid / WAVE), waves = nt / WAVE;
    const uint32_t W = a.W, K = a.K, T = a.T, row = it.row;
    const uint32_t q = W / 64, r = W % 64, hist = q + (r ? 1 : 0);     // whole blocks, steps of a tail, slots before a block
    const int32_t first = (int32_t)a.first_step;                       // (first + T below 2^31)
    const uint32_t s0 = blockIdx.x * stretch * 64;
    const uint32_t blocks = min((T - s0 + 63) / 64, stretch);
    const bool last = s0 + blocks * 64 >= T;
    const uint32_t last_start = s0 + (blocks - 1) * 64;                // (the batch's last block, where `last`)
    const uint32_t wc = min(w0 + lane, row - 1);                       // (lanes past the row repeat its last word, and store nothing)
    const bool mine = w0 + lane < row;
    // a slot's planes lie one behind another: of the whole block, then of its tail
    const uint32_t slot_words = (r ? 2 * GD_BLOCK_PLANES - 1 : GD_BLOCK_PLANES) * TILE;
    auto planes_of = [&](uint32_t slot) -> uint32_t* { return lds + slot * slot_words + lane; };

    // Slots [0, hist): the blocks before the stretch; [hist, hist + blocks): its own; one more
    // for the steps that leave the window during the batch's last block.
    for (uint32_t slot = wv; slot < hist + blocks + (last ? 1 : 0); slot += waves) {
        const bool leaving = slot == hist + blocks;
        const int32_t start = leaving ? (int32_t)last_start - (int32_t)W : (int32_t)(s0 + slot * 64) - (int32_t)(hist * 64);
        const uint32_t n = leaving ? T - last_start : 64u;             // steps that count
        // Lane j works out where step j's row lies -- in the batch, before it in the ring, or
        // nowhere (row 0 of the batch is read then and dropped) -- and the rows' addresses are
        // read from the lanes one after another: worked out in scalars they are a chain of
        // dependent instructions as long as the loads themselves.
        const int32_t s = start + (int32_t)lane;
        const bool ok = lane < n && s < (int32_t)T && s >= -(int32_t)W && first + s >= 0;
        const uint32_t* of_lane = it.anom + (ok && s >= 0 ? (size_t)(uint32_t)s * row : 0);
        if (ok && s < 0) of_lane = it.ring + (size_t)((uint32_t)(first + s) % W) * row;
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
                v[g][j] = reinterpret_cast<const uint32_t*>((uintptr_t)hi << 32 | lo)[wc];
            }
        }
        uint32_t all[GD_BLOCK_PLANES] = {}, end[GD_BLOCK_PLANES] = {};
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t on = (uint32_t)(valid >> (16 * g)) & 0xFFFFu, tail = (uint32_t)(in_tail >> (16 * g)) & on;
            if (on == 0) continue;
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
    if (tid == 0) walked = 0;
    for (uint32_t x = tid; x < 8 * FOUND_PITCH; x += nt)
        reinterpret_cast<uint4*>(found)[x] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
    // The ring's new words (the batch's last min(T, W) steps) are the first stretch's to
    // store: some of them are fetched now.
    const uint32_t keep = T < W ? T : W;
    constexpr uint32_t EARLY = 16;
    uint32_t early[EARLY];
    if (s0 == 0) {
#pragma unroll
        for (uint32_t e = 0; e < EARLY; ++e)
            early[e] = it.anom[(size_t)(T - keep + min(wv + e * waves, keep - 1)) * row + wc];
    }
    __syncthreads();

    // counts where each block begins, and the items that may reach k inside it
    for (uint32_t b = wv; b < blocks; b += waves) {
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
        const uint32_t cand = mine ? gd_planes_reach(u, K) & ~gd_planes_reach(c, K) : 0u;
        const int32_t start = (int32_t)(s0 + b * 64), s = start + (int32_t)lane;       // this lane's step in a walk
        uint64_t todo = __ballot(cand != 0);
        if (__builtin_expect(__popcll(todo) > FEW_WORDS || __ballot(__popc(cand) > FEW_ITEMS) != 0, 0)) {
            walk_all(it, c, cand, (uint32_t)start, first, T, W, K, wc, lane, found);
            if (lane == 0) walked = 1;
            todo = 0;
        }
        for (; todo; todo &= todo - 1) {
            const int src = __builtin_ctzll(todo);
            const uint32_t w = w0 + (uint32_t)src;
            uint32_t enters = 0, leaves = 0;
            if (s < (int32_t)T) {
                enters = it.anom[(size_t)(uint32_t)s * row + w];
                const int32_t o = s - (int32_t)W;
                if (o >= 0) leaves = it.anom[(size_t)(uint32_t)o * row + w];
                else if (first + o >= 0) leaves = it.ring[(size_t)((uint32_t)(first + o) % W) * row + w];
            }
            // items flagged before this batch are left alone, as are those beyond the last one
            const uint32_t item = w * 32 + (lane & 31);
            const int32_t seen = item < it.n ? it.first[item] : 1;
            const uint32_t done = (uint32_t)__ballot(item >= it.n || (seen != 0 && seen <= first));
            const uint64_t upto = (2ull << lane) - 1;
            for (uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)cand, src) & ~done; bits; bits &= bits - 1) {
                const uint32_t bit = (uint32_t)__builtin_ctz(bits);
                const uint64_t in = __ballot((enters >> bit) & 1u), out = __ballot((leaves >> bit) & 1u);
                const uint32_t cnt = gd_planes_count(c, src, bit) + (uint32_t)__popcll(in & upto) -
                                     (uint32_t)__popcll(out & upto);
                const uint64_t reach = __ballot(cnt >= K && s < (int32_t)T);
                if (reach && lane == 0) lower_first(&it.first[w * 32 + bit], first + start + __builtin_ctzll(reach) + 1);
            }
        }
    }
    __syncthreads();                                                   // (and the ring has been read for the last time)
    for (uint32_t x = walked ? tid : TILE * 32; x < TILE * 32; x += nt) {
        const uint32_t at = found[(x % 32) * FOUND_PITCH + x / 32], item = w0 * 32 + x;
        if (at == 0xFFFFFFFFu || item >= it.n) continue;
        lower_first(&it.first[item], first + (int32_t)at + 1);
    }
    if (!last && s0 != 0) return;
    if (last) {
        for (uint32_t x = tid; x < TILE * 32; x += nt) {
            const uint32_t item = w0 * 32 + x;
            if (item >= it.n) break;
            uint32_t c = 0;
#pragma unroll
            for (int p = 0; p < GD_COUNT_PLANES; ++p) c |= ((final_planes[p][x / 32] >> (x % 32)) & 1u) << p;
            it.count[item] = (uint16_t)c;
            if (is_node)
                reinterpret_cast<float*>(a.state + a.lay.node_z_last)[item] = a.node_z[(size_t)(T - 1) * a.N + item];
        }
    }
    if (s0 == 0) {
        const uint32_t ring0 = (uint32_t)(first + (int32_t)(T - keep)) % W;
        auto into_ring = [&](uint32_t j, uint32_t v) {
            const uint32_t to = ring0 + j < W ? ring0 + j : ring0 + j - W;
            if (mine) it.ring[(size_t)to * row + w0 + lane] = v;
        };
#pragma unroll
        for (uint32_t e = 0; e < EARLY; ++e)
            if (wv + e * waves < keep) into_ring(wv + e * waves, early[e]);
        for (uint32_t j = wv + EARLY * waves; j < keep; j += waves)
            into_ring(j, it.anom[(size_t)(T - keep + j) * row + wc]);
    }
}

__global__ __launch_bounds__(WIN_NT) void flags_kernel(const gd_flags_args a) {
    const uint32_t i = blockIdx.x * WIN_NT + threadIdx.x;
    const uint16_t* rc = reinterpret_cast<const uint16_t*>(a.state + a.lay.rank_count);
    const int32_t* rf = reinterpret_cast<const int32_t*>(a.state + a.lay.rank_first);
    const uint16_t* nc = reinterpret_cast<const uint16_t*>(a.state + a.lay.node_count);
    const int32_t* nf = reinterpret_cast<const int32_t*>(a.state + a.lay.node_first);
    if (i < a.R) {
        const uint32_t c = rc[i];
        if (a.rank_flag) a.rank_flag[i] = c >= a.K ? 1 : 0;
        if (a.rank_count) a.rank_count[i] = (uint16_t)c;
        if (a.rank_first) a.rank_first[i] = rf[i] - 1;
    }
    if (i < a.N) {
        const uint32_t c = nc[i];
        if (a.node_flag) {
            uint8_t b = c >= a.K ? 1 : 0;
            // 8 GPUs per node: two 8-byte loads of the ranks' counts
            const uint4 q = *reinterpret_cast<const uint4*>(rc + (size_t)i * 8);
            const uint32_t v[4] = {q.x, q.y, q.z, q.w};
            bool any = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) any |= (v[j] & 0xFFFFu) >= a.K || (v[j] >> 16) >= a.K;
            if (any) b |= 2;
            a.node_flag[i] = b;
        }
        if (a.node_count) a.node_count[i] = (uint16_t)c;
        if (a.node_first) a.node_first[i] = nf[i] - 1;
    }
}

}  // namespace

hipError_t gd_launch_window(const gd_window_args& a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    if (a.T == 1) {
        const uint32_t blocks = (a.R + WIN_NT - 1) / WIN_NT + (a.N + WIN_NT - 1) / WIN_NT;
        hipLaunchKernelGGL(window_step_kernel, dim3(blocks), dim3(WIN_NT), 0, s, a);
        return hipGetLastError();
    }
    // Walking the steps costs by the step, and the more the more waves share a SIMD; the blocks
    // load the whole window whatever the batch.  us by steps / by blocks, 65 536 ranks: window
    // 1 024, 64 steps 5.2 / 13.5, 256 13.1 / 15.1, 512 22 / 20; window 256, 256 steps 12.9 / 12.0,
    // 300 13.8 / 10.0; 16 384 ranks: window 512, 300 steps 9.9 / 12.7, 512 15.0 / 16.0, 700 18.2 /
    // 14.9; window 1 024, 512 steps 14.8 / 19.5, 1 024 27 / 30; 64 ranks: window 256, 300 steps
    // 6.8 / 9.7; window 511, 511 steps 9.9 / 18.5.
    const uint32_t walked = a.W > SHORT_BATCH && a.R <= 32768 ? a.W : SHORT_BATCH;
    if (a.T <= walked) {
        const uint32_t blocks = (a.R + WIN_NT - 1) / WIN_NT + (a.N + WIN_NT - 1) / WIN_NT;
        hipLaunchKernelGGL(window_short_kernel, dim3(blocks), dim3(WIN_NT), 0, s, a);
        return hipGetLastError();
    }
    const uint32_t rank_tiles = (2 * ((a.R + 63) / 64) + TILE - 1) / TILE;
    const uint32_t node_tiles = (2 * ((a.N + 63) / 64) + TILE - 1) / TILE;
    const uint32_t q = a.W / 64, r = a.W % 64, hist = q + (r ? 1 : 0), blocks = (a.T + 63) / 64;
    // The shortest stretches that make at most 256 workgroups (one per CU), but of at least
    // the window (only the first stretch may look at the ring) and four blocks, and no longer
    // than gives every wave of a 16-wave workgroup one block: 65 536 ranks x 4 096 steps
    // takes 18 us with 10 or 11 blocks, 21 with 5 (two workgroups after another on most CUs).
    const uint32_t tiles = rank_tiles + node_tiles;
    const uint32_t fits = WIN_MAX_NT / WAVE - 1 > hist ? WIN_MAX_NT / WAVE - 1 - hist : 0;
    uint32_t stretch = hist > MIN_STRETCH ? hist : MIN_STRETCH;
    while (stretch < fits && (uint64_t)((blocks + stretch - 1) / stretch) * tiles > 256) ++stretch;
    if (stretch > blocks) stretch = blocks;
    const uint32_t stretches = (blocks + stretch - 1) / stretch;
    const uint32_t slots = hist + stretch + 1;
    const uint32_t nt = (slots < (uint32_t)WIN_MAX_NT / WAVE ? slots : (uint32_t)WIN_MAX_NT / WAVE) * WAVE;
    const size_t lds = (size_t)(r ? 2 * GD_BLOCK_PLANES - 1 : GD_BLOCK_PLANES) * slots * TILE * 4;
    constexpr size_t most = (size_t)(2 * GD_BLOCK_PLANES - 1) * (MAX_HISTORY + MAX_STRETCH + 1) * TILE * 4;
    static_assert(most + sizeof(uint32_t) * (GD_COUNT_PLANES * TILE + 32 * FOUND_PITCH) <= 160 * 1024,
                  "LDS budget of one CU");
    static std::atomic<uint64_t> granted{0};
    const hipError_t e = gd_grant_lds(granted, reinterpret_cast<const void*>(window_blocks_kernel), most);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(window_blocks_kernel, dim3(stretches, tiles), dim3(nt), lds, s, a, rank_tiles, stretch);
    return hipGetLastError();
}

hipError_t gd_launch_flags(const gd_flags_args& a, hipStream_t s) {
    const uint32_t blocks = (a.R + WIN_NT - 1) / WIN_NT;
    hipLaunchKernelGGL(flags_kernel, dim3(blocks), dim3(WIN_NT), 0, s, a);
    return hipGetLastError();
}
