// Parallel random walk (Section 5) on the reuse machinery: an agent's
// "index" is its packed cell key x | y << 16, and the expensive per-index
// program is the search of the cell's most likely moves, which agents on the
// same cell share.  One workgroup deduplicates the cells of a batch of
// agents in an LDS hash table, evaluates each distinct cell once and then
// moves every agent of the batch.
#pragma once

#include "vr_device.h"
#include "vr_walk_pieces.h"

namespace vr {

constexpr uint32_t kWalkKeep = 8;          // options kept per cell
constexpr uint32_t kWalkMaxBatch = 512;    // agents per workgroup
constexpr uint32_t kWalkThreads = 512;     // threads per batch workgroup (4 per cell searched)

struct WalkArgs {
    const uint32_t *keys_in;
    uint32_t *keys_out;
    const float *activity;   // grid * grid, cell (x, y) at y * grid + x
    const int8_t *moves;     // (dx, dy) per move
    const float *weights;    // per move
    const float *uniforms;   // per agent, [0, 1)
    uint32_t n, grid, num_moves, batch;
    uint32_t parts;                 // workgroups per batch: 1, 4 or 16
    unsigned long long *agg;        // per workgroup: (its batch, once, << 32) | evaluations
    unsigned long long *counters;   // {evaluations, units, 0, 0} or NULL
    unsigned long long *total_inv;
    uint32_t *err;
};

// The kept list: kWalkKeep keys in descending order.  A key holds the
// likelihood in its upper half, mapped so that unsigned order is float order,
// and the complement of the move index in its lower half, so that one 64-bit
// comparison orders by likelihood, ties to the lower move index, whatever
// order the moves are visited in.
struct WalkList {
    uint64_t k[kWalkKeep];
};

// An empty entry: likelihood -1 (below every likelihood kept: activities and
// weights are >= 0), move 0.
constexpr uint64_t kWalkNone = ((uint64_t)0x407FFFFFu << 32) | 0xFFFFFFFFu;

__device__ __forceinline__ uint64_t walk_key(float l, uint32_t m) {
    const uint32_t u = __float_as_uint(l + 0.0f);   // -0 compares equal to 0
    return ((uint64_t)((int32_t)u < 0 ? ~u : u | 0x80000000u) << 32) | (uint32_t)~m;
}
__device__ __forceinline__ float walk_likelihood(uint64_t key) {
    const uint32_t u = (uint32_t)(key >> 32);
    return __uint_as_float((int32_t)u < 0 ? u & 0x7FFFFFFFu : ~u);
}
__device__ __forceinline__ uint32_t walk_move(uint64_t key) { return ~(uint32_t)key; }

__device__ __forceinline__ void walk_clear(WalkList &K) {
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) K.k[j] = kWalkNone;
}

// Puts a key above the last kept one in its place by a fixed network, so that
// no index is dynamic and the list stays in registers.
__device__ __forceinline__ void walk_insert(WalkList &K, uint64_t key) {
    K.k[kWalkKeep - 1] = key;
#pragma unroll
    for (uint32_t j = kWalkKeep - 1; j >= 1; --j) {
        const bool up = K.k[j] > K.k[j - 1];
        const uint64_t hi = up ? K.k[j] : K.k[j - 1], lo = up ? K.k[j - 1] : K.k[j];
        K.k[j - 1] = hi;
        K.k[j] = lo;
    }
}

// The first kWalkKeep keys of this lane's list and that of lane (lane ^ MASK)
// of its quad (MASK 1 or 2): the larger of entry j and the other's entry
// 7 - j are those, in bitonic order, and three compare-exchange stages sort
// them.  Both lanes end with the same list.
template <int MASK>
__device__ __forceinline__ void walk_merge_quad(WalkList &K) {
    constexpr int kPerm = MASK == 1 ? 0xB1 : 0x4E;   // quad_perm [1,0,3,2] or [2,3,0,1]
    uint64_t o[kWalkKeep];
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)K.k[j], kPerm, 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(K.k[j] >> 32), kPerm, 0xf, 0xf, true);
        o[j] = ((uint64_t)hi << 32) | lo;
    }
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) {
        const uint64_t other = o[kWalkKeep - 1 - j];
        K.k[j] = K.k[j] > other ? K.k[j] : other;
    }
#pragma unroll
    for (uint32_t d = kWalkKeep / 2; d >= 1; d /= 2) {
#pragma unroll
        for (uint32_t j = 0; j < kWalkKeep; ++j) {
            if (j & d) continue;
            const bool down = K.k[j] < K.k[j + d];
            const uint64_t hi = down ? K.k[j + d] : K.k[j], lo = down ? K.k[j] : K.k[j + d];
            K.k[j] = hi;
            K.k[j + d] = lo;
        }
    }
}

// The same for likelihoods and moves met in index order, where ties settle
// themselves: l above position j moves entry j - 1 there, and the median of it,
// l and entry j is what position j then holds.
__device__ __forceinline__ void walk_insert(float (&L)[kWalkKeep], uint32_t (&mi)[kWalkKeep], float l, uint32_t m) {
    if (!(l > L[kWalkKeep - 1])) return;
#pragma unroll
    for (uint32_t j = kWalkKeep - 1; j >= 1; --j) {
        // one select after the other: nested they become branches
        const uint32_t mj = l > L[j] ? m : mi[j];
        mi[j] = l > L[j - 1] ? mi[j - 1] : mj;
        L[j] = __builtin_amdgcn_fmed3f(L[j - 1], l, L[j]);   // L[j - 1] >= L[j]
    }
    mi[0] = l > L[0] ? m : mi[0];
    L[0] = fmaxf(l, L[0]);
}

// The kWalkKeep most likely moves among moves [m0, m1) from cell (x, y):
// likelihood = activity of the target times the move's weight (one FP32
// product), moves leaving the grid skipped, descending with ties to the lower
// move index.  The activity is read from `act`, with row pitch `pitch` and first
// cell (ox, oy), which holds every in-grid target (the whole field, or a tile of
// it in LDS).  Returns the number of moves that stay in the grid.
//
// The moves come in index order, so likelihoods and moves are kept as they are
// and made keys at the end (100,000 agents, 1,788 moves, a search each: 492 us
// with 64-bit keys inserted, 463 us so).
__device__ __forceinline__ uint32_t walk_search(const WalkArgs &W, uint32_t x, uint32_t y, uint32_t m0, uint32_t m1,
                                                WalkList &K, const float *act, uint32_t pitch, int32_t ox, int32_t oy) {
    float L[kWalkKeep];
    uint32_t mi[kWalkKeep];
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) {
        L[j] = -1.0f;   // kWalkNone
        mi[j] = 0;
    }
    uint32_t valid = 0;
    for (uint32_t m = m0; m < m1; ++m) {
        const int32_t tx = (int32_t)x + W.moves[2 * m], ty = (int32_t)y + W.moves[2 * m + 1];
        if (tx < 0 || ty < 0 || tx >= (int32_t)W.grid || ty >= (int32_t)W.grid) continue;
        ++valid;
        const float l = act[(uint32_t)(ty - oy) * pitch + (uint32_t)(tx - ox)] * W.weights[m];
        walk_insert(L, mi, l, m);
    }
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) K.k[j] = walk_key(L[j], mi[j]);
    return valid;
}

// ---------------------------------------------------------------------------
// Moves by descending weight.  A workgroup of NT threads counts the moves per
// weight class (the float's exponent and two mantissa bits; negative weights
// come last) and lists them in LDS in that order: heavy moves first means that
// a cell's list is nearly final after a few of them and insertions, which
// cost an order of magnitude more than a comparison, are rare afterwards; and
// with a bound on the activity the search can stop.  Up to kWalkListed moves,
// where the list fits beside the rest of a workgroup's LDS; more are read from
// memory in the order given.  A listed move is (move index | dy << 16 | dx <<
// 24, weight).
// ---------------------------------------------------------------------------
constexpr uint32_t kWalkListed = 1024, kWalkClasses = 1024;
// A search per agent lists from so many moves on: 300,000 agents, 12 moves 10.0
// us listed and 8.9 us from memory, 28 moves 13.4 and 15.6 us (1,000 agents 6.9
// and 6.7, 9.5 and 12.1 us).
constexpr uint32_t kWalkNaiveListed = 20;
constexpr uint32_t kWalkTile = 4096;   // cells of a batch's tile (see k_walk_hash)

__device__ __forceinline__ uint32_t walk_class(float w) {
    const uint32_t u = __float_as_uint(w);
    return (int32_t)u < 0 ? kWalkClasses - 1 : kWalkClasses - 1 - (u >> 21);   // u >> 21 < 1024 for u >= 0
}

// The largest weight a move listed at or after one of weight w can have (the
// last class holds the smallest weights beside the negative ones).
__device__ __forceinline__ float walk_class_top(float w) {
    const uint32_t u = __float_as_uint(w);
    return __uint_as_float(((int32_t)u < 0 ? 0u : u) | 0x1FFFFFu);
}

// s_list holds num_moves entries, s_hist kWalkClasses words (free again
// afterwards), s_tmp NT / 64 words.  Contains barriers: call uniformly.
template <int NT>
__device__ __forceinline__ void walk_list_moves(const WalkArgs &W, uint2 *s_list, uint32_t *s_hist, uint32_t *s_tmp) {
    constexpr uint32_t kPer = kWalkListed / NT, kBins = kWalkClasses / NT;
    const uint32_t tid = threadIdx.x;
    for (uint32_t c = tid; c < kWalkClasses; c += NT) s_hist[c] = 0;
    __syncthreads();
    float w[kPer];
    uint32_t at[kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t m = tid + k * NT;
        if (m < W.num_moves) {
            w[k] = W.weights[m];
            at[k] = atomicAdd(&s_hist[walk_class(w[k])], 1u);
        }
    }
    __syncthreads();
    uint32_t c[kBins], sum = 0, total;
#pragma unroll
    for (uint32_t j = 0; j < kBins; ++j) {
        c[j] = s_hist[tid * kBins + j];
        sum += c[j];
    }
    uint32_t run = block_excl_scan<NT>(sum, s_tmp, total);
#pragma unroll
    for (uint32_t j = 0; j < kBins; ++j) {
        s_hist[tid * kBins + j] = run;
        run += c[j];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t m = tid + k * NT;
        if (m < W.num_moves)
            s_list[s_hist[walk_class(w[k])] + at[k]] =
                make_uint2(m | (uint32_t)(uint8_t)W.moves[2 * m + 1] << 16 | (uint32_t)(uint8_t)W.moves[2 * m] << 24,
                           __float_as_uint(w[k]));
    }
    __syncthreads();
}

// walk_search over listed moves q, q + step, .. of [0, num_moves), the
// activity read from the whole field.
__device__ __forceinline__ uint32_t walk_search_listed(const WalkArgs &W, const uint2 *s_list, uint32_t x, uint32_t y,
                                                       uint32_t q, uint32_t step, WalkList &K) {
    uint32_t valid = 0;
    float last = walk_likelihood(K.k[kWalkKeep - 1]);
    for (uint32_t i0 = q; i0 < W.num_moves; i0 += 4 * step) {   // four targets in flight
        uint2 e[4];
        float a[4];
        bool in[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t i = i0 + r * step;
            e[r] = s_list[min(i, W.num_moves - 1)];
            const int32_t tx = (int32_t)x + ((int32_t)e[r].x >> 24), ty = (int32_t)y + (int8_t)(e[r].x >> 16);
            in[r] = i < W.num_moves && tx >= 0 && ty >= 0 && tx < (int32_t)W.grid && ty < (int32_t)W.grid;
            a[r] = in[r] ? W.activity[(uint32_t)ty * W.grid + (uint32_t)tx] : 0.0f;
            valid += in[r];
        }
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const float l = a[r] * __uint_as_float(e[r].y);
            if (in[r] && l >= last) {
                const uint64_t key = walk_key(l, e[r].x & 0xFFFFu);
                if (key > K.k[kWalkKeep - 1]) walk_insert(K, key);
                last = walk_likelihood(K.k[kWalkKeep - 1]);
            }
        }
    }
    return valid;
}

// One agent's move: the first option whose running FP32 sum exceeds u times
// the options' sum (the last one when rounding leaves none); an agent whose
// options sum to zero stays.  The loops run over all kWalkKeep positions
// with the count as a predicate, so the arrays stay in registers.
__device__ __forceinline__ uint32_t walk_choose(const WalkArgs &W, uint32_t key, float u, const WalkList &K,
                                                uint32_t k) {
    float L[kWalkKeep];
    float S = 0.0f;
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) {
        L[j] = walk_likelihood(K.k[j]);
        if (j < k) S += L[j];
    }
    if (k == 0 || !(S > 0.0f)) return key;
    const float t = u * S;
    float run = 0.0f;
    bool found = false;
    uint32_t m = 0;
#pragma unroll
    for (uint32_t j = 0; j < kWalkKeep; ++j) {
        if (j < k) {
            run += L[j];
            if (!found) m = walk_move(K.k[j]);   // ends on the first option past the target, else the last one
            found = found || run > t;
        }
    }
    const uint32_t x = (key & 0xFFFFu) + (uint32_t)(int32_t)W.moves[2 * m];
    const uint32_t y = (key >> 16) + (uint32_t)(int32_t)W.moves[2 * m + 1];
    return (x & 0xFFFFu) | (y << 16);
}

// A key outside the grid raises VR_ERR_INDEX_RANGE; the agent stays.
__device__ __forceinline__ bool walk_key_ok(const WalkArgs &W, uint32_t key) {
    if ((key & 0xFFFFu) < W.grid && (key >> 16) < W.grid) return true;
    raise_error(W.err, VR_ERR_INDEX_RANGE);
    return false;
}

// No reuse: every agent evaluates its own cell (LISTED: from the moves in
// weight order).  300,000 agents, 796 moves: 290 us with the moves read from
// memory in their own order, 222 us listed.
template <bool LISTED>
__global__ __launch_bounds__(256) void k_walk_naive(WalkArgs W) {
    extern __shared__ __attribute__((aligned(16))) uint2 s_list[];
    __shared__ uint32_t s_hist[LISTED ? kWalkClasses : 1], s_tmp[4];
    if (LISTED) walk_list_moves<256>(W, s_list, s_hist, s_tmp);
    const uint32_t a = blockIdx.x * 256 + threadIdx.x;
    if (a < W.n) {
        const uint32_t key = W.keys_in[a];
        uint32_t out = key;
        if (walk_key_ok(W, key)) {
            const uint32_t x = key & 0xFFFFu, y = key >> 16;
            WalkList K;
            walk_clear(K);
            const uint32_t valid = LISTED ? walk_search_listed(W, s_list, x, y, 0, 1, K)
                                          : walk_search(W, x, y, 0, W.num_moves, K, W.activity, W.grid, 0, 0);
            out = walk_choose(W, key, W.uniforms[a], K, min(valid, kWalkKeep));
        }
        W.keys_out[a] = out;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (W.counters) {
            W.counters[0] = W.n;
            W.counters[1] = W.n;
            W.counters[2] = 0;
            W.counters[3] = 0;
        }
        atomicAdd(W.total_inv, (unsigned long long)W.n);
    }
}

// One batch of up to kWalkMaxBatch agents per workgroup of NT threads: the
// batch's cells go into an LDS hash table (linear probing, 2 x kWalkMaxBatch
// slots); the lane that inserts a cell takes the next id; each distinct cell
// is evaluated once into LDS, by the four lanes of a quad taking every fourth
// move each; every agent then takes its move from its cell's options.
//
// LISTED (see walk_list_moves): the cells' bounding box is cut into split x
// split pieces, as few as let each piece, grown by the longest move, fit the
// staged window, and a piece's cells are searched in its window.  A quad stops
// at the first move whose weight class times the window's largest activity is
// below the last likelihood it keeps (only where no activity of the window is
// negative).  Window cells outside the grid hold NaN, whose product is never
// kept: no test per move.  With W.parts workgroups per batch (few batches),
// each takes every parts-th piece and the agents on its cells.
//
// Not LISTED (more than kWalkListed moves): the cells are searched in one staged
// tile, their bounding box grown by the longest move and clipped to the grid,
// where that holds at most kWalkTile cells, else in memory (300,000 agents, 1,788
// moves: 305 us from memory alone, 227 us with tiles).
//
// Insertions (45 instructions, when any lane of the wavefront makes one) and
// two LDS reads per move bound the search.  300,000 agents on 65,536 cells, 796
// moves, batches of 512: 136 us with the moves read from memory in their own
// order and no window where the whole box does not fit one, 39 us so; 5,000
// agents 399 us, 33 us so.
template <int NT, bool LISTED>
__global__ __launch_bounds__(NT) void k_walk_hash(WalkArgs W) {
    constexpr uint32_t S = 2 * kWalkMaxBatch, mask = S - 1;
    // s_raw holds the hash table, the slot ids and the weight classes while
    // the batch's cells are inserted, then the staged window
    __shared__ uint32_t s_raw[kWalkSide * kWalkPitch];
    uint32_t *s_table = s_raw, *s_id = s_raw + S;
    float *s_win = (float *)s_raw;
    extern __shared__ __attribute__((aligned(16))) uint2 s_list[];
    __shared__ uint32_t s_uniq[kWalkMaxBatch];
    __shared__ uint16_t s_slot[kWalkMaxBatch], s_sel[kWalkMaxBatch];
    // the cells' options: a key's upper half, and its move (below 65536)
    __shared__ uint32_t s_like[kWalkKeep][kWalkMaxBatch];
    __shared__ uint16_t s_move[kWalkKeep][kWalkMaxBatch];
    __shared__ uint8_t s_k[kWalkMaxBatch];       // options kept; kElsewhere: another workgroup's cell
    constexpr uint8_t kElsewhere = 0xFF;
    __shared__ uint32_t s_count, s_box[5];       // min x, min y, max x, max y, longest move
    __shared__ uint32_t s_top, s_neg, s_nsel;    // the window's largest activity (as bits); any negative; cells selected
    __shared__ uint32_t s_tmp[NT / kWave];
    static_assert(2 * S + kWalkClasses <= kWalkSide * kWalkPitch, "table, ids and weight classes share the window's space");
    const uint32_t tid = threadIdx.x, b = blockIdx.x / W.parts, part = blockIdx.x % W.parts;
    if (blockIdx.x == 0 && tid < 4 && W.counters) W.counters[tid] = 0;   // k_finish adds to them afterwards
    const uint32_t a0 = b * W.batch, cnt = min(W.batch, W.n - a0);
    for (uint32_t s = tid; s < S; s += NT) s_table[s] = kEmpty;
    if (tid == 0) {
        s_count = 0;
        s_box[0] = s_box[1] = 0xFFFFFFFFu;
        s_box[2] = s_box[3] = s_box[4] = 0;
        s_nsel = 0;
    }
    if (LISTED) walk_list_moves<NT>(W, s_list, s_raw + 2 * S, s_tmp);
    else __syncthreads();
    for (uint32_t i = tid; i < cnt; i += NT) {
        const uint32_t key = W.keys_in[a0 + i];
        uint32_t p = hash_slot(key, 10);   // S = 1024 slots
        for (;;) {                          // at most cnt <= S / 2 distinct keys: a free slot exists
            const uint32_t prev = atomicCAS(&s_table[p], kEmpty, key);
            if (prev == kEmpty) {
                const uint32_t id = atomicAdd(&s_count, 1u);
                s_id[p] = id;
                s_uniq[id] = key;
                break;
            }
            if (prev == key) break;
            p = (p + 1) & mask;
        }
        s_slot[i] = (uint16_t)p;
    }
    {
        uint32_t longest = 0;
        for (uint32_t m = tid; m < W.num_moves; m += NT) {
            const int32_t dx = W.moves[2 * m], dy = W.moves[2 * m + 1];
            longest = max(longest, (uint32_t)max(max(dx, -dx), max(dy, -dy)));
        }
        longest = wave_max(longest);
        if (lane_id() == 0) atomicMax(&s_box[4], longest);
    }
    __syncthreads();
    const uint32_t inv = s_count;
    for (uint32_t i = tid; i < cnt; i += NT) s_slot[i] = (uint16_t)s_id[s_slot[i]];   // slot -> id
    for (uint32_t j0 = 0; j0 < inv; j0 += NT) {   // uniform: every lane takes part in the reductions
        const uint32_t j = j0 + tid;
        const uint32_t key = j < inv ? s_uniq[j] : 0xFFFFFFFFu, x = key & 0xFFFFu, y = key >> 16;
        const bool in = x < W.grid && y < W.grid;   // grids have at most 32768 cells a side
        const uint32_t mnx = wave_min(in ? x : 0xFFFFFFFFu), mny = wave_min(in ? y : 0xFFFFFFFFu);
        const uint32_t mxx = wave_max(in ? x : 0u), mxy = wave_max(in ? y : 0u);
        if (lane_id() == 0) {
            atomicMin(&s_box[0], mnx);
            atomicMin(&s_box[1], mny);
            atomicMax(&s_box[2], mxx);
            atomicMax(&s_box[3], mxy);
        }
        if (j < inv) {
            s_k[j] = !in && part == 0 ? 0 : kElsewhere;
            if (!in && part == 0) {   // its agents stay
                raise_error(W.err, VR_ERR_INDEX_RANGE);
                atomicAdd(&s_nsel, 1u);
            }
        }
    }
    __syncthreads();   // the table and ids are dead from here on
    const int32_t R = (int32_t)s_box[4];
    const uint32_t bx = s_box[0], by = s_box[1], outside = s_nsel;
    const bool any = bx <= s_box[2];
    const uint32_t bw = any ? s_box[2] - bx + 1 : 0u, bh = any ? s_box[3] - by + 1 : 0u;
    const WalkPieces pieces = walk_pieces(bw, bh, (uint32_t)R, W.parts, W.num_moves);
    const uint32_t split = pieces.split;
    const bool windowed = LISTED && pieces.windowed;
    // unlisted moves: the whole box grown by the longest move and clipped to the
    // grid, if that fits
    const int32_t tx0 = max(0, (int32_t)bx - R), ty0 = max(0, (int32_t)by - R);
    const uint32_t tw = (uint32_t)(min((int32_t)W.grid, (int32_t)(bx + bw) + R) - tx0);
    const uint32_t th = (uint32_t)(min((int32_t)W.grid, (int32_t)(by + bh) + R) - ty0);
    const bool tiled = !LISTED && any && tw * th <= kWalkTile;
    if (tiled)   // the pieces below begin with a barrier
        for (uint32_t c = tid; c < tw * th; c += NT) {
            const uint32_t r = c / tw;
            s_win[c] = W.activity[((uint32_t)ty0 + r) * W.grid + (uint32_t)tx0 + (c - r * tw)];
        }
    const uint32_t pw = max(1u, (bw + split - 1) / split), ph = max(1u, (bh + split - 1) / split);
    uint32_t evaluated = outside;
    for (uint32_t piece = part; any && piece < (windowed ? split * split : W.parts); piece += W.parts) {
        // the piece's cells (without windows: a share of the cells by hash)
        const uint32_t px = piece % split, py = piece / split;
        __syncthreads();   // the previous piece's window and selection are done with
        if (tid == 0) s_nsel = s_top = s_neg = 0;
        __syncthreads();
        for (uint32_t j = tid; j < inv; j += NT) {
            const uint32_t key = s_uniq[j], x = key & 0xFFFFu, y = key >> 16;
            if (x >= W.grid || y >= W.grid) continue;
            const bool mine = windowed ? (x - bx) / pw == px && (y - by) / ph == py
                                       : hash_slot(key, 4) % W.parts == piece;
            if (mine) s_sel[atomicAdd(&s_nsel, 1u)] = (uint16_t)j;
        }
        const int32_t ox = (int32_t)(bx + px * pw) - R, oy = (int32_t)(by + py * ph) - R;
        const int32_t ww = (int32_t)pw + 2 * R, wh = (int32_t)ph + 2 * R;   // <= kWalkSide
        __syncthreads();
        const uint32_t nsel = s_nsel;
        evaluated += nsel;
        if (nsel == 0) continue;
        if (windowed) {
            float top = 0.0f;
            bool neg = false;
            for (int32_t r = (int32_t)(tid / kWalkSide); r < wh; r += NT / kWalkSide) {
                const int32_t c = (int32_t)(tid % kWalkSide), x = ox + c, y = oy + r;
                float v = __uint_as_float(0x7FC00000u);
                if (c < ww && x >= 0 && y >= 0 && x < (int32_t)W.grid && y < (int32_t)W.grid)
                    v = W.activity[(uint32_t)y * W.grid + (uint32_t)x];
                s_win[r * kWalkPitch + c] = v;
                top = v > top ? v : top;
                neg = neg || v < 0.0f;
            }
            const uint32_t bits = wave_max(__float_as_uint(top));   // top >= 0: bits order as floats
            if (lane_id() == 0) atomicMax(&s_top, bits);
            if (neg) s_neg = 1;
            __syncthreads();
        }
        const float top = s_neg ? __uint_as_float(0x7F800000u) : __uint_as_float(s_top);
        const uint32_t quarter = (W.num_moves + 3) / 4;
        for (uint32_t base = 0; base < nsel; base += NT / 4) {   // uniform trip count: every lane merges
            const uint32_t q = tid % 4;
            const bool has = base + tid / 4 < nsel;
            const uint32_t j = has ? s_sel[base + tid / 4] : 0u;
            const uint32_t key = s_uniq[j], x = key & 0xFFFFu, y = key >> 16;
            WalkList K;
            walk_clear(K);
            uint32_t valid = 0;
            if (has && windowed) {
                const int32_t at = ((int32_t)y - oy) * kWalkPitch + ((int32_t)x - ox);
                // nothing below `last` can be among the quad's options; it is
                // the same in the quad's lanes, and so is the trip count
                float last = walk_likelihood(K.k[kWalkKeep - 1]);
                for (uint32_t i0 = 0; i0 < W.num_moves; i0 += 16) {   // four targets in flight
                    const float w0 = __uint_as_float(s_list[i0].y);
                    if (top * walk_class_top(w0) < last) break;   // nothing listed from here on can be kept
                    uint2 e[4];
                    float a[4];
#pragma unroll
                    for (uint32_t r = 0; r < 4; ++r) e[r] = s_list[min(i0 + 4 * r + q, W.num_moves - 1)];
#pragma unroll
                    for (uint32_t r = 0; r < 4; ++r)
                        a[r] = s_win[at + (int32_t)(int8_t)(e[r].x >> 16) * kWalkPitch + ((int32_t)e[r].x >> 24)];
#pragma unroll
                    for (uint32_t r = 0; r < 4; ++r) {
                        const float l = a[r] * __uint_as_float(e[r].y);
                        if (l >= last && i0 + 4 * r + q < W.num_moves) {
                            const uint64_t k = walk_key(l, e[r].x & 0xFFFFu);
                            if (k > K.k[kWalkKeep - 1]) walk_insert(K, k);
                        }
                    }
                    if (i0 == 16 || i0 == 80 || i0 == 272) {
                        // the quad's list so far: lane 0 keeps it, its last
                        // likelihood is what later moves have to reach
                        walk_merge_quad<1>(K);
                        walk_merge_quad<2>(K);
                        last = walk_likelihood(K.k[kWalkKeep - 1]);
                        if (q != 0) walk_clear(K);
                    }
                }
                // moves that stay in the grid: all of them from an inner cell,
                // else counted up to kWalkKeep (the heavy ones are short and
                // mostly stay, so few are looked at)
                if ((int32_t)x >= R && (int32_t)y >= R && (int32_t)x + R < (int32_t)W.grid &&
                    (int32_t)y + R < (int32_t)W.grid)
                    valid = q == 0 ? W.num_moves : 0u;
                else if (q == 0)
                    for (uint32_t m = 0; m < W.num_moves && valid < kWalkKeep; ++m) {
                        const uint32_t e = s_list[m].x;
                        const int32_t tx = (int32_t)x + ((int32_t)e >> 24), ty = (int32_t)y + (int8_t)(e >> 16);
                        valid += tx >= 0 && ty >= 0 && tx < (int32_t)W.grid && ty < (int32_t)W.grid;
                    }
            } else if (has && LISTED) {
                valid = walk_search_listed(W, s_list, x, y, q, 4, K);
            } else if (has) {
                const uint32_t m0 = min(W.num_moves, q * quarter), m1 = min(W.num_moves, (q + 1) * quarter);
                valid = tiled ? walk_search(W, x, y, m0, m1, K, s_win, tw, tx0, ty0)
                              : walk_search(W, x, y, m0, m1, K, W.activity, W.grid, 0, 0);
            }
            walk_merge_quad<1>(K);
            walk_merge_quad<2>(K);
            valid += (uint32_t)__shfl_xor((int)valid, 1, kWave);
            valid += (uint32_t)__shfl_xor((int)valid, 2, kWave);
            if (has && q == 0) {
#pragma unroll
                for (uint32_t r = 0; r < kWalkKeep; ++r) {
                    s_like[r][j] = (uint32_t)(K.k[r] >> 32);
                    s_move[r][j] = (uint16_t)walk_move(K.k[r]);
                }
                s_k[j] = (uint8_t)min(valid, kWalkKeep);
            }
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += NT) {
        const uint32_t id = s_slot[i];
        const uint32_t kept = s_k[id];
        if (kept == kElsewhere) continue;
        WalkList K;
#pragma unroll
        for (uint32_t r = 0; r < kWalkKeep; ++r) K.k[r] = (uint64_t)s_like[r][id] << 32 | (uint32_t)~(uint32_t)s_move[r][id];
        W.keys_out[a0 + i] = walk_choose(W, s_uniq[id], W.uniforms[a0 + i], K, kept);
    }
    if (tid == 0) W.agg[blockIdx.x] = (part == 0 ? 1ull << 32 : 0ull) | evaluated;
}

}  // namespace vr
