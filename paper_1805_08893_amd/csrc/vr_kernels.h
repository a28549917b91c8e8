// Geometry-stage kernels for gfx950: naive, LDS sort / hash / parallel-hash
// deduplication over static or dynamic batches, and wave64 ballot rounds.
#pragma once

#include <type_traits>

#include "vr_device.h"
#include "vr_stream.h"

namespace vr {

// What a unit writes: per-corner vertices alone, any of a draw's outputs, or
// per-corner vertices and a stream's triangle records.
enum UnitOut { kCorners = 0, kAll = 1, kRecords = 2 };

enum DedupMode { kSort = 0, kHash = 1, kPHash = 2 };

// Everything a draw kernel reads besides the shader parameters.
struct DrawArgs {
    const uint32_t *idx;        // uint32[3T]
    const f4 *vtx;              // [V][2] float4
    uint32_t V, T;
    uint32_t batch_tris;        // static batches: N_p
    uint32_t num_batches;       // static batches: ceil(T / N_p)
    const uint32_t *plan;       // dynamic batches: [B, start_0 .. start_{B-1}, T]
    f4 *corners;                // [3T][3]
    uint32_t *tris;             // [3T]
    f4 *verts;                  // [..][3]
    uint16_t *local_idx;        // [3T]
    uint32_t *unit_offsets;     // [units + 1]
    uint32_t *unit_inv;         // [units]
    unsigned long long *counters;   // [4]
    unsigned long long *agg;    // per batch: (units << 32) | invocations
    unsigned long long *status; // look-back words, zero at launch (cleared by k_finish)
    uint32_t *err;              // first device-side error
    unsigned long long *total_inv;  // invocations since the last vr_sync
    uint32_t hash_bits;         // log2 of the LDS hash-table size
    uint32_t probes;            // parallel hashing: per-lane probes
    uint32_t max_idx;           // LDS capacity in corners (3 * max triangles per unit)
    uint32_t max_uniq;          // LDS capacity in shaded vertices
    uint32_t need_prefix;       // tris / verts / unit arrays requested
    uint32_t status_cap;        // look-back words available
    uint32_t stream_verts;      // no corners: shaded vertices stream out through an NT-row stage
    SetupTarget setup;          // a stream's draw
    unsigned long long *arrivals;   // draws of few batches: the word their batches add to (see batch_done)
};

// Draw arguments and shader parameters in constant memory (a launch's kernel
// arguments, a frame's tables): read with scalar loads where they are used.
#define VR_CONSTANT __attribute__((address_space(4)))
using ArgsPtr = const VR_CONSTANT DrawArgs *;
using ShaderPtr = const VR_CONSTANT vr_shader_params *;

// The same pointer, of unknown origin to the compiler: what is read through
// it is read again instead of being kept from before.  A unit's phases use
// different fields, and kept across them they exceed the scalar registers and
// are spilled into vector lanes, two vector instructions for each.
template <typename T>
__device__ __forceinline__ const VR_CONSTANT T *reread(const VR_CONSTANT T *p) {
    uint64_t a = (uint64_t)p;
    asm volatile("" : "+s"(a));
    return (const VR_CONSTANT T *)a;
}

// Units a launch may take: the plan's count, bounded by the look-back
// capacity (a plan built for other limits raises an error instead of
// overrunning scratch).
__device__ __forceinline__ uint32_t launch_units(const DrawArgs &A, uint32_t nb) {
    if (A.need_prefix && nb > A.status_cap) {
        raise_error(A.err, VR_ERR_CAPACITY);
        return A.status_cap;
    }
    return nb;
}

// Batches that count: those within the draw's bound, all of which a launch
// covers.  A plan built for other limits, or for a longer stream, may list more.
__device__ __forceinline__ uint32_t counted_batches(const DrawArgs &A, uint32_t nb) { return min(nb, A.status_cap); }

__device__ __forceinline__ uint32_t batch_count(const DrawArgs &A) {
    return A.plan ? A.plan[0] : A.num_batches;
}

__device__ __forceinline__ void batch_range(const DrawArgs &A, uint32_t b, uint32_t &t0, uint32_t &t1) {
    if (A.plan) {   // the plan may be that of a longer stream with the same start
        t0 = A.plan[1 + b];
        t1 = min(A.plan[2 + b], A.T);
    } else {
        t0 = b * A.batch_tris;
        t1 = min(A.T, t0 + A.batch_tris);
    }
}

// Workgroup b of a grid of n takes piece xcd_piece(b, n): the hardware deals
// workgroups round robin over the eight XCDs, and this gives each XCD one
// contiguous run of pieces, so that the vertices neighbouring pieces share are
// fetched into one L2 instead of several.  Only where pieces do not wait for
// their predecessors.  Grid of 1.8M triangles, Hilbert order, MVP: naive 51.7
// -> 43.6 us, two-pass 68.9 -> 57.7 us, ballot 60.4 -> 56.3 us; hash 256 / 341
// with Offset-64 on 8.4M triangles 312 -> 297 us.
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t xcd_piece(uint32_t b, uint32_t n) {
    const uint32_t x = b % kXcds;
    return x * (n / kXcds) + min(x, n % kXcds) + b / kXcds;
}

// Index fetch with the range check fused in: an index >= V raises
// VR_ERR_INDEX_RANGE and is replaced by 0 so no access leaves the buffers.
__device__ __forceinline__ uint32_t checked_index(const DrawArgs &A, uint32_t k) {
    if (k >= A.V) {
        raise_error(A.err, VR_ERR_INDEX_RANGE);
        k = 0;
    }
    return k;
}

__device__ __forceinline__ uint32_t fetch_index(const DrawArgs &A, uint64_t pos) {
    return checked_index(A, A.idx[pos]);
}

// The indices idx[base .. base + n) into dst[0 .. n), checked as
// fetch_index does, by NT threads; each thread issues three loads before it
// uses the first, so that their latencies overlap.
template <uint32_t NT>
__device__ __forceinline__ void load_indices(const DrawArgs &A, uint64_t base, uint32_t n, uint32_t *dst,
                                             uint32_t tid) {
    for (uint32_t i0 = 0; i0 < n; i0 += 3 * NT) {
        uint32_t v[3];
#pragma unroll
        for (uint32_t r = 0; r < 3; ++r) {
            const uint32_t i = i0 + r * NT + tid;
            v[r] = i < n ? A.idx[base + i] : 0u;
        }
#pragma unroll
        for (uint32_t r = 0; r < 3; ++r) {
            const uint32_t i = i0 + r * NT + tid;
            if (i < n) dst[i] = checked_index(A, v[r]);
        }
    }
}

// Shades the vertex whose 32 input bytes are (a, b) into dst[0..2].
template <int KIND>
__device__ __forceinline__ void shade_raw_to_lds(const vr_shader_params &sh, f4 a, f4 b, f4 *dst) {
    float4 o0, o1, o2;
    shade_vertex<KIND>(sh, make_float4(a.x, a.y, a.z, a.w), make_float4(b.x, b.y, b.z, b.w), o0, o1, o2);
    dst[0] = f4{o0.x, o0.y, o0.z, o0.w};
    dst[1] = f4{o1.x, o1.y, o1.z, o1.w};
    dst[2] = f4{o2.x, o2.y, o2.z, o2.w};
}

template <int KIND>
__device__ __forceinline__ void shade_to_lds(const DrawArgs &A, const vr_shader_params &sh, uint32_t v,
                                             f4 *dst) {
    const f4 a = A.vtx[2ull * v], b = A.vtx[2ull * v + 1];
    float4 o0, o1, o2;
    shade_vertex<KIND>(sh, make_float4(a.x, a.y, a.z, a.w), make_float4(b.x, b.y, b.z, b.w), o0, o1, o2);
    dst[0] = f4{o0.x, o0.y, o0.z, o0.w};
    dst[1] = f4{o1.x, o1.y, o1.z, o1.w};
    dst[2] = f4{o2.x, o2.y, o2.z, o2.w};
}

// Assembly (Section 4.2): every corner of the unit's triangles receives its
// shaded vertex.  The unit's corner rows are one contiguous span, so lane q
// stores float4 q of the span: fully coalesced 16-byte stores.
template <int NT, int OUT, typename LocalT>
__device__ __forceinline__ void write_unit(const DrawArgs &A, uint32_t t0, uint32_t ntri, const LocalT *s_local,
                                           const f4 *s_sv, uint32_t inv, uint32_t vbase, uint32_t unit,
                                           uint32_t tid, bool verts_written = false) {
    constexpr bool FULL = OUT == kAll;
    const uint32_t ncorner = 3 * ntri;
    if (!FULL || A.corners) {
        // float4 q of the span is part q % 3 of corner q / 3.  Lane tid takes
        // q = tid + NT i; NT is a power of two, so NT = r (mod 3) with r = 1
        // or 2, and for i = 3 m + j the corner is NT m + kj[j] and the part
        // pj[j], both fixed per lane: no division in the loop.  Three rows per
        // lane at a time, so that their LDS reads overlap.
        constexpr uint32_t r = NT % 3;
        static_assert(r != 0, "the workgroup size is a power of two");
        uint32_t kj[3], pj[3];
#pragma unroll
        for (uint32_t j = 0; j < 3; ++j) {
            const uint32_t m = tid + r * j;
            kj[j] = (NT - r) / 3 * j + m / 3;
            pj[j] = m % 3;
        }
        f4 *dst = A.corners + 9ull * t0;
        const uint32_t cnt = 9 * ntri, klast = ncorner - 1;
        for (uint32_t q = tid, kb = 0; q < cnt; q += 3 * NT, kb += NT) {
            uint32_t at[3];
            f4 row[3];
            // rows past the span read the last corner (kept in bounds) and are not stored
#pragma unroll
            for (uint32_t j = 0; j < 3; ++j) at[j] = 3 * (uint32_t)s_local[min(kb + kj[j], klast)] + pj[j];
#pragma unroll
            for (uint32_t j = 0; j < 3; ++j) row[j] = s_sv[at[j]];
#pragma unroll
            for (uint32_t j = 0; j < 3; ++j)
                if (q + j * NT < cnt) __builtin_nontemporal_store(row[j], dst + q + j * NT);
        }
    }
    if (!FULL) return;
    if (A.tris || A.local_idx) {
        for (uint32_t k = tid; k < ncorner; k += NT) {
            const uint32_t l = s_local[k];
            if (A.tris) A.tris[3ull * t0 + k] = vbase + l;
            if (A.local_idx) A.local_idx[3ull * t0 + k] = (uint16_t)l;
        }
    }
    if (A.verts && !verts_written) {
        f4 *dst = A.verts + 3ull * vbase;
        for (uint32_t q = tid; q < 3 * inv; q += NT) __builtin_nontemporal_store(s_sv[q], dst + q);
    }
    if (tid == 0) {
        if (A.unit_offsets) A.unit_offsets[unit] = t0;
        if (A.unit_inv) A.unit_inv[unit] = inv;
    }
}

// ---------------------------------------------------------------------------
// End of a batched draw: each workgroup sums a slice of the per-batch
// aggregates and adds it to the counters (zeroed by the draw's first
// kernel) and to the context total, one atomic per counter and workgroup,
// and clears its slice of the look-back words for the next launch.
__global__ __launch_bounds__(256) void k_finish(const uint32_t *plan, uint32_t num_batches, uint32_t status_cap,
                                                const unsigned long long *agg, unsigned long long *status,
                                                unsigned long long *counters, unsigned long long *total_inv) {
    __shared__ unsigned long long part[4];
    uint32_t nb = plan ? plan[0] : num_batches;
    if (nb > status_cap) nb = status_cap;
    unsigned long long sum = 0;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nb; i += gridDim.x * 256) {
        sum += agg[i];
        if (status) status[i] = 0;
    }
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_down(sum, d, kWave);
    if (lane_id() == 0) part[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long t = part[0] + part[1] + part[2] + part[3];
        const unsigned long long inv = t & 0xFFFFFFFFull, units = t >> 32;
        if (counters) {
            atomicAdd(&counters[0], inv);
            atomicAdd(&counters[1], units);
        }
        atomicAdd(total_inv, inv);
    }
}

// A draw of at most kFewBatches batches needs no k_finish: every batch that
// counts adds (1 << 52 | units << 32 | invocations) to one word of the draw
// (zero between draws), and the batch that finds all others there writes the
// counters and clears the word and the look-back words.  The sums travel in the
// word and need no order with other memory.  The look-back words do: a batch's
// arrival is a release after its last store to them and its last load of
// others', and the batch that clears them acquires every arrival first, so that
// no earlier store can follow the zeros.
//
// A launch costs about 4 us, an addition to one address about 20 ns: at 128
// batches the additions cost at most 2.6 us, and mostly while other batches run
// (7,938 triangles, plan and hash draw: 22.4 -> 21.3 us; 3,000 triangles, hash
// 9.8 -> 7.7 us, ballot 13.8 -> 7.3 us).  A release writes back its XCD's L2 and
// waits: with look-back words k_finish is as quick from about 32 batches on
// (indexed outputs, k_finish and arrivals: 25 batches 12.4 and 11.5 us, 94 10.7
// and 13.3 us, 125 12.4 and 14.8 us).
constexpr uint32_t kFewBatches = 128, kFewPrefixed = 32;   // without look-back words, with them

// PREFIX: the draw may have look-back words.
template <bool PREFIX>
__device__ __forceinline__ void batch_done(const DrawArgs &A, uint32_t b, uint32_t units, uint32_t inv) {
    const uint32_t nb = counted_batches(A, batch_count(A));
    if (b >= nb) return;
    const unsigned long long mine = 1ull << 52 | (unsigned long long)units << 32 | inv;
    const bool prefix = PREFIX && A.need_prefix;
    if (prefix) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned long long all = atomicAdd(A.arrivals, mine) + mine;
    if ((uint32_t)(all >> 52) != nb) return;
    atomicExch(A.arrivals, 0ull);
    if (A.counters) {
        A.counters[0] = all & 0xFFFFFFFFull;
        A.counters[1] = all >> 32 & 0xFFFFFull;
        A.counters[2] = 0;
        A.counters[3] = 0;
    }
    atomicAdd(A.total_inv, all & 0xFFFFFFFFull);
    if (prefix) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        for (uint32_t i = 0; i < nb; ++i) status_store(&A.status[i], 0);
    }
}

// The draw's first kernel clears its counters before k_finish adds to them, or
// where no batch will write them (an empty plan).
__device__ __forceinline__ void clear_counters(const DrawArgs &A) {
    if (blockIdx.x == 0 && threadIdx.x < 4 && A.counters && (!A.arrivals || batch_count(A) == 0))
        A.counters[threadIdx.x] = 0;
}

// ---------------------------------------------------------------------------
// Naive (Section 3.3): no reuse, every corner is shaded.  One lane per
// corner (three invocations per triangle as in the paper's one thread per
// triangle); the block's corner rows are staged in LDS and stored
// contiguously.
// ---------------------------------------------------------------------------
// One chunk of 256 corners (256 threads); s_sv holds 768 float4.  Returns
// the chunk's aggregate ((triangles started) << 32 | invocations).
template <int KIND>
__device__ __forceinline__ unsigned long long naive_chunk(const DrawArgs &A, const vr_shader_params &sh,
                                                          uint32_t chunk, f4 *s_sv) {
    const uint32_t tid = threadIdx.x;
    const uint64_t n = 3ull * A.T;
    const uint64_t c0 = (uint64_t)chunk * 256;
    const uint32_t cnt = (uint32_t)min<uint64_t>(256, n - c0);
    if (tid < cnt) {
        const uint64_t c = c0 + tid;
        const uint32_t v = fetch_index(A, c);
        shade_to_lds<KIND>(A, sh, v, s_sv + 3 * tid);
        const uint32_t corner = (uint32_t)(c % 3);
        if (A.tris) A.tris[c] = (uint32_t)c;
        if (A.local_idx) A.local_idx[c] = (uint16_t)corner;
        if (corner == 0) {
            const uint32_t t = (uint32_t)(c / 3);
            if (A.unit_offsets) A.unit_offsets[t] = t;
            if (A.unit_inv) A.unit_inv[t] = 3;
        }
    }
    __syncthreads();
    for (uint32_t q = tid; q < 3 * cnt; q += 256) {
        if (A.corners) __builtin_nontemporal_store(s_sv[q], A.corners + 3 * c0 + q);
        if (A.verts) __builtin_nontemporal_store(s_sv[q], A.verts + 3 * c0 + q);
    }
    __syncthreads();
    const uint64_t tris_started = (c0 + cnt + 2) / 3 - (c0 + 2) / 3;
    return (tris_started << 32) | cnt;
}

template <int KIND>
__global__ __launch_bounds__(256) void k_naive(DrawArgs A, vr_shader_params sh) {
    __shared__ f4 s_sv[256 * 3];
    naive_chunk<KIND>(A, sh, xcd_piece(blockIdx.x, gridDim.x), s_sv);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const unsigned long long n = 3ull * A.T;
        if (A.unit_offsets) A.unit_offsets[A.T] = A.T;
        if (A.counters) {
            A.counters[0] = n;
            A.counters[1] = A.T;
            A.counters[2] = 0;
            A.counters[3] = 0;
        }
        atomicAdd(A.total_inv, n);
    }
}

// A stream's naive draw: 85 triangles (255 corners) per workgroup, written and
// set up from their shaded corners in LDS.
constexpr uint32_t kNaiveTris = 85;

template <int KIND>
__global__ __launch_bounds__(256) void k_naive_records(DrawArgs A, vr_shader_params sh) {
    __shared__ f4 s_sv[9 * kNaiveTris];
    const uint32_t tid = threadIdx.x, t0 = xcd_piece(blockIdx.x, gridDim.x) * kNaiveTris;
    const uint32_t ntri = min(kNaiveTris, A.T - t0);
    if (tid < 3 * ntri) shade_to_lds<KIND>(A, sh, fetch_index(A, 3ull * t0 + tid), s_sv + 3 * tid);
    __syncthreads();
    f4 *dst = A.corners + 9ull * t0;
    for (uint32_t q = tid; q < 9 * ntri; q += 256) __builtin_nontemporal_store(s_sv[q], dst + q);
    if (tid < 2 * kWave) {   // the wavefronts that hold triangles, whole
        bool vis = false;
        if (tid < ntri) {
            const f4 c[3] = {s_sv[9 * tid], s_sv[9 * tid + 3], s_sv[9 * tid + 6]};
            vis = setup_triangle(A.setup, c, t0 + tid);
        }
        const uint32_t seen = (uint32_t)__popcll(ballot(vis));
        if (lane_id() == 0) setup_totals(A.setup, 2 * blockIdx.x + tid / kWave, seen, tid == 0 ? 3 * ntri : 0u);
    }
}

// ---------------------------------------------------------------------------
// Two-pass reference (Section 4.2, Table 2), not streaming: every vertex of
// the buffer is shaded once by a first kernel, referenced or not; a second
// kernel assembles the corners from the shaded buffer in global memory.
// ---------------------------------------------------------------------------
// 256 vertices per workgroup: shaded into LDS, then stored as one contiguous
// span of rows (plain stores, so the rows stay in the caches for the gather).
template <int KIND>
__global__ __launch_bounds__(256) void k_multi_shade(DrawArgs A, vr_shader_params sh, f4 *shaded) {
    __shared__ f4 s_sv[256 * 3];
    const uint32_t v0 = blockIdx.x * 256, tid = threadIdx.x;
    const uint32_t cnt = min(256u, A.V - v0);
    if (tid < cnt) shade_to_lds<KIND>(A, sh, v0 + tid, s_sv + 3 * tid);
    __syncthreads();
    f4 *dst = shaded + 3ull * v0;
    for (uint32_t q = tid; q < 3 * cnt; q += 256) dst[q] = s_sv[q];
}

// 256 corners per workgroup: each lane gathers its corner's three rows from
// the shaded buffer into LDS, then the block's rows are stored as one
// contiguous span (fully coalesced 16-byte stores).  The single unit's
// counters and offsets come from block 0.
__global__ __launch_bounds__(256) void k_multi_assemble(DrawArgs A, const f4 *shaded) {
    __shared__ f4 s_rows[256 * 3];
    const uint64_t n = 3ull * A.T, c0 = (uint64_t)xcd_piece(blockIdx.x, gridDim.x) * 256;
    const uint32_t tid = threadIdx.x;
    const uint32_t cnt = (uint32_t)min<uint64_t>(256, n - c0);
    if (tid < cnt) {
        const uint32_t v = fetch_index(A, c0 + tid);
        const f4 *src = shaded + 3ull * v;
        s_rows[3 * tid] = src[0];
        s_rows[3 * tid + 1] = src[1];
        s_rows[3 * tid + 2] = src[2];
        if (A.tris) A.tris[c0 + tid] = v;
    }
    __syncthreads();
    if (A.corners)
        for (uint32_t q = tid; q < 3 * cnt; q += 256) __builtin_nontemporal_store(s_rows[q], A.corners + 3 * c0 + q);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (A.counters) {
            A.counters[0] = A.V;
            A.counters[1] = 1;
            A.counters[2] = 0;
            A.counters[3] = 0;
        }
        if (A.unit_offsets) {
            A.unit_offsets[0] = 0;
            A.unit_offsets[1] = A.T;
        }
        if (A.unit_inv) A.unit_inv[0] = A.V;
        atomicAdd(A.total_inv, (unsigned long long)A.V);
    }
}

// ---------------------------------------------------------------------------
// LDS layout of the dedup kernel (bytes), shared with the host launcher.
// ---------------------------------------------------------------------------
struct DedupLds {
    uint32_t local, pairs, stab, table, first, uniq, sv, tmp, total;
};

__host__ __device__ inline uint32_t align16(uint32_t x) { return (x + 15u) & ~15u; }

// Corners a thread keeps in registers during deduplication; a unit of more
// than kRows * NT corners is deduplicated in chunks of that many.
constexpr uint32_t kRows = 4;

// Count groups per digit of the sort's radix passes: rounds x wavefronts,
// padded to whole words.
__host__ __device__ inline uint32_t sort_groups(uint32_t max_keys, uint32_t nt) {
    const uint32_t g = (max_keys + nt - 1) / nt * (nt / 64);
    return (g + 3u) & ~3u;
}

// The local ids and the unique list live from deduplication to the end of
// the unit; the shaded vertices (written after deduplication) share their
// region with what deduplication alone uses: the hash table and each slot's
// id word (or a static sort's indices), then the sort's two position buffers
// and its per-digit counts (uint8) and offsets (uint16).  sv_rows shaded vertices are kept: every
// unique vertex of a unit when corners are assembled, else one stage of nt
// rows through which the shaded vertices stream out.
__host__ __device__ inline DedupLds dedup_lds_layout(int mode, bool dynamic, uint32_t max_idx, uint32_t max_uniq,
                                                     uint32_t hash_bits, uint32_t nt, uint32_t sv_rows) {
    DedupLds L{};
    uint32_t off = 0;
    L.local = off; off += align16(2 * max_idx);   // uint16: hash slots < 8192, then ids < max_idx
    L.uniq = off;  off += align16(4 * max_uniq);
    L.sv = off;
    uint32_t d = off;
    L.table = d;
    if (mode == kSort && !dynamic) {
        d += align16(4 * max_idx);   // every index, as no table drops duplicates
    } else {
        d += align16(4u << hash_bits);
        L.first = d; d += align16(4u << hash_bits);
    }
    if (mode == kSort) {   // of the indices that are sorted: all, or the distinct ones
        const uint32_t m = dynamic ? max_uniq : max_idx;
        L.pairs = d; d += align16(4 * m);   // two uint16 position buffers
        L.stab = d;  d += 3u * 256u * sort_groups(m, nt);
    }
    off = max(align16(off + 48 * sv_rows), align16(d));
    L.tmp = off;  off += 64;   // scan words, or counts (uint8) per row and wavefront; then three words of the unit
    L.total = off;
    return L;
}

// LDS a dedup kernel takes besides that layout, which starts at the next 16 bytes:
// a word of the unit at a fixed address up to 256 threads (with it in the layout
// a frame's hashing variants take 0.5 % longer), and with 1,024 threads, whose
// scan fills the layout's words, all three.
__host__ __device__ constexpr uint32_t dedup_lds_static(uint32_t nt) { return nt <= 256 || nt == 1024 ? 16u : 0u; }

// Bytes a unit counts for against the device's LDS limit: the sizes a call
// may ask for follow from this (never less than the layout above takes), so
// that they do not depend on how the kernel arranges its LDS.
__host__ inline uint32_t dedup_lds_counted(int mode, uint32_t max_idx, uint32_t max_uniq, uint32_t hash_bits,
                                           uint32_t nt, uint32_t sv_rows) {
    const uint32_t ids = align16(2 * max_idx), uniq = align16(4 * max_uniq), keys = align16(4 * max_idx);
    if (mode == kSort) {
        const uint32_t stab = 2 * keys, end = stab + 3u * 256u * sort_groups(max_idx, nt);
        return max(max(align16(48 * sv_rows), stab) + ids + uniq, end) + 64;
    }
    return max(align16(ids + uniq + 48 * sv_rows), align16(ids + uniq + keys + 2 * align16(4u << hash_bits))) + 64;
}

// LSD radix sort of a unit's distinct indices (Algorithm 2's sort): 8-bit
// digits of (index - unit minimum), `passes` of them.  Within a pass, element
// x of the current order is handled in round x / NT by thread x % NT; its
// stable destination is the offset of (digit, round, wavefront) plus its
// rank among the wavefront's lanes with the same digit, found with 8
// ballots.  Counts (uint8) and offsets (uint16) are stored per digit
// contiguously in `tab`, so the thread owning a digit scans them with word
// accesses and clears the counts for the next pass.  RR is the round count
// when known at compile time (R == RR), else 8 (R <= 8).  Returns the sorted
// order (one of the two position buffers).
template <int NT, uint32_t RR>
__device__ __forceinline__ const uint16_t *radix_passes(const uint32_t *s_keys, uint16_t *src, uint16_t *dst,
                                                        uint32_t n, uint32_t R, uint32_t kmin, uint32_t passes,
                                                        uint32_t Gp, unsigned char *tab, uint32_t *s_tmp) {
    constexpr uint32_t NW = NT / kWave;
    constexpr uint32_t DP = NT >= 256 ? 1u : 256u / NT;   // digits per thread in the scan
    const uint32_t tid = threadIdx.x, w = tid / kWave;
    uint32_t *s_c32 = (uint32_t *)tab;              // [256][Gp] uint8 counts
    uint2 *s_o64 = (uint2 *)(tab + 256 * Gp);       // [256][Gp] uint16 offsets
    const uint16_t *s_o16 = (const uint16_t *)s_o64;
    uint8_t *s_c8 = (uint8_t *)s_c32;
    for (uint32_t pass = 0; pass < passes; ++pass) {
        uint32_t dig[RR], rank[RR], pos[RR];
#pragma unroll
        for (uint32_t r = 0; r < RR; ++r) {
            if (RR == 8 && r >= R) break;
            const uint32_t x = r * NT + tid;
            const bool act = x < n;
            const uint32_t p = act ? src[x] : 0u;
            const uint32_t d = act ? ((s_keys[p] - kmin) >> (8 * pass)) & 0xFFu : 0u;
            // lanes with the same digit: for each bit, the lanes that agree
            // on it are m where the bit is set and ~m where it is clear
            const uint64_t act_m = ballot(act);
            uint32_t plo = (uint32_t)act_m, phi = (uint32_t)(act_m >> 32);
            const uint32_t nd = ~d;
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                // nx = ~0 where the bit is clear, 0 where it is set (one signed
                // bit-field extract, kept opaque so that it is not rebuilt from
                // compares and selects)
                uint32_t nx;
                asm volatile("v_bfe_i32 %0, %1, %2, 1" : "=v"(nx) : "v"(nd), "n"(bit));
                const uint64_t m = ballot(nx == 0u);
                plo &= (uint32_t)m ^ nx;
                phi &= (uint32_t)(m >> 32) ^ nx;
            }
            const uint64_t peers = ((uint64_t)phi << 32) | plo;
            const uint32_t rk = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            // digit x group index in 24-bit products (full-rate multiplies)
            if (act && rk == 0) s_c8[__umul24(d, Gp) + r * NW + w] = (uint8_t)__popcll(peers);
            dig[r] = d;
            rank[r] = rk;
            pos[r] = p;
        }
        __syncthreads();
        {   // exclusive offsets in (digit, round, wavefront) order
            const uint32_t d0 = tid * DP, words = Gp / 4;
            uint32_t sum = 0;
            if (d0 < 256)
                for (uint32_t j = 0; j < DP * words; ++j) {
                    const uint32_t c = s_c32[d0 * words + j];
                    sum += (c & 0xFFu) + ((c >> 8) & 0xFFu) + ((c >> 16) & 0xFFu) + (c >> 24);
                }
            uint32_t total;
            uint32_t run = block_excl_scan<NT>(sum, s_tmp, total);
            if (d0 < 256)
                for (uint32_t j = 0; j < DP * words; ++j) {
                    const uint32_t c = s_c32[d0 * words + j];
                    s_c32[d0 * words + j] = 0;   // counts start at zero next pass
                    const uint32_t o0 = run, o1 = o0 + (c & 0xFFu), o2 = o1 + ((c >> 8) & 0xFFu),
                                   o3 = o2 + ((c >> 16) & 0xFFu);
                    run = o3 + (c >> 24);
                    s_o64[d0 * words + j] = make_uint2(o0 | (o1 << 16), o2 | (o3 << 16));
                }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < RR; ++r) {
            if (RR == 8 && r >= R) break;
            const uint32_t x = r * NT + tid;
            if (x < n) dst[s_o16[__umul24(dig[r], Gp) + r * NW + w] + rank[r]] = (uint16_t)pos[r];
        }
        __syncthreads();
        uint16_t *t = src;
        src = dst;
        dst = t;
    }
    return src;
}

// Inserts this thread's corners (row k is pending where bit k is set) into
// the unit's LDS hash table by linear probing and returns in slot[] where
// each key sits; fresh gets a bit per row whose key this lane inserted.  The
// rows advance together, one probe each per round: a round issues every
// row's compare-and-swap before it looks at the first, so that their LDS
// round trips overlap.  With MODE kPHash a row still unplaced after A.probes
// rounds is handed to its whole wavefront, which tests 64 slots at a time.
template <int MODE>
__device__ __forceinline__ void insert_rows(const DrawArgs &A, uint32_t *s_table, const uint32_t (&key)[kRows],
                                            uint32_t (&slot)[kRows], uint32_t pending, uint32_t &fresh) {
    const uint32_t mask = (1u << A.hash_bits) - 1;
    fresh = 0;
#pragma unroll
    for (uint32_t k = 0; k < kRows; ++k) slot[k] = hash_slot(key[k], A.hash_bits);
    for (uint32_t round = 0; MODE == kPHash ? (pending && round < A.probes) : pending != 0; ++round) {
        uint32_t prev[kRows];
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k)
            if (pending & (1u << k)) prev[k] = atomicCAS(&s_table[slot[k]], kEmpty, key[k]);
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k) {
            if (pending & (1u << k)) {
                if (prev[k] == kEmpty) fresh |= 1u << k;
                if (prev[k] == kEmpty || prev[k] == key[k]) pending &= ~(1u << k);
                else slot[k] = (slot[k] + 1) & mask;
            }
        }
        if (MODE != kPHash && round > mask && pending) {   // table full: only with foreign plans
            raise_error(A.err, VR_ERR_CAPACITY);
            break;
        }
    }
    if (MODE != kPHash) return;
    const uint32_t lane = lane_id();
#pragma unroll
    for (uint32_t k = 0; k < kRows; ++k) {
        uint64_t pend = ballot((pending >> k) & 1u);
        while (pend) {
            const uint32_t Lr = (uint32_t)__builtin_ctzll(pend);
            const uint32_t want = __builtin_amdgcn_readlane(key[k], Lr);
            uint32_t start = __builtin_amdgcn_readlane(slot[k], Lr);
            for (uint32_t sweep = 0;; ++sweep) {
                if (sweep > 2 * (mask + 1)) {     // table full: only with foreign plans
                    if (lane == 0) raise_error(A.err, VR_ERR_CAPACITY);
                    break;
                }
                const uint32_t s = (start + lane) & mask;
                const uint32_t val = __hip_atomic_load(&s_table[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const uint64_t hit = ballot(val == kEmpty || val == want);
                if (!hit) {
                    start = (start + kWave) & mask;
                    continue;
                }
                const uint32_t w = (uint32_t)__builtin_ctzll(hit);
                const uint32_t ws = (start + w) & mask;
                uint32_t got = 0;
                if (lane == w) got = atomicCAS(&s_table[ws], kEmpty, want);
                got = __builtin_amdgcn_readlane(got, w);
                if (got == kEmpty || got == want) {
                    if (lane == Lr) {
                        slot[k] = ws;
                        if (got == kEmpty) fresh |= 1u << k;
                    }
                    break;
                }
                start = ws;   // lost the slot to another key: continue past it
            }
            pend &= pend - 1;
        }
    }
}

// ---------------------------------------------------------------------------
// Batched deduplication + shading + assembly (Algorithms 2 and 3, and the
// parallel-hashing variant).  Workgroup u owns unit u (no atomics to pick
// work); a unit of n corners is deduplicated in LDS into inv unique
// vertices with canonical local ids:
//   sort  - ascending rank among distinct indices (Algorithm 2).  A dynamic
//           unit's duplicates are dropped by the table first, so that the
//           radix sort takes its distinct indices only (a quarter of them on
//           an ordered mesh; on a random one the unit is small either way:
//           49.4 -> 45.9 us for 398,000 triangles).  A static unit sorts all
//           of its indices: in random order the table only adds to the sort
//           (batches of 64: 32.4 us without it, 39.2 us with),
//   hash  - first-occurrence order (Algorithm 3, ids made independent of
//           the insertion races by ranking each slot's first position),
//   phash - as hash, but a lane that fails `probes` linear probes hands its
//           key to a wavefront-cooperative probe of 64 slots at a time.
// Corner i of the unit is row i / NT of thread i % NT; a thread's rows stay
// in registers from the index load to the local ids.  OUT says what the unit
// writes.  The sort takes at most SORT_ROUNDS indices per thread.  FEW: the
// unit may be one of a draw of few batches (batch_done).
//
// A unit is a serial chain (index load, insertion, vertex gather, shading,
// stores) between barriers, so its phases are kept few and their loads early:
// the index load covers the clearing of the table, the vertex gather the
// writing of the local ids.  icosphere of 1.31M triangles, Phong-8, 256 / 341:
// with the indices staged in LDS, one row at a time and every kernel argument
// kept in (spilled) scalar registers, hash took 1,245 vector instructions per
// wavefront and 53.3 us, sort 2,220 and 64.0 us, indexed phash 61.2 us; so
// hash takes 945 and 51.2 us, sort 1,344 and 57.4 us, indexed phash 50.1 us.
// ---------------------------------------------------------------------------
template <int NT, int MODE, int KIND, int OUT, uint32_t SORT_ROUNDS, bool FEW>
__device__ __forceinline__ void dedup_unit(ArgsPtr args, ShaderPtr shader, uint32_t u, uint32_t nb,
                                           unsigned char *smem, unsigned long long *agg) {
    constexpr bool FULL = OUT == kAll;
    constexpr uint32_t NW = NT / kWave, kChunk = kRows * NT;
    const DrawArgs &A = *(const DrawArgs *)reread(args);
    // without corners, units whose unique vertices would not leave room for
    // several workgroups per CU stream them out through an NT-row stage
    const bool stream = FULL && A.stream_verts != 0;
    const bool direct = MODE == kSort && !A.plan;   // the sort takes every corner's index
    const DedupLds L = dedup_lds_layout(MODE, !direct, A.max_idx, A.max_uniq, A.hash_bits, NT, stream ? NT : A.max_uniq);
    uint16_t *s_local = (uint16_t *)(smem + L.local);
    uint32_t *s_uniq = (uint32_t *)(smem + L.uniq);
    f4 *s_sv = (f4 *)(smem + L.sv);
    uint32_t *s_table = (uint32_t *)(smem + L.table);
    uint32_t *s_first = (uint32_t *)(smem + L.first);
    uint32_t *s_tmp = (uint32_t *)(smem + L.tmp);
    __shared__ __attribute__((aligned(16))) uint32_t s_static[NT == 512 ? 1 : dedup_lds_static(NT) / 4];
    uint32_t *s_unit = NT < 1024 ? s_tmp + 12 : s_static;
    uint32_t &s_min = s_unit[1], &s_max = s_unit[2];
    uint32_t &s_count = NT == 512 ? s_unit[0] : s_static[0];
    uint32_t &s_vbase = s_count;   // known after the last use of the count

    const uint32_t tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint32_t t0, t1;
    batch_range(A, u, t0, t1);
    uint32_t n = 3 * (t1 - t0);
    const bool fits = t1 >= t0 && n <= A.max_idx;   // false only for a plan built with other limits
    if (!fits) {
        if (tid == 0) raise_error(A.err, VR_ERR_CAPACITY);
        n = 0;
    }
    // Ids are visible only in the indexed outputs and local ids; then the
    // hashes make them canonical (first-occurrence order).  Otherwise a key's
    // id comes from a counter (Algorithm 3), and the corners are the same
    // either way.  The sort ranks the distinct indices in both cases.
    const bool canon = FULL && MODE != kSort && (A.need_prefix || A.local_idx);
    // slots of several chunks wait in LDS; so do the sort's, whose passes need the registers
    const bool chunked = MODE == kSort || n > kChunk;
    const uint64_t base = 3ull * t0;
    uint32_t key[kRows], slot[kRows];
    auto load_keys = [&](uint32_t c0) {
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k) {
            const uint32_t i = c0 + k * NT + tid;
            key[k] = i < n ? A.idx[base + i] : 0u;
        }
    };
    load_keys(0);   // in flight while the table is cleared
    if (!direct) {
        const uint4 e = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
        const uint32_t q1 = (canon ? 2u : 1u) << A.hash_bits;   // the id words follow the table
        for (uint32_t q = 4 * tid; q < q1; q += 4 * NT) *(uint4 *)&s_table[q] = e;
    }
    // the sort takes a dynamic unit's distinct indices, a static unit's every index
    const uint32_t sort_cap = direct ? A.max_idx : A.max_uniq, Gp = sort_groups(sort_cap, NT);
    uint16_t *s_pos0 = (uint16_t *)(smem + L.pairs);
    uint16_t *s_pos1 = s_pos0 + (align16(4 * sort_cap) / 4);
    if (MODE == kSort) {
        uint32_t *s_c32 = (uint32_t *)(smem + L.stab);   // [256][Gp] uint8 counts
        for (uint32_t i = tid; i < sort_cap; i += NT) s_pos0[i] = (uint16_t)i;
        for (uint32_t i = tid; i < 64 * Gp; i += NT) s_c32[i] = 0;
    }
    if (tid == 0) {
        s_count = 0;
        s_min = kEmpty;
        s_max = 0;
    }
    __syncthreads();
    for (uint32_t c0 = 0; c0 < n; c0 += kChunk) {
        if (c0) load_keys(c0);
        uint32_t act = 0, fresh = 0;
        bool bad = false;
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k) {
            if (c0 + k * NT + tid < n) act |= 1u << k;
            if (key[k] >= A.V) {   // replaced by 0, so that no access leaves the buffers
                bad = true;
                key[k] = 0;
            }
        }
        if (bad) raise_error(A.err, VR_ERR_INDEX_RANGE);
        if (direct) {
#pragma unroll
            for (uint32_t k = 0; k < kRows; ++k)
                if (act & (1u << k)) s_table[c0 + k * NT + tid] = key[k];
        } else {
            insert_rows<MODE>(A, s_table, key, slot, act, fresh);
        }
        if (canon) {
#pragma unroll
            for (uint32_t k = 0; k < kRows; ++k)
                if (act & (1u << k)) atomicMin(&s_first[slot[k]], c0 + k * NT + tid);
        } else {
            // the wavefront's new keys take consecutive ids, one counter update per wavefront
            uint64_t b[kRows];
            uint32_t total = 0;
#pragma unroll
            for (uint32_t k = 0; k < kRows; ++k) {
                b[k] = ballot((fresh >> k) & 1u);
                total += (uint32_t)__popcll(b[k]);
            }
            if (total) {
                uint32_t id0 = 0;
                if (lane == 0) id0 = atomicAdd(&s_count, total);
                id0 = __builtin_amdgcn_readfirstlane(id0);
#pragma unroll
                for (uint32_t k = 0; k < kRows; ++k) {
                    if (fresh & (1u << k)) {
                        const uint32_t id = id0 + __builtin_amdgcn_mbcnt_hi(
                                                      (uint32_t)(b[k] >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)b[k], 0u));
                        s_first[slot[k]] = id;
                        if (id < A.max_uniq) s_uniq[id] = key[k];
                    }
                    id0 += (uint32_t)__popcll(b[k]);
                }
            }
            if (MODE == kSort) {   // the range of the unit's indices
                uint32_t mn = kEmpty, mx = 0;
#pragma unroll
                for (uint32_t k = 0; k < kRows; ++k) {
                    if (act & (1u << k)) {
                        mn = min(mn, key[k]);
                        mx = max(mx, key[k]);
                    }
                }
                mn = wave_min(mn);
                mx = wave_max(mx);
                if (lane == 0) {
                    atomicMin(&s_min, mn);
                    atomicMax(&s_max, mx);
                }
            }
        }
        if (chunked && !direct) {
#pragma unroll
            for (uint32_t k = 0; k < kRows; ++k)
                if (act & (1u << k)) s_local[c0 + k * NT + tid] = (uint16_t)slot[k];
        }
    }
    __syncthreads();
    // the rows of chunk c0: their slots, from LDS when there are several chunks
    auto row_slots = [&](uint32_t c0) {
        if (!chunked) return;
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k) {
            const uint32_t i = c0 + k * NT + tid;
            slot[k] = i < n ? (uint32_t)s_local[i] : 0u;
        }
    };
    uint32_t inv = 0;
    if (canon) {
        // a slot's id is the rank of its first position: positions are in
        // (row, wavefront, lane) order, so a ballot per row and the counts of
        // the rows and wavefronts before give it.  The first position then
        // overwrites its slot's word with the rank r <= position, which no
        // later position can mistake for itself.
        uint8_t *s_cnt = (uint8_t *)s_tmp;   // [kRows][NW], at most 64 each
        for (uint32_t c0 = 0; c0 < n; c0 += kChunk) {
            row_slots(c0);
            uint64_t b[kRows];
#pragma unroll
            for (uint32_t k = 0; k < kRows; ++k) {
                const uint32_t i = c0 + k * NT + tid;
                b[k] = ballot(i < n && s_first[slot[k]] == i);
                if (lane == 0) s_cnt[k * NW + w] = (uint8_t)__popcll(b[k]);
            }
            __syncthreads();
#pragma unroll
            for (uint32_t k = 0; k < kRows; ++k) {
                uint32_t before = inv, all = 0;
                if (NW < 4) {
#pragma unroll
                    for (uint32_t j = 0; j < NW; ++j) {
                        const uint32_t c = s_cnt[k * NW + j];
                        before += j < w ? c : 0u;
                        all += c;
                    }
                } else {
#pragma unroll
                    for (uint32_t j = 0; j < NW; j += 4) {   // four wavefronts' counts per word
                        const uint32_t c = ((const uint32_t *)s_cnt)[(k * NW + j) / 4];
                        const uint32_t low = w <= j ? 0u : w - j >= 4 ? ~0u : (1u << (8 * (w - j))) - 1u;
                        before = __builtin_amdgcn_sad_u8(c & low, 0u, before);
                        all = __builtin_amdgcn_sad_u8(c, 0u, all);
                    }
                }
                if ((b[k] >> lane) & 1ull) {
                    const uint32_t r = before + __builtin_amdgcn_mbcnt_hi(
                                                    (uint32_t)(b[k] >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)b[k], 0u));
                    s_first[slot[k]] = r;
                    if (r < A.max_uniq) s_uniq[r] = chunked ? s_table[slot[k]] : key[k];
                }
                inv += all;
            }
            if (chunked) __syncthreads();   // the counts are read before the next chunk's
        }
        __syncthreads();
    } else {
        inv = s_count;
    }
    if (inv > A.max_uniq) {   // only with a plan built for a larger N_u
        if (tid == 0) raise_error(A.err, VR_ERR_CAPACITY);
        inv = 0;
        n = 0;
    }
    // this unit's invocation count is published as soon as it is known, since
    // the units after it wait for it (random order, phash 128 / 128, every
    // output: 80.9 us when published after the local ids, 72.2 us here), and
    // its prefix is resolved after shading (before it when the shaded vertices
    // stream out)
    auto publish = [&]() {
        if (FULL && A.need_prefix && tid == 0) lookback_publish(A.status, u, (1ull << 32) | inv);
    };
    if (!direct) publish();
    const uint16_t *s_rank = nullptr;
    if (MODE == kSort) {
        // LSD radix sort (radix_passes) of the distinct indices, or of a static
        // unit's every index, only as many passes as the unit's index range needs
        const uint32_t m = direct ? n : inv;
        const uint32_t *s_keys = direct ? s_table : s_uniq;
        const uint32_t R = (m + NT - 1) / NT;   // the launcher sizes NT for at most 8
        const uint32_t kmin = s_min, span = m ? s_max - kmin : 0u;
        const uint32_t passes = span ? (32u - __builtin_clz(span) + 7u) / 8u : 0u;
        // the round count fixed at compile time where it is small
        auto sorted_by = [&](auto rr) {
            return radix_passes<NT, decltype(rr)::value>(s_keys, s_pos0, s_pos1, m, R, kmin, passes, Gp,
                                                         smem + L.stab, s_tmp);
        };
        const uint16_t *src;
        if (R <= 1) src = sorted_by(std::integral_constant<uint32_t, 1>{});
        else if (R == 2) src = sorted_by(std::integral_constant<uint32_t, 2>{});
        else if (SORT_ROUNDS == 3 || R == 3) src = sorted_by(std::integral_constant<uint32_t, 3>{});
        else src = sorted_by(std::integral_constant<uint32_t, 8>{});
        if (direct) {
            // run ends of the sorted indices; the exclusive prefix over run
            // ends is the rank of every entry's run (Algorithm 2's marks and
            // prefix sum)
            const uint32_t E = (n + NT - 1) / NT;
            const uint32_t lo = min(n, tid * E), hi = min(n, lo + E);
            uint32_t cnt = 0;
            for (uint32_t i = lo; i < hi; ++i) cnt += (i + 1 == n || s_keys[src[i]] != s_keys[src[i + 1]]);
            uint32_t r = block_excl_scan<NT>(cnt, s_tmp, inv);
            publish();
            for (uint32_t i = lo; i < hi; ++i) {
                const uint32_t p = src[i], k = s_keys[p];
                s_local[p] = (uint16_t)r;
                if (i + 1 == n || k != s_keys[src[i + 1]]) s_uniq[r++] = k;
            }
        } else {
            // an id's place in the sorted order is its rank
            uint16_t *s_out = src == s_pos0 ? s_pos1 : s_pos0;   // free after the last pass
            for (uint32_t i = tid; i < inv; i += NT) {
                const uint32_t id = src[i];
                s_table[i] = s_uniq[id];   // the keys' table is dead, the id words are not
                s_out[id] = (uint16_t)i;
            }
            __syncthreads();   // every index is read before the list is rewritten in order
            for (uint32_t i = tid; i < inv; i += NT) s_uniq[i] = s_table[i];
            s_rank = s_out;
        }
        __syncthreads();   // the list is complete
    }
    // the thread's place, of unknown origin to the compiler: what the phases
    // below derive from it is not kept from before (a sort with more outputs than
    // corners spilled eight such values a lane; 398,000 triangles in random
    // order, static 85: indexed 48.5 -> 46.5 us, every output 60.9 -> 55.9 us)
    uint32_t at = tid;
    if (MODE == kSort && FULL) asm volatile("" : "+v"(at));
    // the first NT unique vertices: their input is loaded while the corners'
    // local ids are written
    f4 va = {}, vb = {};
    if (!stream && at < inv) {
        const uint32_t v = s_uniq[at];
        va = A.vtx[2ull * v];
        vb = A.vtx[2ull * v + 1];
    }
    for (uint32_t c0 = 0; c0 < n && !direct; c0 += kChunk) {
        row_slots(c0);
#pragma unroll
        for (uint32_t k = 0; k < kRows; ++k) {
            const uint32_t i = c0 + k * NT + at;
            if (i < n) {
                uint32_t id = s_first[slot[k]];
                if (MODE == kSort) id = s_rank[id];
                s_local[i] = (uint16_t)id;
            }
        }
    }
    if (!direct) __syncthreads();   // the table is dead: shaded vertices take its space
    const DrawArgs &B = *(const DrawArgs *)reread(args);
    const vr_shader_params &sh = *(const vr_shader_params *)reread(shader);
    if (!stream) {
        if (at < inv) shade_raw_to_lds<KIND>(sh, va, vb, s_sv + 3 * at);
        for (uint32_t j = at + NT; j < inv; j += NT) shade_to_lds<KIND>(B, sh, s_uniq[j], s_sv + 3 * j);
    }
    if (FULL && at < kWave) {   // the first wavefront, whole (NT >= 64)
        uint32_t vb0 = 0;
        if (B.need_prefix) vb0 = (uint32_t)lookback_resolve(B.status, u, (1ull << 32) | inv, B.err);
        if (at == 0) {
            s_vbase = vb0;
            if (B.unit_offsets && u + 1 == nb) B.unit_offsets[nb] = B.T;
        }
    }
    __syncthreads();
    if (stream) {
        // NT unique vertices at a time: shaded into the stage, then stored as
        // one contiguous span of rows while the next ones' input is loaded
        f4 *dst = B.verts ? B.verts + 3ull * s_vbase : nullptr;
        f4 ra = {}, rb = {};
        auto load_next = [&](uint32_t j) {
            if (j >= inv) return;
            const uint32_t v = s_uniq[j];
            ra = B.vtx[2ull * v];
            rb = B.vtx[2ull * v + 1];
        };
        load_next(at);
        for (uint32_t j0 = 0; j0 < inv; j0 += NT) {
            const uint32_t rows = min((uint32_t)NT, inv - j0);
            if (at < rows) shade_raw_to_lds<KIND>(sh, ra, rb, s_sv + 3 * at);
            __syncthreads();
            load_next(j0 + NT + at);
            if (dst)
                for (uint32_t q = at; q < 3 * rows; q += NT)
                    __builtin_nontemporal_store(s_sv[q], dst + 3ull * j0 + q);
            __syncthreads();
        }
    }
    if (fits && (inv > 0 || t1 == t0))
        write_unit<NT, OUT>(B, t0, t1 - t0, s_local, s_sv, inv, FULL ? s_vbase : 0u, u, at, stream);
    if (OUT == kRecords) {
        const uint32_t seen = fits && inv > 0 ? setup_unit<NT>(B.setup, t0, t1 - t0, s_local, s_sv, at) : 0u;
        if (lane == 0) setup_totals(B.setup, u * NW + w, seen, at == 0 ? inv : 0u);
    } else if (at == 0) {
        // read again here, so that nothing is kept for it; a frame's units come
        // with their place
        const DrawArgs &F = *(const DrawArgs *)reread(args);
        if (FEW && F.arrivals) batch_done<FULL>(F, u, 1, inv);
        else if (u < F.status_cap) (agg ? agg : F.agg)[u] = (1ull << 32) | inv;   // no room past the bound
    }
    __syncthreads();   // the caller may reuse the LDS for the next unit
}

// Wavefronts per SIMD the occupancy-bound kernels are held to: as many as
// their registers allow without spilling to scratch (FULL at 8 spilled 40 B a
// lane: indexed phash 128 / 128 36.7 us at 8, 35.0 us at 7).
__host__ __device__ constexpr int dedup_waves(int mode, bool full) { return mode == kSort || full ? 7 : 8; }

// The other kernels: as many as their LDS mostly leaves anyway.  A sort of 64
// threads with more outputs than corners is given six instead of five (static
// 32, 398,000 triangles in random order, Phong-9: indexed 73.2 -> 69.9 us, every
// output 83.7 -> 78.5 us; with corners alone 37.8 -> 45.6 us with MVP).
__host__ __device__ constexpr int dedup_waves_free(int mode, bool full, int nt) {
    return mode != kSort || (full && nt == 64) ? 6 : 5;
}

struct DedupLaunch {
    DrawArgs A;
    vr_shader_params sh;
    uint32_t base, stride;
};

// Units from base on: unit base + workgroup index (stride 0), or
// grid-stride over every unit from base on (stride = the grid).  Grid-stride
// serves the units of a dynamic draw beyond the fewest it can have within
// the same launch; it is used without prefix outputs only, since the
// look-back needs each unit's predecessor running or done.  With OCC the
// kernel is held to eight wavefronts per SIMD (seven for the sort, whose
// registers would otherwise spill): the host picks it only when the unit's
// LDS lets that many workgroups reside, and then the extra wavefronts hide
// more of a unit's serial latency; otherwise the bound would only add
// spills.
template <int NT, int MODE, int KIND, bool OCC, int OUT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(OCC ? dedup_waves(MODE, OUT == kAll) : dedup_waves_free(MODE, OUT == kAll, NT)))) void k_dedup(DedupLaunch) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // the launch's only argument, at the start of the kernel-argument segment
    const VR_CONSTANT DedupLaunch *P = (const VR_CONSTANT DedupLaunch *)__builtin_amdgcn_kernarg_segment_ptr();
    const DrawArgs &A = *(const DrawArgs *)&P->A;
    if (P->base == 0) clear_counters(A);
    const uint32_t nb = launch_units(A, batch_count(A));
    // units with prefix outputs wait for their predecessors: in dispatch order;
    // so are the units past the first of each workgroup, which are few and
    // would otherwise all fall to one XCD
    uint64_t u = (uint64_t)P->base + (OUT == kAll ? blockIdx.x : xcd_piece(blockIdx.x, gridDim.x));
    for (uint64_t next = (uint64_t)P->base + blockIdx.x; u < nb; u = next) {
        dedup_unit<NT, MODE, KIND, OUT, OCC ? 3 : 8, !OCC>(&P->A, &P->sh, (uint32_t)u, nb, smem, nullptr);
        next += P->stride ? P->stride : nb;
    }
}

// ---------------------------------------------------------------------------
// Wave64 rounds (Algorithm 1 on a 64-lane wavefront).  One wavefront owns a
// batch and cuts it into rounds: it takes 21 whole triangles (63 indices, one
// per lane) at a time, finds the lanes that hold an index the round has not
// met (a small table in the wavefront's LDS brings equal indices together, the
// lowest lane of each counts as its first), and a ballot of those lanes gives
// each the next free lane, which will shade it.  The first triangle that would
// need a 65th lane ends the round; lanes taken by rejected triangles are
// released, so a round shades exactly its distinct indices.
// ---------------------------------------------------------------------------
struct RoundState {
    uint32_t my_id;   // the vertex this lane shades in the round
    uint32_t fill;    // lanes in use (= invocations of the round)
    f4 va, vb;        // its input, loaded when the lane took it (output sweep only)
};

// Indices of a batch a wavefront keeps in LDS (the rest, for batches of more
// than 256 triangles, is fetched per group of 21 triangles).
constexpr uint32_t kBallotPrefetch = 768;

// LDS of one ballot wavefront: 64 shaded vertices, the prefetched indices, a
// hand-over area for new values (2 x 64 words) and a lane number per corner.
__host__ __device__ inline uint32_t ballot_lds_bytes(uint32_t batch_tris) {
    const uint32_t pre = 3 * batch_tris < kBallotPrefetch ? 3 * batch_tris : kBallotPrefetch;
    return 64 * 48 + 4 * pre + 2 * 64 * 4 + ((3 * batch_tris + 15u) & ~15u);
}

// Processes one round starting at triangle `cur` of the batch starting at
// t0; returns the round's end.  The batch's first `pre` indices are in
// s_keys; s_new is the wavefront's hand-over area, s_table kRoundSlots index
// words and as many position words (the space of the round's shaded
// vertices).  When s_map is not NULL it receives each corner's lane (local id).
//
// Within a group equal indices meet in one slot of s_table; the smallest
// position that reached the slot is the index's first occurrence, and its
// lane then leaves the lane number there (never above the position, so later
// positions change neither).  Resolving a group by one vote per distinct index
// instead (broadcast, compare, ballot, about 14 instructions each in one
// dependent chain) took 1,639 vector and 906 scalar instructions per batch of
// 64 triangles and 63.7 us for the icosphere's 20,480 batches (Phong-8); the
// table's few LDS round trips take 1,051 and 577, and 52.8 us.
constexpr uint32_t kRoundBits = 8, kRoundSlots = 1u << kRoundBits;   // at most 64 + 63 indices at once

__device__ __forceinline__ uint32_t ballot_round(const DrawArgs &A, uint32_t t0, uint32_t cur, uint32_t t1,
                                                 const uint32_t *s_keys, uint32_t pre, uint32_t *s_new,
                                                 uint32_t *s_table, uint8_t *s_map, RoundState &st) {
    static_assert(8 * kRoundSlots <= 64 * 48, "the table fits the shaded vertices' space");
    const uint32_t lane = lane_id();
    uint32_t my_id = kEmpty, my_intro = kEmpty, fill = 0, done = 0;
    f4 va = {}, vb = {};
    uint32_t *s_first = s_table + kRoundSlots;
#pragma unroll
    for (uint32_t q = 0; q < 2 * kRoundSlots / 256; ++q)
        ((uint4 *)s_table)[q * kWave + lane] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    wave_sync_lds();
    for (;;) {
        const uint32_t gt = min(21u, t1 - cur);
        const uint32_t nc = 3 * gt;
        const bool act = lane < nc;
        const uint32_t pos = __umul24(3u, cur - t0) + lane;   // cur - t0 < 2^24 (a batch)
        const uint32_t k = act ? (pos < pre ? s_keys[pos] : fetch_index(A, 3ull * cur + lane)) : kEmpty;
        uint32_t at = hash_slot(k, kRoundBits);
        for (bool todo = act; todo;) {   // linear probing; the table is at most half full
            const uint32_t prev = atomicCAS(&s_table[at], kEmpty, k);
            todo = prev != kEmpty && prev != k;
            if (todo) at = (at + 1) & (kRoundSlots - 1);
        }
        const uint32_t mine = done + lane;   // position in the round
        if (act) atomicMin(&s_first[at], mine);
        wave_sync_lds();
        const bool first = act && s_first[at] == mine;
        // first occurrences of indices no lane owns yet
        const uint64_t fresh = ballot(first);
        const uint32_t next = fill + __builtin_amdgcn_mbcnt_hi((uint32_t)(fresh >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)fresh, 0u));
        wave_sync_lds();
        if (first) {
            s_first[at] = next;
            if (next < (uint32_t)kWave) {
                s_new[next] = k;
                s_new[kWave + next] = mine;
            }
        }
        wave_sync_lds();
        const uint32_t slot = act ? s_first[at] : 0u;
        const uint32_t f = fill + (uint32_t)__popcll(fresh);
        if (lane >= fill && lane < f) {
            my_id = s_new[lane];
            my_intro = s_new[kWave + lane];
            if (s_map) {   // the output sweep: the load overlaps the rest of the round
                va = A.vtx[2ull * my_id];
                vb = A.vtx[2ull * my_id + 1];
            }
        }
        const uint64_t bad = ballot(act && slot >= (uint32_t)kWave);
        const uint32_t acc = bad ? ((uint32_t)__ffsll((long long)bad) - 1) / 3 : gt;
        if (s_map && lane < 3 * acc) s_map[done + lane] = (uint8_t)slot;
        done += 3 * acc;
        cur += acc;
        if (bad) {
            const uint64_t keep = ballot(my_intro < done);
            fill = (uint32_t)__popcll(keep);
            if (!((keep >> lane) & 1ull)) my_id = kEmpty;
            break;
        }
        fill = f;
        if (cur >= t1) break;
    }
    st.my_id = my_id;
    st.fill = fill;
    st.va = va;
    st.vb = vb;
    return cur;
}

// One batch processed by one wavefront in its private LDS area of
// ballot_lds_bytes(batch_tris) bytes.  The batch's indices are loaded once,
// up front; only wavefront-level synchronisation is used, so several
// wavefronts of a workgroup can work on different batches.
template <int KIND, int OUT, bool FEW>
__device__ __forceinline__ void ballot_batch(const DrawArgs &A, const vr_shader_params &sh, uint32_t b, uint32_t nb,
                                             unsigned char *lds, unsigned long long *agg_out) {
    const uint32_t lane = lane_id();
    uint32_t t0, t1;
    batch_range(A, b, t0, t1);
    if (t1 < t0 || 3 * (t1 - t0) > A.max_idx) {   // only with a plan built for other limits
        if (lane == 0) raise_error(A.err, VR_ERR_CAPACITY);
        t1 = t0;
    }
    const uint32_t cap = A.max_idx < kBallotPrefetch ? A.max_idx : kBallotPrefetch;
    f4 *s_sv = (f4 *)lds;
    uint32_t *s_keys = (uint32_t *)(lds + 64 * 48);
    uint32_t *s_new = s_keys + cap;
    uint8_t *s_map = (uint8_t *)(s_new + 2 * kWave);
    const uint32_t pre = min(3 * (t1 - t0), cap);
    load_indices<kWave>(A, 3ull * t0, pre, s_keys, lane);
    wave_sync_lds();
    uint32_t vbase = 0, ubase = b;
    RoundState st;
    if (OUT == kAll && A.need_prefix) {
        // counting sweep: the batch's rounds and invocations, published
        // before any output so later batches can resolve their prefix
        uint32_t rounds = 0, inv = 0;
        for (uint32_t cur = t0; cur < t1; ++rounds) {
            cur = ballot_round(A, t0, cur, t1, s_keys, pre, s_new, (uint32_t *)s_sv, nullptr, st);
            inv += st.fill;
        }
        const uint64_t agg = ((uint64_t)rounds << 32) | inv;
        if (lane == 0) lookback_publish(A.status, b, agg);
        const uint64_t ex = lookback_resolve(A.status, b, agg, A.err);
        vbase = __builtin_amdgcn_readfirstlane((uint32_t)ex);
        ubase = __builtin_amdgcn_readfirstlane((uint32_t)((ex >> 32) & 0x3FFFFFFFu));
    }
    uint32_t r = 0, inv = 0, seen = 0;
    for (uint32_t cur = t0; cur < t1; ++r) {
        const uint32_t end = ballot_round(A, t0, cur, t1, s_keys, pre, s_new, (uint32_t *)s_sv, s_map, st);
        if (lane < st.fill) shade_raw_to_lds<KIND>(sh, st.va, st.vb, s_sv + 3 * lane);
        wave_sync_lds();
        if (OUT == kRecords) seen += setup_unit<64>(A.setup, cur, end - cur, s_map, s_sv, lane);
        write_unit<64, OUT>(A, cur, end - cur, s_map, s_sv, st.fill, vbase, ubase + r, lane);
        wave_sync_lds();
        vbase += st.fill;
        inv += st.fill;
        cur = end;
    }
    if (OUT == kRecords) {
        if (lane == 0) setup_totals(A.setup, b, seen, inv);
        return;
    }
    if (OUT == kAll && A.unit_offsets && b + 1 == nb && lane == 0) A.unit_offsets[ubase + r] = A.T;
    if (lane == 0) {
        if (FEW && A.arrivals) batch_done<OUT == kAll>(A, b, r, inv);
        else if (b < A.status_cap) agg_out[b] = ((unsigned long long)r << 32) | inv;   // no room past the bound
    }
}

// Two wavefronts per workgroup, one batch each (batch 2 * workgroup +
// wavefront); `stride` is the per-wavefront LDS area.  Two measured faster
// than four and eight, and about as fast as one.
constexpr uint32_t kBallotWaves = 2;

template <int KIND, int OUT>
__global__ __launch_bounds__(kBallotWaves * 64) void k_ballot(DrawArgs A, vr_shader_params sh, uint32_t stride) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    clear_counters(A);
    const uint32_t nb = launch_units(A, batch_count(A));
    const uint32_t w = threadIdx.x / kWave;
    // in dispatch order where batches wait for their predecessors; a dynamic
    // launch has more workgroups than there are batches, or fewer (a plan built
    // for other limits: the launch covers the draw's bound)
    const uint32_t pieces = (min(nb, A.status_cap) + kBallotWaves - 1) / kBallotWaves;
    if (blockIdx.x >= pieces) return;
    const uint32_t b = (A.need_prefix ? blockIdx.x : xcd_piece(blockIdx.x, pieces)) * kBallotWaves + w;
    if (b >= nb) return;   // only wavefront-level synchronisation follows
    ballot_batch<KIND, OUT, true>(A, sh, b, nb, smem + w * stride, A.agg);
}

}  // namespace vr
