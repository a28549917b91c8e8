// Triangle setup: the stage that consumes the geometry stage's output in a
// streaming pipeline (Section 4.2).  Runs inside the draw kernels of a stream
// on a unit's shaded vertices while they are in LDS, beside the writing of its
// corners: perspective divide, viewport mapping, {xmin, ymin, xmax, ymax} and
// {area, flags, 0, 0} as two float4 per triangle.  A chunk is then one launch,
// and latency, not traffic, bounds a chunk: with a kernel, a reduction and a
// consumer on a second HIP stream per chunk, ordered by events, 20 chunks of
// 65,536 triangles (ballot, Phong-8) took 812 us, so 310 us (400 before the rounds
// of k_ballot got shorter).
#pragma once

#include "vr_device.h"

namespace vr {

typedef float f4 __attribute__((ext_vector_type(4)));

// Totals are spread over kSpread rows, 64 B apart, so that workgroups do not
// queue at one address (same-address atomics take about 20 ns each).
constexpr uint32_t kSpread = 64, kSpreadWords = 8;

// Where a stream's draws put their records.
struct SetupTarget {
    f4 *records;                        // of the chunk's first triangle
    uint32_t width, height;
    unsigned long long *totals;         // [kSpread][kSpreadWords]: visible, invocations
    unsigned long long *invocations;    // [kSpread][kSpreadWords]: the context's
};

// One triangle from the clip-space rows of its corners; returns visibility.
__device__ __forceinline__ bool setup_triangle(const SetupTarget &S, const f4 (&c)[3], uint32_t t) {
    const float hw = 0.5f * (float)S.width, hh = 0.5f * (float)S.height;
    float sx[3], sy[3];
    bool front = true, vis = false;
#pragma unroll
    for (uint32_t k = 0; k < 3; ++k) {
        front = front && c[k].w > 0.0f;
        sx[k] = (c[k].x / c[k].w + 1.0f) * hw;
        sy[k] = (c[k].y / c[k].w + 1.0f) * hh;
    }
    f4 box = {0.0f, 0.0f, 0.0f, 0.0f}, rest = {0.0f, 0.0f, 0.0f, 0.0f};
    if (front) {
        const float area = (sx[1] - sx[0]) * (sy[2] - sy[0]) - (sx[2] - sx[0]) * (sy[1] - sy[0]);
        const float x0 = fmaxf(fminf(fminf(sx[0], sx[1]), sx[2]), 0.0f);
        const float x1 = fminf(fmaxf(fmaxf(sx[0], sx[1]), sx[2]), (float)S.width);
        const float y0 = fmaxf(fminf(fminf(sy[0], sy[1]), sy[2]), 0.0f);
        const float y1 = fminf(fmaxf(fmaxf(sy[0], sy[1]), sy[2]), (float)S.height);
        vis = area > 0.0f && x0 < x1 && y0 < y1;
        box = f4{x0, y0, x1, y1};
        rest = f4{area, __uint_as_float(vis ? 1u : 0u), 0.0f, 0.0f};
    }
    S.records[2ull * t] = box;
    S.records[2ull * t + 1] = rest;
    return vis;
}

// Triangles [t0, t0 + ntri) by NT threads, corner k's shaded vertex being
// s_sv[3 * s_local[k]] (row 0: clip x, y, z, w).  Returns the number of
// visible triangles this wavefront saw.
template <int NT, typename LocalT>
__device__ __forceinline__ uint32_t setup_unit(const SetupTarget &S, uint32_t t0, uint32_t ntri, const LocalT *s_local,
                                               const f4 *s_sv, uint32_t tid) {
    uint32_t seen = 0;
    for (uint32_t b = 0; b < ntri; b += NT) {
        const uint32_t t = b + tid;
        bool vis = false;
        if (t < ntri) {
            const f4 c[3] = {s_sv[3 * (uint32_t)s_local[3 * t]], s_sv[3 * (uint32_t)s_local[3 * t + 1]],
                             s_sv[3 * (uint32_t)s_local[3 * t + 2]]};
            vis = setup_triangle(S, c, t0 + t);
        }
        seen += (uint32_t)__popcll(ballot(vis));
    }
    return seen;
}

// Adds to the totals of workgroup (or wavefront) `who`; called by one lane.
__device__ __forceinline__ void setup_totals(const SetupTarget &S, uint32_t who, uint32_t visible, uint32_t inv) {
    const uint32_t row = who % kSpread * kSpreadWords;
    if (visible) atomicAdd(&S.totals[row], (unsigned long long)visible);
    if (inv) {
        atomicAdd(&S.totals[row + 1], (unsigned long long)inv);
        atomicAdd(&S.invocations[row], (unsigned long long)inv);
    }
}

}  // namespace vr
