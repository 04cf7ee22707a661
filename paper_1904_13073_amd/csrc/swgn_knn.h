// Nearest nodes of the points of a wave, for the skinning of surfels (setup.hip)
// and of append candidates (append.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "swgn_impl.h"

namespace swgn {

// ---------------------------------------------------------------------------
// Nearest nodes. Key ((dx*dx + dy*dy) + dz*dz), dx = x_query - x_node; the 4
// nearest are the 4 smallest (key, caller index) pairs, which is what a scan
// in ascending caller index that admits a candidate only strictly below the
// current fourth key gives. Here the nodes are scanned in the library's
// (Morton) order with candidates ordered by (key, caller index), so the
// result is the same whatever the order, and whole runs of 32 nodes are
// skipped when no lane of the wave can admit any of them: the wave first
// takes the runs whose bounding box meets its surfels' box (else the nearest
// one), then skips every other run whose box distance, less a margin above
// FP32 rounding, exceeds every lane's current fourth key (a candidate enters
// only at or below it).
// A non-finite position enters no list (its keys are NaN or infinite).
// ---------------------------------------------------------------------------
constexpr int kKnnRun = 32;             // nodes per bounding box
inline size_t knn_box_count(int nn) { return 2 * (size_t)((nn + kKnnRun - 1) / kKnnRun); }   // float4s
// boxes of the runs of nodes[nn]
void launch_node_boxes(int nn, const float4* nodes, float4* boxes, hipStream_t st);

__device__ __forceinline__ float wave_minf(float v) {
    v = fminf(v, xchg<32>(v)); v = fminf(v, xchg<16>(v)); v = fminf(v, xchg<8>(v));
    v = fminf(v, xchg<4>(v)); v = fminf(v, xchg<2>(v)); v = fminf(v, xchg<1>(v));
    return v;
}
__device__ __forceinline__ float wave_maxf(float v) {
    v = fmaxf(v, xchg<32>(v)); v = fmaxf(v, xchg<16>(v)); v = fmaxf(v, xchg<8>(v));
    v = fmaxf(v, xchg<4>(v)); v = fmaxf(v, xchg<2>(v)); v = fmaxf(v, xchg<1>(v));
    return v;
}

// A lower bound of every key between the wave's box (lo, hi) and a node box:
// each point pair is at least the boxes' gap apart per axis; the computed key
// is within 5 roundings of the exact sum of squares and so is this bound, so
// shrinking it by 2^-20 (and 1e-30 for tiny values) keeps it below every key.
__device__ __forceinline__ float box_key_bound(float3 lo, float3 hi, float4 blo, float4 bhi) {
    const float gx = fmaxf(fmaxf(lo.x - bhi.x, blo.x - hi.x), 0.f);
    const float gy = fmaxf(fmaxf(lo.y - bhi.y, blo.y - hi.y), 0.f);
    const float gz = fmaxf(fmaxf(lo.z - bhi.z, blo.z - hi.z), 0.f);
    const float d2 = (gx * gx + gy * gy) + gz * gz;
    return d2 * (1.0f - 0x1p-20f) - 1e-30f;
}

// A candidate as one 64-bit word, (key bits, index): keys are >= +0 or +inf
// or NaN, whose bit patterns order as the values do and sort NaN last, so
// comparing words compares (key, index) pairs, ties to the lower index.
__device__ __forceinline__ uint64_t knn_word(float key, int j) {
    return ((uint64_t)__float_as_uint(key) << 32) | (uint32_t)j;
}

// A word into the 4 smallest kept ascending, by selects only (the list stays
// in registers): the words below it stay, it takes the first place above
// them, the rest move down one.
__device__ __forceinline__ void admit4(uint64_t (&kk)[4], uint64_t c) {
    if (c >= kk[3]) return;
    const bool c0 = c < kk[0], c1 = c < kk[1], c2 = c < kk[2];
    kk[3] = c2 ? kk[2] : c;
    kk[2] = c1 ? kk[1] : (c2 ? c : kk[2]);
    kk[1] = c0 ? kk[0] : (c1 ? c : kk[1]);
    kk[0] = c0 ? c : kk[0];
}

// The nodes of run q (uniform over the wave) as candidates of every lane.
__device__ __forceinline__ void admit_run(uint64_t (&kk)[4], float x, float y, float z, int nn, int q,
                                          const float4* __restrict__ nodes, const int* __restrict__ caller) {
    const int t0 = q * kKnnRun, t1 = min(nn, t0 + kKnnRun);
#pragma unroll 8
    for (int t = t0; t < t1; ++t) {
        const float4 p = nodes[t];
        const float dx = x - p.x, dy = y - p.y, dz = z - p.z;
        admit4(kk, knn_word((dx * dx + dy * dy) + dz * dz, caller[t]));
    }
}

__device__ __forceinline__ float worst_key(const uint64_t (&kk)[4], bool fin) {
    return wave_maxf(fin ? __uint_as_float((uint32_t)(kk[3] >> 32)) : -INFINITY);
}

// A wave tests 64 boxes at a time, one per lane, and visits the runs that are
// left in a bit mask; the nodes come by scalar loads, for a run is the same for
// all lanes. (One box after the other by the whole wave, twice, and the nodes
// staged in LDS: 98 us for 248k surfels and 1,788 nodes, 70 us so.)
// Words of the 4 nearest of nodes[nn] (numbered by caller[]) of every lane's
// point, nearest first; (INFINITY, 0) where there is none. Lanes without fin take part with
// no point of their own. All lanes of the wave call this.
__device__ __forceinline__ void nearest4(uint64_t (&kk)[4], float x, float y, float z, bool fin, int nn,
                                         const float4* __restrict__ nodes, const int* __restrict__ caller,
                                         const float4* __restrict__ boxes) {
    const int lane = threadIdx.x % kWave;
    // (INFINITY, 0) admits no infinite key
#pragma unroll
    for (int q = 0; q < 4; ++q) kk[q] = knn_word(INFINITY, 0);
    if (!__any(fin)) return;
    // the box of the wave's finite surfels (empty: every run is skipped)
    const float3 lo = make_float3(wave_minf(fin ? x : INFINITY), wave_minf(fin ? y : INFINITY),
                                  wave_minf(fin ? z : INFINITY));
    const float3 hi = make_float3(wave_maxf(fin ? x : -INFINITY), wave_maxf(fin ? y : -INFINITY),
                                  wave_maxf(fin ? z : -INFINITY));
    const int nruns = (nn + kKnnRun - 1) / kKnnRun;
    auto bound = [&](int q) {                // (past the last run, and of an empty run: none)
        return q < nruns ? box_key_bound(lo, hi, boxes[2 * q], boxes[2 * q + 1]) : INFINITY;
    };
    // first the runs whose box meets the wave's, or else the nearest one
    bool met = false;
    float least = INFINITY;
    int seed = 0;
    for (int q0 = 0; q0 < nruns; q0 += kWave) {
        const float b = bound(q0 + lane);
        unsigned long long todo = __ballot(b <= 0.f);
        met = met || todo != 0;
        for (; todo; todo &= todo - 1) admit_run(kk, x, y, z, nn, q0 + __builtin_ctzll(todo), nodes, caller);
        const float m = -wave_maxf(-b);
        if (m < least) {
            least = m;
            seed = q0 + __builtin_ctzll(__ballot(b == m));
        }
    }
    if (met) seed = -1;
    else admit_run(kk, x, y, z, nn, __builtin_amdgcn_readfirstlane(seed), nodes, caller);
    // then every run within the lanes' fourth keys (a candidate enters only at or below it)
    float worst = worst_key(kk, fin);
    for (int q0 = 0; q0 < nruns; q0 += kWave) {
        const float b = bound(q0 + lane);
        const bool open = b > 0.f && q0 + lane < nruns && q0 + lane != seed;
        for (unsigned long long todo = __ballot(open && b <= worst); todo;) {
            const int l = __builtin_ctzll(todo);
            admit_run(kk, x, y, z, nn, q0 + l, nodes, caller);
            worst = worst_key(kk, fin);
            todo &= todo - 1;
            todo &= __ballot(open && b <= worst);
        }
    }
}

}  // namespace swgn
