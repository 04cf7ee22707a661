// Setup kernels, run once per node set (Sec. 6.5, Initialization): skinning of
// every surfel to its nearest nodes, the node graph, and the block pattern of
// J^T J with the per-block lists the assembly walks.
//
// Every integer result is deterministic: nearest-node order is decided by an
// FP32 key with a fixed operation order and ties to the lower index; sorts
// compare full (key, value) pairs that are unique; the atomics are integer OR /
// ADD whose results do not depend on order, or give places that are put in
// order afterwards.
#include "swgn_frame.h"
#include "swgn_impl.h"
#include "swgn_knn.h"
#include "swgn_launch.h"
#include "swgn_setup.h"

namespace swgn {

// ---------------------------------------------------------------------------
// Skinning: the 4 nearest nodes of every surfel and their weights.
// ---------------------------------------------------------------------------
__global__ void k_node_boxes(int nn, const float4* __restrict__ nodes, float4* __restrict__ boxes) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q * kKnnRun >= nn) return;
    float3 lo = make_float3(INFINITY, INFINITY, INFINITY), hi = make_float3(-INFINITY, -INFINITY, -INFINITY);
    for (int t = q * kKnnRun; t < min(nn, (q + 1) * kKnnRun); ++t) {
        const float4 p = nodes[t];
        lo.x = fminf(lo.x, p.x); lo.y = fminf(lo.y, p.y); lo.z = fminf(lo.z, p.z);
        hi.x = fmaxf(hi.x, p.x); hi.y = fmaxf(hi.y, p.y); hi.z = fmaxf(hi.z, p.z);
    }
    boxes[2 * q] = make_float4(lo.x, lo.y, lo.z, 0.f);
    boxes[2 * q + 1] = make_float4(hi.x, hi.y, hi.z, 0.f);
}

__global__ void __launch_bounds__(256) k_knn_skin(int ns, const float* __restrict__ pos, int nn,
        const float4* __restrict__ nodes, const int* __restrict__ caller, const float4* __restrict__ boxes,
        float inv_two_sigma2, int4* __restrict__ out_idx, float4* __restrict__ out_w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    float x = 0.f, y = 0.f, z = 0.f;
    if (i < ns) { x = pos[3 * i]; y = pos[3 * i + 1]; z = pos[3 * i + 2]; }
    uint64_t kk[4];
    nearest4(kk, x, y, z, i < ns && isfinite(x) && isfinite(y) && isfinite(z), nn, nodes, caller, boxes);
    float kd[4];
    int ki[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        kd[q] = __uint_as_float((uint32_t)(kk[q] >> 32));
        ki[q] = (int)(uint32_t)kk[q];
    }
    if (i >= ns) return;
    // weights exp(-(d_k^2 - d_0^2) / (2 sigma^2)), normalised
    float e0 = 1.0f;
    float e1 = expf(-(kd[1] - kd[0]) * inv_two_sigma2);
    float e2 = expf(-(kd[2] - kd[0]) * inv_two_sigma2);
    float e3 = expf(-(kd[3] - kd[0]) * inv_two_sigma2);
    float inv = 1.0f / (((e0 + e1) + e2) + e3);
    out_idx[i] = make_int4(ki[0], ki[1], ki[2], ki[3]);
    out_w[i] = make_float4(e0 * inv, e1 * inv, e2 * inv, e3 * inv);
}

// One wave per node j: lane l keeps the 8 nearest of the nodes l, l + 64, ...
// (ascending index, so equal keys keep the lower index first), then the wave
// merges its 64 sorted lists by taking, 8 times, the smallest (key, index)
// head: the same set and order as one sequential scan. A node with fewer than
// 8 others at a finite distance sets *lone (and lists node 0 in their place).
constexpr int kGraphNodesPerBlock = 4;

__global__ void __launch_bounds__(64 * kGraphNodesPerBlock) k_node_graph(int nn, const float4* __restrict__ nodes,
                                                                         int* __restrict__ nbr,
                                                                         int* __restrict__ lone) {
    const int lane = threadIdx.x % kWave;
    const int j = blockIdx.x * kGraphNodesPerBlock + threadIdx.x / kWave;
    if (j >= nn) return;                     // whole waves: no barrier follows
    const float4 me = nodes[j];
    float kd[8];
    int ki[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) { kd[q] = INFINITY; ki[q] = 0x7fffffff; }
    for (int t = lane; t < nn; t += kWave) {
        if (t == j) continue;
        const float4 p = nodes[t];
        const float dx = me.x - p.x, dy = me.y - p.y, dz = me.z - p.z;
        knn_insert<8>(kd, ki, (dx * dx + dy * dy) + dz * dz, t);
    }
    int out = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        float bk = kd[0];
        int bi = ki[0];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ok = __shfl_xor(bk, o, kWave);
            const int oi = __shfl_xor(bi, o, kWave);
            if (ok < bk || (ok == bk && oi < bi)) { bk = ok; bi = oi; }
        }
        if (lane == r) out = bi;
        if (ki[0] == bi) {                   // this lane's head was taken: shift its list
#pragma unroll
            for (int q = 0; q < 7; ++q) { kd[q] = kd[q + 1]; ki[q] = ki[q + 1]; }
            kd[7] = INFINITY;
            ki[7] = 0x7fffffff;
        }
    }
    if (lane < 8) {
        const bool none = out == 0x7fffffff;
        if (none) *lone = 1;
        nbr[8 * j + lane] = none ? 0 : out;
    }
}

// ---------------------------------------------------------------------------
// Bitonic sort of (u64 key, u32 val) pairs, ascending in (key, val).
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool pair_less(uint64_t ka, uint32_t va, uint64_t kb, uint32_t vb) {
    return ka < kb || (ka == kb && va < vb);
}

// S consecutive stages j, j/2, ..., j/2^(S-1) of block size k in one pass:
// each thread holds the 2^S elements whose indices differ only in those S
// bits (all in one k-block, so one direction) and applies the stages to them
// in order, as the one-stage passes would.
template <int S>
__global__ void k_bitonic_global(uint64_t* __restrict__ key, uint32_t* __restrict__ val, int n, int k, int jlow) {
    constexpr int E = 1 << S;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (n >> S)) return;
    // insert S zero bits at the stage bits (jlow is the lowest stage)
    const int a = ((t & ~(jlow - 1)) << S) | (t & (jlow - 1));
    const bool asc = (a & k) == 0;
    uint64_t kk[E];
    uint32_t vv[E];
#pragma unroll
    for (int m = 0; m < E; ++m) {
        kk[m] = key[a + m * jlow];
        vv[m] = val[a + m * jlow];
    }
#pragma unroll
    for (int st = S - 1; st >= 0; --st) {
        const int d = 1 << st;              // partner offset in units of jlow
#pragma unroll
        for (int m = 0; m < E; ++m) {
            if (m & d) continue;
            const uint64_t ka = kk[m], kb = kk[m | d];
            const uint32_t va = vv[m], vb = vv[m | d];
            const bool sw = asc ? pair_less(kb, vb, ka, va) : pair_less(ka, va, kb, vb);
            kk[m] = sw ? kb : ka; kk[m | d] = sw ? ka : kb;
            vv[m] = sw ? vb : va; vv[m | d] = sw ? va : vb;
        }
    }
#pragma unroll
    for (int m = 0; m < E; ++m) {
        key[a + m * jlow] = kk[m];
        val[a + m * jlow] = vv[m];
    }
}

constexpr int kSortLds = 1024;  // elements per block in the LDS stages

// All stages with j < kSortLds for a given k (and, when k <= kSortLds, all k
// up to it) on one 1024-element slice held in LDS, 512 threads.
static_assert(kSortLds == 2 * 512, "one compare-exchange per thread and stage");
__global__ void __launch_bounds__(512) k_bitonic_lds(uint64_t* __restrict__ key,
        uint32_t* __restrict__ val, int n, int k_from, int k_to) {
    __shared__ uint64_t sk[kSortLds];
    __shared__ uint32_t sv[kSortLds];
    int base = blockIdx.x * kSortLds;
    for (int t = threadIdx.x; t < kSortLds; t += blockDim.x) {
        sk[t] = key[base + t];
        sv[t] = val[base + t];
    }
    __syncthreads();
    for (int k = k_from; k <= k_to; k <<= 1) {
        int jstart = min(k >> 1, kSortLds >> 1);
        for (int j = jstart; j > 0; j >>= 1) {
            // one pair per thread: the lower index has a 0 at bit j
            const int q = threadIdx.x;
            const int t = ((q & ~(j - 1)) << 1) | (q & (j - 1)), p = t + j;
            const bool asc = ((base + t) & k) == 0;
            const uint64_t ka = sk[t], kb = sk[p];
            const uint32_t va = sv[t], vb = sv[p];
            const bool sw = asc ? pair_less(kb, vb, ka, va) : pair_less(ka, va, kb, vb);
            if (sw) { sk[t] = kb; sk[p] = ka; sv[t] = vb; sv[p] = va; }
            __syncthreads();
        }
    }
    for (int t = threadIdx.x; t < kSortLds; t += blockDim.x) {
        key[base + t] = sk[t];
        val[base + t] = sv[t];
    }
}

void sort_pairs(uint64_t* key, uint32_t* val, int n_pow2, hipStream_t st) {
    // n_pow2 is a power of two >= kSortLds
    int blocks = n_pow2 / kSortLds;
    hipLaunchKernelGGL(k_bitonic_lds, dim3(blocks), dim3(512), 0, st, key, val, n_pow2, 2, kSortLds);
    for (int k = 2 * kSortLds; k <= n_pow2; k <<= 1) {
        // the stages j >= kSortLds, up to three per pass
        for (int j = k >> 1; j >= kSortLds;) {
            if (j >= 4 * kSortLds) {
                hipLaunchKernelGGL(k_bitonic_global<3>, dim3((n_pow2 / 8 + 255) / 256), dim3(256), 0, st,
                                   key, val, n_pow2, k, j / 4);
                j /= 8;
            } else if (j >= 2 * kSortLds) {
                hipLaunchKernelGGL(k_bitonic_global<2>, dim3((n_pow2 / 4 + 255) / 256), dim3(256), 0, st,
                                   key, val, n_pow2, k, j / 2);
                j /= 4;
            } else {
                hipLaunchKernelGGL(k_bitonic_global<1>, dim3((n_pow2 / 2 + 255) / 256), dim3(256), 0, st,
                                   key, val, n_pow2, k, j);
                j /= 2;
            }
        }
        hipLaunchKernelGGL(k_bitonic_lds, dim3(blocks), dim3(512), 0, st, key, val, n_pow2, k, k);
    }
}

// ---------------------------------------------------------------------------
// Exclusive scan of int32 (n elements -> out[0..n], out[n] = total): tiles of
// 4,096 elements scanned by themselves, then every tile adds the sum of the
// tiles before it, which it forms itself from their totals (up to
// kScanFlat tiles; beyond, the totals are scanned the same way). Setup is bound by
// the number of its launches: one or two here (tiles of 1,024, a scan of their
// totals and a launch for the total: five).
// ---------------------------------------------------------------------------
constexpr int kScanBlock = 1024, kScanItems = 4, kScanTile = kScanBlock * kScanItems;
constexpr int kScanFlat = 256;

// Exclusive prefix of v over the 1024 threads of a workgroup; total = the sum.
__device__ __forceinline__ int block_prefix(int v, int* sh, int& total) {
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    __syncthreads();                         // (sh may still be read from the last call)
    if (lane == kWave - 1) sh[wave] = inc;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / kWave; ++w) {
        const int t = sh[w];
        if (w < wave) before += t;
        total += t;
    }
    return before + inc - v;
}

// (blockIdx.y: one of up to two arrays of the same length)
struct ScanArrays {
    const int* in[2];
    int *out[2], *sums[2];
};

__global__ void __launch_bounds__(kScanBlock) k_scan_tiles(ScanArrays a, int n) {
    __shared__ int sh[kScanBlock / kWave];
    const int* in = a.in[blockIdx.y];
    int *out = a.out[blockIdx.y], *sums = a.sums[blockIdx.y];
    const int64_t i = ((int64_t)blockIdx.x * kScanBlock + threadIdx.x) * kScanItems;
    int v[kScanItems], own = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        v[q] = i + q < n ? in[i + q] : 0;
        own += v[q];
    }
    int total;
    int run = block_prefix(own, sh, total);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        if (i + q < n) out[i + q] = run;
        run += v[q];
    }
    if (threadIdx.x == 0) {
        if (gridDim.x == 1) out[n] = total;
        else sums[blockIdx.x] = total;
    }
}

// sums: the tiles' totals, or (scanned) their exclusive scan
__global__ void __launch_bounds__(kScanBlock) k_scan_add(ScanArrays a, int scanned, int n) {
    __shared__ int sh[kScanBlock / kWave];
    int* out = a.out[blockIdx.y];
    const int* sums = a.sums[blockIdx.y];
    const int b = blockIdx.x;
    int before = 0;
    if (scanned) {
        before = sums[b];
        if (b == (int)gridDim.x - 1 && threadIdx.x == 0) out[n] = sums[b + 1];
    } else {
        int own = 0;
        for (int q = threadIdx.x; q < b; q += kScanBlock) own += sums[q];
        block_prefix(own, sh, before);
        if (b == (int)gridDim.x - 1 && threadIdx.x == 0) out[n] = before + sums[b];
    }
    const int64_t i = ((int64_t)b * kScanBlock + threadIdx.x) * kScanItems;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q)
        if (i + q < n) out[i + q] += before;
}

static void scan_arrays(ScanArrays a, int arrays, int n, int* tmp, hipStream_t st) {
    const int nb = n > 0 ? (int)(((int64_t)n + kScanTile - 1) / kScanTile) : 1;
    for (int q = 0; q < arrays; ++q) a.sums[q] = tmp + (size_t)q * nb;
    hipLaunchKernelGGL(k_scan_tiles, dim3(nb, arrays), dim3(kScanBlock), 0, st, a, n);
    if (nb == 1) return;
    tmp += (size_t)arrays * nb;
    if (nb <= kScanFlat) {
        hipLaunchKernelGGL(k_scan_add, dim3(nb, arrays), dim3(kScanBlock), 0, st, a, 0, n);
        return;
    }
    ScanArrays t{};
    for (int q = 0; q < arrays; ++q) {
        t.in[q] = a.sums[q];
        a.sums[q] = t.out[q] = tmp + (size_t)q * (nb + 1);
    }
    scan_arrays(t, arrays, nb, tmp + (size_t)arrays * (nb + 1), st);
    hipLaunchKernelGGL(k_scan_add, dim3(nb, arrays), dim3(kScanBlock), 0, st, a, 1, n);
}

void exclusive_scan(const int* in, int* out, int n, int* tmp, hipStream_t st) {
    scan_arrays(ScanArrays{{in, nullptr}, {out, nullptr}, {nullptr, nullptr}}, 1, n, tmp, st);
}

void exclusive_scan2(const int* in0, int* out0, const int* in1, int* out1, int n, int* tmp, hipStream_t st) {
    scan_arrays(ScanArrays{{in0, in1}, {out0, out1}, {nullptr, nullptr}}, 2, n, tmp, st);
}

// (for one array; twice that for two)
size_t scan_tmp_size(int n) {
    size_t total = 0;
    while (n > kScanTile) {
        const int nb = (int)(((int64_t)n + kScanTile - 1) / kScanTile);
        total += 2 * (size_t)nb + 1;
        n = nb;
    }
    return total + 4;
}

// ---------------------------------------------------------------------------
// Surfel ordering by node set
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sort4(int& a, int& b, int& c, int& d) {
    int t;
#define SWGN_CS(p, q) if (p > q) { t = p; p = q; q = t; }
    SWGN_CS(a, b) SWGN_CS(c, d) SWGN_CS(a, c) SWGN_CS(b, d) SWGN_CS(b, c)
#undef SWGN_CS
}

__global__ void k_tuple_keys(int ns, int npad, const int4* __restrict__ idx, uint64_t* __restrict__ key,
                             uint32_t* __restrict__ val) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npad) return;
    if (i >= ns) {
        key[i] = ~0ull;
        val[i] = 0xffffffffu;
        return;
    }
    int4 q = idx[i];
    int a = q.x, b = q.y, c = q.z, d = q.w;
    sort4(a, b, c, d);
    key[i] = ((uint64_t)a << 48) | ((uint64_t)b << 32) | ((uint64_t)c << 16) | (uint64_t)d;
    val[i] = (uint32_t)i;
}

// Surfels by node set without a sort over all of them: a bucket per value of
// the leading bits of the four ascending node numbers (kBucketBits of them, no
// gaps between the numbers' bits), a place in the bucket from an atomic
// counter (any order will do), then each bucket sorted on chip by (key, surfel).
// Pairs are unique, so the result is the sort's. A bucket of more than
// kBucketCap surfels sets *over; the host then runs the bitonic sort
// instead, which takes any distribution (248k surfels, 1,788 nodes: 5 launches,
// 53 us of the device, against 27 launches and 190 us).
constexpr int kBucketBits = 13, kBucketCap = 2048, kBucketBlock = 256;

struct BucketOf {
    int bits, shift;                         // of a node number; of the joined numbers to the bucket
};

static BucketOf bucket_of(int nn) {
    int w = 1;
    while ((1 << w) < nn) ++w;
    return BucketOf{w, 4 * w > kBucketBits ? 4 * w - kBucketBits : 0};
}

// Renumbers the surfels' nodes (from the caller's numbering), keys, buckets
// and places. Lanes of a wave with one bucket take their places together.
__global__ void __launch_bounds__(256) k_bucket_count(int ns, int4* __restrict__ idx, const int* __restrict__ inv,
        BucketOf o, uint64_t* __restrict__ key, int* __restrict__ bucket, int* __restrict__ place,
        int* __restrict__ count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, lane = threadIdx.x % kWave;
    const bool in = i < ns;
    int b = -1;
    if (in) {
        int4 q = idx[i];
        q = make_int4(inv[q.x], inv[q.y], inv[q.z], inv[q.w]);
        idx[i] = q;
        int t0 = q.x, t1 = q.y, t2 = q.z, t3 = q.w;
        sort4(t0, t1, t2, t3);
        key[i] = ((uint64_t)t0 << 48) | ((uint64_t)t1 << 32) | ((uint64_t)t2 << 16) | (uint64_t)t3;
        const uint64_t joined = ((((uint64_t)t0 << o.bits | (uint64_t)t1) << o.bits | (uint64_t)t2) << o.bits) |
                                (uint64_t)t3;
        b = (int)(joined >> o.shift);
        bucket[i] = b;
    }
    // the first lane of each bucket speaks for it
    int first = lane, before = 0, n = 1;
    for (unsigned long long todo = __ballot(in); todo;) {
        const int l = __builtin_ctzll(todo);
        const unsigned long long same = __ballot(in && b == __builtin_amdgcn_readlane(b, l));
        if ((same >> lane) & 1ull) {
            first = l;
            before = __popcll(same & ((1ull << lane) - 1ull));
            n = __popcll(same);
        }
        todo &= ~same;
    }
    int base = 0;
    if (in && first == lane) base = atomicAdd(&count[b], n);
    base = __shfl(base, first, kWave);
    if (in) place[i] = base + before;
}

// Exclusive scan of n counts by one workgroup (start[n] = the total); *over is
// set where a count is above cap.
__global__ void __launch_bounds__(kScanBlock) k_bucket_scan(int n, const int* __restrict__ count, int cap,
                                                            int* __restrict__ start, int* __restrict__ over) {
    __shared__ int sh[kScanBlock / kWave];
    int carry = 0;
    for (int base = 0; base < n; base += kScanTile) {
        const int i = base + (int)threadIdx.x * kScanItems;
        int v[kScanItems], own = 0;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            v[q] = i + q < n ? count[i + q] : 0;
            own += v[q];
            if (v[q] > cap) *over = 1;
        }
        int total;
        int run = carry + block_prefix(own, sh, total);
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            if (i + q < n) start[i + q] = run;
            run += v[q];
        }
        carry += total;
    }
    if (threadIdx.x == 0) start[n] = carry;
}

__global__ void __launch_bounds__(256) k_bucket_scatter(int ns, const uint64_t* __restrict__ key,
        const int* __restrict__ bucket, const int* __restrict__ place, const int* __restrict__ start,
        uint64_t* __restrict__ skey, uint32_t* __restrict__ sval) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ns) return;
    const int p = start[bucket[i]] + place[i];
    skey[p] = key[i];
    sval[p] = (uint32_t)i;
}

// One workgroup per bucket: up to 256 pairs by counting the smaller ones, more
// by a bitonic sort in LDS.
__global__ void __launch_bounds__(kBucketBlock) k_bucket_sort(const int* __restrict__ start, uint64_t* __restrict__ key,
                                                              uint32_t* __restrict__ val) {
    __shared__ uint64_t sk[kBucketCap];
    __shared__ uint32_t sv[kBucketCap];
    const int s0 = start[blockIdx.x], n = start[blockIdx.x + 1] - s0, t = threadIdx.x;
    if (n <= 1 || n > kBucketCap) return;
    if (n <= kBucketBlock) {
        uint64_t k = 0;
        uint32_t v = 0;
        if (t < n) {
            k = key[s0 + t];
            v = val[s0 + t];
            sk[t] = k;
            sv[t] = v;
        }
        __syncthreads();
        if (t >= n) return;
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += pair_less(sk[j], sv[j], k, v) ? 1 : 0;
        key[s0 + rank] = k;
        val[s0 + rank] = v;
        return;
    }
    int p2 = 2 * kBucketBlock;
    while (p2 < n) p2 <<= 1;
    for (int j = t; j < p2; j += kBucketBlock) {
        sk[j] = j < n ? key[s0 + j] : ~0ull;
        sv[j] = j < n ? val[s0 + j] : 0xffffffffu;
    }
    __syncthreads();
    for (int k = 2; k <= p2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int q = t; q < p2 / 2; q += kBucketBlock) {
                const int a = ((q & ~(j - 1)) << 1) | (q & (j - 1)), b = a + j;
                const uint64_t ka = sk[a], kb = sk[b];
                const uint32_t va = sv[a], vb = sv[b];
                const bool sw = (a & k) == 0 ? pair_less(kb, vb, ka, va) : pair_less(ka, va, kb, vb);
                if (sw) { sk[a] = kb; sk[b] = ka; sv[a] = vb; sv[b] = va; }
            }
            __syncthreads();
        }
    for (int j = t; j < n; j += kBucketBlock) {
        key[s0 + j] = sk[j];
        val[s0 + j] = sv[j];
    }
}

// Gather surfel arrays into sorted order; flag run starts. Where *over is set
// (given and not zero) the keys are out of order and the whole is done again
// after another sort: nothing is gathered, and all surfels count as one run,
// for unsorted ones would be a run each, and what lists the runs' node sets
// would set the same few bits for every surfel (2M surfels, 9 nodes: 44 ms).
__global__ void k_permute_surfels(int ns, const int* __restrict__ over, const uint64_t* __restrict__ key, const uint32_t* __restrict__ val,
        const float* __restrict__ ipos, const float* __restrict__ inrm, const int4* __restrict__ iidx,
        const float4* __restrict__ iw, float* __restrict__ px, float* __restrict__ py, float* __restrict__ pz,
        float* __restrict__ nx, float* __restrict__ ny, float* __restrict__ nz, int4* __restrict__ oidx,
        float4* __restrict__ ow, int* __restrict__ orig, int* __restrict__ flag) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ns) return;
    if (over && *over != 0) {
        flag[i] = i == 0 ? 1 : 0;
        return;
    }
    int o = (int)val[i];
    px[i] = ipos[3 * o + 0]; py[i] = ipos[3 * o + 1]; pz[i] = ipos[3 * o + 2];
    nx[i] = inrm[3 * o + 0]; ny[i] = inrm[3 * o + 1]; nz[i] = inrm[3 * o + 2];
    oidx[i] = iidx[o];
    ow[i] = iw[o];
    orig[i] = o;
    // run starts: a new node set
    flag[i] = (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
}

// First surfel and node set of every run of equal node sets; pos[ns] runs.
__global__ void k_run_starts(int ns, const int* __restrict__ flag, const int* __restrict__ pos,
                             const uint64_t* __restrict__ key, int* __restrict__ run_start,
                             uint64_t* __restrict__ run_key) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ns && flag[i]) {
        run_start[pos[i]] = i;
        run_key[pos[i]] = key[i];
    }
    if (i == 0) run_start[pos[ns]] = ns;
}

// Positions (3 bits each) of surfel i's 4 nodes, in its slot order, among
// its segment's nodes; the segment is found by binary search over the
// segment starts. A node missing from the segment sets *bad.
__global__ void k_seg_pos4(int ns, int nseg, const int* __restrict__ seg_start, const int* __restrict__ seg_nodes,
                           const int4* __restrict__ idx, uint16_t* __restrict__ pos4, int* __restrict__ bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ns) return;
    int lo = 0, hi = nseg - 1;                 // largest g with seg_start[g] <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg_start[mid] <= i) lo = mid;
        else hi = mid - 1;
    }
    int nd[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) nd[q] = seg_nodes[5 * lo + q];
    const int4 t = idx[i];
    const int id[4] = {t.x, t.y, t.z, t.w};
    int code = 0;
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int p = 5;
#pragma unroll
        for (int q = 4; q >= 0; --q)
            if (nd[q] == id[k]) p = q;
        ok = ok && p < 5;
        code |= (p < 5 ? p : 0) << (3 * k);
    }
    pos4[i] = (uint16_t)code;
    if (!ok) atomicOr(bad, 1);
}

// ---------------------------------------------------------------------------
// Block pattern: a bitmap row of nn bits per node with the columns of its full
// block row, and one with the nodes whose edges end in it. Everything that
// lists them in ascending order (upper blocks, full rows, in-edges) is then a
// walk of a wave over the row's bits; sorting the transposed blocks and the
// in-edges instead took 20 launches.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void set_bit(uint32_t* bm, int words, int r, int c) {
    atomicOr(&bm[(size_t)r * words + (c >> 5)], 1u << (c & 31));
}

// The node pairs of every run's node set (its first surfel's).
__global__ void k_pattern_sets(int ns, const uint64_t* __restrict__ key, const int* __restrict__ flag,
                               uint32_t* __restrict__ bm, int words) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ns || !flag[i]) return;
    const uint64_t k = key[i];
    int t[4] = {(int)(k >> 48), (int)((k >> 32) & 0xffff), (int)((k >> 16) & 0xffff), (int)(k & 0xffff)};
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (a != b) set_bit(bm, words, t[a], t[b]);
}

// Edge e = 8 j + q of the graph: both blocks of j and its neighbour, the
// diagonal, and the neighbour's in-edge.
__global__ void k_pattern_nodes(int nn, const int* __restrict__ nbr, uint32_t* __restrict__ bm,
                                uint32_t* __restrict__ in_bm, int words) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 8 * nn) return;
    const int j = e >> 3, m = nbr[e];
    if ((e & 7) == 0) set_bit(bm, words, j, j);
    set_bit(bm, words, j, m);
    set_bit(bm, words, m, j);
    set_bit(in_bm, words, m, j);
}

constexpr int kRowBlock = 256;               // 4 rows per workgroup, one per wave

// Bits of word w at columns >= r.
__device__ __forceinline__ uint32_t from_column(uint32_t m, int w, int r) {
    return w < (r >> 5) ? 0u : (w == (r >> 5) ? m & (~0u << (r & 31)) : m);
}

// Per node: upper blocks, all blocks of its row, in-edges.
__global__ void __launch_bounds__(kRowBlock) k_row_counts(int nn, const uint32_t* __restrict__ bm,
        const uint32_t* __restrict__ in_bm, int words, int* __restrict__ upper, int* __restrict__ full,
        int* __restrict__ in_cnt) {
    const int r = blockIdx.x * (kRowBlock / kWave) + threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (r >= nn) return;
    int u = 0, f = 0, n = 0;
    for (int w = lane; w < words; w += kWave) {
        const uint32_t m = bm[(size_t)r * words + w];
        f += __popc(m);
        u += __popc(from_column(m, w, r));
        n += __popc(in_bm[(size_t)r * words + w]);
    }
    u = wave_sumi(u); f = wave_sumi(f); n = wave_sumi(n);
    if (lane == 0) { upper[r] = u; full[r] = f; in_cnt[r] = n; }
}

// One workgroup each: row_ptr and in_ptr (exclusive scans with their totals),
// the longest full row.
__global__ void __launch_bounds__(kScanBlock) k_row_scan(int nn, const int* __restrict__ upper,
        const int* __restrict__ full, const int* __restrict__ in_cnt, int* __restrict__ row_ptr,
        int* __restrict__ in_ptr, int* __restrict__ longest) {
    __shared__ int sh[kScanBlock / kWave];
    if (blockIdx.x == 2) {
        int m = 1;
        for (int k = threadIdx.x; k < nn; k += kScanBlock) m = max(m, full[k]);
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
        if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = m;
        __syncthreads();
        for (int w = 0; w < kScanBlock / kWave; ++w) m = max(m, sh[w]);
        if (threadIdx.x == 0) *longest = m;
        return;
    }
    const int* in = blockIdx.x == 0 ? upper : in_cnt;
    int* out = blockIdx.x == 0 ? row_ptr : in_ptr;
    int carry = 0;
    for (int base = 0; base < nn; base += kScanTile) {
        const int i = base + (int)threadIdx.x * kScanItems;
        int v[kScanItems], own = 0;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            v[q] = i + q < nn ? in[i + q] : 0;
            own += v[q];
        }
        int total;
        int run = carry + block_prefix(own, sh, total);
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            if (i + q < nn) out[i + q] = run;
            run += v[q];
        }
        carry += total;
    }
    if (threadIdx.x == 0) out[nn] = carry;
}

// Exclusive prefix of v over the wave, and its sum.
__device__ __forceinline__ int wave_prefix(int v, int& total) {
    const int lane = threadIdx.x % kWave;
    int inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    total = __shfl(inc, kWave - 1, kWave);
    return inc - v;
}

// Upper blocks of every row (columns, rows, the list of off-diagonal ones)
// and the in-edges, ascending.
__global__ void __launch_bounds__(kRowBlock) k_row_fill(int nn, const uint32_t* __restrict__ bm,
        const uint32_t* __restrict__ in_bm, int words, const int* __restrict__ row_ptr,
        const int* __restrict__ in_ptr, int* __restrict__ col_idx, int* __restrict__ blk_row,
        int* __restrict__ offlist, int* __restrict__ in_list) {
    const int r = blockIdx.x * (kRowBlock / kWave) + threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (r >= nn) return;
    int p0 = row_ptr[r], n0 = in_ptr[r];
    for (int w0 = 0; w0 < words; w0 += kWave) {
        const int w = w0 + lane;
        uint32_t m = w < words ? from_column(bm[(size_t)r * words + w], w, r) : 0u;
        uint32_t n = w < words ? in_bm[(size_t)r * words + w] : 0u;
        int total;
        int p = p0 + wave_prefix(__popc(m), total);
        p0 += total;
        for (; m; m &= m - 1, ++p) {
            const int c = w * 32 + __ffs(m) - 1;
            col_idx[p] = c;
            blk_row[p] = r;
            if (c != r) offlist[p - r - 1] = p;   // (the diagonal is first in each row)
        }
        p = n0 + wave_prefix(__popc(n), total);
        n0 += total;
        for (; n; n &= n - 1, ++p) in_list[p] = w * 32 + __ffs(n) - 1;
    }
}

// Full rows in ELL layout (width ell_w, left-aligned, ~0 padding): the
// transposed blocks (columns below the row, found in the column's own row),
// then the upper ones; and the slot of every block and of its transpose (-1: diagonal).
__global__ void __launch_bounds__(kRowBlock) k_ell(int nn, int ell_w, const uint32_t* __restrict__ bm, int words,
        const int* __restrict__ row_ptr, const int* __restrict__ full, const int* __restrict__ col_idx,
        uint32_t* __restrict__ ell_blk, int* __restrict__ ell_col, int* __restrict__ slot_u,
        int* __restrict__ slot_t) {
    const int r = blockIdx.x * (kRowBlock / kWave) + threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (r >= nn) return;
    const int b0 = row_ptr[r], low = full[r] - (row_ptr[r + 1] - b0);     // columns below the row
    int s0 = 0;
    for (int w0 = 0; w0 < words; w0 += kWave) {
        const int w = w0 + lane;
        uint32_t m = w < words ? bm[(size_t)r * words + w] : 0u;
        int total;
        int s = s0 + wave_prefix(__popc(m), total);
        s0 += total;
        for (; m; m &= m - 1, ++s) {
            const int c = w * 32 + __ffs(m) - 1, e = r * ell_w + s;
            int b = b0 + s - low;
            if (c < r) {
                int lo = row_ptr[c], hi = row_ptr[c + 1];
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (col_idx[mid] < r) lo = mid + 1;
                    else hi = mid;
                }
                b = lo;
                slot_t[b] = e;
            } else {
                slot_u[b] = e;
                if (c == r) slot_t[b] = -1;
            }
            ell_blk[e] = c < r ? (uint32_t)b | kTransposed : (uint32_t)b;
            ell_col[e] = c;
        }
    }
    for (int s = s0 + lane; s < ell_w; s += kWave) {
        ell_blk[(size_t)r * ell_w + s] = 0xffffffffu;
        ell_col[(size_t)r * ell_w + s] = 0;
    }
}

// The library's neighbour lists from the caller's.
__global__ void k_map_graph(int nn, const int* __restrict__ nbr_call, const int* __restrict__ perm,
                            const int* __restrict__ inv, int* __restrict__ nbr) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < 8 * nn) nbr[e] = inv[nbr_call[8 * perm[e >> 3] + (e & 7)]];
}

// Up to kInfo device integers to pinned host memory (null: 0).
__global__ void k_info(InfoList l, int* __restrict__ out) {
    const int i = threadIdx.x;
    if (i < kInfo) out[i] = l.p[i] ? *l.p[i] : 0;
}

// The whole-solve kernel's view of the rows: per workgroup of 8 WAVES rows
// the foreign nodes its slots touch, ascending (at most kHalo are kept, the rest is -1),
// and per slot the column's place among the workgroup's local nodes
// (its own rows first, then the foreign ones; kLocal: the slot is not in use). One workgroup per tile: the
// columns are marked in a bitmap over the nodes, a column's place is its rank.
// need becomes the largest number of foreign nodes, or 2^20 when they or the
// slots from 16 on of 8 rows are more than the kernel holds.
template <int WAVES>
__global__ void __launch_bounds__(256) k_pcg_local(int nn, int ell_w, const uint32_t* __restrict__ ell_blk,
                                                   const int* __restrict__ ell_col, uint16_t* __restrict__ loc,
                                                   int* __restrict__ halo, int* __restrict__ halo_n,
                                                   int* __restrict__ need) {
    constexpr int kRows = pcg_rows(WAVES), kLocal = pcg_local(WAVES), kHalo = pcg_halo(WAVES);
    constexpr int kWords = 1024;                        // 32768 nodes
    __shared__ uint32_t bits[kWords];
    __shared__ int before[kWords];
    __shared__ int sums[256];
    const int row0 = blockIdx.x * kRows, row1 = min(nn, row0 + kRows);
    const int nslots = (row1 - row0) * ell_w;
    const size_t slot0 = (size_t)row0 * ell_w;
    const int words = (nn + 31) / 32;
    for (int w = threadIdx.x; w < kWords; w += 256) bits[w] = 0;
    __syncthreads();
    for (int t = threadIdx.x; t < nslots; t += 256) {
        const int c = ell_col[slot0 + t];
        if (ell_blk[slot0 + t] != 0xffffffffu && (c < row0 || c >= row1)) atomicOr(&bits[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    // exclusive prefix of the words' counts, four consecutive words per thread
    const int w0 = 4 * threadIdx.x;
    int own = 0;
    for (int q = 0; q < 4; ++q) own += __popc(bits[w0 + q]);
    sums[threadIdx.x] = own;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
        const int v = (int)threadIdx.x >= d ? sums[threadIdx.x - d] : 0;
        __syncthreads();
        sums[threadIdx.x] += v;
        __syncthreads();
    }
    int run = sums[threadIdx.x] - own;
    for (int q = 0; q < 4; ++q) {
        before[w0 + q] = run;
        run += __popc(bits[w0 + q]);
    }
    __syncthreads();
    const int total = sums[255];
    if (threadIdx.x == 0) {
        halo_n[blockIdx.x] = min(total, kHalo);
        atomicMax(need, total > kHalo ? 1 << 20 : total);
    }
    if (threadIdx.x < WAVES) {
        int nfar = 0;
        for (int j = 0; j < 8; ++j) {
            const int row = row0 + 8 * threadIdx.x + j;
            for (int f = 16; row < row1 && f < ell_w; ++f)
                nfar += ell_blk[(size_t)row * ell_w + f] != 0xffffffffu ? 1 : 0;
        }
        if (nfar > kPcgFar) atomicMax(need, 1 << 20);
    }
    for (int r = min(total, kHalo) + threadIdx.x; r < kHalo; r += 256) halo[(size_t)blockIdx.x * kHalo + r] = -1;
    for (int w = threadIdx.x; w < words; w += 256) {
        int rank = before[w];
        for (uint32_t m = bits[w]; m != 0u; m &= m - 1u, ++rank)
            if (rank < kHalo) halo[(size_t)blockIdx.x * kHalo + rank] = 32 * w + __ffs(m) - 1;
    }
    for (int t = threadIdx.x; t < nslots; t += 256) {
        const int c = ell_col[slot0 + t];
        int l = kLocal;                              // not in use
        if (ell_blk[slot0 + t] != 0xffffffffu) {
            l = (c >= row0 && c < row1) ? c - row0
                                        : kRows + before[c >> 5] + __popc(bits[c >> 5] & ((1u << (c & 31)) - 1u));
        }
        loc[slot0 + t] = (uint16_t)min(l, kLocal);
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
void launch_node_boxes(int nn, const float4* nodes, float4* boxes, hipStream_t st) {
    const int nruns = (nn + kKnnRun - 1) / kKnnRun;
    if (nruns > 0)
        hipLaunchKernelGGL(k_node_boxes, dim3((nruns + 255) / 256), dim3(256), 0, st, nn, nodes, boxes);
}

void launch_knn_skin(int ns, const float* pos_aos, int nn, const float4* nodes, const int* caller, float4* boxes,
                     float inv_two_sigma2, int4* idx, float4* w, hipStream_t st) {
    if (ns <= 0 || nn <= 0) return;
    launch_node_boxes(nn, nodes, boxes, st);
    hipLaunchKernelGGL(k_knn_skin, dim3((ns + 255) / 256), dim3(256), 0, st, ns, pos_aos, nn, nodes, caller, boxes,
                       inv_two_sigma2, idx, w);
}

void launch_node_graph(int nn, const float4* nodes, int* nbr, int* lone, hipStream_t st) {
    hipLaunchKernelGGL(k_node_graph, dim3((nn + kGraphNodesPerBlock - 1) / kGraphNodesPerBlock),
                       dim3(64 * kGraphNodesPerBlock), 0, st, nn, nodes, nbr, lone);
}

size_t bucket_work_ints(int ns) { return 2 * (size_t)ns + 2 * ((size_t)1 << kBucketBits) + 1; }

void launch_bucket_sort(int ns, int nn, int4* idx, const int* inv, uint64_t* key_in, int* work, uint64_t* key,
                        uint32_t* val, int* over, hipStream_t st) {
    const BucketOf o = bucket_of(nn);
    const int nb = 1 << (4 * o.bits - o.shift);
    int *bucket = work, *place = work + ns, *count = work + 2 * (size_t)ns, *start = count + nb;
    const dim3 grid((ns + 255) / 256);
    launch_fill_i32(count, nb, 0, st);
    hipLaunchKernelGGL(k_bucket_count, grid, dim3(256), 0, st, ns, idx, inv, o, key_in, bucket, place, count);
    hipLaunchKernelGGL(k_bucket_scan, dim3(1), dim3(kScanBlock), 0, st, nb, count, kBucketCap, start, over);
    hipLaunchKernelGGL(k_bucket_scatter, grid, dim3(256), 0, st, ns, key_in, bucket, place, start, key, val);
    hipLaunchKernelGGL(k_bucket_sort, dim3(nb), dim3(kBucketBlock), 0, st, start, key, val);
}

void launch_tuple_keys(int ns, int npad, const int4* idx, uint64_t* key, uint32_t* val, hipStream_t st) {
    hipLaunchKernelGGL(k_tuple_keys, dim3((npad + 255) / 256), dim3(256), 0, st, ns, npad, idx, key, val);
}

void launch_permute_surfels(int ns, const int* over, const uint64_t* key, const uint32_t* val, const float* ipos,
                            const float* inrm, const int4* iidx, const float4* iw, float* px, float* py,
                            float* pz, float* nx, float* ny, float* nz, int4* oidx, float4* ow, int* orig,
                            int* flag, hipStream_t st) {
    hipLaunchKernelGGL(k_permute_surfels, dim3((ns + 255) / 256), dim3(256), 0, st, ns, over, key, val, ipos, inrm,
                       iidx, iw, px, py, pz, nx, ny, nz, oidx, ow, orig, flag);
}

void launch_seg_pos4(int ns, int nseg, const int* seg_start, const int* seg_nodes, const int4* idx, uint16_t* pos4,
                     int* bad, hipStream_t st) {
    if (ns > 0 && nseg > 0)
        hipLaunchKernelGGL(k_seg_pos4, dim3((ns + 255) / 256), dim3(256), 0, st, ns, nseg, seg_start, seg_nodes, idx,
                           pos4, bad);
}

void launch_run_starts(int ns, const int* flag, const int* pos, const uint64_t* key, int* run_start,
                       uint64_t* run_key, hipStream_t st) {
    hipLaunchKernelGGL(k_run_starts, dim3((ns + 255) / 256), dim3(256), 0, st, ns, flag, pos, key, run_start, run_key);
}

void launch_pattern(int ns, const uint64_t* key, const int* flag, int nn, const int* nbr, uint32_t* bm,
                    uint32_t* in_bm, int words, hipStream_t st) {
    hipLaunchKernelGGL(k_pattern_sets, dim3((ns + 255) / 256), dim3(256), 0, st, ns, key, flag, bm, words);
    hipLaunchKernelGGL(k_pattern_nodes, dim3((8 * nn + 255) / 256), dim3(256), 0, st, nn, nbr, bm, in_bm, words);
}

static dim3 row_grid(int nn) { return dim3((nn + kRowBlock / kWave - 1) / (kRowBlock / kWave)); }

void launch_row_counts(int nn, const uint32_t* bm, const uint32_t* in_bm, int words, int* upper, int* full,
                       int* in_cnt, int* row_ptr, int* in_ptr, int* longest, hipStream_t st) {
    hipLaunchKernelGGL(k_row_counts, row_grid(nn), dim3(kRowBlock), 0, st, nn, bm, in_bm, words, upper, full, in_cnt);
    hipLaunchKernelGGL(k_row_scan, dim3(3), dim3(kScanBlock), 0, st, nn, upper, full, in_cnt, row_ptr, in_ptr,
                       longest);
}

void launch_row_fill(int nn, const uint32_t* bm, const uint32_t* in_bm, int words, const int* row_ptr,
                     const int* in_ptr, int* col_idx, int* blk_row, int* offlist, int* in_list, hipStream_t st) {
    hipLaunchKernelGGL(k_row_fill, row_grid(nn), dim3(kRowBlock), 0, st, nn, bm, in_bm, words, row_ptr, in_ptr,
                       col_idx, blk_row, offlist, in_list);
}

void launch_ell(int nn, int ell_w, const uint32_t* bm, int words, const int* row_ptr, const int* full,
                const int* col_idx, uint32_t* ell_blk, int* ell_col, int* slot_u, int* slot_t, hipStream_t st) {
    hipLaunchKernelGGL(k_ell, row_grid(nn), dim3(kRowBlock), 0, st, nn, ell_w, bm, words, row_ptr, full, col_idx,
                       ell_blk, ell_col, slot_u, slot_t);
}

void launch_map_graph(int nn, const int* nbr_call, const int* perm, const int* inv, int* nbr, hipStream_t st) {
    hipLaunchKernelGGL(k_map_graph, dim3((8 * nn + 255) / 256), dim3(256), 0, st, nn, nbr_call, perm, inv, nbr);
}

void launch_info(const InfoList& l, int* out, hipStream_t st) {
    hipLaunchKernelGGL(k_info, dim3(1), dim3(kWave), 0, st, l, out);
}

void launch_pcg_local(int waves, int nn, int ell_w, const uint32_t* ell_blk, const int* ell_col, uint16_t* loc,
                      int* halo, int* halo_n, int* need, hipStream_t st) {
    const dim3 grid(cdiv(nn, pcg_rows(waves)));
    if (waves == 4)
        hipLaunchKernelGGL(k_pcg_local<4>, grid, dim3(256), 0, st, nn, ell_w, ell_blk, ell_col, loc, halo, halo_n, need);
    else
        hipLaunchKernelGGL(k_pcg_local<8>, grid, dim3(256), 0, st, nn, ell_w, ell_blk, ell_col, loc, halo, halo_n, need);
}

}  // namespace swgn
