// The segment layout on the device (Sec. 6.5, Initialization: the per-node-set
// structures the assembly of J^T J walks every iteration).
//
// Surfels sorted by node set are cut into segments: greedy runs of at most M
// consecutive surfels whose node sets together name at most 5 nodes, so that
// a segment's Gram matrix is at most 31 x 31 (three 16x16 MFMA tiles); packs are greedy runs of
// whole segments with at most M surfels. A greedy cut is a chain: a segment
// that opens at surfel s always starts with the node set of s's run, so the
// next opening after s is a function next(s) of s alone, with
// s < next(s) <= s + M. next is formed for every surfel at once; the chain
// from surfel 0 is then walked in chunks of C positions, M <= C <= kChainChunk
// (each chunk from each of the M positions a chain can enter it by, in
// parallel; the chunks linked by one thread; the chosen walk of each chunk
// written out).
// Packs are the same chain over segments. Every result is an integer that
// does not depend on the order of any atomic.
#include "swgn_impl.h"
#include "swgn_launch.h"
#include "swgn_setup.h"

namespace swgn {

namespace {

constexpr int kChainChunk = 8192;   // most positions per workgroup of the chain walk (LDS ints)
constexpr int kChainBlock = 256;    // threads per workgroup; >= M

__device__ __forceinline__ void set_nodes(uint64_t k, int (&t)[4]) {
    t[0] = (int)(k >> 48);
    t[1] = (int)((k >> 32) & 0xffff);
    t[2] = (int)((k >> 16) & 0xffff);
    t[3] = (int)(k & 0xffff);
}

// Adds the 4 distinct nodes t to the set cur (cn entries, 5 slots); returns
// the new size, or 6 once it would exceed 5 (cur is then no longer used).
__device__ __forceinline__ int merge_set(int (&cur)[5], int cn, const int (&t)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bool have = false;
#pragma unroll
        for (int q = 0; q < 5; ++q) have = have || (q < cn && cur[q] == t[k]);
        if (!have) {
            if (cn == 5) return 6;
#pragma unroll
            for (int q = 0; q < 5; ++q)
                if (q == cn) cur[q] = t[k];
            ++cn;
        }
    }
    return cn;
}

__device__ __forceinline__ int first_pair(int pa) { return 5 * pa - pa * (pa - 1) / 2; }

// next(s): where the segment opening at surfel s ends. run_pos is the
// exclusive scan of the run-start flags (s lies in run run_pos[s + 1] - 1).
// Within s's run only the length cuts; each following run joins while the
// node union stays within 5 nodes and the segment within M surfels, and a run
// that would take it past M surfels cuts it at s + M.
__global__ void k_seg_next(int ns, const uint64_t* __restrict__ set_key, const int* __restrict__ set_start,
                           const int* __restrict__ run_pos, int M, int* __restrict__ next) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ns) return;
    const int r = run_pos[s + 1] - 1, nsets = run_pos[ns];
    int nx = ns;
    if (set_start[r + 1] - s > M) {
        nx = s + M;
    } else {
        int t[4];
        set_nodes(set_key[r], t);
        int cur[5] = {t[0], t[1], t[2], t[3], -1};
        int cn = 4;
        for (int r2 = r + 1; r2 < nsets; ++r2) {
            const int a2 = set_start[r2];
            if (a2 - s >= M) { nx = a2; break; }
            set_nodes(set_key[r2], t);
            cn = merge_set(cur, cn, t);
            if (cn > 5) { nx = a2; break; }
            if (set_start[r2 + 1] - s > M) { nx = s + M; break; }
        }
    }
    next[s] = nx;
}

// next over segments for packs: the first segment g2 > g whose end lies more
// than M surfels past the start of g (binary search), else nseg.
__global__ void k_pack_next(int nseg, const int* __restrict__ seg_start, int M, int* __restrict__ next) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nseg) return;
    const int lim = seg_start[g] + M;
    int lo = g + 2, hi = nseg + 1;            // smallest k in [g + 2, nseg] with seg_start[k] > lim, else nseg + 1
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (seg_start[mid] > lim) hi = mid;
        else lo = mid + 1;
    }
    next[g] = lo <= nseg ? lo - 1 : nseg;
}

__device__ __forceinline__ void stage_chunk(const int* __restrict__ next, int lo, int hi, int* nx) {
    // (8 loads of a thread on their way at once)
    for (int i0 = lo + (int)threadIdx.x; i0 < hi; i0 += 8 * kChainBlock) {
        int v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = next[min(i0 + q * kChainBlock, hi - 1)];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (i0 + q * kChainBlock < hi) nx[i0 + q * kChainBlock - lo] = v[q];
    }
    __syncthreads();
}

// Per chunk q and entry position lo + t (t < M): where the walk from it leaves
// the chunk and how many positions it visits inside. A successor that does not
// move forward ends the walk and flags the input.
__global__ void __launch_bounds__(kChainBlock) k_chain_chunks(const int* __restrict__ next, int n, int M, int C,
                                                               int* __restrict__ exit_pos, int* __restrict__ hops,
                                                               int* __restrict__ bad) {
    __shared__ int nx[kChainChunk];
    const int q = blockIdx.x, lo = q * C, hi = min(n, lo + C);
    stage_chunk(next, lo, hi, nx);
    const int t = threadIdx.x;
    if (t >= M) return;
    int pos = lo + t, cnt = 0;
    while (pos < hi) {
        const int np = nx[pos - lo];
        if (np <= pos) { atomicOr(bad, 1); break; }
        pos = np;
        ++cnt;
    }
    exit_pos[q * M + t] = pos;
    hops[q * M + t] = cnt;
}

// The chunks linked in order from position 0: each chunk's entry position and
// the number of chain positions before it; *count = the chain's length. An
// entry outside the chunk's M entry positions flags the input and marks the
// remaining chunks unused (entry -1). One thread walks; the chunks' walks come
// to LDS first, kLinkWords / M chunks at a time, a word each (positions past
// the chunk's start in the low half, hops in the high one: both below 2^15),
// so that a step is an LDS read (61 chunks read from memory: 28 us).
constexpr int kLinkWords = 15360;
static_assert(kChainChunk + kChainBlock < 32768, "a chunk's walk in two 16-bit halves");
__global__ void __launch_bounds__(1024) k_chain_link(int nchunks, int n, int M, int C, const int* __restrict__ exit_pos,
                             const int* __restrict__ hops, int* __restrict__ entry, int* __restrict__ base,
                             int* __restrict__ count, int* __restrict__ bad) {
    __shared__ uint32_t walk[kLinkWords];
    const int per = kLinkWords / M;
    int e = 0, b = 0;
    bool ok = true;
    for (int q0 = 0; q0 < nchunks; q0 += per) {
        const int q1 = min(nchunks, q0 + per);
        __syncthreads();
        for (int t = threadIdx.x; t < (q1 - q0) * M; t += 1024) {
            const int64_t src = (int64_t)q0 * M + t;
            const int64_t over = (int64_t)exit_pos[src] - (int64_t)(q0 + t / M) * C;
            // (a walk that broke the rule is flagged already; any value does)
            walk[t] = (uint32_t)(over < 0 ? 0 : (over > 32767 ? 32767 : over)) | ((uint32_t)hops[src] << 16);
        }
        __syncthreads();
        if (threadIdx.x != 0) continue;
        for (int q = q0; q < q1; ++q) {
            const int t = e - q * C;
            ok = ok && t >= 0 && t < M;
            entry[q] = ok ? e : -1;
            base[q] = b;
            if (ok) {
                const uint32_t w = walk[(q - q0) * M + t];
                b += (int)(w >> 16);
                e = q * C + (int)(w & 0xffffu);
            }
        }
    }
    if (threadIdx.x != 0) return;
    if (!ok || e != n) *bad = 1;
    *count = ok ? b : 0;
}

// The chain's positions inside each chunk, from its entry, at out[base ...].
__global__ void __launch_bounds__(kChainBlock) k_chain_emit(const int* __restrict__ next, int n, int C,
                                                             const int* __restrict__ entry,
                                                             const int* __restrict__ base, int* __restrict__ out) {
    __shared__ int nx[kChainChunk];
    const int q = blockIdx.x, lo = q * C, hi = min(n, lo + C);
    stage_chunk(next, lo, hi, nx);
    if (threadIdx.x != 0 || entry[q] < 0) return;
    int pos = entry[q], j = base[q];
    while (pos < hi && j < n) {
        out[j++] = pos;
        const int np = nx[pos - lo];
        if (np <= pos) break;
        pos = np;
    }
}

// Per segment: its nodes (ascending, -1 padded), the mask of its node pairs
// that share a surfel (bit first(pa) + pb - pa, pa <= pb positions in the
// node list), its Gram output in 4-float units (36 per pair + 32) and its
// pair count; the units' 64-bit total. More than 5 nodes flags the input.
__global__ void __launch_bounds__(256) k_seg_info(int nseg, const int* __restrict__ seg_start,
                                                  const int* __restrict__ run_pos, const uint64_t* __restrict__ set_key,
                                                  int* __restrict__ seg_nodes, uint16_t* __restrict__ mask,
                                                  int* __restrict__ units, int* __restrict__ npairs,
                                                  unsigned long long* __restrict__ total_units, int* __restrict__ bad) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    int u = 0;
    if (g < nseg) {
        const int r0 = run_pos[seg_start[g] + 1] - 1, r1 = run_pos[seg_start[g + 1]] - 1;
        int t[4];
        set_nodes(set_key[r0], t);
        int cur[5] = {t[0], t[1], t[2], t[3], 0x7fffffff};
        int cn = 4;
        for (int r = r0 + 1; r <= r1 && cn <= 5; ++r) {
            set_nodes(set_key[r], t);
            cn = merge_set(cur, cn, t);
        }
        if (cn > 5) {
            atomicOr(bad, 1);
            cn = 4;
            set_nodes(set_key[r0], t);
            cur[0] = t[0]; cur[1] = t[1]; cur[2] = t[2]; cur[3] = t[3]; cur[4] = 0x7fffffff;
        }
        // ascending (an unused slot holds the largest int and sorts last)
        int tmp;
#define SWGN_CS(p, q) if (cur[p] > cur[q]) { tmp = cur[p]; cur[p] = cur[q]; cur[q] = tmp; }
        SWGN_CS(0, 1) SWGN_CS(3, 4) SWGN_CS(2, 4) SWGN_CS(2, 3) SWGN_CS(0, 3)
        SWGN_CS(0, 2) SWGN_CS(1, 4) SWGN_CS(1, 3) SWGN_CS(1, 2)
#undef SWGN_CS
        uint32_t m = 0;
        for (int r = r0; r <= r1; ++r) {
            set_nodes(set_key[r], t);
            int p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                p[k] = 0;
#pragma unroll
                for (int q = 0; q < 5; ++q) p[k] += cur[q] < t[k] ? 1 : 0;
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = x; y < 4; ++y) m |= 1u << (first_pair(p[x]) + p[y] - p[x]);
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) seg_nodes[5 * g + q] = q < cn ? cur[q] : -1;
        mask[g] = (uint16_t)m;
        const int np = __popc(m);
        u = 9 * np + 8;
        units[g] = u;
        npairs[g] = np;
    }
    u = wave_sumi(u);
    if ((threadIdx.x % kWave) == 0 && u != 0) atomicAdd(total_units, (unsigned long long)u);
}

// The cuts as segment starts, closed by ns.
__global__ void k_seg_starts(int nseg, const int* __restrict__ cuts, int ns, int* __restrict__ seg_start) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g <= nseg) seg_start[g] = g < nseg ? cuts[g] : ns;
}

// Per segment 16 lanes, one entry per pair of its mask (in mask order): the
// block of the pair (binary search in the node's row of the upper pattern), the
// float offsets of its sub-block and, on the diagonal, of the J^T r piece; the
// entry's place in the block is an atomic counter's (ordered by
// k_ent_order). A pair missing from the pattern flags the input and has no
// block (-1). Also the segments' float offsets. (One thread per segment
// searched its pairs one after the other: 28.7 us for 3,000 segments.)
__global__ void __launch_bounds__(256) k_seg_entries(int nseg, const int* __restrict__ seg_nodes,
        const uint16_t* __restrict__ mask, const int* __restrict__ off_units, uint32_t* __restrict__ off,
        const int* __restrict__ ebase, const int* __restrict__ row_ptr, const int* __restrict__ col_idx,
        int* __restrict__ eblk, int* __restrict__ eplace, uint32_t* __restrict__ esub, uint32_t* __restrict__ egrad,
        int* __restrict__ bcount, int* __restrict__ bad) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x, g = t >> 4, bit = t & 15;
    if (g > nseg) return;
    const uint32_t o = 4u * (uint32_t)off_units[g];
    if (bit == 15) off[g] = o;
    if (g == nseg || bit == 15) return;
    const uint32_t m = mask[g];
    if (!((m >> bit) & 1u)) return;
    int pa = 0;
    while (pa < 4 && first_pair(pa + 1) <= bit) ++pa;
    const int pb = pa + bit - first_pair(pa);
    const uint32_t rank = (uint32_t)__popc(m & ((1u << bit) - 1u)), np = (uint32_t)__popc(m);
    const int e = ebase[g] + (int)rank;
    const int ra = seg_nodes[5 * g + pa], cb = seg_nodes[5 * g + pb];
    const int end = row_ptr[ra + 1];
    int lo = row_ptr[ra], hi = end;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (col_idx[mid] < cb) lo = mid + 1;
        else hi = mid;
    }
    int blk = lo, place = 0;
    if (lo >= end || col_idx[lo] != cb) {
        atomicOr(bad, 1);
        blk = -1;
    } else {
        place = atomicAdd(&bcount[blk], 1);
    }
    eblk[e] = blk;
    eplace[e] = place;
    esub[e] = o + 36u * rank;
    egrad[e] = pa == pb ? o + 36u * np + 6u * (uint32_t)pa : 0xffffffffu;
}

__global__ void __launch_bounds__(256) k_ent_scatter(int ne, const int* __restrict__ eblk, const int* __restrict__ eplace,
                                                     const int* __restrict__ ent_ptr, int* __restrict__ list) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < ne && eblk[e] >= 0) list[ent_ptr[eblk[e]] + eplace[e]] = e;
}

// Each block's entries in ascending order (segment order): a wave per block of
// up to 64, by counting the smaller ones, then the workgroup together for its
// longer ones, by a bitonic sort in LDS (counting took 1,178 us for 45 blocks
// of 2,300 entries); above kEntCap *over is set (the host
// sorts them instead).
constexpr int kEntCap = 4096;
__global__ void __launch_bounds__(256) k_ent_order(int nb, const int* __restrict__ ent_ptr,
        const int* __restrict__ list, const uint32_t* __restrict__ esub, const uint32_t* __restrict__ egrad,
        uint32_t* __restrict__ ent_sub, uint32_t* __restrict__ ent_grad, int* __restrict__ over) {
    __shared__ int ids[kEntCap];
    constexpr int kBlocks = 256 / kWave;
    const int lane = threadIdx.x % kWave, b = blockIdx.x * kBlocks + threadIdx.x / kWave;
    if (b < nb) {
        const int p = ent_ptr[b], n = ent_ptr[b + 1] - p;
        if (n <= kWave) {
            const int e = lane < n ? list[p + lane] : 0x7fffffff;
            int rank = 0;
            for (int j = 0; j < n; ++j) rank += __builtin_amdgcn_readlane(e, j) < e ? 1 : 0;
            if (lane < n) {
                ent_sub[p + rank] = esub[e];
                ent_grad[p + rank] = egrad[e];
            }
        }
    }
    for (int w = 0; w < kBlocks; ++w) {                  // (the same for all threads)
        const int bb = blockIdx.x * kBlocks + w;
        if (bb >= nb) break;
        const int p = ent_ptr[bb], n = ent_ptr[bb + 1] - p;
        if (n <= kWave) continue;
        if (n > kEntCap) {
            if (threadIdx.x == 0) *over = 1;
            continue;
        }
        __syncthreads();                                 // (ids may still be read for the last block)
        int p2 = 2 * kWave;
        while (p2 < n) p2 <<= 1;
        for (int j = threadIdx.x; j < p2; j += 256) ids[j] = j < n ? list[p + j] : 0x7fffffff;
        __syncthreads();
        for (int k = 2; k <= p2; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int q = threadIdx.x; q < p2 / 2; q += 256) {
                    const int a = ((q & ~(j - 1)) << 1) | (q & (j - 1)), b2 = a + j;
                    const int ea = ids[a], eb = ids[b2];
                    if ((a & k) == 0 ? eb < ea : ea < eb) { ids[a] = eb; ids[b2] = ea; }
                }
                __syncthreads();
            }
        for (int q = threadIdx.x; q < n; q += 256) {
            const int e = ids[q];
            ent_sub[p + q] = esub[e];
            ent_grad[p + q] = egrad[e];
        }
    }
}

// Keys (block, entry) of all entries for sort_pairs, padded to npad.
__global__ void k_ent_keys(int ne, int npad, const int* __restrict__ eblk, uint64_t* __restrict__ key,
                           uint32_t* __restrict__ val) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= npad) return;
    key[e] = e < ne ? ((uint64_t)(uint32_t)eblk[e] << 32) | (uint32_t)e : ~0ull;
    val[e] = e < ne ? (uint32_t)e : 0xffffffffu;
}

__global__ void k_ent_gather(int ne, const uint32_t* __restrict__ order, const uint32_t* __restrict__ esub,
                             const uint32_t* __restrict__ egrad, uint32_t* __restrict__ ent_sub,
                             uint32_t* __restrict__ ent_grad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const uint32_t v = order[i];
    ent_sub[i] = esub[v];
    ent_grad[i] = egrad[v];
}

// First segment and first surfel of every pack; the closing entries nseg and ns.
__global__ void k_pack_arrays(int npack, int nseg, int ns, const int* __restrict__ cuts,
                              const int* __restrict__ seg_start, int* __restrict__ pack_seg,
                              int* __restrict__ pack_start) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > npack) return;
    const int g = i < npack ? cuts[i] : nseg;
    pack_seg[i] = g;
    pack_start[i] = i < npack ? seg_start[g] : ns;
}

inline int grid_of(int64_t n, int block) { return (int)((n + block - 1) / block); }

}  // namespace

// Chunk size: a walk inside a chunk costs a dependent LDS read per step and
// the link a dependent global read per chunk, so C ~ sqrt(32 n) (a power of
// two in [256, kChainChunk]; at least M, so that a chain enters every chunk).
int chain_chunk(int n, int M) {
    int c = 256;
    while (c < kChainChunk && (int64_t)c * c < 32 * (int64_t)n) c <<= 1;
    return c < M ? kChainChunk : c;
}

size_t chain_work_ints(int n, int M) {
    const int64_t nchunks = (n + 255) / 256;
    return (size_t)(nchunks * (2 * (int64_t)M + 2) + 1);
}

void chain_from_zero(const int* next, int n, int M, int* out, int* count, int* work, int* bad, hipStream_t st) {
    const int C = chain_chunk(n, M);
    const int nchunks = (n + C - 1) / C;
    int* exit_pos = work;
    int* hops = exit_pos + (size_t)nchunks * M;
    int* entry = hops + (size_t)nchunks * M;
    int* base = entry + nchunks;
    hipLaunchKernelGGL(k_chain_chunks, dim3(nchunks), dim3(kChainBlock), 0, st, next, n, M, C, exit_pos, hops, bad);
    hipLaunchKernelGGL(k_chain_link, dim3(1), dim3(1024), 0, st, nchunks, n, M, C, exit_pos, hops, entry, base,
                       count, bad);
    hipLaunchKernelGGL(k_chain_emit, dim3(nchunks), dim3(kChainBlock), 0, st, next, n, C, entry, base, out);
}

int chain_max_hop() { return kChainBlock; }

void launch_seg_next(int ns, const uint64_t* set_key, const int* set_start, const int* run_pos, int M,
                     int* next, hipStream_t st) {
    hipLaunchKernelGGL(k_seg_next, dim3(grid_of(ns, 256)), dim3(256), 0, st, ns, set_key, set_start, run_pos, M,
                       next);
}

void launch_pack_next(int nseg, const int* seg_start, int M, int* next, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_next, dim3(grid_of(nseg, 256)), dim3(256), 0, st, nseg, seg_start, M, next);
}

void launch_seg_info(int nseg, const int* seg_start, const int* run_pos, const uint64_t* set_key, int* seg_nodes,
                     uint16_t* mask, int* units, int* npairs, unsigned long long* total_units, int* bad,
                     hipStream_t st) {
    hipLaunchKernelGGL(k_seg_info, dim3(grid_of(nseg, 256)), dim3(256), 0, st, nseg, seg_start, run_pos, set_key,
                       seg_nodes, mask, units, npairs, total_units, bad);
}

void launch_seg_starts(int nseg, const int* cuts, int ns, int* seg_start, hipStream_t st) {
    hipLaunchKernelGGL(k_seg_starts, dim3(grid_of(nseg + 1, 256)), dim3(256), 0, st, nseg, cuts, ns, seg_start);
}

void launch_seg_entries(int nseg, const int* seg_nodes, const uint16_t* mask, const int* off_units, uint32_t* off,
                        const int* ebase, const int* row_ptr, const int* col_idx, int* eblk, int* eplace,
                        uint32_t* esub, uint32_t* egrad, int* bcount, int* bad, hipStream_t st) {
    hipLaunchKernelGGL(k_seg_entries, dim3(grid_of(16 * ((int64_t)nseg + 1), 256)), dim3(256), 0, st, nseg, seg_nodes,
                       mask, off_units, off, ebase, row_ptr, col_idx, eblk, eplace, esub, egrad, bcount, bad);
}

void launch_ent_order(int ne, int nb, const int* eblk, const int* eplace, const int* ent_ptr, const uint32_t* esub,
                      const uint32_t* egrad, int* list, uint32_t* ent_sub, uint32_t* ent_grad, int* over,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_ent_scatter, dim3(grid_of(ne, 256)), dim3(256), 0, st, ne, eblk, eplace, ent_ptr, list);
    hipLaunchKernelGGL(k_ent_order, dim3(grid_of(nb, 4)), dim3(256), 0, st, nb, ent_ptr, list, esub, egrad, ent_sub,
                       ent_grad, over);
}

void sort_entries(int ne, int npad, const int* eblk, uint64_t* key, uint32_t* val, const uint32_t* esub,
                  const uint32_t* egrad, uint32_t* ent_sub, uint32_t* ent_grad, hipStream_t st) {
    hipLaunchKernelGGL(k_ent_keys, dim3(grid_of(npad, 256)), dim3(256), 0, st, ne, npad, eblk, key, val);
    sort_pairs(key, val, npad, st);
    hipLaunchKernelGGL(k_ent_gather, dim3(grid_of(ne, 256)), dim3(256), 0, st, ne, val, esub, egrad, ent_sub,
                       ent_grad);
}

void launch_pack_arrays(int npack, int nseg, int ns, const int* cuts, const int* seg_start, int* pack_seg,
                        int* pack_start, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_arrays, dim3(grid_of(npack + 1, 256)), dim3(256), 0, st, npack, nseg, ns, cuts,
                       seg_start, pack_seg, pack_start);
}

}  // namespace swgn
