// A whole linear solve (all PCG iterations and the node update) in one launch.
//
// The step-wise kernels (solve.hip) pay a launch boundary and the dependent
// loads of the blocks, the columns' vectors and their inverses in every
// iteration, although nothing of the matrix changes. Here a workgroup keeps
// its 32 block rows in registers for the whole solve (8 rows per wave, lane
// = row sub of a slot's block), the vectors and inverses of its local nodes
// (its rows and the columns they touch) on the chip, and the workgroups of a
// stream meet once per iteration: each publishes u, v of its rows and the
// partial sums of its parts, and takes the sums of all parts and u, v of its
// foreign columns. With those it repeats the finish of the foreign columns
// itself, so one exchange per iteration is enough.
//
// What bounds it: the latency of that exchange (a store to and a load from
// the memory side: 1.5 us for 2 workgroups and 1.8 us for 56 over 8 XCDs, of
// 4.4 us per iteration), then the wave's own chain of products (0.8 us), sums
// and publication (0.55 us), scalars (0.2 us) and finishes (0.6 us). Measured,
// 10 iterations: 640x480, 1,788 nodes: 51.9 us, as 11 step-wise launches
// 84 us; 16 uneven streams, 41,000 nodes: 225 us against 385 us. Of the 52 us
// about 9 are the way to the first product (all loads of the blocks issued
// before any is waited for: 54.6 -> 51.9 us).
//
// Why 32 rows per workgroup (4 waves): alone on its SIMD a wave runs its chain
// fastest and a stream spreads over more CUs (4.4 us per iteration against
// 5.2 us with 64 rows); with more waves than SIMDs, 64 rows (8 waves) make
// half the workgroups to meet and each foreign column serves more rows (16
// streams: 86 us against 88 us for a third of them, and fewer launches). That
// holds also where a tile has so many foreign columns that its workgroup takes
// a CU's LDS for itself (1,788 nodes, up to 136 of them: 56.5 us, 64.2 us with
// 64 rows). A node set of 64 nodes at most is one workgroup of 8 waves, which
// has nobody to wait for (40 nodes: 41.4 us, two workgroups 43.4 us).
//
// The exchange. A value travels as 64-bit words, each the iteration's tag in
// the upper half and 32 bits of payload in the lower, written and read by
// relaxed agent-scope atomics: a word is its own flag, so no fence, no cache
// write-back and no second round trip is needed. Every fold counts (also one
// whose solve then runs step by step, and a replayed one), and a tag is the
// iteration in the range of that count, so nothing has to be cleared between
// solves. A tag comes again after 2^32 / kPcgTags folds; the host clears the
// words before that many have passed. Words are double-buffered by iteration
// parity: a workgroup writes iteration i + 2 only after it has every part of
// iteration i + 1, which their owners publish after they have read all of
// iteration i.
//
// Every workgroup of a stream must be resident for the others to get on, so
// the host launches no more of them than find a place on the chip however they
// are placed (a lease on their number, taken per device for as long as they
// run; swgn_lease.h), and every wait is
// bounded: a workgroup that waits longer than the stream allows raises the
// stream's stall flag and stops waiting, and so does every workgroup of the
// frame that finds the flag raised, in this launch and in the frame's later
// ones. The host then solves the frame again step by step.
//
// Arithmetic. Every value is formed by the step-wise kernels' operations in
// their order (slot order, butterfly sums over a row's lane groups, sums of
// 8 rows, the 256-leaf sum over parts), so the results agree bit for bit.
#include "swgn_frame.h"
#include "swgn_impl.h"
#include "swgn_launch.h"
#include "swgn_pcg.h"

#include <initializer_list>

namespace swgn {

namespace {

typedef unsigned long long u64;

// Two adjacent words, 16-byte aligned, read past the caches of this XCD (the
// scope bit of an agent-scope load): each word is whole, for it is written by
// one 8-byte store and lies in one aligned 8 bytes of one request.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t XchgBuf;
constexpr int kAgentScope = 16;
__device__ __forceinline__ XchgBuf xchg_buffer(const u64* base, size_t words) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<u64*>(base), 0, (int)(words * 8), 0x00027000);
}
__device__ __forceinline__ u32x4 xchg_load2(XchgBuf b, int word) {
    return __builtin_amdgcn_raw_buffer_load_b128(b, word * 8, 0, kAgentScope);
}
__device__ __forceinline__ void xchg_store(u64* p, unsigned tag, unsigned payload) {
    typedef __attribute__((address_space(1))) u64 G;
    __hip_atomic_store((G*)p, ((u64)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int agent_load(const int* p) {
    typedef __attribute__((address_space(1))) const int G;
    return __hip_atomic_load((G*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sums of 8 rows over the wave's 8 lane groups: acc[j] is row j's term of the
// lane's group; returns the total of row `group` in every group, each the
// butterfly sum over the groups (distance 1, 2, 4). Rows trade places while
// the sums halve, so the 8 rows take 7 additions instead of 24.
__device__ __forceinline__ float group_rows(const float (&acc)[8], int lane) {
    const bool b0 = (lane & 8) != 0;
    float w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float keep = b0 ? acc[2 * q + 1] : acc[2 * q];
        const float send = b0 ? acc[2 * q] : acc[2 * q + 1];
        w[q] = keep + xchg<8>(send);
    }
    float y[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        // odd rows (of 16 lanes) of the first trade places with even rows of the second
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(w[2 * q]), __float_as_int(w[2 * q + 1]),
                                                        false, false);
        y[q] = __int_as_float(p[0]) + __int_as_float(p[1]);
    }
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(y[0]), __float_as_int(y[1]), false, false);
    return __int_as_float(p[0]) + __int_as_float(p[1]);
}

// One slot each of two rows: u += B z, v += B p for the lane's row of the
// block h (g), with c (d) the column's z, p of the components q and 4 + (q & 1)
// in quad position q. The broadcast rides on the multiply-add (the
// compiler forms the accumulating instruction too late to fold a DPP move
// into it and would issue twice as many), and the four sums take turns, so
// none waits for its own last addition. s_nop: two wait states before a DPP
// source that a vector instruction may just have written.
__device__ __forceinline__ void slot_step2(float& u0, float& v0, float& u1, float& v1, const float (&h)[6],
                                           const float (&g)[6], float4 c, float4 d) {
#define SWGN_MAC(acc, src, w, c) "v_fmac_f32_dpp %" #acc ", %" #src ", %" #w " quad_perm:[" c "," c "," c "," c "] row_mask:0xf bank_mask:0xf\n\t"
#define SWGN_MAC4(z0, p0, z1, p1, w0, w1, c) SWGN_MAC(0, z0, w0, c) SWGN_MAC(1, p0, w0, c) SWGN_MAC(2, z1, w1, c) SWGN_MAC(3, p1, w1, c)
    asm("s_nop 1\n\t"
        SWGN_MAC4(4, 5, 8, 9, 12, 18, "0") SWGN_MAC4(4, 5, 8, 9, 13, 19, "1")
        SWGN_MAC4(4, 5, 8, 9, 14, 20, "2") SWGN_MAC4(4, 5, 8, 9, 15, 21, "3")
        SWGN_MAC4(6, 7, 10, 11, 16, 22, "0") SWGN_MAC4(6, 7, 10, 11, 17, 23, "1")
        : "+v"(u0), "+v"(v0), "+v"(u1), "+v"(v1)
        : "v"(c.x), "v"(c.y), "v"(c.z), "v"(c.w), "v"(d.x), "v"(d.y), "v"(d.z), "v"(d.w),
          "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]), "v"(h[4]), "v"(h[5]),
          "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(g[4]), "v"(g[5]));
#undef SWGN_MAC4
#undef SWGN_MAC
}
// Component `sub` of a node's z and p into its vec entries (components 4 and 5
// at two quad positions each; the lanes that have nothing to write, write the
// node's fifth float4).
__device__ __forceinline__ void put_vec(float4* node, int sub, float z, float p) {
    float2* f = reinterpret_cast<float2*>(node);
    const bool two = sub == 4 || sub == 5;
    f[sub < 4 ? 2 * sub : (two ? 2 * sub - 7 : 8)] = make_float2(z, p);
    f[two ? 2 * sub - 3 : 9] = make_float2(z, p);
}
__device__ __forceinline__ float2 get_vec(const float4* node, int sub) {
    const float2* f = reinterpret_cast<const float2*>(node);
    return f[sub < 4 ? 2 * sub : 2 * (sub & 1) + 1];
}

// Sums over the wave of two values at once, as wave_sum4 forms four: value 0
// in lanes 0-31, value 1 in lanes 32-63.
__device__ __forceinline__ double wave_sum2(double a, double b) {
    swap32(a, b);
    a += b;
    a += xchg<16>(a);
    a += xchg<8>(a);
    a += xchg<4>(a);
    a += xchg<2>(a);
    a += xchg<1>(a);
    return a;
}

// kWaves: waves (of 8 block rows) per workgroup; kSets: sets of local nodes,
// one node of a set per lane group, that the launch's largest workgroup needs.
template <int kWaves, int kSets>
__global__ void __launch_bounds__(64 * kWaves, kWaves == 4 && kSets > kPcgPairSets ? 1 : 2) k_pcg_solve(Batch b) {
    // kNone: the local column of a slot that is not in use; kLocal: local nodes held, the zero node's place
    constexpr int kRows = pcg_rows(kWaves), kNone = pcg_local(kWaves), kHalo = pcg_halo(kWaves);
    constexpr int kLocal = kSets * kRows;
    static_assert(kLocal <= kNone && kLocal < 512, "the local columns' layout and their 9 bits");
    // the sums over parts have the shape of a 256-thread sum of four values:
    // with 8 waves each half of the workgroup forms two of them
    constexpr int kValues = 16 / kWaves;
    constexpr int kTogether = kSets > 4 ? 2 : (kWaves == 8 ? 2 : 4);
    constexpr int kLeafParts = 4 / kValues;            // parts of a leaf taken at once (more: in rounds)
    constexpr unsigned kPartBit = 1u << 30;
    static_assert(kWaves == 4 || kWaves == 8, "256 threads, or 256 for each half of the sums");
    // (z, p) of the local nodes as a lane's quad position q needs them: those of
    // components q and 4 + (q & 1); the last node is zero. 5 float4 per node,
    // so that the columns of a wave spread over the banks.
    constexpr int kVecStride = 5;
    __shared__ float4 vec[(kLocal + 1) * kVecStride];
    __shared__ float res[kLocal * 8];              // r of the local nodes
    __shared__ double minv[kLocal * 36];
    __shared__ float2 far[kWaves * kPcgFar + 1][18];   // blocks of the rows' slots from 16 on; the last one is zero
    __shared__ double red[kWaves][4];
    __shared__ double rowdot[kWaves][3][8];
    __shared__ int stalled;
    const Where at = locate(b);
    const FrameDesc a = *b.d[at.s];
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int sub = lane & 7, grp = lane >> 3, gi = tid >> 3;
    const int base = lane & ~7, quad = lane & 3;
    const int ntiles = pcg_tiles(a, kWaves), iters = a.pcg_iters, nparts = solve_parts(a);
    const int row0 = at.tile * kRows;
    const uint16_t* loc = kWaves == 4 ? a.loc4 : a.loc8;
    const int* halo = (kWaves == 4 ? a.halo4 : a.halo8) + at.tile * kHalo;
    const int part = at.tile * kWaves + wave;
    // (a wait of the frame already given up: this launch waits for nothing)
    int* const flags = a.flags;
    const int given_up = tid == 0 ? agent_load(flags + 1) : 0;

    // Loads that need no other load's result first: the local columns and the
    // blocks of the wave's 8 rows (slots grp and grp + 8 in registers), the
    // foreign nodes' numbers, the own node's state.
    const bool own = row0 + gi < a.nn && sub < 6;
    const int sl = sub < 6 ? sub : 0;
    unsigned lcol[8][3];
    float h[8][2][6];
    int node[kSets];                                   // set m of lane group gi is local node 32 m + gi: the own
#pragma unroll                                         // row, then foreign columns
    for (int m = 0; m < kSets; ++m) {
        const int l = m * kRows + gi;
        node[m] = m == 0 ? (row0 + gi < a.nn ? row0 + gi : -1) : gld(halo + l - kRows);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = row0 + 8 * wave + j;
        const size_t e0 = (size_t)(row < a.nn ? row : a.nn - 1) * a.ell_w;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int f = grp + 8 * s;
            lcol[j][s] = gld(loc + e0 + (f < a.ell_w ? f : 0));
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int f = grp + 8 * s;
            const float2* B = reinterpret_cast<const float2*>(a.Hf + (e0 + (f < a.ell_w ? f : 0)) * 36 + sl * 6);
            const float2 q0 = gld2(B), q1 = gld2(B + 1), q2 = gld2(B + 2);
            h[j][s][0] = q0.x; h[j][s][1] = q0.y; h[j][s][2] = q1.x;
            h[j][s][3] = q1.y; h[j][s][4] = q2.x; h[j][s][5] = q2.y;
        }
    }
    double rho_own = part < nparts ? gld(a.part_rho.b0 + part) : 0.0;
    // the local nodes' state, which needs their numbers: z_0 = M r_0, p_{-1} = 0,
    // x = 0 (written by the fold), the inverses
    int word[kSets];                                   // the lane's exchange words in set m; -1: none
    float z0[kSets], r0[kSets];
    double mr[kSets][6];
#pragma unroll
    for (int m = 0; m < kSets; ++m) {
        word[m] = -1;
        z0[m] = r0[m] = 0.f;
#pragma unroll
        for (int j = 0; j < 6; ++j) mr[m][j] = 0.0;    // (a row past the last node stays zero)
        if (node[m] >= 0 && sub < 6) {
            word[m] = (6 * node[m] + sub) * 2;
            z0[m] = gld(a.z.b0 + 6 * node[m] + sub);
            r0[m] = gld(a.r.b0 + 6 * node[m] + sub);
#pragma unroll
            for (int j = 0; j < 6; ++j) mr[m][j] = gld(a.Minv + (size_t)node[m] * 36 + sub * 6 + j);
        }
    }
    const int nlocal = kRows + gld((kWaves == 4 ? a.halo_n4 : a.halo_n8) + at.tile);
    // a slot that is not in use is a zero block on the zero node; local columns packed 9 bits each
    unsigned col[8];
    unsigned farx[2];                                  // rows' blocks from slot 16 on in LDS, 8 bits each
    farx[0] = farx[1] = (unsigned)(kWaves * kPcgFar) * 0x01010101u;
    unsigned third = 0;                                // rows with a slot from 16 on (uniform over the wave)
    int nfar = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = row0 + 8 * wave + j;
        col[j] = 0;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const bool use = row < a.nn && grp + 8 * s < a.ell_w && lcol[j][s] != (unsigned)kNone;
            col[j] |= (use ? lcol[j][s] : (unsigned)kLocal) << (9 * s);
            if (s < 2) {
#pragma unroll
                for (int c = 0; c < 6; ++c) h[j][s][c] = use ? h[j][s][c] : 0.f;
            } else {
                // the few slots from 16 on: to LDS, in the order of the rows
                const u64 m = __ballot(use && sub == 0);
                if (m == 0) continue;
                third |= 1u << j;
                const unsigned at_far = wave * kPcgFar + nfar + __popcll(m & ((1ull << base) - 1ull));
                if (use) farx[j / 4] ^= (at_far ^ (unsigned)(kWaves * kPcgFar)) << (8 * (j % 4));
                if (use && sub < 6) {
                    const float2* B = reinterpret_cast<const float2*>(
                        a.Hf + ((size_t)row * a.ell_w + grp + 16) * 36 + sub * 6);
                    float2* dst = far[at_far] + 3 * sub;
                    dst[0] = gld2(B); dst[1] = gld2(B + 1); dst[2] = gld2(B + 2);
                }
                nfar += __popcll(m);
            }
        }
    }
    float z = z0[0], p = 0.f, r = r0[0], x = 0.f;
#pragma unroll
    for (int m = 0; m < kSets; ++m) {
        const int l = m * kRows + gi;
        if (sub < 6) {
#pragma unroll
            for (int j = 0; j < 6; ++j) minv[l * 36 + sub * 6 + j] = mr[m][j];
        }
        put_vec(vec + l * kVecStride, sub, z0[m], 0.f);
        res[l * 8 + sub] = r0[m];
    }
    if (tid < 4) vec[kLocal * kVecStride + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < 18) far[kWaves * kPcgFar][tid] = make_float2(0.f, 0.f);
    const unsigned tag0 = (unsigned)__builtin_amdgcn_readfirstlane(gld(a.xepoch)) * (unsigned)kPcgTags + 1u;
    double rho_prev = 0.0;
    float4 nq = make_float4(0.f, 0.f, 0.f, 0.f), nt = nq, npos = nq;
    const size_t part_words = pcg_part_words(a);      // of one copy
    const int copy = at.tile % kPcgCopies;
    const long long t_limit = a.pcg_wait;
    if (tid == 0) stalled = given_up;
    __syncthreads();

    for (int i = 0; i < iters; ++i) {
        // the lane's numbers formed anew in every iteration, so that none of
        // the addresses that follow from them stays in a register across it
        int tl = tid;
        asm volatile("" : "+v"(tl));
        const int lane = tl % kWave, sub = lane & 7, grp = lane >> 3, gi = tl >> 3, quad = lane & 3;
        const int sl = sub < 6 ? sub : 0;
        const int par = i & 1;
        const unsigned tag = tag0 + (unsigned)i;
        const bool last = i == iters - 1;
        u64* xp = a.xpart + (size_t)par * kPcgCopies * part_words;
        u64* xu = a.xuv + (size_t)par * a.nn * 12;
        // u = A z_i, v = A p_{i-1} of the wave's rows
        float au[8], av[8];
        float4 c[2][2][2];                             // two rows' columns while the next two's are on their way
        auto fetch = [&](int j) {
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                asm volatile("" : "+v"(col[j + n]));   // (its addresses are formed anew, not kept)
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    c[(j / 2) & 1][n][s] = vec[((col[j + n] >> (9 * s)) & 511u) * kVecStride + quad];
            }
        };
        fetch(0);
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            if (j + 2 < 8) fetch(j + 2);
            __builtin_amdgcn_sched_barrier(0);
            au[j] = av[j] = au[j + 1] = av[j + 1] = 0.f;
#pragma unroll
            for (int s = 0; s < 2; ++s)
                slot_step2(au[j], av[j], au[j + 1], av[j + 1], h[j][s], h[j + 1][s], c[(j / 2) & 1][0][s],
                           c[(j / 2) & 1][1][s]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // slots from 16 on, four rows at a time (blocks from LDS; an unused one is the zero block on the zero node)
#pragma unroll
        for (int j0 = 0; j0 < 8; j0 += 4) {
            if (((third >> j0) & 15u) == 0u) continue;
            float hb[4][6];
            float4 cb[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2* B = far[(farx[j0 / 4] >> (8 * j)) & 255u] + 3 * sl;
                const float2 q0 = B[0], q1 = B[1], q2 = B[2];
                hb[j][0] = q0.x; hb[j][1] = q0.y; hb[j][2] = q1.x; hb[j][3] = q1.y; hb[j][4] = q2.x; hb[j][5] = q2.y;
                cb[j] = vec[((col[j0 + j] >> 18) & 511u) * kVecStride + quad];
            }
#pragma unroll
            for (int j = 0; j < 4; j += 2)
                slot_step2(au[j0 + j], av[j0 + j], au[j0 + j + 1], av[j0 + j + 1], hb[j], hb[j + 1], cb[j], cb[j + 1]);
        }
        // lane group grp now takes row grp of the wave: its own node (set 0)
        float u = group_rows(au, lane), v = group_rows(av, lane);
        u = own ? u : 0.f;
        v = own ? v : 0.f;
        if (ntiles > 1 && own && !last) {
            xchg_store(xu + word[0], tag, __float_as_uint(u));
            xchg_store(xu + word[0] + 1, tag, __float_as_uint(v));
        }
        // the row's three products, then the in-order sums of the wave's 8 rows
        const double c1 = low6_sum((double)z * (double)u);
        const double c2 = low6_sum((double)z * (double)v + (double)p * (double)u);
        const double c3 = low6_sum((double)p * (double)v);
        if (sub < 3) rowdot[wave][sub][grp] = sub == 0 ? c1 : (sub == 1 ? c2 : c3);
        wave_fence();
        if (lane < 8 * kPcgCopies) {
            const int q = (lane >> 1) & 3;             // of 8 lanes, 2 q and 2 q + 1: the low and high half of value q
            double d = rho_own;
            if (q > 0) {
                d = 0.0;
#pragma unroll
                for (int w = 0; w < 8; ++w) d += rowdot[wave][q - 1][w];
            }
            const u64 bits = (u64)__double_as_longlong(d);
            if (ntiles == 1) {
                if ((lane & 1) == 0 && lane < 8) red[wave][q] = d;  // (the parts of a single workgroup stay in LDS)
            } else if (part < nparts) {
                xchg_store(xp + (lane >> 3) * part_words + pcg_part_word(part, lane & 7), tag,
                           (unsigned)((lane & 1) ? bits >> 32 : bits));
            }
        }
        if (last && sub == 0 && row0 + gi < a.nn) {    // (for the node update, while the others' words are on their way)
            nq = gld4(a.rq + row0 + gi);
            nt = gld4(a.tt + row0 + gi);
            npos = gld4(a.pref + row0 + gi);
        }
        // the index map of the next Gauss-Newton iteration (this one's is done
        // with), while the others' words are on their way
        if (i == 0) reset_index_map(a, at.tile, ntiles);
        // the sums of all parts (thread t: parts t, t + 256, ...) and u, v of the foreign columns
        double sum[kValues];
#pragma unroll
        for (int q = 0; q < kValues; ++q) sum[q] = 0.0;
        const int leaf = tl & 255, v0 = kWaves == 8 ? (wave >> 2) * kValues : 0;   // the thread's leaf and first value
        u32x4 wuv[kSets] = {};
        const XchgBuf bp = xchg_buffer(xp + copy * part_words, part_words), bu = xchg_buffer(xu, (size_t)a.nn * 12);
        if (ntiles == 1) {
            __syncthreads();
            if (leaf < nparts) {
#pragma unroll
                for (int q = 0; q < kValues; ++q) sum[q] += red[leaf][v0 + q];
            }
            __syncthreads();
        } else {
            long long t0 = 0;
            for (int p0 = 0; p0 < nparts; p0 += 256 * kLeafParts) {
                u32x4 ws[kLeafParts][kValues];
                // what the lane still waits for: its parts (bits 30, 31), its columns (bit m); only that is read again
                unsigned need = 0u;
#pragma unroll
                for (int g = 0; g < kLeafParts; ++g)
                    if (p0 + 256 * g + leaf < nparts) need |= kPartBit << g;
#pragma unroll
                for (int m = 1; m < kSets; ++m)
                    if (p0 == 0 && !last && word[m] >= 0) need |= 1u << m;
                for (int spin = 0;; ++spin) {
                    asm volatile("" ::: "memory");   // (every round reads anew)
                    // (the flag's load goes out with the words')
                    const bool look = (spin & 15) == 15 || t_limit < 0;
                    const int raised = look ? agent_load(flags + 1) : 0;
#pragma unroll
                    for (int g = 0; g < kLeafParts; ++g)
                        if (need & (kPartBit << g)) {
                            const int wp = (int)pcg_part_word(p0 + 256 * g + leaf, 2 * v0);
#pragma unroll
                            for (int q = 0; q < kValues; ++q) ws[g][q] = xchg_load2(bp, wp + 8 * q);
                        }
#pragma unroll
                    for (int m = 1; m < kSets; ++m)
                        if ((need >> m) & 1u) wuv[m] = xchg_load2(bu, word[m]);
#pragma unroll
                    for (int g = 0; g < kLeafParts; ++g)
                        if (need & (kPartBit << g)) {
                            unsigned miss = 0;
#pragma unroll
                            for (int q = 0; q < kValues; ++q) miss |= (ws[g][q].y ^ tag) | (ws[g][q].w ^ tag);
                            if (miss == 0u) need &= ~(kPartBit << g);
                        }
#pragma unroll
                    for (int m = 1; m < kSets; ++m)
                        if ((need >> m) & 1u) {
                            if (((wuv[m].y ^ tag) | (wuv[m].w ^ tag)) == 0u) need &= ~(1u << m);
                        }
                    if (__ballot(need != 0u) == 0) break;
                    if (look) {
                        // bounded: nobody waits past the limit, and nobody of the frame once one has
                        const long long now = wall_clock64();
                        if (t0 == 0) t0 = now;
                        if (raised != 0) {
                            *(volatile int*)&stalled = 1;
                        } else if (now - t0 > t_limit) {
                            *(volatile int*)&stalled = 1;
                            if (lane == 0) atomicAdd(flags + 1, 1);
                        }
                    }
                    if (*(volatile int*)&stalled != 0) break;
                }
#pragma unroll
                for (int g = 0; g < kLeafParts; ++g)
                    if (p0 + 256 * g + leaf < nparts) {
#pragma unroll
                        for (int q = 0; q < kValues; ++q)
                            sum[q] += __longlong_as_double((long long)(((u64)ws[g][q].z << 32) | ws[g][q].x));
                    }
            }
        }
        {
            if constexpr (kWaves == 4) {
                const double t = wave_sum4(sum);
                if ((lane & 15) == 0) red[wave][((lane >> 5) & 1) | ((lane >> 3) & 2)] = t;
            } else {
                const double t = wave_sum2(sum[0], sum[1]);
                if ((lane & 31) == 0) red[wave & 3][v0 + (lane >> 5)] = t;
            }
        }
        __syncthreads();
        double tot[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            tot[q] = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) tot[q] += red[w][q];
        }
        const PcgScalars s = pcg_scalars_of(i, tot[0], tot[1], tot[2], tot[3], rho_prev);
        rho_prev = tot[0];
        // finish of iteration i: the own node and (for the next products) the
        // foreign columns, a few sets side by side
#pragma unroll
        for (int m0 = 0; m0 < kSets; m0 += kTogether) {
            if (m0 * kRows >= nlocal) break;
            double mrow[kTogether][6];
            float zk[kTogether], pk[kTogether], rk[kTogether];
#pragma unroll
            for (int n = 0; n < kTogether && m0 + n < kSets; ++n) {
                // (a lane group without a node in the set works on what its place
                // holds, which no product reads)
                const int m = m0 + n, l = m * kRows + gi;
#pragma unroll
                for (int j = 0; j < 6; ++j) mrow[n][j] = minv[l * 36 + sl * 6 + j];
                if (m == 0) {
                    zk[0] = z; pk[0] = p; rk[0] = r;
                } else {
                    const float2 zp = get_vec(vec + l * kVecStride, sub);
                    zk[n] = zp.x; pk[n] = zp.y; rk[n] = res[l * 8 + sub];
                }
            }
#pragma unroll
            for (int n = 0; n < kTogether && m0 + n < kSets; ++n) {
                const int m = m0 + n, l = m * kRows + gi;
                const float um = m == 0 ? u : __uint_as_float(wuv[m].x), vm = m == 0 ? v : __uint_as_float(wuv[m].z);
                const Finished f = finish_lane(zk[n], pk[n], um, vm, rk[n], x, mrow[n], s);
                if (m == 0) { z = f.z; p = f.p; r = f.r; x = f.x; }
                put_vec(vec + l * kVecStride, sub, f.z, f.p);
                if (m > 0) res[l * 8 + sub] = f.r;
            }
            __builtin_amdgcn_sched_barrier(0);         // (more sets at once would not fit the registers)
        }
        rho_own = wave_sum(own ? (double)r * (double)z : 0.0);
        __syncthreads();
    }
    // the stream's last finish: |r|^2 partials, x, the node update (the
    // descriptor read anew: its pointers need not stay in registers through
    // the iterations)
    const FrameDesc* dp = b.d[at.s];
    asm volatile("" : "+s"(dp));
    const FrameDesc e = *dp;
    const double rr = wave_sum(own ? (double)r * (double)r : 0.0);
    if (lane == 0 && part < nparts) by_parity(e.part_rr, iters & 1)[part] = rr;
    if (own) e.x[6 * (row0 + gi) + sub] = x;
    float xs[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) xs[j] = bcast8(x, j);
    if (sub == 0 && row0 + gi < e.nn) update_node_x(e, row0 + gi, xs, nq, nt, npos);
}

}  // namespace

void launch_pcg_solve(const Batch& b, hipStream_t st) {
    const int grid = b.off[b.n];
    if (grid <= 0) return;
    // (most node sets need few sets; the kernels for more hold fewer of them side by side)
    static_assert(kPcgPairSets == 5, "the sets of the kernels below");
    if (b.wide) {
        if (b.sets <= 4) hipLaunchKernelGGL((k_pcg_solve<8, 4>), dim3(grid), dim3(512), 0, st, b);
        else hipLaunchKernelGGL((k_pcg_solve<8, 5>), dim3(grid), dim3(512), 0, st, b);
    } else {
        if (b.sets <= 4) hipLaunchKernelGGL((k_pcg_solve<4, 4>), dim3(grid), dim3(256), 0, st, b);
        else if (b.sets <= 5) hipLaunchKernelGGL((k_pcg_solve<4, 5>), dim3(grid), dim3(256), 0, st, b);
        else hipLaunchKernelGGL((k_pcg_solve<4, 8>), dim3(grid), dim3(256), 0, st, b);
    }
}

void pcg_workgroups_per_cu(int& pair, int& alone) {
    auto least = [](std::initializer_list<const void*> kernels, int threads) {
        int n = 1 << 20;
        for (const void* k : kernels) {
            int m = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&m, k, threads, 0) != hipSuccess) m = 0;
            n = m < n ? m : n;
        }
        return n;
    };
    pair = least({(const void*)k_pcg_solve<4, 4>, (const void*)k_pcg_solve<4, 5>}, 256);
    const int many = least({(const void*)k_pcg_solve<4, 8>}, 256);
    alone = least({(const void*)k_pcg_solve<8, 4>, (const void*)k_pcg_solve<8, 5>}, 512);
    alone = many < alone ? many : alone;
}

}  // namespace swgn
