// Device code shared by the step-wise PCG kernels (solve.hip) and the kernel
// that runs a whole linear solve (pcg.hip): the finish of an iteration, the
// scalars, the node update of a stream's last finish. Both evaluate the same
// operations in the same order, so they agree bit for bit.
#pragma once

#include "swgn_frame.h"
#include "swgn_impl.h"

namespace swgn {

// T_k <- Delta_k(x) o T_k from the node's state q, t4 and reference position p.
__device__ __forceinline__ void update_node_x(const FrameDesc& a, int k, const float (&x)[6], float4 q4f, float4 t4,
                                              float4 p) {
    float3 w = make_float3(x[0], x[1], x[2]);
    float3 tau = make_float3(x[3], x[4], x[5]);
    float th = sqrtf(dot3(w, w));
    Q4 e;
    if (th < 1e-8f) {
        e = Q4{1.f, 0.5f * w.x, 0.5f * w.y, 0.5f * w.z};
    } else {
        float sn, cs;
        sincosf(0.5f * th, &sn, &cs);
        float sc = sn / th;
        e = Q4{cs, sc * w.x, sc * w.y, sc * w.z};
    }
    float en = sqrtf(((e.w * e.w + e.x * e.x) + e.y * e.y) + e.z * e.z);
    e = Q4{e.w / en, e.x / en, e.y / en, e.z / en};
    Q4 r = q4(q4f);
    float3 t = make_float3(t4.x, t4.y, t4.z);
    float3 c = add3(qrot(r.w, make_float3(r.x, r.y, r.z), make_float3(p.x, p.y, p.z)), t);
    Q4 rn = qmul(e, r);
    float nr = sqrtf(((rn.w * rn.w + rn.x * rn.x) + rn.y * rn.y) + rn.z * rn.z);
    float sg = rn.w < 0.f ? -1.f : 1.f;
    rn = Q4{sg * rn.w / nr, sg * rn.x / nr, sg * rn.y / nr, sg * rn.z / nr};
    float3 tn = add3(add3(qrot(e.w, make_float3(e.x, e.y, e.z), sub3(t, c)), c), tau);
    bool fin = fabsf(rn.w) <= 1.f && fabsf(tn.x) < INFINITY && fabsf(tn.y) < INFINITY && fabsf(tn.z) < INFINITY;
    if (!fin) atomicOr(a.flags, 4);
    a.rq[k] = f4(rn);
    a.tt[k] = make_float4(tn.x, tn.y, tn.z, 0.f);
    node_tables(p, rn, tn, a.dq, a.cl, k);
}

// Index map of the next iteration: tile `tile` of a launch with `ntiles`
// tiles for the stream clears its share of the pixels.
__device__ __forceinline__ void reset_index_map(const FrameDesc& a, int tile, int ntiles) {
    const int chunk = cdiv(a.npx, ntiles);
    const int p0 = tile * chunk, p1 = min(a.npx, p0 + chunk);
    for (int p = p0 + (int)threadIdx.x; p < p1; p += (int)blockDim.x) a.zbuf[p] = ~0ull;
}

// The node update of a stream's last PCG finish, inside the finishing lane
// group (lane c holds component c of x_k): the group's 6 entries of x to
// every lane, lane 0 moves node k.
__device__ __forceinline__ void update_from_lanes(const FrameDesc& a, int k, int c, float xc) {
    float x[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) x[j] = bcast8(xc, j);
    if (c == 0 && k < a.nn) update_node_x(a, k, x, a.rq[k], a.tt[k], a.pref[k]);
}


struct PcgScalars {
    float alpha, beta;
};

// beta_k and alpha_k from the sums of iteration k (rho = r_k.z_k, c1 = z.u,
// c2 = z.v + p.u, c3 = p.v) and rho_{k-1}.
__device__ __forceinline__ PcgScalars pcg_scalars_of(int k, double rho, double c1, double c2, double c3,
                                                     double rho_prev) {
    const bool stop = (rho == 0.0);
    const float beta = (k > 0 && !stop) ? (float)(rho / rho_prev) : 0.f;
    const double bd = (double)beta;
    const double pq = (c1 + bd * c2) + (bd * bd) * c3;
    const float alpha = stop ? 0.f : (float)(rho / pq);
    return PcgScalars{alpha, beta};
}

// Lane C (of 4) of each quad, to the whole quad (bound_ctrl set, so that the
// move can fold into the instruction that uses it).
template <int C>
__device__ __forceinline__ float quad_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), C * 0x55, 0xF, 0xF, true));
}

// The finish of iteration k for one component of one node (8 lanes per node,
// component c = lane & 7 < 6, lanes 6 and 7 carry zeros): p_k, r_{k+1},
// z_{k+1} = M r_{k+1} (FP64 sum of the node's 6 entries, read by DPP within
// the lane group) and x_{k+1}. A fused step repeats the same
// operations for the nodes of its rows' columns, so both agree bit for bit.
struct Finished {
    float p, r, z, x;
};

__device__ __forceinline__ Finished finish_lane(float zk, float pprev, float uk, float vk, float rk, float xk,
                                                const double (&mrow)[6], PcgScalars s) {
    Finished f;
    f.p = zk + s.beta * pprev;
    const float q = uk + s.beta * vk;
    f.x = xk + s.alpha * f.p;
    f.r = rk - s.alpha * q;
    // the group's r, components 0-3 and 4, 5 in each quad, then by quad broadcasts
    const int ri = __float_as_int(f.r);
    const float lo = __int_as_float(dpp_mov<0x114, 0xA>(ri, ri)), hi = __int_as_float(dpp_mov<0x104, 0x5>(ri, ri));
    double zc = 0.0;
    zc += mrow[0] * (double)quad_bcast<0>(lo);
    zc += mrow[1] * (double)quad_bcast<1>(lo);
    zc += mrow[2] * (double)quad_bcast<2>(lo);
    zc += mrow[3] * (double)quad_bcast<3>(lo);
    zc += mrow[4] * (double)quad_bcast<0>(hi);
    zc += mrow[5] * (double)quad_bcast<1>(hi);
    f.z = (float)zc;
    return f;
}

// Sum of a value that only lanes 0-5 hold (every other lane holds +0): the
// value the wave butterfly 32, 16, ..., 1 gives, valid in lanes 0-7. Its
// first three steps only add +0, which turns -0 into +0, as one addition of
// +0 does.
__device__ __forceinline__ double low6_sum(double v) {
    v += 0.0;
    v += xchg<4>(v);
    v += xchg<2>(v);
    v += xchg<1>(v);
    return v;
}

}  // namespace swgn
