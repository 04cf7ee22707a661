// Host-side launchers of the setup kernels and the node-state helpers; the
// per-frame stages are launched through swgn_frame.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace swgn {

// setup
// 4 nearest nodes (caller indices) and weights of every surfel; nodes in the
// library's order with their caller indices; boxes holds knn_box_count(nn)
// float4 of scratch.
void launch_knn_skin(int ns, const float* pos_aos, int nn, const float4* nodes, const int* caller, float4* boxes,
                     float inv_two_sigma2, int4* idx, float4* w, hipStream_t st);
// *lone is set if some node has fewer than 8 others at a finite distance
void launch_node_graph(int nn, const float4* nodes, int* nbr, int* lone, hipStream_t st);
void sort_pairs(uint64_t* key, uint32_t* val, int n_pow2, hipStream_t st);
// in[n] -> out[n + 1], out[n] = the total; tmp (scan_tmp_size(n) ints) is read until the last launch ends
void exclusive_scan(const int* in, int* out, int n, int* tmp, hipStream_t st);
// two arrays of one length (2 scan_tmp_size(n) ints of scratch)
void exclusive_scan2(const int* in0, int* out0, const int* in1, int* out1, int n, int* tmp, hipStream_t st);
size_t scan_tmp_size(int n);
// Renumbers idx (caller's numbers to inv's) and sorts the surfels by (node
// set, number) into key, val; key_in[ns] and work (bucket_work_ints(ns) ints) are
// scratch. *over is set if they have to be sorted by sort_pairs instead.
size_t bucket_work_ints(int ns);
void launch_bucket_sort(int ns, int nn, int4* idx, const int* inv, uint64_t* key_in, int* work, uint64_t* key,
                        uint32_t* val, int* over, hipStream_t st);
void launch_tuple_keys(int ns, int npad, const int4* idx, uint64_t* key, uint32_t* val, hipStream_t st);
void launch_permute_surfels(int ns, const int* over, const uint64_t* key, const uint32_t* val, const float* ipos, const float* inrm,
                            const int4* iidx, const float4* iw, float* px, float* py, float* pz, float* nx,
                            float* ny, float* nz, int4* oidx, float4* ow, int* orig, int* flag, hipStream_t st);
// first surfel and node set of every run of equal node sets (run_pos[ns] runs)
void launch_run_starts(int ns, const int* flag, const int* pos, const uint64_t* key, int* run_start,
                       uint64_t* run_key, hipStream_t st);
// bitmaps (zero before) of the full block rows and of the in-edges
void launch_pattern(int ns, const uint64_t* key, const int* flag, int nn, const int* nbr, uint32_t* bm,
                    uint32_t* in_bm, int words, hipStream_t st);
// counts per row, their scans (row_ptr, in_ptr: [nn + 1]) and the longest full row
void launch_row_counts(int nn, const uint32_t* bm, const uint32_t* in_bm, int words, int* upper, int* full,
                       int* in_cnt, int* row_ptr, int* in_ptr, int* longest, hipStream_t st);
void launch_row_fill(int nn, const uint32_t* bm, const uint32_t* in_bm, int words, const int* row_ptr,
                     const int* in_ptr, int* col_idx, int* blk_row, int* offlist, int* in_list, hipStream_t st);
void launch_ell(int nn, int ell_w, const uint32_t* bm, int words, const int* row_ptr, const int* full,
                const int* col_idx, uint32_t* ell_blk, int* ell_col, int* slot_u, int* slot_t, hipStream_t st);
void launch_map_graph(int nn, const int* nbr_call, const int* perm, const int* inv, int* nbr, hipStream_t st);

// what the host has to know of a setup's sizes, written to pinned host memory
constexpr int kInfo = 8;
struct InfoList {
    const int* p[kInfo];
};
void launch_info(const InfoList& l, int* out, hipStream_t st);

// the whole-solve kernel's local columns and foreign nodes per workgroup of
// 4 or 8 waves;
// need (zero before) becomes the largest number of foreign nodes, or a number
// beyond any when a wave's slots from 16 on are more than the kernel holds
void launch_pcg_local(int waves, int nn, int ell_w, const uint32_t* ell_blk, const int* ell_col, uint16_t* loc,
                      int* halo, int* halo_n, int* need, hipStream_t st);

// node state and capture helpers
void launch_nodes_from_se3(int nn, const float* se3, const float4* pref, float4* rq, float4* tt, float4* dq,
                           float4* cl, hipStream_t st);
void launch_node_se3_out(int nn, const float4* rq, const float4* tt, const int* caller, float4* out, hipStream_t st);
void launch_export_index_map(int npx, const unsigned long long* z, int* out, hipStream_t st);
void launch_positions_to_f4(int n, const float* pos, float4* out, hipStream_t st);

}  // namespace swgn

namespace swgn {
void launch_fill_i32(int* p, int n, int v, hipStream_t st);
void launch_tables_from_state(int nn, const float4* pref, const float4* rq, const float4* tt, float4* dq, float4* cl,
                              hipStream_t st);
}  // namespace swgn
