// Launchers of the setup kernels that build the segment layout on the device
// (setup.hip, segwalk.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swgn {

// pos4[i]: positions (3 bits each, slot order) of surfel i's nodes among the
// 5 nodes of its segment (seg_start[nseg + 1], seg_nodes[5 nseg]); *bad is set
// if a node is missing.
void launch_seg_pos4(int ns, int nseg, const int* seg_start, const int* seg_nodes, const int4* idx, uint16_t* pos4,
                     int* bad, hipStream_t st);

// Successor chains: for next[i] with i < next[i] <= min(n, i + M) (M at most
// chain_max_hop()), out[0 .. *count) = 0, next[0], next[next[0]], ... (every
// position below n the chain from 0 visits). work holds chain_work_ints(n, M)
// ints; *bad is set if next breaks the rule (out and *count are then not the
// chain).
size_t chain_work_ints(int n, int M);
int chain_max_hop();
void chain_from_zero(const int* next, int n, int M, int* out, int* count, int* work, int* bad, hipStream_t st);

// next[s]: the surfel where the greedy segment opening at surfel s ends (at
// most M surfels, at most 5 nodes; runs of equal node sets from set_start[] with
// node sets set_key[]; run_pos[ns + 1] the exclusive scan of the run-start
// flags, so run_pos[ns] runs).
void launch_seg_next(int ns, const uint64_t* set_key, const int* set_start, const int* run_pos, int M,
                     int* next, hipStream_t st);

// next[g]: the segment where the greedy pack of at most M surfels opening at
// segment g ends.
void launch_pack_next(int nseg, const int* seg_start, int M, int* next, hipStream_t st);

// Per segment: nodes (5, ascending, -1 padded), pair mask, Gram output size
// in 4-float units and pair count; *total_units accumulates the sizes (64-bit);
// *bad is set for a segment of more than 5 nodes.
void launch_seg_info(int nseg, const int* seg_start, const int* run_pos, const uint64_t* set_key, int* seg_nodes,
                     uint16_t* mask, int* units, int* npairs, unsigned long long* total_units, int* bad,
                     hipStream_t st);

// seg_start[0 .. nseg] = the cuts and ns.
void launch_seg_starts(int nseg, const int* cuts, int ns, int* seg_start, hipStream_t st);

// The block fold's entries: ne = sum of the pair counts, entry e of segment g
// at ebase[g] + rank, its block (-1: none, and *bad is set) and its place among
// the block's; bcount[nb] counts entries per block (zero before);
// off[g] = 4 off_units[g] for g <= nseg (float offsets from 4-float units).
void launch_seg_entries(int nseg, const int* seg_nodes, const uint16_t* mask, const int* off_units, uint32_t* off,
                        const int* ebase, const int* row_ptr, const int* col_idx, int* eblk, int* eplace,
                        uint32_t* esub, uint32_t* egrad, int* bcount, int* bad, hipStream_t st);

// ent_sub/ent_grad: the entries in block order (ent_ptr = scan of bcount),
// each block's ascending; list[ne] is scratch. *over is set where a block has too
// many for that: sort_entries gives the same from any.
void launch_ent_order(int ne, int nb, const int* eblk, const int* eplace, const int* ent_ptr, const uint32_t* esub,
                      const uint32_t* egrad, int* list, uint32_t* ent_sub, uint32_t* ent_grad, int* over,
                      hipStream_t st);
void sort_entries(int ne, int npad, const int* eblk, uint64_t* key, uint32_t* val, const uint32_t* esub,
                  const uint32_t* egrad, uint32_t* ent_sub, uint32_t* ent_grad, hipStream_t st);

// pack_seg = the cuts and nseg; pack_start[i] = seg_start[pack_seg[i]], closed by ns.
void launch_pack_arrays(int npack, int nseg, int ns, const int* cuts, const int* seg_start, int* pack_seg,
                        int* pack_start, hipStream_t st);

}  // namespace swgn
