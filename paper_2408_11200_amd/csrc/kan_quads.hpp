// Walk over cell lists whose cells are padded to groups of four samples ("quads"): arguments and launch functions
// (plain types; the kernels are built for windows of four and of six rows, kan_quads_kernel.hpp).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kan {

// Sorted lists of one (chunk, input) each, L entries apart: the samples of the chunk ordered by window row (equal rows in
// batch order), every row's run filled up to a multiple of four with kQuadPad entries.
constexpr unsigned kQuadPad = 0xffffu;
struct CellLists {
    float *x;                   // the sample's input value
    uint16_t *sample;           // its index in the chunk, or kQuadPad
    int *n_quads;               // [chunk][input]: entries in use / 4
    int L;
};

struct QuadWalkArgs {
    // the layer (SplineGeom)
    int n_in, n_out, rows, slab_rows, k;
    float lo, inv_h;
    const int32_t *cell_base;
    int base_act;
    CellLists lists;
    const float *gy, *cf, *w_b;
    float *part_c, *part_b, *gx;        // part_c, part_b, gx may be null
    float *carry;
    int *seg_row;
    int64_t B;
    int S, n_seg, n_jt;
    int chunk0, n_chunks;               // chunks of this launch
    int blocks_per_chunk, xcd_groups;
    int prezeroed, shared;
};

// entries a list may need: S samples in at most min(S, window rows) runs
inline int quad_list_entries(int S, int rows, int window)
{
    const int cells = rows - window + 1 < S ? rows - window + 1 : S;
    return (S + 3 * cells + 63) / 64 * 64;
}

hipError_t launch_cell_lists(const QuadWalkArgs &a, const float *xT, int row_bits, hipStream_t st);
hipError_t launch_cell_lists6(const QuadWalkArgs &a, const float *xT, int row_bits, hipStream_t st);

// layers of one output: one launch over all chunks, lists of one segment
constexpr int kOneWaves = 8;
inline size_t walk_one_lds_bytes(int rows, int S) { return ((size_t)4 * kOneWaves * (rows - 3) + S + rows) * sizeof(float); }
hipError_t walk_one(const QuadWalkArgs &a, hipStream_t st);

// name: streams a wave, outputs a lane; 6: window of six rows (degrees 4 and 5)
void quad_walk_s1t8(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk_s1t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk_s2t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk_s4t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk_s4t2(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk_s4t1(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk6_s1t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk6_s2t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk6_s4t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk6_s4t2(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);
void quad_walk6_s4t1(const QuadWalkArgs &a, unsigned blocks, hipStream_t st);

}  // namespace kan
