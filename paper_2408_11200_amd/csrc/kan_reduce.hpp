// Last stage of the parameter gradients, for every layer kind and window width (plain argument types).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kan {

// What the segments of a sorted list left behind for the rows of the segment after them (kan_walk.hip): carry row s of
// segment k of list l belongs to table row seg_row[l * n_seg + k] + s, s < window.  n_seg == 1: nothing.
struct CarryRows {
    const int *seg_row;
    const float *carry;
    int n_seg;
    int window;
};

// Sums n_chunks partial tables part_c[c][n_in][rows][n_out] (with their carry rows) and n_slices_b slices part_b[s][n_in][n_out]
// (may be null) in fp64 and writes
//   gcoef = w_s * sum,   gw_s = sum over rows of coef * sum,   gw_b = sum of the slices (zero without)
// Any of the three may be null.  scratch: reduce_scratch_bytes(...) bytes, or null (then the rows of an edge are not split).
size_t reduce_scratch_bytes(int n_in, int rows, int n_out);
hipError_t launch_dparam_reduce(const float *part_c, const float *part_b, const CarryRows &cr, const float *coef,
                                const float *w_s, float *gcoef, float *gw_s, float *gw_b, int n_in, int rows, int n_out,
                                int n_chunks, int n_slices_b, void *scratch, hipStream_t st);

}  // namespace kan
