// backward_walk_kernel with 1 stream per wave and 4 outputs per lane (see kan_walk.hip).
#include "kan_walk_kernel.hpp"

namespace kan {

void walk_launch_s1t4_ragged(bool dx, unsigned blocks, hipStream_t st, const SplineGeom &g, const WalkRecords &rec,
                      const float *gy, const float *cf, const float *w_b, float *part_c, float *part_b, float *gx,
                      int64_t B, const WalkPlan &p, int bpc, int m, int prezeroed, float *carry, int *seg_row, int chunk0,
                      int n_chunks)
{
    walk_launch<1, 4, true>(dx, blocks, st, g, rec, gy, cf, w_b, part_c, part_b, gx, B, p, bpc, m, prezeroed, carry, seg_row, chunk0,
                      n_chunks);
}

}  // namespace kan
