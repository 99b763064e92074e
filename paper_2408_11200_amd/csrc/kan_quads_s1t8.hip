// quad_walk_kernel with 1 stream per wave and 8 outputs per lane (kan_quads_kernel.hpp).
#include "kan_quads_kernel.hpp"

namespace kan {

void quad_walk_s1t8(const QuadWalkArgs &a, unsigned blocks, hipStream_t st) { quad_walk_launch<1, 8>(a, blocks, st); }

}  // namespace kan
