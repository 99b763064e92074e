// quad_walk_kernel with 4 streams per wave and 1 output per lane (kan_quads_kernel.hpp).
#include "kan_quads_kernel.hpp"

namespace kan {

void quad_walk_s4t1(const QuadWalkArgs &a, unsigned blocks, hipStream_t st) { quad_walk_launch<4, 1>(a, blocks, st); }

}  // namespace kan
