// quad_walk_kernel with 4 streams per wave and 4 outputs per lane (kan_quads_kernel.hpp).
#include "kan_quads_kernel.hpp"

namespace kan {

void quad_walk_s4t4(const QuadWalkArgs &a, unsigned blocks, hipStream_t st) { quad_walk_launch<4, 4>(a, blocks, st); }

}  // namespace kan
