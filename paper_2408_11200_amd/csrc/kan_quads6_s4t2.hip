// quad_walk_kernel for windows of six rows (degrees 4 and 5), 4 streams per wave and 2 outputs per lane (kan_quads_kernel.hpp).
#define KAN_MAXK 6
#define KAN_NS kan_k5
#include "kan_quads_kernel.hpp"

namespace kan {

void quad_walk6_s4t2(const QuadWalkArgs &a, unsigned blocks, hipStream_t st) { kan_k5::quad_walk_launch<4, 2>(a, blocks, st); }

}  // namespace kan
