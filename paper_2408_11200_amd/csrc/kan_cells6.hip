// Cell lists of the quad walk, windows of six rows (degrees 4 and 5; kan_cells_kernel.hpp).
#define KAN_MAXK 6
#define KAN_NS kan_k5
#include "kan_cells_kernel.hpp"

namespace kan {

hipError_t launch_cell_lists6(const QuadWalkArgs &a, const float *xT, int row_bits, hipStream_t st)
{
    return kan_k5::launch_cell_list_by_size(a, xT, row_bits, st);
}

}  // namespace kan
