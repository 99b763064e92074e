// Cell lists of the quad walk, windows of four rows (kan_cells_kernel.hpp).
#include "kan_cells_kernel.hpp"

namespace kan {

hipError_t launch_cell_lists(const QuadWalkArgs &a, const float *xT, int row_bits, hipStream_t st)
{
    return launch_cell_list_by_size(a, xT, row_bits, st);
}

}  // namespace kan
