// The split iteration kernel (mppi_split.hpp) at 4 and 8 lanes per sample.
#include "mppi_split.hpp"

namespace mppi_impl {

hipError_t launch_split_wide(int lanes, int ne, int model, const InstDesc* d0, const BatchHdr* hdr_dev, int cls,
                             int grid, size_t smem, hipStream_t stream)
{
    switch (lanes) {
    case 4: return launch_split_g<4, false>(ne, model, d0, hdr_dev, cls, grid, smem, stream);
    case 8: return launch_split_g<8, false>(ne, model, d0, hdr_dev, cls, grid, smem, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mppi_impl
