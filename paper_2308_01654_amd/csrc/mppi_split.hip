// The split iteration kernel (mppi_split.hpp) at 16 lanes per sample.
#include "mppi_split.hpp"

namespace mppi_impl {

hipError_t launch_split(int lanes, int ne, int model, int per_step, const InstDesc* d0, const BatchHdr* hdr_dev,
                        int cls, int grid, size_t smem, hipStream_t stream)
{
    if (lanes != 16) return launch_split_wide(lanes, ne, model, d0, hdr_dev, cls, grid, smem, stream);
    return per_step ? launch_split_g<16, true>(ne, model, d0, hdr_dev, cls, grid, smem, stream)
                    : launch_split_g<16, false>(ne, model, d0, hdr_dev, cls, grid, smem, stream);
}

}  // namespace mppi_impl
