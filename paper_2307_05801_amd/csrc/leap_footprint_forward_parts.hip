// The column-wise footprint forward kernels, a bundle's layers shared by the waves of a workgroup.
#include <hip/hip_runtime.h>

#include "sf_project_launch.h"

bool leap_launch_footprint_slab_parts(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, int waves, float *d_sino, hipStream_t stream, int items)
{
    return launch_fp_slab<FP_PARTS>(G, S, slab, waves, d_sino, stream, items);
}
