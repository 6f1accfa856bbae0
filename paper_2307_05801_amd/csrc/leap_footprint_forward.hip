// The column-wise footprint forward kernels, a bundle per wave.
#include <hip/hip_runtime.h>

#include "sf_project_launch.h"

bool leap_launch_footprint_slab(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    if (G->fp_parts > 1) return leap_launch_footprint_slab_parts(G, S, slab, d_sino, stream, items);
    return launch_fp_slab<1>(G, S, slab, d_sino, stream, items);
}
