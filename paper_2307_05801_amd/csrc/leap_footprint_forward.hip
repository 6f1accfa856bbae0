// The column-wise footprint forward kernels, a bundle per wave.
#include <hip/hip_runtime.h>

#include "sf_project_launch.h"

bool leap_launch_footprint_slab(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    const int n = slab.xmajor < 0 ? (G->g.nx > G->g.ny ? G->g.nx : G->g.ny) : slab.n1 - slab.n0;
    const int waves = fp_waves_for(n, 64 / G->fp_nq, G->fp_parts, G->fp_rows != 0);
    if (waves > 1) return leap_launch_footprint_slab_parts(G, S, slab, waves, d_sino, stream, items);
    return launch_fp_slab<1>(G, S, slab, 1, d_sino, stream, items);
}
