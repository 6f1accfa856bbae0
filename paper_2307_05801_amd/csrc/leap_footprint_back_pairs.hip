// Launchers of the tiled footprint back projection with two volumes per workgroup (sf_backproject_tiled.h).
#include <hip/hip_runtime.h>

#include "leap_internal.h"
#include "sf_backproject_tiled.h"

template <int NC, int NV, int SH>
static bool launch_instance(const leap_geometry *G, const float *d_sino, float *d_vol, int blocks, hipStream_t stream)
{
    if constexpr (bp_pair_instance_exists(NC, NV, SH)) {
        constexpr SfBpShape S = BP_PAIR_SHAPES[SH];
        const SfGeom &g = G->g;
        const SfBpSets sets = {G->bp_mirror ? 1 : 0, G->bp_mirror ? sf_mirror_first_voxel_above(g.nz) : 0};
        const unsigned tiles_x = (unsigned)(g.nx + BP_T - 1) / BP_T, tiles_y = (unsigned)(g.ny + BP_T - 1) / BP_T;
        const dim3 grid(tiles_x * tiles_y, (unsigned)(g.nz - sets.kfirst + S.zc - 1) / S.zc, (unsigned)blocks);
        if (g.type == SF_CONE_CURVED)
            hipLaunchKernelGGL((sf_backproject_tiled<NC, NV, S.zc, S.pw, S.ph, 1, 2>), grid, dim3(256), 0, stream, g, G->d_views, d_sino, d_vol,
                               (int)tiles_x, G->bp_wh, (const void *)G->d_colcs, sets);
        else
            hipLaunchKernelGGL((sf_backproject_tiled<NC, NV, S.zc, S.pw, S.ph, 0, 2>), grid, dim3(256), 0, stream, g, G->d_views, d_sino, d_vol,
                               (int)tiles_x, G->bp_wh, (const void *)nullptr, sets);
        return true;
    } else {
        return false;
    }
}

template <int NC, int NV>
static bool launch_shape(const leap_geometry *G, const float *d_sino, float *d_vol, int blocks, hipStream_t stream)
{
    static_assert(BP_NPAIR_SHAPES == 4, "every shape has a case");
    switch (G->bp_pair_shape) {
    case 0: return launch_instance<NC, NV, 0>(G, d_sino, d_vol, blocks, stream);
    case 1: return launch_instance<NC, NV, 1>(G, d_sino, d_vol, blocks, stream);
    case 2: return launch_instance<NC, NV, 2>(G, d_sino, d_vol, blocks, stream);
    case 3: return launch_instance<NC, NV, 3>(G, d_sino, d_vol, blocks, stream);
    default: return false;
    }
}

bool leap_launch_backproject_pairs(const leap_geometry *G, const float *d_sino, float *d_vol, int blocks, hipStream_t stream)
{
    switch (G->bp_nc * 10 + G->bp_nv) {
    case 22: return launch_shape<2, 2>(G, d_sino, d_vol, blocks, stream);
    case 23: return launch_shape<2, 3>(G, d_sino, d_vol, blocks, stream);
    case 32: return launch_shape<3, 2>(G, d_sino, d_vol, blocks, stream);
    case 33: return launch_shape<3, 3>(G, d_sino, d_vol, blocks, stream);
    case 42: return launch_shape<4, 2>(G, d_sino, d_vol, blocks, stream);
    case 43: return launch_shape<4, 3>(G, d_sino, d_vol, blocks, stream);
    case 52: return launch_shape<5, 2>(G, d_sino, d_vol, blocks, stream);
    case 53: return launch_shape<5, 3>(G, d_sino, d_vol, blocks, stream);
    default: return false;
    }
}
