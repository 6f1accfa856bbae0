// Launchers of the tiled footprint back projection with four groups of threads per workgroup that share the views; parts > 1: that many
// workgroups of them, by way of the handle's room for their volumes.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "leap_internal.h"
#include "sf_backproject_tiled.h"

template <int NC, int NV, int SH, int NS>
static bool launch_instance(const leap_geometry *G, int parts, const float *d_sino, float *room, float *d_vol, int blocks, hipStream_t stream)
{
    if constexpr (bp_split_instance_exists(NC, NV, SH)) {
        constexpr SfBpShape S = BP_SPLIT_SHAPES[SH];
        const SfGeom &g = G->g;
        const bool mirror = NS == 2 && G->bp_mirror;
        const SfBpSets sets = {mirror ? 1 : 0, mirror ? sf_mirror_first_voxel_above(g.nz) : 0, parts};
        const unsigned tiles_x = cdiv(g.nx, BP_T), tiles_y = cdiv(g.ny, BP_T);
        const dim3 grid(tiles_x * tiles_y, cdiv(g.nz - sets.kfirst, S.zc), (unsigned)(blocks * parts));
        float *const to = parts > 1 ? room : d_vol;
        auto go = [&](auto kernel, const void *aux) {
            hipLaunchKernelGGL(kernel, grid, dim3(256 * BP_SPLIT), 0, stream, g, G->d_views, d_sino, to, (int)tiles_x, G->bp_wh, aux, sets);
        };
        auto launch = [&](auto gt, const void *aux) {
            constexpr int GT = decltype(gt)::value;
            if (parts > 1) go(sf_backproject_tiled<NC, NV, S.zc, S.pw, S.ph, GT, NS, BP_SPLIT, true>, aux);
            else go(sf_backproject_tiled<NC, NV, S.zc, S.pw, S.ph, GT, NS, BP_SPLIT, false>, aux);
        };
        if (g.type == SF_CONE_CURVED) {
            launch(std::integral_constant<int, 1>(), G->d_colcs);
        } else if (g.type == SF_MODULAR) {
            if constexpr (NS == 1) launch(std::integral_constant<int, 2>(), G->d_geoms);
            else return false;
        } else {
            launch(std::integral_constant<int, 0>(), nullptr);
        }
        if (parts > 1) {
            const unsigned nvol = (unsigned)g.nx * (unsigned)g.ny * (unsigned)g.nz;
            const int per = mirror ? 1 : NS;
            hipLaunchKernelGGL(sf_sum_parts, dim3(cdiv(nvol, 256), (unsigned)(blocks * per)), dim3(256), 0, stream, room, d_vol, nvol, parts, per);
        }
        return true;
    } else {
        return false;
    }
}

template <int NC, int NV, int NS>
static bool launch_shape(const leap_geometry *G, int shape, int parts, const float *d_sino, float *room, float *d_vol, int blocks, hipStream_t stream)
{
    static_assert(BP_NSPLIT_SHAPES == 3, "every shape has a case");
    switch (shape) {
    case 0: return launch_instance<NC, NV, 0, NS>(G, parts, d_sino, room, d_vol, blocks, stream);
    case 1: return launch_instance<NC, NV, 1, NS>(G, parts, d_sino, room, d_vol, blocks, stream);
    case 2: return launch_instance<NC, NV, 2, NS>(G, parts, d_sino, room, d_vol, blocks, stream);
    default: return false;
    }
}

template <int NC, int NV>
static bool launch_sets(const leap_geometry *G, int shape, int parts, const float *d_sino, float *room, float *d_vol, int items, hipStream_t stream)
{
    const int pairs = leap_back_split_pairs(G, items), left = G->bp_mirror ? 0 : items - 2 * pairs;
    if (pairs && !launch_shape<NC, NV, 2>(G, shape, parts, d_sino, room, d_vol, pairs, stream)) return false;
    d_sino += (size_t)(items - left) * G->g.nviews * G->g.nrows * G->g.ncols;
    d_vol += (size_t)(items - left) * G->g.nx * G->g.ny * G->g.nz;
    return !left || launch_shape<NC, NV, 1>(G, shape, parts, d_sino, room, d_vol, left, stream);
}

bool leap_launch_backproject_split(const leap_geometry *G, int shape, int parts, const float *d_sino, float *room, float *d_vol, int items, hipStream_t stream)
{
    switch (G->bp_nc * 10 + G->bp_nv) {
    case 22: return launch_sets<2, 2>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 23: return launch_sets<2, 3>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 32: return launch_sets<3, 2>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 33: return launch_sets<3, 3>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 42: return launch_sets<4, 2>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 43: return launch_sets<4, 3>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 52: return launch_sets<5, 2>(G, shape, parts, d_sino, room, d_vol, items, stream);
    case 53: return launch_sets<5, 3>(G, shape, parts, d_sino, room, d_vol, items, stream);
    default: return false;
    }
}
