// Launchers of the tiled Siddon back projection with four groups of threads per workgroup that share the views; parts
// > 1: that many workgroups of them, into a volume each behind d_vol.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "leap_internal.h"
#include "sd_backproject_tiled.h"

template <int NCS, int SH>
static void launch_instance(const leap_geometry *G, int parts, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    constexpr SfBpShape S = SD_BP_SPLIT_SHAPES[SH];
    constexpr int VS = SD_BP_SPLIT;
    const SfGeom &g = G->g;
    const unsigned tiles_x = cdiv(g.nx, BP_T), tiles_y = cdiv(g.ny, BP_T);
    const dim3 grid(tiles_x * tiles_y, cdiv(g.nz, S.zc), (unsigned)(items * parts));
    auto go = [&](auto kernel, const SfGeom *geoms) {
        hipLaunchKernelGGL(kernel, grid, dim3(256 * VS), 0, stream, g, G->d_views, G->d_raycols, d_sino, d_vol, (int)tiles_x, geoms, parts);
    };
    const bool apart = G->sd_min_row_step > 1.0 + 1e-6;
    auto launch = [&](auto shared) {
        constexpr bool PARTS = decltype(shared)::value;
        if (g.type == SF_MODULAR) {
            if (apart) go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, true, true, VS, PARTS>, G->d_geoms);
            else go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, true, false, VS, PARTS>, G->d_geoms);
        } else {
            if (apart) go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, false, true, VS, PARTS>, nullptr);
            else go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, false, false, VS, PARTS>, nullptr);
        }
    };
    if (parts > 1) launch(std::true_type());
    else launch(std::false_type());
}

template <int NCS>
static bool launch_shape(const leap_geometry *G, int shape, int parts, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    static_assert(SD_BP_NSPLIT_SHAPES == 2, "every shape has a case");
    switch (shape) {
    case 0: launch_instance<NCS, 0>(G, parts, d_sino, d_vol, items, stream); return true;
    case 1: launch_instance<NCS, 1>(G, parts, d_sino, d_vol, items, stream); return true;
    default: return false;
    }
}

bool leap_launch_siddon_back_split(const leap_geometry *G, int shape, int parts, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    switch (G->bp_nc) {
    case 2: return launch_shape<2>(G, shape, parts, d_sino, d_vol, items, stream);
    case 3: return launch_shape<3>(G, shape, parts, d_sino, d_vol, items, stream);
    case 4: return launch_shape<4>(G, shape, parts, d_sino, d_vol, items, stream);
    default: return false;
    }
}
