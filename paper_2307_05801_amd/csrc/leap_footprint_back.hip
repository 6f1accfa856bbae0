// Launchers of the tiled footprint back projection, one volume per workgroup.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "leap_internal.h"
#include "sf_backproject_tiled.h"

template <int NC, int NV, int SH, int GT>
static void launch_bp_tiled_gt(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    constexpr SfBpShape S = BP_SHAPES[SH];
    const SfGeom &g = G->g;
    const unsigned tiles_x = cdiv(g.nx, BP_T), tiles_y = cdiv(g.ny, BP_T);
    dim3 grid(tiles_x * tiles_y, cdiv(g.nz, S.zc), (unsigned)items);
    hipLaunchKernelGGL((sf_backproject_tiled<NC, NV, S.zc, S.pw, S.ph, GT, 1>), grid, dim3(256, 1, 1), 0, stream, g, G->d_views,
                       d_sino, d_vol, (int)tiles_x, G->bp_wh, GT == 1 ? (const void *)G->d_colcs : (const void *)G->d_geoms, SfBpSets{0, 0});
}

template <int NC, int NV, int SH>
static bool launch_bp_instance(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    if constexpr (bp_instance_exists(NC, NV, SH)) {
        if (G->g.type == SF_CONE_CURVED) launch_bp_tiled_gt<NC, NV, SH, 1>(G, d_sino, d_vol, stream, items);
        else if (G->g.type == SF_MODULAR) launch_bp_tiled_gt<NC, NV, SH, 2>(G, d_sino, d_vol, stream, items);
        else launch_bp_tiled_gt<NC, NV, SH, 0>(G, d_sino, d_vol, stream, items);
        return true;
    } else {
        return false;
    }
}

template <int NC, int NV>
static bool launch_bp_shape(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    switch (G->bp_shape) {
    case 0: return launch_bp_instance<NC, NV, 0>(G, d_sino, d_vol, stream, items);
    case 1: return launch_bp_instance<NC, NV, 1>(G, d_sino, d_vol, stream, items);
    case 2: return launch_bp_instance<NC, NV, 2>(G, d_sino, d_vol, stream, items);
    case 3: return launch_bp_instance<NC, NV, 3>(G, d_sino, d_vol, stream, items);
    case 4: return launch_bp_instance<NC, NV, 4>(G, d_sino, d_vol, stream, items);
    case BP_TALL_SHAPE: return launch_bp_instance<NC, NV, BP_TALL_SHAPE>(G, d_sino, d_vol, stream, items);
    case BP_WIDE_SHAPE: return launch_bp_instance<NC, NV, BP_WIDE_SHAPE>(G, d_sino, d_vol, stream, items);
    default: return false;
    }
}

// As many items at a time as the handle's room for the parts' volumes holds; in one slot of it where that holds them all.
static int launch_in_parts(const leap_geometry *G, const LeapBackParts &plan, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    const size_t nvol = (size_t)G->g.nx * G->g.ny * G->g.nz, nsino = (size_t)G->g.nviews * G->g.nrows * G->g.ncols;
    const bool one = items <= std::min(plan.items, G->back_slot_items);
    const int slot = one ? G->back.pick(stream) : 0;
    LeapTurn turn = one ? G->back.turn(slot, stream) : G->back.turn_at_all(stream);
    LEAP_HIP_CHECK(turn.begin());
    float *const room = G->d_back + (size_t)slot * G->back_slot_items * nvol * plan.parts;
    for (int b = 0; b < items;) {
        const int n = std::min(items - b, plan.items);
        if (!leap_launch_backproject_split(G, plan.shape, plan.parts, d_sino + b * nsino, room, d_vol + b * nvol, n, stream)) {
            leap_set_error("internal: no back-projection instance that shares the views for this footprint");
            return LEAP_UNSUPPORTED;
        }
        LEAP_HIP_CHECK(hipGetLastError());
        b += n;
    }
    LEAP_HIP_CHECK(turn.end());
    return LEAP_OK;
}

// The tiled footprint back projection on `items` consecutive sinograms of a batch in one launch.
int leap_launch_footprint_back(const leap_geometry *G, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    bool ok = false;
    const LeapBackParts plan = leap_back_parts(G, items);
    if (plan.parts > 1 && !leap_capturing(stream)) return launch_in_parts(G, plan, d_sino, d_vol, items, stream);
    const int split = leap_back_split_shape(G, items);
    if (split >= 0) {
        if (!leap_launch_backproject_split(G, split, 1, d_sino, nullptr, d_vol, items, stream)) {
            leap_set_error("internal: no back-projection instance that shares the views for this footprint");
            return LEAP_UNSUPPORTED;
        }
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    if (G->bp_pair_shape >= 0) {
        // two volumes per workgroup: an item and its mirror image, or two items of the batch; an odd last item by itself
        const int blocks = leap_back_pairs(G, items);
        if (blocks && !leap_launch_backproject_pairs(G, d_sino, d_vol, blocks, stream)) {
            leap_set_error("internal: no back-projection instance of two volumes for this footprint");
            return LEAP_UNSUPPORTED;
        }
        LEAP_HIP_CHECK(hipGetLastError());
        const int done = G->bp_mirror ? items : 2 * blocks;
        if (done == items) return LEAP_OK;
        d_sino += (size_t)done * G->g.nviews * G->g.nrows * G->g.ncols;
        d_vol += (size_t)done * G->g.nx * G->g.ny * G->g.nz;
        items -= done;
    }
    switch (G->bp_nc * 10 + G->bp_nv) {
    case 22: ok = launch_bp_shape<2, 2>(G, d_sino, d_vol, stream, items); break;
    case 23: ok = launch_bp_shape<2, 3>(G, d_sino, d_vol, stream, items); break;
    case 32: ok = launch_bp_shape<3, 2>(G, d_sino, d_vol, stream, items); break;
    case 33: ok = launch_bp_shape<3, 3>(G, d_sino, d_vol, stream, items); break;
    case 24: ok = launch_bp_shape<2, 4>(G, d_sino, d_vol, stream, items); break;
    case 34: ok = launch_bp_shape<3, 4>(G, d_sino, d_vol, stream, items); break;
    case 42: ok = launch_bp_shape<4, 2>(G, d_sino, d_vol, stream, items); break;
    case 43: ok = launch_bp_shape<4, 3>(G, d_sino, d_vol, stream, items); break;
    case 44: ok = launch_bp_shape<4, 4>(G, d_sino, d_vol, stream, items); break;
    case 52: ok = launch_bp_shape<5, 2>(G, d_sino, d_vol, stream, items); break;
    case 53: ok = launch_bp_shape<5, 3>(G, d_sino, d_vol, stream, items); break;
    case 54: ok = launch_bp_shape<5, 4>(G, d_sino, d_vol, stream, items); break;
    default: break;
    }
    if (!ok) {
        leap_set_error("internal: no tiled back-projection instance for this footprint");
        return LEAP_UNSUPPORTED;
    }
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}
