// HIP kernels (gfx950) and launchers of the projector pairs (separable footprint and Siddon).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <mutex>

#include "leap_internal.h"
#include "sf_general.h"
#include "sf_backproject_tiled.h"
#include "sf_project_columns.h"
#include "sf_project_rows.h"
#include "sf_flat.h"
#include "sd_project_columns.h"
#include "md_project_columns.h"
#include "sd_backproject_tiled.h"
#include "md_backproject_tiled.h"
#include "md_footprint_tiled.h"

// ------------------------------------------------------------------------------------------------
// General kernels: plain loop nests over global memory, valid for every validated geometry.
// ------------------------------------------------------------------------------------------------

constexpr int GEN_ZC = 8;   // voxels along z per back-projection thread
constexpr int GEN_RC = 8;   // detector rows per forward-projection thread

// grid: x = ceil(nx/64), y = ceil(ny/4), z = ceil(nz/GEN_ZC); block 64x4.
__global__ __launch_bounds__(256) void sf_backproject_general(SfGeom g, const SfView *__restrict__ views,
                                                              const float *__restrict__ sino, float *__restrict__ vol)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    const int j = blockIdx.y * 4 + threadIdx.y;
    const int k0 = blockIdx.z * GEN_ZC;
    if (i >= g.nx || j >= g.ny) return;
    float acc[GEN_ZC];
#pragma unroll
    for (int kk = 0; kk < GEN_ZC; ++kk) acc[kk] = 0.0f;
    sf_backproject_column_chunk<GEN_ZC>(g, views, sino, i, j, k0, acc);
#pragma unroll
    for (int kk = 0; kk < GEN_ZC; ++kk)
        if (k0 + kk < g.nz) vol[((size_t)(k0 + kk) * g.ny + j) * g.nx + i] = acc[kk];
}

// grid: x = ceil(ncols/64), y = ceil(ceil(nrows/GEN_RC)/4), z = nviews; block 64x4.
__global__ __launch_bounds__(256) void sf_project_general(SfGeom g, const SfView *__restrict__ views,
                                                          const float *__restrict__ vol, float *__restrict__ sino)
{
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int r0 = (blockIdx.y * 4 + threadIdx.y) * GEN_RC;
    const int a = blockIdx.z;
    if (c >= g.ncols || r0 >= g.nrows) return;
    const SfView v = views[a];
    float out[GEN_RC];
    sf_project_ray_chunk<GEN_RC>(g, v, vol, c, r0, out);
    float *__restrict__ y = sino + ((size_t)a * g.nrows) * g.ncols + c;
#pragma unroll
    for (int rr = 0; rr < GEN_RC; ++rr)
        if (r0 + rr < g.nrows) y[(size_t)(r0 + rr) * g.ncols] = out[rr];
}

// Modular geometry, footprint model on upright modules: the general bodies with one parameter block per view.
__global__ __launch_bounds__(256) void sf_backproject_general_modular(SfGeom g, const SfGeom *__restrict__ geoms,
                                                                      const SfView *__restrict__ views,
                                                                      const float *__restrict__ sino, float *__restrict__ vol)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    const int j = blockIdx.y * 4 + threadIdx.y;
    const int k0 = blockIdx.z * GEN_ZC;
    if (i >= g.nx || j >= g.ny) return;
    float acc[GEN_ZC];
#pragma unroll
    for (int kk = 0; kk < GEN_ZC; ++kk) acc[kk] = 0.0f;
    sf_backproject_column_chunk<GEN_ZC>(g, views, sino, i, j, k0, acc, geoms);
#pragma unroll
    for (int kk = 0; kk < GEN_ZC; ++kk)
        if (k0 + kk < g.nz) vol[((size_t)(k0 + kk) * g.ny + j) * g.nx + i] = acc[kk];
}

__global__ __launch_bounds__(256) void sf_project_general_modular(const SfGeom *__restrict__ geoms,
                                                                  const SfView *__restrict__ views,
                                                                  const float *__restrict__ vol, float *__restrict__ sino)
{
    const int a = blockIdx.z;
    const SfGeom g = geoms[a];
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int r0 = (blockIdx.y * 4 + threadIdx.y) * GEN_RC;
    if (c >= g.ncols || r0 >= g.nrows) return;
    const SfView v = views[a];
    float out[GEN_RC];
    sf_project_ray_chunk<GEN_RC>(g, v, vol, c, r0, out);
    float *__restrict__ y = sino + ((size_t)a * g.nrows) * g.ncols + c;
#pragma unroll
    for (int rr = 0; rr < GEN_RC; ++rr)
        if (r0 + rr < g.nrows) y[(size_t)(r0 + rr) * g.ncols] = out[rr];
}

// Modular geometry, footprint model on tilted modules (md_footprint.h): one thread per MF_RC rows of a detector column /
// per voxel.  Forward grid: x = ceil(ncols/64), y = ceil(ceil(nrows/MF_RC)/4), z = nviews; back grid as for the general
// Siddon kernel below.
#ifndef MF_RC_VALUE
#define MF_RC_VALUE 8
#endif
constexpr int MF_RC = MF_RC_VALUE;
__global__ __launch_bounds__(256) void mf_project_general(SfGeom g, const MfView *__restrict__ views,
                                                          const float *__restrict__ vol, float *__restrict__ sino)
{
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int r0 = (blockIdx.y * 4 + threadIdx.y) * MF_RC;
    const int a = blockIdx.z;
    if (c >= g.ncols || r0 >= g.nrows) return;
    float out[MF_RC];
    mf_project_rows<MF_RC>(g, views[a], vol, r0, c, out);
    float *__restrict__ y = sino + ((size_t)a * g.nrows) * g.ncols + c;
#pragma unroll
    for (int rr = 0; rr < MF_RC; ++rr)
        if (r0 + rr < g.nrows) y[(size_t)(r0 + rr) * g.ncols] = out[rr];
}

__global__ __launch_bounds__(256) void mf_backproject_general(SfGeom g, const MfView *__restrict__ views,
                                                              const float *__restrict__ sino, float *__restrict__ vol)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    const int j = blockIdx.y * 4 + threadIdx.y;
    const int k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    vol[((size_t)k * g.ny + j) * g.nx + i] = mf_backproject_voxel(g, views, sino, i, j, k);
}

// Siddon model, general kernels: one thread per ray / per voxel.
// grid: x = ceil(ncols/64), y = ceil(nrows/4), z = nviews; block 64x4.
__global__ __launch_bounds__(256) void sd_project_general(SfGeom g, const SdRayCol *__restrict__ rays,
                                                          const float *__restrict__ vol, float *__restrict__ sino)
{
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int r = blockIdx.y * 4 + threadIdx.y;
    const int a = blockIdx.z;
    if (c >= g.ncols || r >= g.nrows) return;
    const SdRayCol R = rays[(size_t)a * g.ncols + c];
    sino[((size_t)a * g.nrows + r) * g.ncols + c] = sd_project_ray(g, R, vol, r);
}

// grid: x = ceil(nx/64), y = ceil(ny/4), z = nz; block 64x4.
__global__ __launch_bounds__(256) void sd_backproject_general(SfGeom g, const SfView *__restrict__ views,
                                                              const SdRayCol *__restrict__ rays,
                                                              const float *__restrict__ sino, float *__restrict__ vol)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    const int j = blockIdx.y * 4 + threadIdx.y;
    const int k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    vol[((size_t)k * g.ny + j) * g.nx + i] = sd_backproject_voxel(g, views, rays, sino, i, j, k);
}

// Modular geometry, Siddon model: one thread per ray / per voxel.  Same grids as the general Siddon kernels.
__global__ __launch_bounds__(256) void md_project_general(SfGeom g, const MdPose *__restrict__ poses,
                                                          const float *__restrict__ vol, float *__restrict__ sino)
{
    const int c = blockIdx.x * 64 + threadIdx.x;
    const int r = blockIdx.y * 4 + threadIdx.y;
    const int a = blockIdx.z;
    if (c >= g.ncols || r >= g.nrows) return;
    const MdPose P = poses[a];
    sino[((size_t)a * g.nrows + r) * g.ncols + c] = md_project_ray(g, P, vol, r, c);
}

__global__ __launch_bounds__(256) void md_backproject_general(SfGeom g, const MdPose *__restrict__ poses,
                                                              const float *__restrict__ sino, float *__restrict__ vol)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    const int j = blockIdx.y * 4 + threadIdx.y;
    const int k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    vol[((size_t)k * g.ny + j) * g.nx + i] = md_backproject_voxel(g, poses, sino, i, j, k);
}

constexpr int SD_WAVES = 4;   // adjacent detector columns per workgroup of the Siddon forward kernel

template <int RG>
static void launch_sd_columns(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    const SfGeom &g = G->g;
    const int col_tiles = (int)cdiv(g.ncols, SD_WAVES), bands = (int)cdiv(g.nrows, RG * 64);
    const int vb = G->fp_vb, tb = G->fp_tb;
    const int views_pad = (int)cdiv(g.nviews, vb) * vb;
    const int tiles_per_xcd_pad = (int)cdiv(cdiv(col_tiles, 8), tb) * tb;
    const unsigned zero_col = (unsigned)(S.item_floats - (size_t)G->nzp);      // the copy's last column, which every copy clears
    dim3 grid((unsigned)(8 * tiles_per_xcd_pad * views_pad * bands), (unsigned)items, 1);
    if (G->md_tilted) {
        if constexpr (RG <= 4)        // (the selection offers the per-lane kernel 1, 2 or 4 row groups)
            hipLaunchKernelGGL((md_project_columns<RG, SD_WAVES>), grid, dim3(SD_WAVES * 64, 1, 1), 0, stream, g,
                               (const MdPose *)G->d_poses, S.volz, d_sino, G->nzp, S.item_floats, zero_col, col_tiles, bands, vb, tb, G->fp_turn,
                               views_pad, tiles_per_xcd_pad, slab);
    } else if (g.type == SF_MODULAR)
        hipLaunchKernelGGL((sd_project_columns<RG, SD_WAVES, true>), grid, dim3(SD_WAVES * 64, 1, 1), 0, stream, g, G->d_raycols,
                           S.volz, d_sino, G->nzp, S.item_floats, zero_col, col_tiles, bands, vb, tb, G->fp_turn, views_pad, tiles_per_xcd_pad,
                           slab, (const SfGeom *)G->d_geoms);
    else
        hipLaunchKernelGGL((sd_project_columns<RG, SD_WAVES, false>), grid, dim3(SD_WAVES * 64, 1, 1), 0, stream, g, G->d_raycols,
                           S.volz, d_sino, G->nzp, S.item_floats, zero_col, col_tiles, bands, vb, tb, G->fp_turn, views_pad, tiles_per_xcd_pad,
                           slab, (const SfGeom *)nullptr);
}

// Two rows per lane; RG pair groups of 128 rows.
template <int RG>
static void launch_sd_pairs(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    const SfGeom &g = G->g;
    const int col_tiles = (int)cdiv(g.ncols, 4), bands = (int)cdiv(g.nrows, RG * 128);
    const int vb = G->fp_vb, tb = G->fp_tb;
    const int views_pad = (int)cdiv(g.nviews, vb) * vb;
    const int tiles_per_xcd_pad = (int)cdiv(cdiv(col_tiles, 8), tb) * tb;
    dim3 grid((unsigned)(8 * tiles_per_xcd_pad * views_pad * bands), (unsigned)items, 1);
    auto go = [&](auto kernel, const SfGeom *geoms) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, g, G->d_raycols, S.volz, d_sino, G->nzp, S.item_floats, col_tiles, bands, vb,
                           tb, G->fp_turn, views_pad, tiles_per_xcd_pad, slab, geoms);
    };
    if (g.type == SF_MODULAR) {
        if (G->sd_pairs == 2) go(sd_project_pairs<RG, true, true>, G->d_geoms);
        else go(sd_project_pairs<RG, false, true>, G->d_geoms);
    } else {
        if (G->sd_pairs == 2) go(sd_project_pairs<RG, true, false>, nullptr);
        else go(sd_project_pairs<RG, false, false>, nullptr);
    }
}

static bool launch_sd_slab(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    if (G->sd_pairs) {
        switch (G->fp_rg) {
        case 2: launch_sd_pairs<1>(G, S, slab, d_sino, stream, items); return true;
        case 4: launch_sd_pairs<2>(G, S, slab, d_sino, stream, items); return true;
        case 8: launch_sd_pairs<4>(G, S, slab, d_sino, stream, items); return true;
        default: return false;
        }
    }
    switch (G->fp_rg) {
    case 1: launch_sd_columns<1>(G, S, slab, d_sino, stream, items); return true;
    case 2: launch_sd_columns<2>(G, S, slab, d_sino, stream, items); return true;
    case 4: launch_sd_columns<4>(G, S, slab, d_sino, stream, items); return true;
    case 8: launch_sd_columns<8>(G, S, slab, d_sino, stream, items); return true;
    default: return false;
    }
}

static int run_forward_columns(const leap_geometry *G, const FwdScratch &S, const float *d_vol, float *d_sino, int batch,
                               hipStream_t stream);

// On the general kernel, whatever the handle's fast one.
static int launch_sd_project(const leap_geometry *G, const float *d_vol, float *d_sino, hipStream_t stream)
{
    const SfGeom &g = G->g;
    if (g.type == SF_MODULAR) {                       // sizes were checked against the grid limits at creation
        dim3 grid(cdiv(g.ncols, 64), cdiv(g.nrows, 4), g.nviews);
        hipLaunchKernelGGL(md_project_general, grid, dim3(64, 4, 1), 0, stream, g, G->d_poses, d_vol, d_sino);
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    dim3 grid(cdiv(g.ncols, 64), cdiv(g.nrows, 4), g.nviews);
    if (grid.y > 65535u) {
        leap_set_error("detector has too many rows for one launch");
        return LEAP_UNSUPPORTED;
    }
    hipLaunchKernelGGL(sd_project_general, grid, dim3(64, 4, 1), 0, stream, g, G->d_raycols, d_vol, d_sino);
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

template <int NCS, int SH>
static void launch_sd_tiled(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    constexpr SfBpShape S = BP_SHAPES[SH];
    const SfGeom &g = G->g;
    const unsigned tiles_x = cdiv(g.nx, BP_T), tiles_y = cdiv(g.ny, BP_T);
    dim3 grid(tiles_x * tiles_y, cdiv(g.nz, S.zc), (unsigned)items);
    auto go = [&](auto kernel, const SfGeom *geoms) {
        hipLaunchKernelGGL(kernel, grid, dim3(256, 1, 1), 0, stream, g, G->d_views, G->d_raycols, d_sino, d_vol, (int)tiles_x, geoms, 1);
    };
    const bool apart = G->sd_min_row_step > 1.0 + 1e-6;
    if (g.type == SF_MODULAR) {
        if (apart) go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, true, true>, G->d_geoms);
        else go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, true, false>, G->d_geoms);
    } else {
        if (apart) go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, false, true>, nullptr);
        else go(sd_backproject_tiled<NCS, S.zc, S.pw, S.ph, false, false>, nullptr);
    }
}

template <int NCS>
static bool launch_sd_shape(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    switch (G->bp_shape) {
    case 1: launch_sd_tiled<NCS, 1>(G, d_sino, d_vol, stream, items); return true;
    case 2: launch_sd_tiled<NCS, 2>(G, d_sino, d_vol, stream, items); return true;
    case 3: launch_sd_tiled<NCS, 3>(G, d_sino, d_vol, stream, items); return true;
    case 4: launch_sd_tiled<NCS, 4>(G, d_sino, d_vol, stream, items); return true;
    default: return false;
    }
}

template <int SH>
static void launch_md_tiled(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    constexpr SfBpShape S = MD_BP_SHAPES[SH];
    const SfGeom &g = G->g;
    const unsigned tiles_x = cdiv(g.nx, BP_T), tiles_y = cdiv(g.ny, BP_T);
    dim3 grid(tiles_x * tiles_y, cdiv(g.nz, S.zc), (unsigned)items);
    hipLaunchKernelGGL((md_backproject_tiled<S.zc, S.pw, S.ph>), grid, dim3(256, 1, 1), 0, stream, g, (const MdBpView *)G->d_mdbp,
                       d_sino, d_vol, (int)tiles_x, 1);
}

template <int SH>
static void launch_md_split(const leap_geometry *G, int parts, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    constexpr SfBpShape S = MD_BP_SPLIT_SHAPES[SH];
    const SfGeom &g = G->g;
    const unsigned tiles_x = cdiv(g.nx, BP_T), tiles_y = cdiv(g.ny, BP_T);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(tiles_x * tiles_y, cdiv(g.nz, S.zc), (unsigned)(items * parts)), dim3(256 * MD_BP_SPLIT[SH]), 0, stream, g,
                           (const MdBpView *)G->d_mdbp, d_sino, d_vol, (int)tiles_x, parts);
    };
    if (parts > 1) go(md_backproject_tiled<S.zc, S.pw, S.ph, MD_BP_SPLIT[SH], true>);
    else go(md_backproject_tiled<S.zc, S.pw, S.ph, MD_BP_SPLIT[SH], false>);
}

static void launch_md_split_shape(const leap_geometry *G, int shape, int parts, const float *d_sino, float *d_vol, hipStream_t stream, int items)
{
    static_assert(MD_BP_NSPLIT_SHAPES == 3, "every shape has a case");
    if (shape == 0) launch_md_split<0>(G, parts, d_sino, d_vol, stream, items);
    else if (shape == 1) launch_md_split<1>(G, parts, d_sino, d_vol, stream, items);
    else launch_md_split<2>(G, parts, d_sino, d_vol, stream, items);
}

// The views of few tiles shared among workgroups: as leap_launch_footprint_back does it.
static int launch_sd_bp_parts(const leap_geometry *G, const LeapBackParts &plan, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    const unsigned nvol = (unsigned)G->g.nx * (unsigned)G->g.ny * (unsigned)G->g.nz;
    const size_t nsino = (size_t)G->g.nviews * G->g.nrows * G->g.ncols;
    const bool one = items <= plan.items && items <= G->back_slot_items;
    const int slot = one ? G->back.pick(stream) : 0;
    LeapTurn turn = one ? G->back.turn(slot, stream) : G->back.turn_at_all(stream);
    LEAP_HIP_CHECK(turn.begin());
    float *const room = G->d_back + (size_t)slot * G->back_slot_items * nvol * plan.parts;
    for (int b = 0; b < items; b += plan.items) {
        const int n = items - b < plan.items ? items - b : plan.items;
        bool ok = true;
        if (!G->d_mdbp) ok = leap_launch_siddon_back_split(G, plan.shape, plan.parts, d_sino + b * nsino, room, n, stream);
        else launch_md_split_shape(G, plan.shape, plan.parts, d_sino + b * nsino, room, stream, n);
        if (!ok) {
            leap_set_error("internal: no Siddon back-projection instance that shares the views");
            return LEAP_UNSUPPORTED;
        }
        hipLaunchKernelGGL(sf_sum_parts, dim3(cdiv(nvol, 256), (unsigned)n), dim3(256), 0, stream, room, d_vol + (size_t)b * nvol, nvol, plan.parts, 1);
        LEAP_HIP_CHECK(hipGetLastError());
    }
    LEAP_HIP_CHECK(turn.end());
    return LEAP_OK;
}

// The tiled Siddon back projection on `items` consecutive sinograms of a batch in one launch.
static int launch_sd_bp_items(const leap_geometry *G, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    bool ok = false;
    const LeapBackParts plan = leap_siddon_parts(G, items);
    if (plan.parts > 1 && !leap_capturing(stream)) return launch_sd_bp_parts(G, plan, d_sino, d_vol, items, stream);
    const int split = leap_siddon_split_shape(G, items);
    if (G->d_mdbp && split >= 0) {
        launch_md_split_shape(G, split, 1, d_sino, d_vol, stream, items);
        ok = true;
    } else if (G->md_tilted || G->d_mdbp) {
        switch (G->d_mdbp ? G->bp_shape : -1) {
        case 0: launch_md_tiled<0>(G, d_sino, d_vol, stream, items); ok = true; break;
        case 1: launch_md_tiled<1>(G, d_sino, d_vol, stream, items); ok = true; break;
        case 2: launch_md_tiled<2>(G, d_sino, d_vol, stream, items); ok = true; break;
        case 3: launch_md_tiled<3>(G, d_sino, d_vol, stream, items); ok = true; break;
        case 4: launch_md_tiled<4>(G, d_sino, d_vol, stream, items); ok = true; break;
        case 5: launch_md_tiled<5>(G, d_sino, d_vol, stream, items); ok = true; break;
        default: break;
        }
    } else if (split >= 0) {
        ok = leap_launch_siddon_back_split(G, split, 1, d_sino, d_vol, items, stream);
    } else
    switch (G->bp_nc) {
    case 2: ok = launch_sd_shape<2>(G, d_sino, d_vol, stream, items); break;
    case 3: ok = launch_sd_shape<3>(G, d_sino, d_vol, stream, items); break;
    case 4: ok = launch_sd_shape<4>(G, d_sino, d_vol, stream, items); break;
    default: break;
    }
    if (!ok) {
        leap_set_error("internal: no tiled Siddon back-projection instance for this geometry");
        return LEAP_UNSUPPORTED;
    }
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

static int launch_sd_backproject(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream)
{
    const SfGeom &g = G->g;
    if (g.type == SF_MODULAR && !G->bp_tiled) {
        dim3 grid(cdiv(g.nx, 64), cdiv(g.ny, 4), g.nz);
        hipLaunchKernelGGL(md_backproject_general, grid, dim3(64, 4, 1), 0, stream, g, G->d_poses, d_sino, d_vol);
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    if (G->bp_tiled) return launch_sd_bp_items(G, d_sino, d_vol, 1, stream);
    dim3 grid(cdiv(g.nx, 64), cdiv(g.ny, 4), g.nz);
    if (grid.y > 65535u || grid.z > 65535u) {
        leap_set_error("volume has too many voxels along y or z for one launch");
        return LEAP_UNSUPPORTED;
    }
    hipLaunchKernelGGL(sd_backproject_general, grid, dim3(64, 4, 1), 0, stream, g, G->d_views, G->d_raycols, d_sino, d_vol);
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

// Copies voxel columns [i0, i0 + ni) x [j0, j0 + nj) of `items` volumes into the scratch: z-fastest, or by detector rows.
static void copy_slab(const leap_geometry *G, const FwdScratch &S, const float *vol, int span, int i0, int j0, int ni, int nj, int items,
                      hipStream_t stream)
{
    const SfGeom &g = G->g;
    if (G->fp_rows) {
        hipLaunchKernelGGL(sf_volume_to_rows, dim3(cdiv(span, 32), cdiv(g.nrows, 32), (unsigned)(nj * items)), dim3(32, 8, 1), 0, stream, g, vol,
                           S.volz, G->nzp, i0, j0, ni, nj, S.item_floats);
        return;
    }
    hipLaunchKernelGGL(sf_volume_to_columns, dim3(cdiv(span, 32), cdiv(g.nz, 32), (unsigned)(nj * items)), dim3(32, 8, 1), 0,
                       stream, vol, S.volz, g.nx, g.ny, g.nz, G->nzp, i0, j0, ni, nj, S.item_floats);
}

// The column-wise forward projection (footprint or Siddon weights) of a batch: up to S.items volumes at a time, each
// walked slab by slab -- first the slabs across x for the rays that advance fastest along x, then the slabs across y
// for the others.  Per slab: copy it z-fastest into the scratch, then every ray adds the slab's share to its sample.
static int run_forward_columns(const leap_geometry *G, const FwdScratch &S, const float *d_vol, float *d_sino, int batch,
                               hipStream_t stream)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.nviews * g.nrows * g.ncols;
    const bool siddon = g.model == SF_MODEL_SIDDON;
    for (int b = 0; b < batch; b += S.items) {
        const int items = batch - b < S.items ? batch - b : S.items;
        const float *vol = d_vol + (size_t)b * nvol;
        float *sino = d_sino + (size_t)b * nsino;
        if (S.width >= (g.nx > g.ny ? g.nx : g.ny)) {
            // The whole volume fits: one copy, and one launch for the rays of either axis.  (As two slabs the copy was made
            // twice and each launch had half the rays to fill the chip with.)
            const SfSlab whole = {0, 0, -1, 1, g.nx};
            copy_slab(G, S, vol, g.nx, 0, 0, g.nx, g.ny, items, stream);
            const bool ok = siddon ? launch_sd_slab(G, S, whole, sino, stream, items) : leap_launch_footprint_slab(G, S, whole, sino, stream, items);
            if (!ok) {
                leap_set_error("internal: no column-wise forward instance for this geometry");
                return LEAP_UNSUPPORTED;
            }
            continue;
        }
        for (int xmajor = 1; xmajor >= 0; --xmajor) {
            const int n_major = xmajor ? g.nx : g.ny;
            for (int n0 = 0; n0 < n_major; n0 += S.width) {
                const int n1 = n0 + S.width < n_major ? n0 + S.width : n_major;
                const SfSlab slab = {n0, n1, xmajor, n0 == 0 ? 1 : 0, S.width};
                const int i0 = xmajor ? n0 : 0, ni = xmajor ? S.width : g.nx, nj = xmajor ? g.ny : n1 - n0;
                copy_slab(G, S, vol, xmajor ? n1 - n0 : g.nx, i0, xmajor ? 0 : n0, ni, nj, items, stream);
                const bool ok = siddon ? launch_sd_slab(G, S, slab, sino, stream, items) : leap_launch_footprint_slab(G, S, slab, sino, stream, items);
                if (!ok) {
                    leap_set_error("internal: no column-wise forward instance for this geometry");
                    return LEAP_UNSUPPORTED;
                }
            }
        }
    }
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

// ------------------------------------------------------------------------------------------------
// Flat scans (sf_flat.h).
// ------------------------------------------------------------------------------------------------

// Waves of a workgroup that share one output tile's slabs or views: as many as it takes to put about eight waves on each of
// the chip's 1024 SIMDs, while each keeps at least four of its `steps` (slabs, views).  A 64^2 slice has 64 tiles and 180
// beams' waves: one wave each took 112 us (A) and 131 us (A^T), 16 of them 11 us each with their launches.  tiles: those of one
// item.  The split orders the sums, so it depends on the scan alone: an item comes out the same bits in any batch, with and
// without the copy.
static int flat_waves(double tiles, int steps)
{
    int w = 1;
    while (w < FLAT_MAX_WAVES && tiles * w < 8192.0 && steps / (2 * w) >= 4) w *= 2;
    return w;
}

template <int NB>
static void launch_project_flat(const leap_geometry *G, const float *src, const float *turned, float *d_sino, int items, hipStream_t stream)
{
    const SfGeom &g = G->g;
    const int tiles = (int)cdiv(g.ncols, FLAT_RAYS);
    const unsigned groups = cdiv((unsigned)items, NB);
    const bool parallel = g.type == SF_PARALLEL;
    int waves = flat_waves((double)tiles * g.nviews, g.nx < g.ny ? g.nx : g.ny);
    while ((size_t)waves * G->flat_span * sizeof(SfFlatRec) > 65536) waves /= 2;        // (spans of up to 256: at least 8 fit)
    const size_t lds = (size_t)waves * (parallel ? 64 * NB * sizeof(float) : G->flat_span * sizeof(SfFlatRec));
    const int grid_tiles = flat_tiles(g.ncols, g.nviews);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid_tiles * (unsigned)g.nviews, groups), dim3(64 * waves), lds, stream, g, G->d_views, src, turned,
                           d_sino, grid_tiles, G->flat_span, items, G->flat_fv);
    };
    if (parallel) go(sf_project_flat<NB, true>);
    else go(sf_project_flat<NB, false>);
}

// `items` slices by way of the handle's scratch: the copy by rows and, behind it, the turned one.
template <int NB>
static void launch_interleaved_flat(const leap_geometry *G, const float *d_vol, float *d_sino, int items, hipStream_t stream)
{
    const SfGeom &g = G->g;
    const unsigned nvol = (unsigned)g.nx * (unsigned)g.ny, groups = cdiv((unsigned)items, NB);
    hipLaunchKernelGGL(sf_interleave<NB>, dim3(cdiv(nvol, 256), groups), dim3(256), 0, stream, d_vol, G->d_volz, nvol, items);
    float *turned = nullptr;
    if ((double)cdiv(g.ncols, FLAT_RAYS) * g.nviews * (g.nx < g.ny ? g.nx : g.ny) * groups >= (g.type == SF_PARALLEL ? FLAT_TURN_STEPS_PARALLEL : FLAT_TURN_STEPS)) {
        turned = G->d_volz + (size_t)groups * NB * nvol;
        hipLaunchKernelGGL(sf_interleave_turned<NB>, dim3(cdiv(g.nx, 32), cdiv(g.ny, 32), groups), dim3(32, 8), 0, stream, d_vol, turned, g.nx, g.ny, items);
    }
    launch_project_flat<NB>(G, G->d_volz, turned, d_sino, items, stream);
}

// Launches of so few workgroups with eight items each take four: half the units idle otherwise, and the voxels fetched ahead cost a wave of eight
// items 4 to 7 % there.  Four over eight items, by workgroups of eight: 40 to 110 0.55 to 0.9, 136 to 160 0.8 to 1.05.  An item comes out the same bits
// either way.
constexpr double FLAT_FEW_GROUPS = 128.0;

// The forward projection of `batch` slices.  With the handle's scratch a weight serves up to eight items; calls on one
// handle then share the scratch and are ordered on the device.  A call that is being captured, or that must not touch the
// scratch (scratch == false), takes the slices one by one as they lie: the same sums in the same order, bit for bit.
static int project_flat(const leap_geometry *G, const float *d_vol, float *d_sino, int batch, hipStream_t stream, bool scratch)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny, nsino = (size_t)g.nviews * g.ncols;
    if (scratch && batch > 1 && G->d_volz) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        LEAP_HIP_CHECK(hipStreamIsCapturing(stream, &capture));
        scratch = capture == hipStreamCaptureStatusNone;
    }
    if (!scratch || batch == 1 || !G->d_volz) {
        for (int b = 0; b < batch; b += 32768) {
            const int items = batch - b < 32768 ? batch - b : 32768;
            launch_project_flat<1>(G, d_vol + b * nvol, nullptr, d_sino + b * nsino, items, stream);
        }
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    LeapTurn turn = G->scratch.turn(0, stream);
    LEAP_HIP_CHECK(turn.begin());
    const int room = (int)(G->scratch_bytes / (2 * nvol * sizeof(float)));      // whole slices the scratch holds, twice each
    for (int b = 0; b < batch;) {
        const float *vol = d_vol + b * nvol;
        float *sino = d_sino + b * nsino;
        const int left = batch - b;
        const int most = left < room ? left : room;
        int items;
        if (most > 4 && (double)cdiv(g.ncols, FLAT_RAYS) * g.nviews * cdiv((unsigned)most, 8) <= FLAT_FEW_GROUPS) {
            items = left < room / 4 * 4 ? left : room / 4 * 4;
            launch_interleaved_flat<4>(G, vol, sino, items, stream);
        } else if (left >= 8 && room >= 8) {                                            // whole groups of eight
            items = (left < room ? left : room) / 8 * 8;
            launch_interleaved_flat<8>(G, vol, sino, items, stream);
        } else if (left > 4 && room >= 8) {
            items = left;
            launch_interleaved_flat<8>(G, vol, sino, items, stream);
        } else if (left > 2 && room >= 4) {
            items = left < 4 ? left : 4;
            launch_interleaved_flat<4>(G, vol, sino, items, stream);
        } else if (left > 1) {
            items = 2;
            launch_interleaved_flat<2>(G, vol, sino, items, stream);
        } else {
            items = 1;
            launch_project_flat<1>(G, vol, nullptr, sino, items, stream);
        }
        b += items;
    }
    LEAP_HIP_CHECK(hipGetLastError());
    LEAP_HIP_CHECK(turn.end());
    return LEAP_OK;
}

// Slices of up to 64 or 128 tiles of 8 x 8 voxels leave most of the compute units idle: their waves take the views in runs of four or two,
// and in a launch of so few tiles (those of its groups of items together) four or two views of a run at a time, on tiles of 4 x 4 or
// 8 x 4 voxels.  Four / two over one view at a time: 16 tiles 0.86 / 0.85, 64 (90 to 400 views) 0.44 to 0.78 / 0.69 to 0.82, 81 to 121
// 0.65 to 1.16 / 0.68 to 0.75, 162 1.72 / 1.36, 169 to 256 0.83 to 1.20 / 1.04 to 1.09.
constexpr double FLAT_FOUR_TILES = 64.0, FLAT_TWO_TILES = 128.0;

template <int NB>
static void launch_backproject_flat(const leap_geometry *G, const float *d_sino, float *d_vol, int items, hipStream_t stream)
{
    const SfGeom &g = G->g;
    const unsigned groups = cdiv((unsigned)items, NB);
    const double tiles = (double)cdiv(g.nx, FLAT_T) * cdiv(g.ny, FLAT_T);
    const int waves = flat_waves(tiles, g.nviews);
    const auto few = [&](double n) { return waves < FLAT_MAX_WAVES || n > FLAT_TWO_TILES ? 1 : (n > FLAT_FOUR_TILES ? 2 : 4); };
    const int shares = few(tiles);                // (of the scan alone: an item comes out the same bits in any batch)
    auto go = [&](auto kernel, auto tile, size_t lds) {
        const unsigned tiles_x = cdiv(g.nx, decltype(tile)::TX), tiles_y = cdiv(g.ny, decltype(tile)::TY);
        hipLaunchKernelGGL(kernel, dim3(tiles_x * tiles_y, groups), dim3(64 * waves), lds, stream, g, G->d_views, d_sino, d_vol, (int)tiles_x, items,
                           shares, G->flat_fv);
    };
    switch (few(tiles * groups)) {
    case 4: go(sf_backproject_flat<NB, 4, true>, FlatTile<4>(), 0); break;
    case 2: go(sf_backproject_flat<NB, 2, true>, FlatTile<2>(), 0); break;
    default:
        const size_t lds = (size_t)waves * 64 * NB * sizeof(float);
        if (NB > 1 || shares > 1) go(sf_backproject_flat<NB, 1, true>, FlatTile<1>(), lds);
        else go(sf_backproject_flat<1, 1, false>, FlatTile<1>(), lds);
    }
}

static int backproject_flat(const leap_geometry *G, const float *d_sino, float *d_vol, int batch, hipStream_t stream)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny, nsino = (size_t)g.nviews * g.ncols;
    for (int b = 0; b < batch;) {
        const float *sino = d_sino + b * nsino;
        float *vol = d_vol + b * nvol;
        const int left = batch - b;
        int items = left < 8 * 4096 ? left : 8 * 4096;
        if (left >= 8) launch_backproject_flat<8>(G, sino, vol, items = items / 8 * 8, stream);
        else if (left > 4) launch_backproject_flat<8>(G, sino, vol, items, stream);
        else if (left > 2) launch_backproject_flat<4>(G, sino, vol, items, stream);
        else if (left > 1) launch_backproject_flat<2>(G, sino, vol, items, stream);
        else launch_backproject_flat<1>(G, sino, vol, items, stream);
        b += items;
    }
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

// Voxels per thread and groups of threads that share the views, for the tilted footprints' tiled back projection: the shape of least
// estimated time, in us.  A view costs a workgroup its staging and a time per voxel and pixel of a voxel's rectangle, alone on a compute unit or one of
// four of 256 threads (one of 1024).  The constants are fitted to 525 scans (12^2 to 230^2 x 140 voxels, 1 to 200 views, rectangles of 4 to 11 pixels; all seven
// shapes each, 20 % rms): the chosen shape takes 1.015 times the best one's time, 1.45 at most.  Against the choice among 8, 2 and 1 voxels by
// workgroups alone 0.76, at most 1.10.  60 views' worth per shape (8, 4, 1 voxels; four groups 4, 2, 1), us per view: 48^2 x 38 voxels 6.4, 3.9, 2.4; 2.0,
// 1.3, 1.8; 64^2 x 51 6.4, 3.9, 3.5; 2.0, 2.5, 3.5; 96^2 x 76 8.4, 6.3, 8.4; 5.7, 7.0, 9.5; 128^2 x 102 12.1, 12.6, 18.7; 13.2, 15.7, 22.8.  Two voxels in
// one group are for few views: 64 x 73 x 67, 6 views 38 us, four groups of 4 or 2 44 and 40; 51 x 60 x 81, 9 views 57, 69 and 62.
static int mf_back_choice(const leap_geometry *G, double tiles)
{
    static const struct {
        int zc, groups;
    } shapes[] = {{8, 1}, {4, 1}, {2, 1}, {1, 1}, {4, 4}, {2, 4}, {1, 4}};
    const double pixels = (G->max_cols_per_voxel + 1.0) * (G->max_rows_per_voxel + 1.0), views = G->g.nviews;
    int best = 0;
    double least = 1e300;
    for (int n = 0; n < 7; ++n) {
        const double per_unit = tiles * cdiv(G->g.nz, shapes[n].zc) / 256.0, work = (shapes[n].zc < G->g.nz ? shapes[n].zc : G->g.nz) * pixels;
        double time = 4.5;
        if (shapes[n].groups > 1) {
            const double rounds = 0.56 * std::ceil(per_unit) + 0.44 * per_unit;
            time += (rounds > 1.0 ? rounds : 1.0) * (std::ceil(views / shapes[n].groups) * (1.8 + 0.169 * work) + 0.85);
        } else {
            const double alone = 1.19 + 0.085 * work, full = 1.58 + 0.152 * work;
            if (per_unit <= 4.0) time += views * (alone + (full - alone) * (std::ceil(per_unit) - 1.0) / 3.0) + 1.25;
            else time += views * full * (0.29 * std::ceil(per_unit / 4.0) + 0.71 * per_unit / 4.0) + 1.25 * per_unit / 4.0;
        }
        if (time < 0.97 * least) {
            least = time;
            best = n;
        }
    }
    return best;
}

// One volume on the kernels that read it as it lies: the flat ones, the tiled footprints', the general ones.
static int launch_project_direct(const leap_geometry *G, const float *d_vol, float *d_sino, hipStream_t stream)
{
    const SfGeom &g = G->g;
    if (g.model == SF_MODEL_SIDDON) return launch_sd_project(G, d_vol, d_sino, stream);
    if (G->flat) return project_flat(G, d_vol, d_sino, 1, stream, false);
    if (G->mf_tiles) {
        // Waves per tile: as many as it takes to supply the chip; four also where there are tiles in plenty (a tile's time is that of its
        // beams' layers, which differ from tile to tile).  us, one / four / eight waves per tile, by tiles: 80 137 / 39 / 30; 200 940 / 241 /
        // 174; 480 1965 / 517 / 523; 560 1023 / 270 / 234; 1200 1226 / 568 / 566; 3360 1269 / 738 / 842; 11520 13991 / 11187 / 13789.
        const unsigned tiles = cdiv(g.ncols, MF_TC), bands = cdiv(g.nrows, MF_TR);
        auto go = [&](auto kernel, unsigned waves) {
            hipLaunchKernelGGL(kernel, dim3(tiles | 1u, bands, g.nviews), dim3(64 * waves), 0, stream, g, G->d_mfviews, d_vol, d_sino);
        };
        if ((double)tiles * bands * g.nviews <= 400.0) go(mf_project_tiles<8>, 8);
        else go(mf_project_tiles<4>, 4);
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    if (G->d_mfviews) {                     // sizes were checked against the grid limits at creation
        dim3 grid(cdiv(g.ncols, 64), cdiv(cdiv(g.nrows, MF_RC), 4), g.nviews);
        hipLaunchKernelGGL(mf_project_general, grid, dim3(64, 4, 1), 0, stream, g, G->d_mfviews, d_vol, d_sino);
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    dim3 block(64, 4, 1);
    dim3 grid(cdiv(g.ncols, 64), cdiv(cdiv(g.nrows, GEN_RC), 4), g.nviews);
    if (grid.y > 65535u) {
        leap_set_error("detector has too many rows for one launch");
        return LEAP_UNSUPPORTED;
    }
    if (g.type == SF_MODULAR)
        hipLaunchKernelGGL(sf_project_general_modular, grid, block, 0, stream, G->d_geoms, G->d_views, d_vol, d_sino);
    else
        hipLaunchKernelGGL(sf_project_general, grid, block, 0, stream, g, G->d_views, d_vol, d_sino);
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

int leap_launch_project_batch(const leap_geometry *G, const float *d_vol, float *d_sino, int batch, hipStream_t stream)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.nviews * g.nrows * g.ncols;
    if (G->flat) return project_flat(G, d_vol, d_sino, batch, stream, true);
    const bool footprint_fast = g.model != SF_MODEL_SIDDON && G->fp_columns;
    const bool siddon_fast = g.model == SF_MODEL_SIDDON && G->sd_columns;
    bool direct = !footprint_fast && !siddon_fast;
    if (!direct && g.nrows < FP_FREE_ROWS) direct = leap_capturing(stream);
    if (!direct) {
        FwdScratch S;
        if (!leap_plan_scratch(G, G->scratch_bytes / sizeof(float), batch, S.width, S.items)) {
            leap_set_error("internal: the handle's scratch holds no slab");
            return LEAP_UNSUPPORTED;
        }
        S.item_floats = ((size_t)S.width * (size_t)(g.nx > g.ny ? g.nx : g.ny) + 1) * (size_t)G->nzp;
        const bool one = G->scratch.slots > 1 && batch <= S.items && batch * S.item_floats <= G->scratch_slot_floats;
        const int slot = one ? G->scratch.pick(stream) : 0;
        S.volz = G->d_volz + slot * G->scratch_slot_floats;
        LeapTurn turn = one ? G->scratch.turn(slot, stream) : G->scratch.turn_at_all(stream);
        LEAP_HIP_CHECK(turn.begin());
        const int rc = run_forward_columns(G, S, d_vol, d_sino, batch, stream);
        if (rc != LEAP_OK) return rc;
        LEAP_HIP_CHECK(turn.end());
        return LEAP_OK;
    }
    for (int b = 0; b < batch; ++b) {
        const int rc = launch_project_direct(G, d_vol + b * nvol, d_sino + b * nsino, stream);
        if (rc != LEAP_OK) return rc;
    }
    return LEAP_OK;
}

int leap_launch_backproject_batch(const leap_geometry *G, const float *d_sino, float *d_vol, int batch, hipStream_t stream)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.nviews * g.nrows * g.ncols;
    if (G->flat) return backproject_flat(G, d_sino, d_vol, batch, stream);
    if (G->bp_tiled) {
        // up to 16 items per launch (a batch of small training volumes fills the chip better that way)
        for (int b = 0; b < batch; b += 16) {
            const int items = batch - b < 16 ? batch - b : 16;
            const int rc = g.model != SF_MODEL_SIDDON ? leap_launch_footprint_back(G, d_sino + b * nsino, d_vol + b * nvol, items, stream)
                                                      : launch_sd_bp_items(G, d_sino + b * nsino, d_vol + b * nvol, items, stream);
            if (rc != LEAP_OK) return rc;
        }
        return LEAP_OK;
    }
    for (int b = 0; b < batch; ++b) {
        const int rc = leap_launch_backproject(G, d_sino + b * nsino, d_vol + b * nvol, stream);
        if (rc != LEAP_OK) return rc;
    }
    return LEAP_OK;
}

int leap_launch_backproject(const leap_geometry *G, const float *d_sino, float *d_vol, hipStream_t stream)
{
    const SfGeom &g = G->g;
    if (g.model == SF_MODEL_SIDDON) return launch_sd_backproject(G, d_sino, d_vol, stream);
    if (G->flat) return backproject_flat(G, d_sino, d_vol, 1, stream);
    if (G->bp_tiled) return leap_launch_footprint_back(G, d_sino, d_vol, 1, stream);
    if (G->mf_tiled) {
        const unsigned tiles_x = cdiv(g.nx, MF_T), tiles_y = cdiv(g.ny, MF_T);
        auto go = [&](auto kernel, int zc, int groups) {
            hipLaunchKernelGGL(kernel, dim3(tiles_x * tiles_y, cdiv(g.nz, zc)), dim3(256 * groups), 0, stream, g, G->d_mfviews, d_sino, d_vol, (int)tiles_x);
        };
        switch (mf_back_choice(G, (double)tiles_x * tiles_y)) {
        case 0: go(mf_backproject_tiled<8, 1>, 8, 1); break;
        case 1: go(mf_backproject_tiled<4, 1>, 4, 1); break;
        case 2: go(mf_backproject_tiled<2, 1>, 2, 1); break;
        case 3: go(mf_backproject_tiled<1, 1>, 1, 1); break;
        case 4: go(mf_backproject_tiled<4, 4>, 4, 4); break;
        case 5: go(mf_backproject_tiled<2, 4>, 2, 4); break;
        default: go(mf_backproject_tiled<1, 4>, 1, 4); break;
        }
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    if (G->d_mfviews) {
        dim3 grid(cdiv(g.nx, 64), cdiv(g.ny, 4), g.nz);
        hipLaunchKernelGGL(mf_backproject_general, grid, dim3(64, 4, 1), 0, stream, g, G->d_mfviews, d_sino, d_vol);
        LEAP_HIP_CHECK(hipGetLastError());
        return LEAP_OK;
    }
    dim3 block(64, 4, 1);
    dim3 grid(cdiv(g.nx, 64), cdiv(g.ny, 4), cdiv(g.nz, GEN_ZC));
    if (grid.y > 65535u || grid.z > 65535u) {
        leap_set_error("volume has too many voxels along y or z for one launch");
        return LEAP_UNSUPPORTED;
    }
    if (g.type == SF_MODULAR)
        hipLaunchKernelGGL(sf_backproject_general_modular, grid, block, 0, stream, g, G->d_geoms, G->d_views, d_sino, d_vol);
    else
        hipLaunchKernelGGL(sf_backproject_general, grid, block, 0, stream, g, G->d_views, d_sino, d_vol);
    LEAP_HIP_CHECK(hipGetLastError());
    return LEAP_OK;
}

// ------------------------------------------------------------------------------------------------
// Forward projection on a fixed scratch array, for callers that must not allocate.
// ------------------------------------------------------------------------------------------------
//
// The column-wise forward kernels read a z-fastest copy of the volume.  A handle normally owns that copy (allocated
// in leap_geometry_create).  leap_project_static_scratch keeps it in the file-scope device array below instead, so
// the call itself, and everything it launches, touches no allocator.  In host code the array's name is only a
// stand-in for the symbol: its device address is asked for once per device (hipGetSymbolAddress, with that device
// current) and only that address is ever handed to kernels.
static __device__ __align__(256) unsigned char scratch[LEAP_STATIC_SCRATCH_BYTES];

constexpr int LEAP_MAX_DEVICES = 64;
static float *g_static_scratch[LEAP_MAX_DEVICES];     // device address of `scratch`, per device (nullptr: not asked yet)
static std::mutex g_static_scratch_mutex;

int leap_static_scratch_init(int device)
{
    if (device < 0 || device >= LEAP_MAX_DEVICES) {
        leap_set_error("device index beyond the static scratch table");
        return LEAP_UNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_static_scratch_mutex);
    if (g_static_scratch[device]) return LEAP_OK;
    int current = -1;
    LEAP_HIP_CHECK(hipGetDevice(&current));
    if (current != device) {
        leap_set_error("the handle's device is not the current device");
        return LEAP_INVALID_ARG;
    }
    void *p = nullptr;
    LEAP_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_static_scratch[device] = static_cast<float *>(p);
    return LEAP_OK;
}

extern "C" int leap_project_static_scratch(const leap_geometry *G, const float *d_vol, float *d_sino, int32_t batch, void *hip_stream)
{
    if (!G || !d_vol || !d_sino) {
        leap_set_error("null handle or data pointer");
        return LEAP_INVALID_ARG;
    }
    if (batch <= 0) {
        leap_set_error("batch must be positive");
        return LEAP_INVALID_ARG;
    }
    if ((const void *)d_vol == (const void *)d_sino) {
        leap_set_error("input and output must not alias");
        return LEAP_INVALID_ARG;
    }
    hipStream_t stream = (hipStream_t)hip_stream;
    const SfGeom &g = G->g;
    const bool footprint_fast = g.model != SF_MODEL_SIDDON && G->fp_columns;
    const bool siddon_fast = g.model == SF_MODEL_SIDDON && G->sd_columns;
    if ((!footprint_fast && !siddon_fast) || g.nrows < FP_FREE_ROWS) {
        // this geometry runs on kernels that read the caller's volume directly: no scratch is involved at all
        if (G->flat) return project_flat(G, d_vol, d_sino, batch, stream, false);
        const size_t nvol = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.nviews * g.nrows * g.ncols;
        for (int b = 0; b < batch; ++b) {
            const int rc = launch_project_direct(G, d_vol + b * nvol, d_sino + b * nsino, stream);
            if (rc != LEAP_OK) return rc;
        }
        return LEAP_OK;
    }
    const int n_side = g.nx > g.ny ? g.nx : g.ny;
    FwdScratch S;
    if (!leap_plan_scratch(G, LEAP_STATIC_SCRATCH_BYTES / sizeof(float), batch, S.width, S.items)) {
        char msg[200];
        std::snprintf(msg, sizeof msg, "volume too large for the static scratch: four voxel layers of its z-fastest copy need %.0f bytes, "
                      "the array holds %zu", 4.0 * G->nzp * (4.0 * n_side + 1.0), (size_t)LEAP_STATIC_SCRATCH_BYTES);
        leap_set_error(msg);
        return LEAP_UNSUPPORTED;
    }
    float *volz = (G->device >= 0 && G->device < LEAP_MAX_DEVICES) ? g_static_scratch[G->device] : nullptr;
    if (!volz) {
        leap_set_error("static scratch address unknown for the handle's device");
        return LEAP_HIP_ERROR;
    }
    S.volz = volz;
    S.item_floats = ((size_t)S.width * n_side + 1) * (size_t)G->nzp;
    const int width = S.width, per = S.items;
    // the array keeps what the last call (of any handle) left in it: restore the zeros around this geometry's columns
    const unsigned ncolumns = (unsigned)width * (unsigned)n_side;
    const unsigned nthreads = ncolumns * 2u * FP_PAD > (unsigned)G->nzp ? ncolumns * 2u * FP_PAD : (unsigned)G->nzp;
    for (int it = 0; it < per && !G->fp_rows; ++it)          // (a copy by detector rows has no pads)
        hipLaunchKernelGGL(sf_clear_column_pads, dim3(cdiv(nthreads, 256)), dim3(256), 0, stream, volz + (size_t)it * S.item_floats,
                           ncolumns, g.nz, G->nzp);
    LEAP_HIP_CHECK(hipGetLastError());
    return run_forward_columns(G, S, d_vol, d_sino, batch, stream);
}
