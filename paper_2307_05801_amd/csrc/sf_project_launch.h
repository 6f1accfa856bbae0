// Launchers of the column-wise footprint forward kernels, for PARTS waves per bundle.
#pragma once

#include "leap_internal.h"
#include "sf_project_columns.h"
#include "sf_project_rows.h"

// Two volumes per wave where a batch brings them; an odd last item by itself.
template <int HC, int RG, int CW, int GT, int NS, int PARTS>
static void launch_fp_columns(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int first,
                              int blocks)
{
    const SfGeom &g = G->g;
    const int col_tiles = (int)cdiv(g.ncols, (PARTS > 1 ? 1 : FP_WAVES) * CW), bands = (int)cdiv(g.nrows, RG * 128);
    // XCD-aware block order (see the kernel): pad views to blocks of vb and each XCD's tiles to chunks of tb
    const int vb = G->fp_vb, tb = G->fp_tb;
    const int vgroups_pad = (int)cdiv(g.nviews, vb) * vb;
    const int tiles_per_xcd_pad = (int)cdiv(cdiv(col_tiles, 8), tb) * tb;
    int nq_log2 = 2;
    while ((1 << nq_log2) < G->fp_nq) ++nq_log2;
    dim3 grid((unsigned)(8 * tiles_per_xcd_pad * vgroups_pad * bands), (unsigned)blocks, 1);
    hipLaunchKernelGGL((sf_project_columns<HC, RG, CW, GT, NS, PARTS>), grid, dim3((PARTS > 1 ? PARTS : FP_WAVES) * 64, 1, 1), 0, stream, g, G->d_views,
                       S.volz + (size_t)first * S.item_floats, d_sino + (size_t)first * g.nviews * g.nrows * g.ncols, G->d_major, G->nzp,
                       S.item_floats, nq_log2, col_tiles, bands, vb, tb, G->fp_turn, vgroups_pad, tiles_per_xcd_pad, slab,
                       (const SfGeom *)G->d_geoms);
}

template <int HC, int RG, int CW, int GT, int NS, int PARTS>
static bool launch_fp_instance(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int first,
                               int blocks)
{
    if constexpr (fp_instance_exists(HC, RG, CW, GT, NS, PARTS)) {
        launch_fp_columns<HC, RG, CW, GT, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
        return true;
    } else {
        return false;
    }
}

template <int HC, int RG, int NS, int PARTS>
static bool launch_fp_w(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int first, int blocks)
{
    const int gt = G->g.type == SF_CONE_CURVED ? 1 : (G->g.type == SF_MODULAR ? 2 : 0);
    switch (gt * 10 + G->fp_cw) {
    case 1: return launch_fp_instance<HC, RG, 1, 0, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 2: return launch_fp_instance<HC, RG, 2, 0, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 4: return launch_fp_instance<HC, RG, 4, 0, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 12: return launch_fp_instance<HC, RG, 2, 1, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 14: return launch_fp_instance<HC, RG, 4, 1, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 22: return launch_fp_instance<HC, RG, 2, 2, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 24: return launch_fp_instance<HC, RG, 4, 2, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    default: return false;
    }
}

template <int HC, int NS, int PARTS>
static bool launch_fp_rg(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int first, int blocks)
{
    switch (NS == 2 ? G->fp_pair_rg : G->fp_rg) {
    case 1: return launch_fp_w<HC, 1, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 2: return launch_fp_w<HC, 2, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 3: return launch_fp_w<HC, 3, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    case 4: return launch_fp_w<HC, 4, NS, PARTS>(G, S, slab, d_sino, stream, first, blocks);
    default: return false;
    }
}

template <int HC, int PARTS>
static bool launch_fp_sets(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    const int paired = leap_forward_paired(G, items);
    return (!paired || launch_fp_rg<HC, 2, PARTS>(G, S, slab, d_sino, stream, 0, paired / 2)) &&
           (paired == items || launch_fp_rg<HC, 1, PARTS>(G, S, slab, d_sino, stream, paired, items - paired));
}

template <int RV, int RG, int CW, int PARTS>
static void launch_fp_rows(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    const SfGeom &g = G->g;
    const int col_tiles = (int)cdiv(g.ncols, (PARTS > 1 ? 1 : FP_WAVES) * CW), bands = (int)cdiv(g.nrows, RG * 64 * RV);
    const int vb = G->fp_vb, tb = G->fp_tb;
    const int vgroups_pad = (int)cdiv(g.nviews, vb) * vb;
    const int tiles_per_xcd_pad = (int)cdiv(cdiv(col_tiles, 8), tb) * tb;
    int nq_log2 = 2;
    while ((1 << nq_log2) < G->fp_nq) ++nq_log2;
    dim3 grid((unsigned)(8 * tiles_per_xcd_pad * vgroups_pad * bands), (unsigned)items, 1);
    hipLaunchKernelGGL((sf_project_rows<RV, RG, CW, PARTS>), grid, dim3((PARTS > 1 ? PARTS : FP_WAVES) * 64, 1, 1), 0, stream, g, G->d_views, S.volz, d_sino, G->d_major,
                       G->nzp, S.item_floats, nq_log2, col_tiles, bands, vb, tb, G->fp_turn, vgroups_pad, tiles_per_xcd_pad, slab);
}

template <int PARTS>
static bool launch_fp_rows_slab(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items)
{
    switch (G->fp_rows * 100 + G->fp_row_groups * 10 + G->fp_cw) {
    case 112: launch_fp_rows<1, 1, 2, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 114: launch_fp_rows<1, 1, 4, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 212: launch_fp_rows<2, 1, 2, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 214: launch_fp_rows<2, 1, 4, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 412: launch_fp_rows<4, 1, 2, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 414: launch_fp_rows<4, 1, 4, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 422: launch_fp_rows<4, 2, 2, PARTS>(G, S, slab, d_sino, stream, items); return true;
    case 424: launch_fp_rows<4, 2, 4, PARTS>(G, S, slab, d_sino, stream, items); return true;
    default: return false;
    }
}

template <int PARTS>
static bool launch_fp_slab(const leap_geometry *G, const FwdScratch &S, const SfSlab &slab, int waves, float *d_sino, hipStream_t stream, int items)
{
    if (G->fp_rows) return waves == 2 ? launch_fp_rows_slab<PARTS == 1 ? 1 : 2>(G, S, slab, d_sino, stream, items) : launch_fp_rows_slab<PARTS>(G, S, slab, d_sino, stream, items);
    switch (fp_height_class(G->fp_nkp)) {
    case 0: return launch_fp_sets<0, PARTS>(G, S, slab, d_sino, stream, items);
    case 1: return launch_fp_sets<1, PARTS>(G, S, slab, d_sino, stream, items);
    case 2: return launch_fp_sets<2, PARTS>(G, S, slab, d_sino, stream, items);
    case 3: return launch_fp_sets<3, PARTS>(G, S, slab, d_sino, stream, items);
    case 4: return launch_fp_sets<4, PARTS>(G, S, slab, d_sino, stream, items);
    default: return false;
    }
}
