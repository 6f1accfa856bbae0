// Forward projection (A) of the footprint model for parallel beams: without magnification a row's overlaps with the voxels
// along z are the same for every voxel column and view, so they are applied once, by the copy that lays a slab of the volume out
// z-fastest (sf_volume_to_rows): the scratch then holds, per voxel column, one number per detector ROW, and what is left per
// view is the in-plane part,
//   y[r, c] = amp sum over voxel columns F_u(c) rows[column][r].
//
// Work split, slabs, candidate records and block order are those of sf_project_columns.h: a wave owns CW adjacent detector
// columns of one view, forms the candidates' F_u lane-parallel and walks them.  A lane owns RV adjacent rows per group of 64 RV
// rows, which one load of 4 RV bytes fetches, and a visit is that load and RV FMAs per group and touched column: no placement,
// no axial sums.  256^3, 180 views of 256^2, A: 1.37 -> 1.21 ms; what is left is the rate at which a visit's kilobyte of rows comes from
// beyond L1 (the whole copy, 70 MB, is larger than the L2s).
#pragma once

#include "sf_project_columns.h"

// Overlap of detector row r with the voxels along z (parallel beams): voxels [kb, kb + n), in voxel units.
struct SfRowOverlap {
    int kb, n;
    float lo, hi;        // the row covers [lo, hi) measured from voxel kb
};

SF_HD SfRowOverlap sf_row_overlap(const SfGeom &g, int r)
{
    SfRowOverlap o;
    const double kap0 = (((double)r - g.row_offd) * g.ikvd - g.zlo0d) * g.iTzd, fl = floor(kap0);
    o.kb = (int)fl;
    o.lo = (float)(kap0 - fl);
    o.hi = (float)(kap0 - fl + g.ikvd * g.iTzd);
    o.n = (int)ceilf(o.hi);
    return o;
}

SF_HD float sf_row_weight(const SfRowOverlap &o, int t)
{
    return fmaxf(fminf((float)(t + 1), o.hi) - fmaxf((float)t, o.lo), 0.0f);
}

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

// vol [nz][ny][nx]  ->  the slab's scratch copy by detector rows: columns (i, j), i0 <= i < i0 + ni, j0 <= j < j0 + nj, at
// rows[((j - j0) ni + (i - i0)) nzp + r].  Block 32 x 8 threads, tile 32 (i) x 32 (r) of one j; blockIdx.z = (j - j0) + nj * item.
static __global__ __launch_bounds__(256) void sf_volume_to_rows(SfGeom g, const float *__restrict__ vol, float *__restrict__ rows, int nzp, int i0,
                                                         int j0, int ni, int nj, size_t item_stride)
{
    __shared__ float tile[32][33];
    const int item = blockIdx.z / nj, jr = blockIdx.z - item * nj, j = j0 + jr;
    const size_t kstride = (size_t)g.nx * g.ny;
    vol += (size_t)item * kstride * g.nz;
    rows += (size_t)item * item_stride;
    const int ib = blockIdx.x * 32, rb = blockIdx.y * 32;
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int ihi = i0 + ni < g.nx ? i0 + ni : g.nx;
    if (j >= g.ny) return;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int r = rb + ty + 8 * s, i = i0 + ib + tx;
        float sum = 0.0f;
        if (r < g.nrows && i < ihi) {
            const SfRowOverlap o = sf_row_overlap(g, r);
            for (int t = 0; t < o.n; ++t) {
                const int k = o.kb + t;
                const float w = sf_row_weight(o, t);
                if ((unsigned)k < (unsigned)g.nz && w > 0.0f) sum = fmaf(w, vol[(size_t)k * kstride + (size_t)j * g.nx + i], sum);
            }
        }
        tile[ty + 8 * s][tx] = sum;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int ir = ib + ty + 8 * s, r = rb + tx;
        if (i0 + ir < ihi && r < g.nrows) rows[((size_t)jr * ni + ir) * nzp + r] = tile[tx][ty + 8 * s];
    }
}

// RV: adjacent rows per lane and group (1, 2, 4); RG: groups of 64 RV rows per wave; CW: detector columns per wave.
template <int RV, int RG, int CW, int PARTS>
__global__ __launch_bounds__((PARTS > 1 ? PARTS : FP_WAVES) * 64) void sf_project_rows(SfGeom g, const SfView *__restrict__ views, const float *__restrict__ rows,
                                                                 float *__restrict__ sino, const unsigned char *__restrict__ major, int nzp,
                                                                 size_t item_stride, int nq_log2, int col_tiles, int bands, int vb, int tb, int turn,
                                                                 int vgroups_pad, int tiles_per_xcd_pad, SfSlab all)
{
    rows += (size_t)blockIdx.y * item_stride;
    sino += (size_t)blockIdx.y * g.nviews * g.nrows * g.ncols;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int ct, band, a;
    if (!fp_block(tb, vb, turn, vgroups_pad, tiles_per_xcd_pad, col_tiles, g.nviews, bands, ct, band, a)) return;      // (whole workgroups)
    const int bundle = PARTS > 1 ? ct : ct * FP_WAVES + wave, part = PARTS > 1 ? wave : 0, c0 = bundle * CW;
    if (c0 >= g.ncols) return;                                               // (waves that share a bundle return together)
    const int nbundles = (g.ncols + CW - 1) / CW;
    const int own = __builtin_amdgcn_readfirstlane((int)major[(size_t)a * nbundles + bundle]);
    const SfSlab slab = sf_slab_for(all, own, g.nx, g.ny);
    if (own != slab.xmajor) return;                                          // this bundle reads the other kind of slab
    const int band0 = band * (RG * 64 * RV);
    const SfView v = views[a];
    const SfRayLines L = sf_ray_lines<0>(g, v, c0, CW, slab.xmajor);
    const int n_minor = slab.xmajor ? g.ny : g.nx;

    float acc[CW][RG][RV];
#pragma unroll
    for (int cw = 0; cw < CW; ++cw)
#pragma unroll
        for (int gq = 0; gq < RG; ++gq)
#pragma unroll
            for (int t = 0; t < RV; ++t) acc[cw][gq][t] = 0.0f;
    const int slot = lane & ((1 << nq_log2) - 1), nrel = lane >> nq_log2, sb_slabs = 64 >> nq_log2;
    const unsigned row_bytes = (unsigned)g.nrows * 4u;                       // rows beyond the detector read as zero
    const int off0 = (band0 + RV * lane) * 4;
    __shared__ float4 recs[PARTS > 1 ? PARTS : FP_WAVES][PARTS > 1 ? 128 : 64];      // (the parts' sums take twice the records' room)
    float4 *rec = recs[wave];

    int nb_first = slab.n0, nb_end = slab.n1;
    if constexpr (PARTS > 1) fp_part_of(slab, sb_slabs, part, PARTS, nb_first, nb_end);
    for (int nb = nb_first; nb < nb_end; nb += sb_slabs) {
        // ---- lane-parallel: one candidate voxel column per lane
        const int n = nb + nrel;
        int qf, ql;
        sf_candidates(L, n, qf, ql);
        const int q = qf + slot;
        const bool valid = n < slab.n1 && q >= 0 && q < n_minor && q <= ql;
        const int i = slab.xmajor ? n : q, j = slab.xmajor ? q : n;
        const int ic = valid ? i : (slab.xmajor ? slab.n0 : 0), jc = valid ? j : (slab.xmajor ? 0 : slab.n0);
        float fa[CW];
        double mu;
        const bool any = sf_candidate_record<CW, 0>(g, v, ic, jc, c0, valid, fa, mu);
        const unsigned colbase = sf_slab_column(slab, g.nx, ic, jc) * (unsigned)nzp;
        rec[lane] = make_float4(fa[0], CW > 1 ? fa[CW > 1 ? 1 : 0] : 0.0f, CW > 2 ? fa[CW > 2 ? 2 : 0] : 0.0f, CW > 3 ? fa[CW > 3 ? 3 : 0] : 0.0f);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        unsigned long long mask = __ballot(any);
        unsigned long long touch[CW];
#pragma unroll
        for (int cw = 0; cw < CW; ++cw) touch[cw] = __ballot(fa[cw] != 0.0f);
        // ---- wave-uniform walk over the candidates that matter, the next one's rows in flight
        float x[RG][RV];
        auto load = [&](int e) {
            const __amdgpu_buffer_rsrc_t col = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(rows + (unsigned)__builtin_amdgcn_readlane((int)colbase, e)), 0, (int)row_bytes, 0x00020000);
            int off = off0;
            asm volatile("" : "+v"(off));    // (or the rows' offsets are worked out before the loop, each for a load of its own)
#pragma unroll
            for (int gq = 0; gq < RG; ++gq)
#pragma unroll
                for (int t = 0; t < RV; ++t)      // the compiler merges these into loads of up to 16 bytes
                    x[gq][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(col, off + (gq * 64 * RV + t) * 4, 0, 0));
        };
        int e = mask ? __builtin_ctzll(mask) : 0;
        if (mask) load(e);
        while (mask) {
            mask &= mask - 1;
            float now[RG][RV];
#pragma unroll
            for (int gq = 0; gq < RG; ++gq)
#pragma unroll
                for (int t = 0; t < RV; ++t) now[gq][t] = x[gq][t];
            const float4 r4 = rec[e];
            const float r[4] = {r4.x, r4.y, r4.z, r4.w};
            const int at = e;
            if (mask) {
                e = __builtin_ctzll(mask);
                load(e);
            }
#pragma unroll
            for (int cw = 0; cw < CW; ++cw) {
                if ((touch[cw] >> at) & 1ull) {
#pragma unroll
                    for (int gq = 0; gq < RG; ++gq)
#pragma unroll
                        for (int t = 0; t < RV; ++t) acc[cw][gq][t] = fmaf(r[cw], now[gq][t], acc[cw][gq][t]);
                }
            }
        }
    }

    if constexpr (PARTS > 1) {
        fp_sum_parts<CW * RG * RV, PARTS>(&acc[0][0][0], &recs[0][0].x, part, lane);
        if (part > 0) return;
    }

    // ---- amplitude and store: CW consecutive floats per row, written together
    float *__restrict__ ya = sino + (size_t)a * g.nrows * g.ncols;
#pragma unroll
    for (int gq = 0; gq < RG; ++gq)
#pragma unroll
        for (int t = 0; t < RV; ++t) {
            const int r = band0 + gq * 64 * RV + RV * lane + t;
            if (r >= g.nrows) continue;
            float *__restrict__ dst = ya + (size_t)r * g.ncols + c0;
            if constexpr (CW == 4) {
                if (c0 + 3 < g.ncols) {
                    fp_store_four(dst, v.par_amp * acc[0][gq][t], v.par_amp * acc[1][gq][t], v.par_amp * acc[2][gq][t],
                                  v.par_amp * acc[3][gq][t], slab.first);
                    continue;
                }
            }
#pragma unroll
            for (int cw = 0; cw < CW; ++cw)
                if (c0 + cw < g.ncols) dst[cw] = slab.first ? v.par_amp * acc[cw][gq][t] : dst[cw] + v.par_amp * acc[cw][gq][t];
        }
}

#endif
