// Forward projection (A) of the Siddon model: ray-driven gather, one wavefront per detector column.
//
// Uses the z-fastest padded scratch copy of one slab of the volume, as the footprint kernel does (sf_project_columns.h:
// slabs across x serve the rays that advance fastest along x, slabs across y the others; every ray adds the slab's share
// to its sample, the first slab of its kind overwrites), plus one all-zero column at the copy's end that stands in for
// every in-plane cell outside the volume.
//
// Work split.  One 64-lane wavefront owns one detector column of one view and a band of RG * 64 detector rows: lane l
// owns rows band0 + 64 g + l, g < RG.  All those rays share their in-plane line, so which voxel columns they cross in
// a slab, and where inside the slab they change from one to the next, is wave-uniform: 64 slabs at a time, lane n
// works that out for slab n, and the wave then walks the slabs, broadcasting the few numbers through v_readlane.
// What differs between the lanes is the axial position: each lane follows its own Z through the slab and splits the
// slab's piece(s) between the two axial cells it can touch (the kernel is only chosen when no ray crosses more than
// one z-face per slab).  A workgroup is SD_WAVES adjacent columns of one view, which share voxel columns in L1.
#pragma once

#include "sd_ray.h"
#include "sf_project_columns.h"

// ---- the axial part of a slab, shared by the kernel and by the host-side re-enactment of its arithmetic ---------------

// Per ray (lane and row group): the row's v, the constant of its lower-Z map, 1 / |dZ per slab|, and the sign of dZ.
struct SdAxial {
    double vr, zadj;
    float inv_amz;
    bool inc;
};

SF_HD SdAxial sd_axial(const SfGeom &g, const SdRayCol &R, int r)
{
    SdAxial A;
    A.vr = sd_row_v(g, r);
    const double mz = A.vr * R.dh;
    A.zadj = g.zk0d + (double)FP_PAD + fmin(mz, 0.0);     // Z of the lower end of the slab's piece, plus the copy's pad
    const float amz = fabsf((float)mz);
    A.inv_amz = amz > 1e-30f ? 1.0f / amz : 1e30f;
    A.inc = mz >= 0.0;
    return A;
}

// Lower axial cell of the slab's piece as an index into the padded z-column (clamped: far outside the column the ray
// reads the zero pads), and the share of the slab spent in that cell.  zlo: Z of the piece's lower end, plus the pad.
SF_HD void sd_axial_cell(double zlo, float inv_amz, int kmax, int &kf, float &tlow)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const float fr = (float)__builtin_amdgcn_fract(zlo);
    kf = (int)zlo;                                       // the conversion saturates
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(kf) : "v"(kf), "s"(kmax));
#else
    const float fr = (float)(zlo - floor(zlo));
    kf = (int)fmin(fmax(zlo, 0.0), (double)kmax);
#endif
    tlow = fminf((1.0f - fr) * inv_amz, 1.0f);
}

// The same for a ray of the circular scanners.  h: h(X) at the slab's entry face.
SF_HD void sd_axial_place(const SdAxial &A, double h, int kmax, int &kf, float &tlow)
{
    sd_axial_cell(fma(A.vr, h, A.zadj), A.inv_amz, kmax, kf, tlow);
}

// A slab whose piece stays in one in-plane cell: xa points at the lower axial cell of that cell's z-column.
SF_HD float sd_gather_one(const float *__restrict__ xa, float tlow, float acc)
{
    return fmaf(tlow, xa[0], fmaf(1.0f - tlow, xa[1], acc));
}

// A slab whose piece changes from in-plane cell a to b at tau = f (omf = 1 - f): rising rays are in the lower axial cell
// first (while still in cell a), falling rays last.
SF_HD float sd_gather_two(const float *__restrict__ xa, const float *__restrict__ xb, bool inc, float f, float omf, float tlow, float acc)
{
    const float p = fminf(inc ? f : omf, tlow), q = tlow - p;
    const float a_low = inc ? p : q, b_low = inc ? q : p;
    float t = acc;
    t = fmaf(a_low, xa[0], t);
    t = fmaf(f - a_low, xa[1], t);
    t = fmaf(b_low, xb[0], t);
    return fmaf(omf - b_low, xb[1], t);
}

// ---- two adjacent rows per lane ("sd_project_pairs" below) -------------------------------------------------------------
//
// The vector cache charges a wave-wide load for its lanes, not for their width (four lanes per clock, 4 bytes or 16), and
// the one-row kernel, with an 8-byte load per row, slab and in-plane cell, is bound by that.  Two adjacent rows lie less
// than two voxels apart where this kernel is chosen, so the two cells of either lie within four consecutive voxels: one
// 16-byte load per pair and cell.
//
// Placement without conversions, from the UPPER end of a row's piece: Z is formed by one double FMA to which 1.5 * 2^20 has
// been added, so the sum's low word is 2^32 times the fraction, which is the way down to the face below, and its high word
// is a constant plus the upper cell.  The share of the slab spent in the upper cell is that way over |dZ|, at most 1; what is
// carried is the rest, spent in the cell below.

struct SdPairRow {
    double vr, zadj;
    float inv;           // 1 / (2^32 |dZ per slab|)
    bool inc;
};

SF_HD SdPairRow sd_pair_row(const SfGeom &g, const SdRayCol &R, int r)
{
    SdPairRow A;
    A.vr = sd_row_v(g, r);
    const double mz = A.vr * R.dh;
    const float amz = fabsf((float)mz);
    const bool level = !(amz > 1e-30f);
    A.zadj = g.zk0d + (double)FP_PAD + FP_KAP_MAGIC + fmax(mz, 0.0);
    // a ray that runs level stays in its upper cell, on a face in the cell above it
    if (level) A.zadj += SD_LEVEL_LIFT;
    A.inv = (level ? 1e30f : 1.0f / amz) * 2.3283064365386963e-10f;
    A.inc = mz >= 0.0;
    return A;
}

// Upper cell (FP_KAP_HI plus its index in the padded column) and the share of the slab spent in the cell below it.
SF_HD void sd_pair_place(const SdPairRow &A, double h, unsigned &hi, float &low)
{
    const double q = fma(A.vr, h, A.zadj);
    unsigned long long bits;
    __builtin_memcpy(&bits, &q, 8);
    hi = (unsigned)(bits >> 32);
    low = sf_clamp(fmaf(-(float)(unsigned)bits, A.inv, 1.0f), 0.0f, 1.0f);
}

// Shares f and omf of the in-plane cells before and after the crossing, both multiples of 2^-24 that add up to 1 exactly, so that
// a cell the ray does not enter comes out with a weight of 0 below.
SF_HD void sd_pair_crossing(float at, float &f, float &omf)
{
    omf = 1.0f - at;
    f = 1.0f - omf;
}

// Lower and upper axial cell of the pair's upper row among the four voxels loaded from the lower row's lower cell on; d: voxels
// between the rows' upper cells (0, 1 or 2; SPREAD: 1 or 2).
template <bool SPREAD>
SF_HD void sd_pair_upper_row(const float (&x)[4], unsigned d, float &lo, float &up)
{
    lo = d > 1u ? x[2] : x[1];
    up = d > 1u ? x[3] : x[2];
    if constexpr (!SPREAD) {
        lo = d == 0u ? x[0] : lo;
        up = d == 0u ? x[1] : up;
    }
}

// A slab whose piece stays in one in-plane cell: lo, up are the lower and the upper axial cell's voxel.  (The slab's value is
// formed by itself, so that the running sum is rounded once per slab: added in two parts, the sums of 160 slabs came out 1.4
// times further off.  Every cell has a weight of its own: as lo + share (up - lo), one instruction less, a voxel that the ray does
// not meet would round the one that it does, and an infinite voxel come out as NaN.)
SF_HD float sd_pair_one(float lo, float up, float low, float acc) { return acc + fmaf(low, lo, (1.0f - low) * up); }

// A slab whose piece changes from in-plane cell a to b at tau = f (omf = 1 - f): rising rays are in the lower axial cell first
// (while still in a, then in b), falling rays last (in b, then in a).
SF_HD float sd_pair_two(float alo, float aup, float blo, float bup, bool inc, float f, float omf, float low, float acc)
{
    const float p = fminf(low, inc ? f : omf), q = low - p;
    const float la = inc ? p : q, lb = inc ? q : p;
    return acc + fmaf(lb, blo, fmaf(omf - lb, bup, fmaf(la, alo, (f - la) * aup)));
}

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

// RG: groups of 128 rows per wave: lane l owns the row pairs band0 + 128 g + 2 l + {0, 1}.  SPREAD: adjacent rows are at least
// one voxel apart everywhere (one test tells where the upper row's cells lie in the load instead of two).  MOD as below.
// Slabs whose cells both lie outside the volume are skipped; a single cell outside is read through an empty buffer
// descriptor, which returns zeros without touching memory.
template <int RG, bool SPREAD, bool MOD>
__global__ __launch_bounds__(256) void sd_project_pairs(SfGeom gk, const SdRayCol *__restrict__ rays, const float *__restrict__ volz,
                                                        float *__restrict__ sino, int nzp, size_t item_stride, int col_tiles, int bands,
                                                        int vb, int tb, int turn, int views_pad, int tiles_per_xcd_pad, SfSlab all,
                                                        const SfGeom *__restrict__ geoms)
{
    constexpr int WAVES = 4, ROWS = RG * 128;
    __shared__ float4 recs[WAVES][64];
    __shared__ float4 out[ROWS];                     // [row][column]: the workgroup's share of the sinogram
    __shared__ int live_waves[WAVES];
    volz += (size_t)blockIdx.y * item_stride;
    sino += (size_t)blockIdx.y * gk.nviews * gk.nrows * gk.ncols;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int ct, band, a;
    if (!fp_block(tb, vb, turn, views_pad, tiles_per_xcd_pad, col_tiles, gk.nviews, bands, ct, band, a)) return;   // whole workgroups
    const int c = ct * WAVES + wave;
    const SfGeom &g = MOD ? geoms[a] : gk;
    const int band0 = band * ROWS;
    const SdRayCol R = rays[(size_t)a * g.ncols + (c < g.ncols ? c : g.ncols - 1)];
    const SfSlab slab = sf_slab_for(all, R.xmajor, g.nx, g.ny);
    const bool live = c < g.ncols && R.xmajor == slab.xmajor;        // this column's rays read this kind of slab

    SdPairRow A[RG][2];
    float acc[RG][2];
#pragma unroll
    for (int gq = 0; gq < RG; ++gq)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            A[gq][p] = sd_pair_row(g, R, band0 + 128 * gq + 2 * lane + p);
            acc[gq][p] = 0.0f;
        }
    if (live) {
        const int n_major = slab.n1, n_minor = R.xmajor ? g.ny : g.nx;
        const unsigned col_bytes = (unsigned)nzp * 4u;
        const unsigned off_k = 0u - (FP_KAP_HI << 2) - 4u;           // byte offset of the cell below the lower row's upper cell
        for (int nb = slab.n0; nb < n_major; nb += 64) {
            // ---- lane-parallel: the in-plane part of slab nb + lane
            const int n = nb + lane;
            const SdSplit s = sd_slab_split(R, n);
            const bool in_n = n < n_major, two = s.qa != s.qb;
            const bool a_ok = in_n && s.qa >= 0 && s.qa < n_minor, b_ok = in_n && two && s.qb >= 0 && s.qb < n_minor;
            const unsigned base_a = a_ok ? sf_slab_column(slab, g.nx, R.xmajor ? n : s.qa, R.xmajor ? s.qa : n) * (unsigned)nzp : 0u;
            const unsigned base_b = b_ok ? sf_slab_column(slab, g.nx, R.xmajor ? n : s.qb, R.xmajor ? s.qb : n) * (unsigned)nzp : 0u;
            const double h = fma((double)n, R.dh, R.h0);
            float f, omf;
            sd_pair_crossing(s.f, f, omf);
            recs[wave][lane] = make_float4(__builtin_bit_cast(float, __double2loint(h)), __builtin_bit_cast(float, __double2hiint(h)), f, omf);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const unsigned long long in_a = __ballot(a_ok), in_b = __ballot(b_ok), cross = __ballot(two);
            // ---- wave-uniform walk over the slabs that meet the volume
            for (unsigned long long mask = in_a | in_b; mask; mask &= mask - 1) {
                const int e = __builtin_ctzll(mask);
                const float4 rec = recs[wave][e];
                const double s_h = __hiloint2double(__builtin_bit_cast(int, rec.y), __builtin_bit_cast(int, rec.x));
                const __amdgpu_buffer_rsrc_t col_a = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(volz + (unsigned)__builtin_amdgcn_readlane((int)base_a, e)), 0, (in_a >> e) & 1ull ? (int)col_bytes : 0, 0x00020000);
                auto place = [&](int gq, float (&low)[2], int &off, unsigned &d) {
                    unsigned hi0, hi1;
                    sd_pair_place(A[gq][0], s_h, hi0, low[0]);
                    sd_pair_place(A[gq][1], s_h, hi1, low[1]);
                    asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(off) : "v"(hi0), "s"(off_k));
                    d = hi1 - hi0;                    // 0, 1 or 2 (SPREAD: 1 or 2) voxels between the rows' upper cells
                };
                auto load = [&](const __amdgpu_buffer_rsrc_t &col, int off, float (&x)[4]) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) x[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(col, off + 4 * t, 0, 0));
                };
                if ((cross >> e) & 1ull) {
                    const __amdgpu_buffer_rsrc_t col_b = __builtin_amdgcn_make_buffer_rsrc(
                        (void *)(volz + (unsigned)__builtin_amdgcn_readlane((int)base_b, e)), 0, (in_b >> e) & 1ull ? (int)col_bytes : 0, 0x00020000);
                    float low[RG][2], xa[RG][4], xb[RG][4];
                    unsigned d[RG];
#pragma unroll
                    for (int gq = 0; gq < RG; ++gq) {
                        int off;
                        place(gq, low[gq], off, d[gq]);
                        load(col_a, off, xa[gq]);
                        load(col_b, off, xb[gq]);
                    }
#pragma unroll
                    for (int gq = 0; gq < RG; ++gq) {
                        acc[gq][0] = sd_pair_two(xa[gq][0], xa[gq][1], xb[gq][0], xb[gq][1], A[gq][0].inc, rec.z, rec.w, low[gq][0], acc[gq][0]);
                        float alo, aup, blo, bup;
                        sd_pair_upper_row<SPREAD>(xa[gq], d[gq], alo, aup);
                        sd_pair_upper_row<SPREAD>(xb[gq], d[gq], blo, bup);
                        acc[gq][1] = sd_pair_two(alo, aup, blo, bup, A[gq][1].inc, rec.z, rec.w, low[gq][1], acc[gq][1]);
                    }
                } else {
                    float low[RG][2], x[RG][4];
                    unsigned d[RG];
#pragma unroll
                    for (int gq = 0; gq < RG; ++gq) {
                        int off;
                        place(gq, low[gq], off, d[gq]);
                        load(col_a, off, x[gq]);
                    }
#pragma unroll
                    for (int gq = 0; gq < RG; ++gq) {
                        float lo, up;
                        sd_pair_upper_row<SPREAD>(x[gq], d[gq], lo, up);
                        acc[gq][0] = sd_pair_one(x[gq][0], x[gq][1], low[gq][0], acc[gq][0]);
                        acc[gq][1] = sd_pair_one(lo, up, low[gq][1], acc[gq][1]);
                    }
                }
            }
        }
    }
    // ---- store: the four columns of a row together (each by itself is a 4-byte write into a line of its own)
    if (lane == 0) live_waves[wave] = live;
#pragma unroll
    for (int gq = 0; gq < RG; ++gq)
#pragma unroll
        for (int p = 0; p < 2; ++p)
            reinterpret_cast<float *>(&out[128 * gq + 2 * lane + p])[wave] = sd_ray_length(R, A[gq][p].vr) * acc[gq][p];
    __syncthreads();
    const bool w0 = live_waves[0], w1 = live_waves[1], w2 = live_waves[2], w3 = live_waves[3];
    if (!(w0 | w1 | w2 | w3)) return;
    float *__restrict__ ya = sino + (size_t)a * g.nrows * g.ncols + (size_t)ct * WAVES;
#pragma unroll
    for (int row = threadIdx.x; row < ROWS; row += 256) {
        const int r = band0 + row;
        if (r >= g.nrows) continue;
        const float4 v = out[row];
        float *__restrict__ dst = ya + (size_t)r * g.ncols;
        if (w0 & w1 & w2 & w3) {
            fp_store_four(dst, v.x, v.y, v.z, v.w, slab.first);
        } else {
            if (w0) dst[0] = slab.first ? v.x : dst[0] + v.x;
            if (w1) dst[1] = slab.first ? v.y : dst[1] + v.y;
            if (w2) dst[2] = slab.first ? v.z : dst[2] + v.z;
            if (w3) dst[3] = slab.first ? v.w : dst[3] + v.w;
        }
    }
}

// MOD: modular geometry with upright modules: the wave's view brings its own parameter block geoms[a] (the scene
// translated so that the view is a circular cone-beam view; gk holds the sizes, which all views share).
template <int RG, int SD_WAVES, bool MOD>
__global__ __launch_bounds__(SD_WAVES * 64) void sd_project_columns(SfGeom gk, const SdRayCol *__restrict__ rays,
                                                                    const float *__restrict__ volz, float *__restrict__ sino,
                                                                    int nzp, size_t item_stride, unsigned zero_col, int col_tiles,
                                                                    int bands, int vb, int tb, int turn, int views_pad,
                                                                    int tiles_per_xcd_pad, SfSlab all,
                                                                    const SfGeom *__restrict__ geoms)
{
    // blockIdx.y: item of a batch (its scratch copy and its sinogram)
    volz += (size_t)blockIdx.y * item_stride;
    sino += (size_t)blockIdx.y * gk.nviews * gk.nrows * gk.ncols;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int ct, band, a;
    if (!fp_block(tb, vb, turn, views_pad, tiles_per_xcd_pad, col_tiles, gk.nviews, bands, ct, band, a)) return;   // padding blocks (no barrier follows)
    const int c = ct * SD_WAVES + wave;
    if (c >= gk.ncols) return;
    const SfGeom &g = MOD ? geoms[a] : gk;
    const int band0 = band * (RG * 64);

    const SdRayCol R = rays[(size_t)a * g.ncols + c];
    const SfSlab slab = sf_slab_for(all, R.xmajor, g.nx, g.ny);
    if (R.xmajor != slab.xmajor) return;             // this column's rays read the other kind of slab
    const int n_major = slab.n1;
    const int n_minor = R.xmajor ? g.ny : g.nx;
    const int kmax = nzp - 2;

    SdAxial A[RG];
    float acc[RG];
#pragma unroll
    for (int gq = 0; gq < RG; ++gq) {
        A[gq] = sd_axial(g, R, band0 + 64 * gq + lane);
        acc[gq] = 0.0f;
    }

    for (int nb = slab.n0; nb < n_major; nb += 64) {
        // ---- lane-parallel: the in-plane part of slab nb + lane
        const int n = nb + lane;
        const SdSplit s = sd_slab_split(R, n);
        const bool in_n = n < n_major;
        const bool a_ok = in_n && s.qa >= 0 && s.qa < n_minor;
        const bool b_ok = in_n && s.qa != s.qb && s.qb >= 0 && s.qb < n_minor;
        const unsigned base_a = a_ok ? sf_slab_column(slab, g.nx, R.xmajor ? n : s.qa, R.xmajor ? s.qa : n) * (unsigned)nzp : zero_col;
        const unsigned base_b = b_ok ? sf_slab_column(slab, g.nx, R.xmajor ? n : s.qb, R.xmajor ? s.qb : n) * (unsigned)nzp : zero_col;
        const double h = fma((double)n, R.dh, R.h0);
        const int h_lo = __double2loint(h), h_hi = __double2hiint(h);
        const float f = s.f, omf = 1.0f - s.f;
        const unsigned long long cross = __ballot(in_n && s.qa != s.qb);
        const int count = n_major - nb < 64 ? n_major - nb : 64;

        // ---- wave-uniform walk over the slabs
        for (int e = 0; e < count; ++e) {
            const double s_h = __hiloint2double(__builtin_amdgcn_readlane(h_hi, e), __builtin_amdgcn_readlane(h_lo, e));
            const float s_f = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f), e));
            const float *__restrict__ col_a = volz + (unsigned)__builtin_amdgcn_readlane((int)base_a, e);
            if ((cross >> e) & 1ull) {
                const float s_omf = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, omf), e));
                const float *__restrict__ col_b = volz + (unsigned)__builtin_amdgcn_readlane((int)base_b, e);
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) {
                    int kf;
                    float tlow;
                    sd_axial_place(A[gq], s_h, kmax, kf, tlow);
                    acc[gq] = sd_gather_two(col_a + kf, col_b + kf, A[gq].inc, s_f, s_omf, tlow, acc[gq]);
                }
            } else {
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) {
                    int kf;
                    float tlow;
                    sd_axial_place(A[gq], s_h, kmax, kf, tlow);
                    acc[gq] = sd_gather_one(col_a + kf, tlow, acc[gq]);
                }
            }
        }
    }

    float *__restrict__ ya = sino + (size_t)a * g.nrows * g.ncols + c;
#pragma unroll
    for (int gq = 0; gq < RG; ++gq) {
        const int r = band0 + 64 * gq + lane;
        if (r < g.nrows) {
            const float part = sd_ray_length(R, A[gq].vr) * acc[gq];
            ya[(size_t)r * g.ncols] = slab.first ? part : ya[(size_t)r * g.ncols] + part;
        }
    }
}

#endif
