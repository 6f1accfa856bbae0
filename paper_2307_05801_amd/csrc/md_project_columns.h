// Forward projection (A) of the Siddon model on tilted modules of the modular geometry ("CT Projection Models and
// Geometries": sources and detectors at any position and orientation): ray-driven gather, one ray per lane.
//
// Same slab formulation, same z-fastest scratch copy of one slab of the volume and same launch order as the circular
// kernel (sd_project_columns.h), but nothing is shared between the rays of a detector column any more: a tilted
// module's column does not lie in a vertical plane, so every ray has its own in-plane line.  A wavefront still owns one
// detector column of one view and RG * 64 of its rows, because those rays run side by side through the volume: at any
// slab they sit in the same or in neighbouring voxel columns and their axial cells are consecutive, which is what
// the z-fastest copy is laid out for.  Each lane derives its ray's constants from the view's pose once, in double
// (minor(X) = m X + b with |m| <= 1 along the in-plane axis the ray advances fastest on, Z(X) = mz X + bz), and then
// walks the slabs of the launch's kind: the in-plane split of the slab (sd_slab_split), the lower axial cell and the
// share of the slab spent in it, four gathers.  Rays whose fastest in-plane axis is the other one sit the launch out.
//
// Chosen on the host only if no ray crosses more than one z-face per slab (|mz| <= 1) and every source keeps more than
// a voxel's distance from the volume's box (then a slab that holds the source contributes nothing and is skipped).
#pragma once

#include "md_siddon.h"
#include "sd_project_columns.h"

// A ray of a tilted module in the slab formulation of sd_ray.h.
struct MdSlabRay {
    SdRayCol R;          // m, b, inv_m, xmajor as for the circular scanners; h0 = Z at X = 0, dh = mz (so v_r = 1, zk0 = 0)
    double xs;           // major index coordinate of the source
    float len;           // mm of ray per unit of X
    int n_lo, n_hi;      // slabs that lie wholly in front of the source: n_lo <= n <= n_hi
};

SF_HD MdSlabRay md_slab_ray(const SfGeom &g, const MdPose &P, int r, int c)
{
    MdSlabRay M;
    const double u = ((double)c - g.col_offd) * g.pu_d, v = fma((double)r, g.pvd, g.v0d);
    double D[3];
    for (int a = 0; a < 3; ++a) D[a] = P.C[a] + u * P.ucol[a] + v * P.vrow[a] - P.S[a];
    const bool xmajor = fabs(D[0]) >= fabs(D[1]);
    const double dmaj = xmajor ? D[0] : D[1], dmin = xmajor ? D[1] : D[0];
    const double lo_maj = (xmajor ? g.x0d : g.y0d) - 0.5 * g.Td, lo_min = (xmajor ? g.y0d : g.x0d) - 0.5 * g.Td;
    const double smaj = xmajor ? P.S[0] : P.S[1], smin = xmajor ? P.S[1] : P.S[0];
    const double iT = 1.0 / g.Td, inv = 1.0 / dmaj;
    M.xs = (smaj - lo_maj) * iT;
    M.R.m = dmin * inv;
    M.R.b = (smin - lo_min) * iT - M.R.m * M.xs;
    M.R.dh = D[2] * inv * g.Td / g.Tzd;
    M.R.h0 = (P.S[2] - g.zlo0d) / g.Tzd - M.R.dh * M.xs;
    const double am = fabs(M.R.m);
    M.R.inv_m = am > 1e-30 ? (float)(1.0 / M.R.m) : 1e30f;
    M.R.lxy = 0.0f; M.R.vscale = 0.0f;
    M.R.xmajor = xmajor ? 1 : 0;
    M.len = (float)(g.Td * sqrt(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]) * fabs(inv));
    // towards larger X the slabs from ceil(xs) on, towards smaller X those up to floor(xs) - 1 (bounds kept within int)
    const double far = 1073741824.0;
    const double xc = fmin(fmax(M.xs, -far), far);
    const bool forward = dmaj > 0.0;
    M.n_lo = forward ? (int)ceil(xc) : -1073741824;
    M.n_hi = forward ? 1073741824 : (int)floor(xc) - 1;
    return M;
}

// Slab n lies wholly in front of the source.
SF_HD bool md_slab_in_front(const MdSlabRay &M, int n) { return n >= M.n_lo && n <= M.n_hi; }

// Per-ray constants of the axial split.
struct MdAxial {
    double zadj;         // Z at X = 0 of the lower end of a slab's piece, plus the pad of the scratch copy's z-columns
    float inv_amz;       // 1 / |dZ per slab|
    bool inc;            // Z rises with X
};

SF_HD MdAxial md_axial(const MdSlabRay &M)
{
    MdAxial A;
    const double mz = M.R.dh;
    A.zadj = M.R.h0 + (double)FP_PAD + fmin(mz, 0.0);
    const float amz = fabsf((float)mz);
    A.inv_amz = amz > 1e-30f ? 1.0f / amz : 1e30f;
    A.inc = mz >= 0.0;
    return A;
}

// Where the voxel columns of a slab's scratch copy (columns of nzp floats) lie as a ray of marching axis x (xmajor) or y sees them:
// column (slab n, minor index q) at base + q pitch_q, base growing by pitch_n per slab from 0 at slab.n0.  One integer
// multiplication per ray and slab instead of four.
struct MdPitch {
    unsigned q, n;
};

SF_HD MdPitch md_pitch(const SfSlab &slab, bool xmajor, int nx, int nzp)
{
    return {(unsigned)nzp * (xmajor ? (unsigned)slab.width : 1u), (unsigned)nzp * (xmajor ? 1u : (unsigned)nx)};
}

// Does the ray meet the volume in cell a (b) of slab n?  now: it reads this kind of slab.
SF_HD void md_slab_meets(const MdSlabRay &M, const SdSplit &s, int n, int n_minor, bool now, bool &a_ok, bool &b_ok)
{
    const bool live = now && md_slab_in_front(M, n);
    a_ok = live & ((unsigned)s.qa < (unsigned)n_minor);
    b_ok = live & (s.qa != s.qb) & ((unsigned)s.qb < (unsigned)n_minor);
}

// Offset of cell a's column, of the neighbouring column that cell b is (only where the ray crosses), and of the lower axial cell
// within a column; the share of the slab spent in it.  A cell outside the volume is read from the zero column instead.
SF_HD unsigned md_cell_a(const SdSplit &s, const MdPitch &pitch, unsigned base) { return (unsigned)s.qa * pitch.q + base; }
SF_HD unsigned md_cell_b(const SdSplit &s, const MdPitch &pitch, unsigned at_a) { return s.qb > s.qa ? at_a + pitch.q : at_a - pitch.q; }
SF_HD void md_axial_place(const MdSlabRay &M, const MdAxial &A, int n, int nzp, unsigned &k, float &tlow)
{
    int kf;
    sd_axial_cell(fma((double)n, M.R.dh, A.zadj), A.inv_amz, nzp - 2, kf, tlow);
    k = (unsigned)kf;
}

// A slab in which the ray stays in one in-plane cell: sd_gather_two's sums without the second cell's, bit for bit.
SF_HD float md_gather_one(float x0, float x1, float tlow, float acc) { return fmaf(1.0f - tlow, x1, fmaf(tlow, x0, acc)); }

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

template <int RG, int SD_WAVES>
__global__ __launch_bounds__(SD_WAVES * 64) void md_project_columns(SfGeom g, const MdPose *__restrict__ poses,
                                                                    const float *__restrict__ volz, float *__restrict__ sino,
                                                                    int nzp, size_t item_stride, unsigned zero_col, int col_tiles,
                                                                    int bands, int vb, int tb, int turn, int views_pad,
                                                                    int tiles_per_xcd_pad, SfSlab all)
{
    volz += (size_t)blockIdx.y * item_stride;
    sino += (size_t)blockIdx.y * g.nviews * g.nrows * g.ncols;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int ct, band, a;
    if (!fp_block(tb, vb, turn, views_pad, tiles_per_xcd_pad, col_tiles, g.nviews, bands, ct, band, a)) return;
    const int c = ct * SD_WAVES + wave;
    if (c >= g.ncols) return;
    const int band0 = band * (RG * 64);
    const MdPose P = poses[a];

    MdSlabRay M[RG];
    MdAxial A[RG];
    float acc[RG];
    bool mine[RG];
    bool inside[RG];
#pragma unroll
    for (int gq = 0; gq < RG; ++gq) {
        const int r = band0 + 64 * gq + lane;
        M[gq] = md_slab_ray(g, P, r < g.nrows ? r : g.nrows - 1, c);
        A[gq] = md_axial(M[gq]);
        inside[gq] = r < g.nrows;
        mine[gq] = false;
        acc[gq] = 0.0f;
    }
    // the slabs of this launch's kind; the whole volume serves the rays of either axis, one after the other
    bool any = false;
    for (int kind = 1; kind >= 0; --kind) {
        const SfSlab slab = sf_slab_for(all, kind, g.nx, g.ny);
        if (slab.xmajor != kind) continue;
        bool now[RG], some = false;
#pragma unroll
        for (int gq = 0; gq < RG; ++gq) {
            now[gq] = inside[gq] && M[gq].R.xmajor == kind;
            mine[gq] = mine[gq] || now[gq];
            some = some || now[gq];
        }
        if (__ballot(some) == 0ull) continue;        // no ray of this wave reads this kind of slab
        any = true;
        // The rays of a detector column run nearly together, so a slab usually finds all of them in the volume or none, and
        // changing their in-plane cell or none: slabs that all miss are skipped, and the second cells are only read where some
        // ray enters one.  256^3 x 360 views x 256^2: 8.35 -> 6.30 ms (8.87 with a branch per row group: the groups' loads must
        // be in flight together).
        const int n_minor = kind ? g.ny : g.nx;
        const MdPitch pitch = md_pitch(slab, kind != 0, g.nx, nzp);
        unsigned base_n = 0;
        for (int n = slab.n0; n < slab.n1; ++n, base_n += pitch.n) {
            SdSplit s[RG];
            bool a_ok[RG], b_ok[RG], meets = false, two = false;
#pragma unroll
            for (int gq = 0; gq < RG; ++gq) {
                s[gq] = sd_slab_split(M[gq].R, n);
                md_slab_meets(M[gq], s[gq], n, n_minor, now[gq], a_ok[gq], b_ok[gq]);
                meets = meets || a_ok[gq] || b_ok[gq];
                two = two || s[gq].qa != s[gq].qb;
            }
            if (__builtin_amdgcn_ballot_w64(meets) == 0) continue;
            float tlow[RG], xa0[RG], xa1[RG];
            unsigned at_a[RG], k[RG];
#pragma unroll
            for (int gq = 0; gq < RG; ++gq) {
                md_axial_place(M[gq], A[gq], n, nzp, k[gq], tlow[gq]);
                at_a[gq] = md_cell_a(s[gq], pitch, base_n);
                const float *__restrict__ xa = volz + ((a_ok[gq] ? at_a[gq] : zero_col) + k[gq]);
                xa0[gq] = xa[0]; xa1[gq] = xa[1];
            }
            if (__builtin_amdgcn_ballot_w64(two)) {
                float xb0[RG], xb1[RG];
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) {
                    const unsigned at_b = md_cell_b(s[gq], pitch, at_a[gq]);
                    const float *__restrict__ xb = volz + ((b_ok[gq] ? at_b : zero_col) + k[gq]);
                    xb0[gq] = xb[0]; xb1[gq] = xb[1];
                }
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) {
                    const float xa[2] = {xa0[gq], xa1[gq]}, xb[2] = {xb0[gq], xb1[gq]};
                    acc[gq] = sd_gather_two(xa, xb, A[gq].inc, s[gq].f, 1.0f - s[gq].f, tlow[gq], acc[gq]);
                }
            } else {
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) acc[gq] = md_gather_one(xa0[gq], xa1[gq], tlow[gq], acc[gq]);
            }
        }
    }
    if (!any) return;

    float *__restrict__ ya = sino + (size_t)a * g.nrows * g.ncols + c;
#pragma unroll
    for (int gq = 0; gq < RG; ++gq) {
        const int r = band0 + 64 * gq + lane;
        if (mine[gq]) {
            const float part = M[gq].len * acc[gq];
            ya[(size_t)r * g.ncols] = all.first ? part : ya[(size_t)r * g.ncols] + part;
        }
    }
}

#endif
