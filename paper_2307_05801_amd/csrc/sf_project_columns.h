// Forward projection (A), ray-driven gather with wave-uniform footprints.
//
// Data layout.  The kernel reads a z-fastest, zero-padded scratch copy of a SLAB of the volume: the voxel columns (i, j)
// whose index along the slab's axis lies in [n0, n0 + width),
//   volz[col * nzp + FP_PAD + k],   nzp = nz + 2 FP_PAD,   col = (j - j0) * ni + (i - i0),
// so that the voxels a ray bundle needs from a voxel column are contiguous whatever the view angle.  A slab across x
// (i0 = n0, ni = width, j0 = 0) serves the ray bundles that advance fastest along x, a slab across y (j0 = n0, ni = nx,
// i0 = 0) those that advance fastest along y; the host walks the volume slab by slab, and every bundle adds the slab's
// share to its sinogram samples (the first slab of its kind overwrites).  The scratch therefore holds a fraction of
// the volume, chosen by the host.  Where the whole volume fits the scratch, its copy has the same layout whichever axis it is
// cut across, and one copy and one launch serve both kinds of bundles.
//
// Work split.  One 64-lane wavefront owns CW adjacent detector columns of one view and a band of RG * 128 detector
// rows: lane l owns the row PAIRS band0 + 128 g + 2 l + {0, 1}, g < RG, of each of its columns.  Because all lanes share
// (view, columns), the whole transaxial part of the weight (which voxel columns the pixels see, F_u, magnification) is
// the same for the 64 lanes, and the axial part (a row's overlaps with the voxels of a voxel column) is the same for
// the CW pixel columns: it is computed once and applied CW times.  The wave therefore computes the transaxial part
// lane-parallel: per block of 64 / nq slabs along the marching axis, lane (slab, slot) evaluates one candidate voxel
// column; a ballot picks the candidates with F_u > 0 and the wave then walks them one by one, reading a candidate's
// record back from LDS at a wave-uniform address (and the two numbers that must be scalar through v_readlane), while
// each lane accumulates its own rows' axial overlaps.
//
// Two adjacent rows per lane, one load.  The vector cache serves a wave-wide load at four lanes per clock whether a
// lane asks for 4 or for 16 bytes (measured), and two adjacent rows overlap in the voxels they need.  One load of P
// consecutive voxels starting at the voxel of the lower row's lower edge serves both rows of a pair: half the cache
// time and half the placement arithmetic of one load per row.
//
// Placement without conversions.  kappa, the axial voxel coordinate of a row's lower edge, is formed by one double
// FMA to which 1.5 * 2^20 has been added: the sum's unit in the last place is 2^-32, so its low word is kappa's
// fraction and the low bits of its high word are floor(kappa) -- no floor, no conversion, no clamp.  The loads are
// raw buffer loads on a descriptor of the candidate's own padded z-column: whatever lies outside it reads as zero,
// which is the truncation rule for rows that miss the volume.
#pragma once

#include "sf_footprint.h"

#include <type_traits>

constexpr int FP_PAD = 8;        // zero voxels before and after every z-column of the scratch copy (>= the voxels a row pair spans)
constexpr int FP_MAX_P = 7;      // most voxels a pair of adjacent rows may overlap (rows of up to 3 voxels)
constexpr int FP_WAVES = 4;      // waves per workgroup: adjacent column bundles of one view (each wave its own LDS, no barrier)

constexpr int FP_PARTS = 4;      // waves of a workgroup that share a bundle's layers where a scan has few bundles
// Fewest detector rows: below, the general kernel's eight rows per thread waste less than the lanes of a wave (5 rows, 716 columns, 512^2 x 5
// voxels: 60 views 3.5 ms against 1.9 here, 360 views 6.6 against 8.8; 8 rows, 720 views 17.1 against 16.8, 24 rows 58.8 against 17.5).
constexpr int FP_MIN_ROWS = 8;
// Largest copy of a volume whose tiles of columns change XCD every eight views (fp_block).  Forward projection with over without: copies of
// 0.9 to 2.8 MB, 7 to 13 tiles 0.73 to 0.99, 6 to 8 MB, 18 and 19 tiles 1.03 to 1.08, 512^3 1.05 (every view 1.36).
constexpr double FP_TURN_BYTES = 3145728.0;
// Scans of fewer rows than this take the general kernels while a stream is being captured and on the fixed scratch array, so that such calls
// need no scratch at all.
constexpr int FP_FREE_ROWS = 32;

// Highest height class (see SfPairClass) of a scan whose pairs of rows overlap up to nkp voxels.
SF_HD int fp_height_class(int nkp) { return nkp <= 5 ? nkp - 2 : 4; }

// Instances of the column-wise kernel by height class, row groups, columns per wave, detector (GT) and volumes per wave.  Two volumes per
// wave: rows of up to a voxel and a half, taller ones where the sums and voxels of two leave enough waves in flight.  Two against one per
// wave, time ratios where the chip is full, one group of rows / more: rows of 1.5 to 2 voxels 0.69 to 0.92 / 0.91 to 1.16, of 2 to 3
// 0.92 to 1.16 / 1.00 to 1.24; on a cylinder (few waves in flight either way) 0.69 to 0.79 / 0.74 to 0.95 and 0.70 to 0.83 / 0.89 to 1.06.
constexpr bool fp_instance_exists(int hc, int rg, int cw, int gt, int ns, int parts = 1)
{
    if (cw == 1) return gt == 0 && ns == 1 && parts == 1;
    if (ns == 1) return true;
    return rg <= 3 && (hc <= 2 || (hc == 3 && (rg == 1 || gt == 1)) || (hc == 4 && rg == 1 && gt == 1));
}

// Candidate voxel columns of pixel columns c .. c+cw-1 in slab n: in-plane lines through the two outer u-edges of
// the bundle, written as "minor index = m * major index + b".  Wave-uniform.
struct SfRayLines {
    float m0, b0, m1, b1, spread;
    int xmajor;
};

// want_major: -1 picks the marching axis from the bundle's central ray, 0 / 1 forces y / x (the kernel takes the host's
// choice, so that both agree on which slabs a bundle reads even where the two directions tie).
template <int GT = -1>
SF_HD SfRayLines sf_ray_lines(const SfGeom &g, const SfView &v, int c, int cw, int want_major = -1)
{
    SfRayLines L;
    const float ue0 = ((float)c - 0.5f - g.col_off) * g.pu, ue1 = ((float)(c + cw) - 0.5f - g.col_off) * g.pu;
    const float x0 = (float)g.x0d, y0 = (float)g.y0d;
    const float iT = 1.0f / g.T;
    if (g.type == SF_PARALLEL) {
        L.xmajor = want_major < 0 ? (int)(fabsf(v.c) >= fabsf(v.s)) : want_major;
        if (L.xmajor) {            // -x s + y c = u  ->  y = (u + x s)/c
            L.m0 = L.m1 = v.s / v.c;
            L.b0 = (ue0 / v.c + x0 * L.m0 - y0) * iT;
            L.b1 = (ue1 / v.c + x0 * L.m1 - y0) * iT;
        } else {                   // x = (y c - u)/s
            L.m0 = L.m1 = v.c / v.s;
            L.b0 = (-ue0 / v.s + y0 * L.m0 - x0) * iT;
            L.b1 = (-ue1 / v.s + y0 * L.m1 - x0) * iT;
        }
    } else {
        const float uc = 0.5f * (ue0 + ue1);
        const float sx = g.sod * v.c, sy = g.sod * v.s;
        float dxc, dyc, dx0, dy0, dx1, dy1;
        if (sf_is_curved<GT>(g)) {      // u is arc length: directions at the fan angles u / sdd
            float sg, cg;
            sincosf(uc / g.sdd, &sg, &cg);
            dxc = -fmaf(cg, v.c, sg * v.s); dyc = fmaf(sg, v.c, -cg * v.s);
            sincosf(ue0 / g.sdd, &sg, &cg);
            dx0 = -fmaf(cg, v.c, sg * v.s); dy0 = fmaf(sg, v.c, -cg * v.s);
            sincosf(ue1 / g.sdd, &sg, &cg);
            dx1 = -fmaf(cg, v.c, sg * v.s); dy1 = fmaf(sg, v.c, -cg * v.s);
        } else {
            dxc = fmaf(-g.sdd, v.c, -uc * v.s); dyc = fmaf(-g.sdd, v.s, uc * v.c);
            dx0 = fmaf(-g.sdd, v.c, -ue0 * v.s); dy0 = fmaf(-g.sdd, v.s, ue0 * v.c);
            dx1 = fmaf(-g.sdd, v.c, -ue1 * v.s); dy1 = fmaf(-g.sdd, v.s, ue1 * v.c);
        }
        L.xmajor = want_major < 0 ? (int)(fabsf(dxc) >= fabsf(dyc)) : want_major;
        if (L.xmajor) {
            L.m0 = dy0 / dx0;
            L.m1 = dy1 / dx1;
            L.b0 = (sy - y0 + (x0 - sx) * L.m0) * iT;
            L.b1 = (sy - y0 + (x0 - sx) * L.m1) * iT;
        } else {
            L.m0 = dx0 / dy0;
            L.m1 = dx1 / dy1;
            L.b0 = (sx - x0 + (y0 - sy) * L.m0) * iT;
            L.b1 = (sx - x0 + (y0 - sy) * L.m1) * iT;
        }
    }
    L.spread = 0.5f * fmaxf(fabsf(L.m0), fabsf(L.m1)) + 2e-3f;
    return L;
}

// First and last candidate (minor index, unclipped) in slab n.
SF_HD void sf_candidates(const SfRayLines &L, int n, int &q_first, int &q_last)
{
    const float qa = fmaf(L.m0, (float)n, L.b0), qb = fmaf(L.m1, (float)n, L.b1);
    q_first = (int)floorf(fminf(qa, qb) - L.spread + 0.5f);
    q_last = (int)floorf(fmaxf(qa, qb) + L.spread + 0.5f);
}

// One slab of the volume as the scratch copy holds it.
struct SfSlab {
    int n0, n1;       // slab indices [n0, n1) along the marching axis
    int xmajor;       // 1: the slab cuts x (serves bundles that advance fastest along x), 0: it cuts y, -1: the whole volume (serves all)
    int first;        // 1: bundles overwrite their sinogram samples, 0: they add to them
    int width;        // slabs the scratch layout is built for (>= n1 - n0)
};

// The slab as a bundle that advances fastest along x (xmajor == 1) or y sees it: the whole volume is cut across its axis.
SF_HD SfSlab sf_slab_for(const SfSlab &s, int xmajor, int nx, int ny)
{
    SfSlab k = s;
    if (s.xmajor < 0) {
        k.xmajor = xmajor;
        k.n1 = xmajor ? nx : ny;
    }
    return k;
}

// Index of voxel column (i, j) among the columns of the slab's scratch copy.
SF_HD unsigned sf_slab_column(const SfSlab &s, int nx, int i, int j)
{
    return s.xmajor ? (unsigned)(j * s.width + (i - s.n0)) : (unsigned)((j - s.n0) * nx + i);
}

// ---- the arithmetic of one lane, shared by the kernel and by the CPU test harness that steps it -----------------------

// Constant of the kappa map: kappa(r) = (r - row_off) mu + zkp is measured from the start of the padded column and
// carries FP_KAP_MAGIC = 1.5 * 2^20 plus half a unit of the 23-bit fraction used below (so that truncating rounds).
constexpr double FP_KAP_MAGIC = 1572864.0;
constexpr unsigned FP_KAP_HI = 0x41380000u;      // high word of FP_KAP_MAGIC: high word of the sum = FP_KAP_HI + floor(kappa)
SF_HD double sf_kappa_const(const SfGeom &g) { return -g.zlo0d * g.iTzd + (double)FP_PAD + FP_KAP_MAGIC + 5.9604644775390625e-08; }

// Lower edge of a row in its candidate column: rd = row - row_off, mu = voxels per row.  fr1 = 1 + the edge's fraction
// inside its voxel (a float in [1, 2) assembled from the sum's bits), hi = FP_KAP_HI + that voxel's index.
SF_HD void sf_place_row(double rd, double mu, double zkp, float &fr1, unsigned &hi)
{
    const double kap = fma(rd, mu, zkp);
    unsigned long long bits;
    __builtin_memcpy(&bits, &kap, 8);
    const unsigned lo = (unsigned)bits;
    hi = (unsigned)(bits >> 32);
#if defined(__HIP_DEVICE_COMPILE__)
    fr1 = __builtin_bit_cast(float, __builtin_amdgcn_alignbit(0x7fu, lo, 9));
#else
    const unsigned f = (0x7fu << 23) | (lo >> 9);
    __builtin_memcpy(&fr1, &f, 4);
#endif
}

// Axial sums of a pair of adjacent rows.  x[0..P-1]: voxels from the one holding the lower row's lower edge; fr1 as
// above; mu = voxels per row.  The lower row A covers [fr, fr + mu) of that run, the upper row B [fr + mu, fr + 2 mu).  With
// a_t = clamp(fr + mu - t) and b_t = clamp(fr + 2 mu - t), the parts of voxel t below either row's upper edge (additions with the clamp
// modifier are the cheapest way to an overlap), and rows shorter than a voxel, with d_t = x_t - x_0,
//   S_A = mu x_0 + sum a_t d_t,    S_B = 2 mu x_0 + sum b_t d_t - S_A     (voxel 0 gets what the others leave of each row),
// rows of a voxel and more
//   S_A = (1 - fr) x_0 + sum a_t x_t,    S_B = sum (b_t - a_t) x_t        (t >= 1; the upper row does not reach voxel 0).
// Rows are sorted into classes by their height, LO2 / 2 <= mu <= HI2 / 2, so that what is known to be 0 or 1 costs nothing: a pair
// of rows of up to half a voxel reads two voxels and takes eight instructions, one of up to a voxel three and eleven, one of up to a voxel
// and a half four and thirteen
// (sixteen while one body served every height up to a voxel and a half).  The clamps and weights depend on no voxel, so a lane that
// carries several volumes forms them once.
// Offsets of the clamps, the same for every row of the detector, worked out once per candidate: ka[t-1] = mu - (t+1), kb[t-1] = 2 mu - (t+1).
struct SfPairOffsets {
    float mu;
    float ka[3], kb[6];
};

SF_HD SfPairOffsets sf_pair_offsets(float mu)
{
    SfPairOffsets k;
    k.mu = mu;
    const float mu2 = mu + mu;
#pragma unroll
    for (int t = 1; t <= 3; ++t) k.ka[t - 1] = mu - (float)(t + 1);
#pragma unroll
    for (int t = 1; t <= 6; ++t) k.kb[t - 1] = mu2 - (float)(t + 1);
    return k;
}

template <int LO2, int HI2>
struct SfPairWeights {
    static constexpr int P = HI2 + 1;                 // voxels a pair can overlap
    static constexpr int NA = (HI2 + 3) / 2;          // voxels the lower row can overlap
    static constexpr bool SHORT = LO2 < 2;            // rows shorter than a voxel: a and b are a_t and b_t, otherwise weights
    float a[NA], b[P];
};

template <int LO2, int HI2>
SF_HD SfPairWeights<LO2, HI2> sf_pair_weights(float fr1, const SfPairOffsets &k)
{
    using W = SfPairWeights<LO2, HI2>;
    W w;
    w.a[0] = W::SHORT ? k.mu : 2.0f - fr1;
    w.b[0] = 0.0f;
#pragma unroll
    for (int t = 1; t < W::NA; ++t) w.a[t] = LO2 >= 2 * (t + 1) ? 1.0f : sf_clamp(fr1 + k.ka[t - 1], 0.0f, 1.0f);
#pragma unroll
    for (int t = 1; t < W::P; ++t) {
        const float upto = LO2 >= t + 1 ? 1.0f : sf_clamp(fr1 + k.kb[t - 1], 0.0f, 1.0f);
        w.b[t] = !W::SHORT && t < W::NA ? upto - w.a[t] : upto;
    }
    return w;
}

template <int LO2, int HI2>
SF_HD void sf_pair_apply(const float *x, const SfPairWeights<LO2, HI2> &w, float &sa, float &sb)
{
    using W = SfPairWeights<LO2, HI2>;
    const float a0 = w.a[0] * x[0];
    sa = a0;
    if constexpr (W::SHORT) {
        float d[W::P];
#pragma unroll
        for (int t = 1; t < W::P; ++t) d[t] = x[t] - x[0];
#pragma unroll
        for (int t = 1; t < W::NA && t < W::P; ++t) sa = fmaf(w.a[t], d[t], sa);
        float b = a0 + a0;                              // 2 mu x_0, exactly
#pragma unroll
        for (int t = 1; t < W::P; ++t) b = fmaf(w.b[t], d[t], b);
        sb = b - sa;
    } else {
#pragma unroll
        for (int t = 1; t < W::NA; ++t) sa = LO2 >= 2 * (t + 1) ? sa + x[t] : fmaf(w.a[t], x[t], sa);
        constexpr int FIRST = LO2 >= 4 ? 2 : 1;         // (the lower row holds all of voxel 1 from two voxels on)
        sb = w.b[FIRST] * x[FIRST];
#pragma unroll
        for (int t = FIRST + 1; t < W::P; ++t) sb = fmaf(w.b[t], x[t], sb);
    }
}

// Height classes: 1 up to a voxel, 2 up to a voxel and a half, 3 up to two, 4 up to three voxels; 0, up to half a voxel, is for scans all
// of whose rows are as short.
template <int CLS>
struct SfPairClass {
    static constexpr int LO2 = CLS <= 1 ? 0 : CLS, HI2 = CLS == 4 ? 6 : CLS + 1, P = HI2 + 1;
};
SF_HD int sf_pair_class(float mu) { return mu <= 1.0f ? 1 : (mu <= 1.5f ? 2 : (mu <= 2.0f ? 3 : 4)); }

// The four numbers that a candidate's visit needs, as its lane leaves them for the wave (cls: its own class, HC: the scan's highest, which also
// takes candidates that rounding puts a class higher) and as the wave reads them in the body of class CLS.  (By value: by reference most
// instances take one register more.)
struct alignas(16) SfOffsetsRecord {
    float x, y, z, w;
};

template <int HC>
SF_HD SfOffsetsRecord sf_pack_offsets(int cls, SfPairOffsets k)
{
    const bool below1 = HC <= 1 || cls <= 1, below2 = HC <= 2 || cls <= 2;
    return {below1 || (HC > 3 && cls > 3) ? k.mu : k.ka[0], below1 ? k.ka[0] : k.ka[1],
            below1 ? k.kb[0] : (below2 ? k.kb[1] : k.kb[2]), below1 ? k.kb[1] : (below2 ? k.kb[2] : k.kb[3])};
}

template <int CLS>
SF_HD void sf_unpack_offsets(const SfOffsetsRecord &r, SfPairOffsets &k)
{
    if constexpr (CLS <= 1) { k.mu = r.x; k.ka[0] = r.y; k.kb[0] = r.z; k.kb[1] = r.w; }
    if constexpr (CLS == 2) { k.ka[0] = r.x; k.ka[1] = r.y; k.kb[1] = r.z; k.kb[2] = r.w; }
    if constexpr (CLS == 3) { k.ka[0] = r.x; k.ka[1] = r.y; k.kb[2] = r.z; k.kb[3] = r.w; }
    if constexpr (CLS == 4) k = sf_pair_offsets(r.x);
}

// Transaxial record of a candidate voxel column with footprint f for the bundle of CW detector columns starting at c0:
// fa[cw] = F_u times rows per voxel, mu = voxels per detector row; returns whether any column is touched.
template <int CW>
SF_HD bool sf_footprint_record(const SfGeom &g, const SfColumn &f, int c0, bool valid, float (&fa)[CW], double &mu)
{
    mu = f.den * (g.ikvd * g.iTzd);
    const float rows_per_voxel = (float)(g.kvd * f.inv * g.Tzd);
    bool any = false;
    float e = sf_pixel_edge(f, c0);
    float g0 = sf_trap_integral(f, e);
#pragma unroll
    for (int cw = 0; cw < CW; ++cw) {
        e += 1.0f;
        const float g1 = sf_trap_integral(f, e);
        const float fu = (valid && c0 + cw < g.ncols) ? fmaxf(g1 - g0, 0.0f) : 0.0f;
        fa[cw] = fu * rows_per_voxel;
        any = any || fu > 0.0f;
        g0 = g1;
    }
    return any;
}

template <int CW, int GT>
SF_HD bool sf_candidate_record(const SfGeom &g, const SfView &v, int i, int j, int c0, bool valid, float (&fa)[CW], double &mu)
{
    return sf_footprint_record<CW>(g, sf_column<GT>(g, v, i, j), c0, valid, fa, mu);
}

// Cylinder: the detector coordinate of a bundle's middle, and how far beside it (pixels) the centre and the corners of a voxel column that
// touches one of its columns can lie.
SF_HD double sf_bundle_middle(int c0, int cw) { return (double)c0 + 0.5 * (cw - 1); }
SF_HD double sf_bundle_reach(int cw, double max_cols_per_voxel) { return 0.5 * cw + max_cols_per_voxel + 0.5; }

// Waves of a workgroup that share a bundle (the rule stands at forward_parts) take consecutive runs of the slab's blocks of 64 / nq layers: those of this part.
SF_HD void fp_part_of(const SfSlab &slab, int block, int part, int parts, int &n_first, int &n_end)
{
    const int blocks = (slab.n1 - slab.n0 + block - 1) / block;
    n_first = slab.n0 + blocks * part / parts * block;
    n_end = slab.n0 + blocks * (part + 1) / parts * block;
    n_end = n_end < slab.n1 ? n_end : slab.n1;
}

// Of `parts` waves those that get a block of a slab of n layers, where a kernel of so many exists (by rows: 1, 2 and 4, else 1 and 4): waves without one
// add zeros, so the sums are the same bits without them, and a batch of volumes of one or two blocks is not held up by idle waves (us, a wave per bundle; four;
// now: 30 x 26 x 79, 37 parallel views, 17 volumes 158, 178, below 165; 14 x 12 x 146, one view, 5 volumes 26, 30, below 27).
SF_HD int fp_waves_for(int n, int block, int parts, bool rows)
{
    const int blocks = (n + block - 1) / block;
    return parts == 1 || blocks <= 1 ? 1 : (rows && blocks == 2 ? 2 : parts);
}

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

// vol [nz][ny][nx]  ->  the slab's scratch copy: columns (i, j), i0 <= i < i0 + ni, j0 <= j < j0 + nj, at
// volz[((j - j0) ni + (i - i0)) nzp + FP_PAD + k].  Block 32 x 8 threads, tile 32 (i) x 32 (k) of one j.
// blockIdx.z = (j - j0) + nj * item: several volumes of a batch go into consecutive scratch copies in one launch.
static __global__ __launch_bounds__(256) void sf_volume_to_columns(const float *__restrict__ vol, float *__restrict__ volz, int nx,
                                                            int ny, int nz, int nzp, int i0, int j0, int ni, int nj,
                                                            size_t item_stride)
{
    __shared__ float tile[32][33];
    const int item = blockIdx.z / nj, jr = blockIdx.z - item * nj, j = j0 + jr;
    vol += (size_t)item * nx * ny * nz;
    volz += (size_t)item * item_stride;
    const int ib = blockIdx.x * 32, k0 = blockIdx.y * 32;
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int ihi = i0 + ni < nx ? i0 + ni : nx;
    if (j >= ny) return;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int k = k0 + ty + 8 * s, i = i0 + ib + tx;
        tile[ty + 8 * s][tx] = (k < nz && i < ihi) ? vol[((size_t)k * ny + j) * nx + i] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int ir = ib + ty + 8 * s, k = k0 + tx;
        if (i0 + ir < ihi && k < nz) volz[((size_t)jr * ni + ir) * nzp + FP_PAD + k] = tile[tx][ty + 8 * s];
    }
    // The spare zero column at the copy's end lies where a copy of another layout (another slab width, chosen by the batch) may
    // have held voxels: every copy clears it, its pads are zero in every layout.
    if (blockIdx.x == 0 && jr == 0 && ty == 0 && k0 + tx < nz) volz[item_stride - nzp + FP_PAD + k0 + tx] = 0.0f;
}

// Zeroes what the column-wise kernels expect to be zero around the voxels that sf_volume_to_columns writes: FP_PAD
// floats before and after each of the ncolumns z-columns and the whole spare column that follows them (a fill kernel,
// not a memset, so that a caller may capture the call in a graph).
static __global__ __launch_bounds__(256) void sf_clear_column_pads(float *__restrict__ volz, unsigned ncolumns, int nz, int nzp)
{
    const unsigned t = blockIdx.x * 256u + threadIdx.x;
    const unsigned col = t / (2u * FP_PAD), e = t % (2u * FP_PAD);
    if (col < ncolumns) volz[(size_t)col * nzp + (e < FP_PAD ? e : nz + e)] = 0.0f;
    if (t < (unsigned)nzp) volz[(size_t)ncolumns * nzp + t] = 0.0f;
}

// Block -> (column tile, band of rows, view), for every column-wise forward kernel.  Workgroups are handed to the 8 XCDs
// round-robin by index, and each XCD has its own L2, so the blocks one XCD runs at the same time are arranged as (a few column
// tiles) x (a run of consecutive views), whose beams overlap almost entirely: index = 8 s + xcd, and within an XCD's sequence s
// the view runs fastest inside a block of vb views, then tb tiles, then blocks of views.  Returns false for padding blocks.
// turn: every 2^turn views the tiles move on by one XCD.  A tile at the detector's edge takes a fraction of the time of one in its middle, and
// with a dozen tiles an XCD has one or two of them for every view; but neighbouring views of a tile read the same voxels, which a copy
// larger than an XCD's L2 then fetches again (the rule stands at FP_TURN_BYTES).
__device__ __forceinline__ bool fp_block(int tb, int vb, int turn, int views_pad, int tiles_per_xcd_pad, int col_tiles, int nviews, int bands, int &ct,
                                         int &band, int &a)
{
    const int xcd = blockIdx.x & 7, sq = blockIdx.x >> 3;
    const int per_chunk = tb * views_pad;                   // tb tiles x all (padded) views
    const int chunk = sq / per_chunk, r = sq - chunk * per_chunk;
    const int vblk = r / (tb * vb), r2 = r - vblk * (tb * vb);
    const int tloc = r2 / vb, v_in = r2 - tloc * vb;
    const int tchunks = tiles_per_xcd_pad / tb;
    band = chunk / tchunks;
    a = vblk * vb + v_in;
    ct = ((chunk - band * tchunks) * tb + tloc) * 8 + ((xcd + (a >> turn)) & 7);
    return ct < col_tiles && a < nviews && band < bands;
}

// Writes a row's samples of four adjacent columns together (first), or adds them to what is there.
__device__ __forceinline__ void fp_store_four(float *__restrict__ dst, float a, float b, float c, float d, bool first)
{
    struct __attribute__((packed, aligned(4))) Quad { float a, b, c, d; };
    Quad q = {a, b, c, d};
    if (!first) {
        const Quad old = *reinterpret_cast<const Quad *>(dst);
        q.a += old.a; q.b += old.b; q.c += old.c; q.d += old.d;
    }
    *reinterpret_cast<Quad *>(dst) = q;
}

// Adds the parts' N sums per lane in the order of the parts; the total is valid in part 0.  red: 8 floats per lane and wave, free to use
// once every wave of the workgroup has arrived.
template <int N, int PARTS>
__device__ __forceinline__ void fp_sum_parts(float *acc, float *__restrict__ red, int part, int lane)
{
#pragma unroll
    for (int s = 0; s < N; s += 8) {
        __syncthreads();
        if (part > 0) {
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (s + t < N) red[(part * 8 + t) * 64 + lane] = acc[s + t];
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int p = 1; p < PARTS; ++p)
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (s + t < N) acc[s + t] += red[(p * 8 + t) * 64 + lane];
        }
    }
}

// HC: highest height class of the scan's rows (0 .. 4); RG: groups of 128 rows per wave; CW: adjacent detector columns per wave;
// GT: 0 flat or parallel, 1 cylindrical detector, 2 modular geometry with upright modules; NS: volumes per wave.
// Cylinder: a candidate's fan angle is taken relative to the bundle's middle ray by a short polynomial.  With a double-precision atan2,
// square root and four atanf per candidate (96 to 168 registers, three to five waves per SIMD, 68 to 127 now) the forward projection of
// 512^3, 720 views of 512^2 took 50.9 ms, now 46.5; 171 x 181 x 96, 323 views of 129 x 270 1.95, now 1.49 ms.
// nq_log2: log2 of the candidate slots per slab (a power of two <= 64).  major[a * nbundles + b]: 1 if bundle b of view
// a advances fastest along x (decided once, on the host, so that both agree on which slabs a bundle reads).
template <int HC, int RG, int CW, int GT, int NS, int PARTS>
__global__ __launch_bounds__((PARTS > 1 ? PARTS : FP_WAVES) * 64, GT == 1 ? (RG * NS <= 2 ? 4 : 3) : 1) void sf_project_columns(SfGeom gk, const SfView *__restrict__ views,
                                                                    const float *__restrict__ volz, float *__restrict__ sino,
                                                                    const unsigned char *__restrict__ major, int nzp,
                                                                    size_t item_stride, int nq_log2, int col_tiles, int bands,
                                                                    int vb, int tb, int turn, int vgroups_pad, int tiles_per_xcd_pad,
                                                                    SfSlab all, const SfGeom *__restrict__ geoms)
{
    // GT == 2 (modular geometry, upright modules): the wave's view brings its own parameter block, the scene
    // translated so that the view is a circular cone-beam view; gk holds the sizes, which all views share.
    const SfGeom &gsz = gk;
    // blockIdx.y: NS items of a batch (their scratch copies and sinograms).  Everything but the voxels and the sums is the same for
    // two items: candidates, records, placement and axial weights are formed once (eight 256^3 volumes of 60 views, 7.6 -> 7.1 ms).
    const size_t nsino = (size_t)gk.nviews * gk.nrows * gk.ncols;
    volz += (size_t)blockIdx.y * NS * item_stride;
    sino += (size_t)blockIdx.y * NS * nsino;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int ct, band, a;
    if (!fp_block(tb, vb, turn, vgroups_pad, tiles_per_xcd_pad, col_tiles, gsz.nviews, bands, ct, band, a)) return;   // (whole workgroups)
    const int bundle = PARTS > 1 ? ct : ct * FP_WAVES + wave, part = PARTS > 1 ? wave : 0;
    const int c0 = bundle * CW;                          // first detector column of this wave
    if (c0 >= gsz.ncols) return;                         // (waves that share a bundle return together)
    const int nbundles = (gsz.ncols + CW - 1) / CW;
    const SfSlab slab = sf_slab_for(all, __builtin_amdgcn_readfirstlane((int)major[(size_t)a * nbundles + bundle]), gsz.nx, gsz.ny);
    if ((int)major[(size_t)a * nbundles + bundle] != slab.xmajor) return;   // this bundle reads the other kind of slab
    const int band0 = band * (RG * 128);

    const SfGeom &g = GT == 2 ? geoms[a] : gk;
    const SfView v = views[a];
    const SfRayLines L = sf_ray_lines<GT>(g, v, c0, CW, slab.xmajor);
    const int n_minor = slab.xmajor ? g.ny : g.nx;
    SfNearRay ray;
    if constexpr (GT == 1) ray = sf_near_ray(g, sf_bundle_middle(c0, CW));

    // the lower row of each of this lane's pairs, as a double relative to the detector's eta origin
    double rd[RG];
#pragma unroll
    for (int gq = 0; gq < RG; ++gq) rd[gq] = (double)(band0 + 128 * gq + 2 * lane) - g.row_offd;
    const double zkp = sf_kappa_const(g);
    // byte offset of voxel floor(kappa) in its column from the high word: (hi << 2) + off_k (mod 2^32); negative
    // kappa wraps to a huge offset, which the buffer load's range check turns into zeros, like kappa beyond the column
    const unsigned off_k = 0u - (FP_KAP_HI << 2);
    const unsigned col_bytes = (unsigned)nzp * 4u;

    float acc[NS][CW][RG][2];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int cw = 0; cw < CW; ++cw)
#pragma unroll
            for (int gq = 0; gq < RG; ++gq) acc[q][cw][gq][0] = acc[q][cw][gq][1] = 0.0f;

    const int slot = lane & ((1 << nq_log2) - 1), nrel = lane >> nq_log2, sb_slabs = 64 >> nq_log2;

    // What a candidate's visit needs as plain vector operands (the CW column factors and the clamp offsets of its height class)
    // goes through LDS: every lane writes its candidate's record, the wave reads the record of the
    // candidate it visits back at a uniform address, which the LDS serves as a broadcast without touching the vector
    // ALU (a v_readlane costs as much issue time as two and a half FMAs, and issue is what binds beside the lane loads).
    // Only what must sit in scalar registers still comes by v_readlane: the column's offset (buffer descriptor) and mu
    // (scalar operand of the placement FMAs).
    __shared__ float4 recs[PARTS > 1 ? PARTS : FP_WAVES][64][2];
    float4 (*rec)[2] = recs[wave];

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
        float fa[CW];                                              // F_u times rows per voxel, per detector column
        double mu;                                                 // voxels per detector row at this column
        bool any;
        if constexpr (GT == 1) any = sf_footprint_record<CW>(g, sf_column_curved_near(g, v, ic, jc, ray), c0, valid, fa, mu);
        else any = sf_candidate_record<CW, GT>(g, v, ic, jc, c0, valid, fa, mu);
        const unsigned colbase = sf_slab_column(slab, g.nx, ic, jc) * (unsigned)nzp;   // start of the padded column
        const int mu_lo = __double2loint(mu), mu_hi = __double2hiint(mu);
        const float muf = (float)mu;
        const int cls = HC > 1 ? sf_pair_class(muf) : HC;
        {
            const SfPairOffsets k = sf_pair_offsets(muf);
            float4 f4 = make_float4(fa[0], 0.0f, 0.0f, 0.0f);
            if constexpr (CW > 1) f4.y = fa[1];
            if constexpr (CW > 2) { f4.z = fa[2]; f4.w = fa[3]; }
            // (the wave has consumed every value it read from the previous block's records)
            rec[lane][0] = f4;
            const SfOffsetsRecord offsets = sf_pack_offsets<HC>(cls, k);
            rec[lane][1] = make_float4(offsets.x, offsets.y, offsets.z, offsets.w);
            // the records are read by the other lanes of this wave only: order the LDS accesses, no barrier
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }

        const unsigned long long mask = __ballot(any);
        unsigned long long touch[CW];                              // candidates that touch detector column cw
#pragma unroll
        for (int cw = 0; cw < CW; ++cw) touch[cw] = __ballot(fa[cw] != 0.0f);
        // ---- wave-uniform walk over the candidates that matter, one height class after the other (a block's candidates
        // lie close together and mostly share theirs).
        auto walk = [&](auto cc, unsigned long long todo) {
            constexpr int CLS = decltype(cc)::value, P = SfPairClass<CLS>::P;
            using C = SfPairClass<CLS>;
            while (todo) {
                const int e = __builtin_ctzll(todo);
                todo &= todo - 1;
                const float4 r0 = rec[e][0], r1 = rec[e][1];
                const float fcol[4] = {r0.x, r0.y, r0.z, r0.w};
                SfPairOffsets k;
                sf_unpack_offsets<CLS>({r1.x, r1.y, r1.z, r1.w}, k);
                const unsigned s_base = (unsigned)__builtin_amdgcn_readlane((int)colbase, e);
                const double s_mu = __hiloint2double(__builtin_amdgcn_readlane(mu_hi, e), __builtin_amdgcn_readlane(mu_lo, e));
                float fr1[RG];
                unsigned ko[RG];
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) {
                    unsigned hi;
                    sf_place_row(rd[gq], s_mu, zkp, fr1[gq], hi);
                    asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(ko[gq]) : "v"(hi), "s"(off_k));
                }
                float xv[NS][RG][P];
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    // buffer resource of this candidate's padded z-column: loads beyond it return zero
                    const __amdgpu_buffer_rsrc_t col =
                        __builtin_amdgcn_make_buffer_rsrc((void *)(volz + s * item_stride + s_base), 0, (int)col_bytes, 0x00020000);
#pragma unroll
                    for (int gq = 0; gq < RG; ++gq)
#pragma unroll
                        for (int t = 0; t < P; ++t)      // the compiler merges these into loads of up to 16 bytes
                            xv[s][gq][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(col, (int)ko[gq] + 4 * t, 0, 0));
                }
                float sa[NS][RG], sb[NS][RG];
#pragma unroll
                for (int gq = 0; gq < RG; ++gq) {
                    const SfPairWeights<C::LO2, C::HI2> w = sf_pair_weights<C::LO2, C::HI2>(fr1[gq], k);
#pragma unroll
                    for (int s = 0; s < NS; ++s) sf_pair_apply<C::LO2, C::HI2>(xv[s][gq], w, sa[s][gq], sb[s][gq]);
                }
                // a candidate usually touches only some of the bundle's columns: skip the others (wave-uniform branches)
#pragma unroll
                for (int cw = 0; cw < CW; ++cw) {
                    if ((touch[cw] >> e) & 1ull) {
#pragma unroll
                        for (int s = 0; s < NS; ++s)
#pragma unroll
                            for (int gq = 0; gq < RG; ++gq) {
                                acc[s][cw][gq][0] = fmaf(fcol[cw], sa[s][gq], acc[s][cw][gq][0]);
                                acc[s][cw][gq][1] = fmaf(fcol[cw], sb[s][gq], acc[s][cw][gq][1]);
                            }
                    }
                }
            }
        };
        unsigned long long todo = mask;
        auto walk_up_to = [&](auto cc) {
            constexpr int CLS = decltype(cc)::value;
            const unsigned long long above = CLS < HC ? __ballot(cls > CLS) : 0ull;
            walk(cc, todo & ~above);
            todo &= above;
        };
        walk_up_to(std::integral_constant<int, (HC < 1 ? HC : 1)>{});
        if constexpr (HC > 1) walk_up_to(std::integral_constant<int, 2>{});
        if constexpr (HC > 2) walk_up_to(std::integral_constant<int, 3>{});
        if constexpr (HC > 3) walk_up_to(std::integral_constant<int, 4>{});
    }

    if constexpr (PARTS > 1) {
        fp_sum_parts<NS * CW * RG * 2, PARTS>(&acc[0][0][0][0], &recs[0][0][0].x, part, lane);
        if (part > 0) return;
    }

    // ---- amplitude and store: CW consecutive floats per lane and row, written together (storing the columns of a
    // bundle one after the other, hundreds of instructions apart, cost 3.7 times the sinogram in partial-line writes)
    SfAmpCol ac[CW];
#pragma unroll
    for (int cw = 0; cw < CW; ++cw) ac[cw] = sf_amp_col<GT>(g, v, c0 + cw < g.ncols ? c0 + cw : g.ncols - 1);
    struct __attribute__((packed, aligned(4))) Pair { float lo, hi; };
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        float *__restrict__ ya = sino + s * nsino + (size_t)a * g.nrows * g.ncols;
#pragma unroll
        for (int gq = 0; gq < RG; ++gq) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = band0 + 128 * gq + 2 * lane + h;
                if (r >= g.nrows) continue;
                float out[CW];
#pragma unroll
                for (int cw = 0; cw < CW; ++cw) out[cw] = sf_amp(g, v, ac[cw], r) * acc[s][cw][gq][h];
                float *__restrict__ dst = ya + (size_t)r * g.ncols + c0;
                if constexpr (CW == 2) {
                    if (c0 + 1 < g.ncols) {
                        Pair pr;
                        if (!slab.first) {
                            pr = *reinterpret_cast<const Pair *>(dst);
                            out[0] += pr.lo; out[1] += pr.hi;
                        }
                        pr.lo = out[0]; pr.hi = out[1];
                        *reinterpret_cast<Pair *>(dst) = pr;
                        continue;
                    }
                }
                if constexpr (CW == 4) {
                    if (c0 + 3 < g.ncols) {
                        fp_store_four(dst, out[0], out[1], out[2], out[3], slab.first);
                        continue;
                    }
                }
#pragma unroll
                for (int cw = 0; cw < CW; ++cw)
                    if (c0 + cw < g.ncols) dst[cw] = slab.first ? out[cw] : dst[cw] + out[cw];
            }
        }
    }
}

#endif
