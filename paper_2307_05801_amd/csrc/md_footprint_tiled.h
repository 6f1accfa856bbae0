// Fast kernels of the footprint pair on tilted modules (md_footprint.h states the model): both are voxel-driven, form every
// voxel's footprint once per view that sees it (once per detector tile in the forward direction) and keep everything in
// double precision, as the general bodies do.
//
// What bounds them is vector-ALU issue on forming the footprints (a voxel's knots change with every voxel and view, nothing is
// shared along a column as it is for upright modules), so the work per voxel is what was cut:
//   - a column of voxels is walked along z: the projections' numerators and denominators advance by one FMA each, and the
//     face between two voxels is projected once;
//   - opposite corners of a voxel share a denominator, (N + n)(N - n) = N^2 - n^2, and the three reciprocals a voxel needs come
//     from one (of their product);
//   - the ray amplitude (a square root and a reciprocal per pixel) is applied once per pixel: to the staged window in the
//     back projection, to the finished sums in the forward projection.
//
// Back (mf_backproject_tiled): 16 x 16 voxel columns of ZC voxels per workgroup, one column per thread, the detector window of
// the workgroup's box staged per view in LDS in double precision, amplitude applied, double-buffered.
// Forward (mf_project_tiles): a wave owns a tile of MF_TC x MF_TR detector pixels whose sums live in LDS, walks the voxel layers
// its beams cross, and adds every voxel's few shares with the LDS's double-precision add.  The 64 lanes take voxels spread
// over the layer's box (16 positions along z times 4 across), so that they rarely meet in a pixel.  A tile belongs to one
// workgroup, whose waves share the layers and keep sums of their own; a wave's LDS operations execute in order, so the sums do not depend
// on scheduling.
//
// Measured at 128^3 x 720 views x 128^2 against one thread per voxel / per eight rows of a column (md_footprint.h): A 60.4 ->
// 13.0 ms, A^T 22.0 -> 7.4 ms, the same bits but for the last; A 11.2 ms since a tile's layers are shared by four waves, and 16 drawn scans of 28^2
// x 14 to 128^3 voxels 0.37 (A) and 0.67 (A^T) of what one wave per tile and views one after the other took.  (Forward tiles of 32 x 32 pixels, with 16 x 4 or 8 x 8 lanes: 15.7 and
// 15.0 ms; fewer than six voxels per lane along z pay too often for starting a column.)
#pragma once

#include "md_footprint.h"

constexpr int MF_T = 16, MF_ZC = 8;              // back projection: tile edge, most voxels per thread
constexpr int MF_PATCH = 2048;                   // doubles per staged window
constexpr int MF_TC = 16, MF_TR = 64;            // forward: detector tile of a wave, columns x rows
constexpr int MF_TG = 2;                         // guard columns and rows around it, which take what falls beside the tile
constexpr int MF_TS = MF_TC + 2 * MF_TG + 1;     // its row stride in LDS (rows a few apart fall on other banks)

// What a voxel column (i, j) contributes to its projections: the parts of the dot products that do not depend on z.
struct MfColumn {
    double N, U, W;
};

SF_HD MfColumn mf_column(const SfGeom &g, const MfView &V, int i, int j)
{
    const double dx = fma((double)i, g.Td, g.x0d) - V.S[0], dy = fma((double)j, g.Td, g.y0d) - V.S[1];
    MfColumn c;
    c.N = fma(dx, V.nP[0], dy * V.nP[1]);
    c.U = fma(dx, V.euP[0], dy * V.euP[1]);
    c.W = fma(dx, V.evP[0], dy * V.evP[1]);
    return c;
}

// Height of the lower face of voxel k above the source.
SF_HD double mf_face_height(const SfGeom &g, const MfView &V, int k) { return fma((double)k, g.Tzd, g.zlo0d - V.S[2]); }

// Row coordinate of the central projection of the column's axis at height dz above the source.
SF_HD double mf_face(const MfView &V, const MfColumn &c, double dz)
{
    return fma(fma(dz, V.evP[2], c.W), mf_rcp(fma(dz, V.nP[2], c.N)), V.eta0);
}

// clamp(a b), clamp(a b + c), clamp(a - b) to [0, 1]: the clamp is a modifier of the instruction.
#if defined(__HIP_DEVICE_COMPILE__)
SF_HD double mf_mul01(double a, double b) { double r; asm("v_mul_f64 %0, %1, %2 clamp" : "=v"(r) : "v"(a), "v"(b)); return r; }
SF_HD double mf_fma01(double a, double b, double c) { double r; asm("v_fma_f64 %0, %1, %2, %3 clamp" : "=v"(r) : "v"(a), "v"(b), "v"(c)); return r; }
SF_HD double mf_sub01(double a, double b) { double r; asm("v_add_f64 %0, %1, -%2 clamp" : "=v"(r) : "v"(a), "v"(b)); return r; }
// (plain instructions: fmin and fmax would first quieten signalling NaNs, an instruction per operand)
SF_HD double mf_min(double a, double b) { double r; asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
SF_HD double mf_max(double a, double b) { double r; asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
#else
SF_HD double mf_clamp01(double x) { return fmin(fmax(x, 0.0), 1.0); }
SF_HD double mf_mul01(double a, double b) { return mf_clamp01(a * b); }
SF_HD double mf_fma01(double a, double b, double c) { return mf_clamp01(fma(a, b, c)); }
SF_HD double mf_sub01(double a, double b) { return mf_clamp01(a - b); }
SF_HD double mf_min(double a, double b) { return fmin(a, b); }
SF_HD double mf_max(double a, double b) { return fmax(a, b); }
#endif

// A voxel on its way up its column: the z-dependent parts of the projections at the voxel's centre (N, U) and at its upper
// face (Nt, Wt), and the row coordinate of the face below.
struct MfWalk {
    double N, U, Nt, Wt, eta;
};

// Starts below voxel k.
SF_HD MfWalk mf_walk(const SfGeom &g, const MfView &V, const MfColumn &c, int k)
{
    const double dz = mf_face_height(g, V, k), dzc = fma(-0.5, g.Tzd, dz);
    MfWalk w;
    w.eta = mf_face(V, c, dz);
    w.N = fma(dzc, V.nP[2], c.N);
    w.U = fma(dzc, V.euP[2], c.U);
    w.Nt = fma(dz, V.nP[2], c.N);
    w.Wt = fma(dz, V.evP[2], c.W);
    return w;
}

// Footprint of a voxel.  Columns: knots k0..k3, ramps and plateau as fractions of their widths (i01, i12, i23: 1 / width; h01,
// h23: half the widths of the ramps).  Rows: [e0, e1).
struct MfFoot {
    double k0, k1, k3, i01, i12, i23, h01, w12, h23, e0, e1;
};

// Steps up to the next voxel and works out its footprint.
SF_HD MfFoot mf_next(const MfView &V, MfWalk &w)
{
    MfFoot f;
    w.N += V.dN; w.U += V.dU; w.Nt += V.dN; w.Wt += V.dW;
    // opposite corners share (N + n)(N - n) = N^2 - n^2; one reciprocal for both pairs and the face
    const double a = fma(w.N, w.N, -V.nA2), b = fma(w.N, w.N, -V.nB2);
    const double ab = a * b, r = mf_rcp(ab * w.Nt);
    const double rab = r * w.Nt, ra = rab * b, rb = rab * a;
    const double top = fma(w.Wt, r * ab, V.eta0);
    f.e0 = mf_min(w.eta, top);
    f.e1 = mf_max(w.eta, top);
    w.eta = top;
    // (U +- u)(N -+ n) / (N^2 - n^2) = middle +- half: the projections of a diagonal's two ends
    const double mA = fma(fma(w.U, w.N, -V.unA), ra, V.xi0), mB = fma(fma(w.U, w.N, -V.unB), rb, V.xi0);
    const double hA = fabs(fma(V.uA, w.N, -(w.U * V.nA)) * ra), hB = fabs(fma(V.uB, w.N, -(w.U * V.nB)) * rb);
    const double loA = mA - hA, hiA = mA + hA, loB = mB - hB, hiB = mB + hB;
    // both diagonals' shadows hold that of the point where they cross, so the inner two knots are in order
    f.k0 = mf_min(loA, loB);
    f.k1 = mf_max(loA, loB);
    const double k2 = mf_min(hiA, hiB);
    f.k3 = mf_max(hiA, hiB);
    const double d01 = f.k1 - f.k0, d23 = f.k3 - k2;
    f.w12 = mf_max(k2 - f.k1, 0.0);
    // (the guards keep the reciprocals finite where a ramp or the plateau has no width; it then contributes nothing)
    const double w01 = mf_max(d01, 1e-12), w12 = mf_max(f.w12, 1e-12), w23 = mf_max(d23, 1e-12);
    const double p = w01 * w12, q = mf_rcp(p * w23), qw = q * w23;
    f.i23 = q * p;
    f.i01 = qw * w12;
    f.i12 = qw * w01;
    f.h01 = 0.5 * d01;
    f.h23 = 0.5 * d23;
    return f;
}

// Integral of the unit-height trapezoid up to a point that lies p of the way up the first ramp, t along the plateau and s
// short of the end of the second ramp (each clamped to [0, 1]).
SF_HD double mf_integral(const MfFoot &f, double p, double t, double s)
{
    return fma(f.h01, p * p, fma(f.w12, t, fma(-f.h23, s * s, f.h23)));
}
SF_HD double mf_integral_at(const MfFoot &f, double x)
{
    return mf_integral(f, mf_mul01(x - f.k0, f.i01), mf_mul01(x - f.k1, f.i12), mf_mul01(f.k3 - x, f.i23));
}
SF_HD double mf_total(const MfFoot &f) { return f.h01 + (f.w12 + f.h23); }

// F_u of the first three columns from the one whose upper edge is x (k0 lies in it); exact if the footprint ends in the third.
SF_HD void mf_fu3(const MfFoot &f, double x, double (&fu)[3])
{
    const double d0 = x - f.k0, d1 = x - f.k1, d3 = f.k3 - x;
    const double g0 = mf_integral(f, mf_mul01(d0, f.i01), mf_mul01(d1, f.i12), mf_mul01(d3, f.i23));
    const double g1 = mf_integral(f, mf_fma01(d0, f.i01, f.i01), mf_fma01(d1, f.i12, f.i12), mf_fma01(d3, f.i23, -f.i23));
    fu[0] = g0;
    fu[1] = g1 - g0;
    fu[2] = mf_total(f) - g1;
}

// Detector window (float bounds, a hundredth of a pixel wide of the truth) that the box of voxels [i0, i1] x [j0, j1] x [k0, k1]
// can touch: the box's corners project to the extremes.  Two columns and rows to spare: the kernel reads three of each from
// the first that a voxel touches.
struct MfWindow {
    int c0, r0, w, h;
};

// Column / row coordinate of the box's corner q (0..7).
SF_HD void mf_box_corner(const SfGeom &g, const MfView &V, int i0, int i1, int j0, int j1, int k0, int k1, int q, float &xi, float &eta)
{
    const double dx = fma((double)((q & 1) ? i1 : i0) + ((q & 1) ? 0.5 : -0.5), g.Td, g.x0d) - V.S[0];
    const double dy = fma((double)((q & 2) ? j1 : j0) + ((q & 2) ? 0.5 : -0.5), g.Td, g.y0d) - V.S[1];
    const double dz = mf_face_height(g, V, (q & 4) ? k1 + 1 : k0);
    const double r = mf_rcp(fma(dx, V.nP[0], fma(dy, V.nP[1], dz * V.nP[2])));
    xi = (float)fma(fma(dx, V.euP[0], fma(dy, V.euP[1], dz * V.euP[2])), r, V.xi0);
    eta = (float)fma(fma(dx, V.evP[0], fma(dy, V.evP[1], dz * V.evP[2])), r, V.eta0);
}

SF_HD MfWindow mf_window(float xlo, float xhi, float elo, float ehi)
{
    MfWindow w;
    w.c0 = sf_f2i(floorf(xlo + 0.49f));
    w.r0 = sf_f2i(floorf(elo - 0.01f));
    w.w = sf_f2i(floorf(xhi + 0.51f)) - w.c0 + 3;
    w.h = sf_f2i(floorf(ehi + 0.01f)) - w.r0 + 3;
    return w;
}

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

// The window of a workgroup's box, the eight corners shared out among the lanes.
__device__ __forceinline__ MfWindow mf_wave_window(const SfGeom &g, const MfView &V, int i0, int i1, int j0, int j1, int k0, int k1, int lane)
{
    float x, e;
    mf_box_corner(g, V, i0, i1, j0, j1, k0, k1, lane & 7, x, e);
    float xlo = x, xhi = x, elo = e, ehi = e;
#pragma unroll
    for (int s = 1; s < 8; s *= 2) {
        xlo = fminf(xlo, __shfl_xor(xlo, s)); xhi = fmaxf(xhi, __shfl_xor(xhi, s));
        elo = fminf(elo, __shfl_xor(elo, s)); ehi = fmaxf(ehi, __shfl_xor(ehi, s));
    }
    MfWindow w = mf_window(xlo, xhi, elo, ehi);
    w.c0 = __builtin_amdgcn_readfirstlane(w.c0);
    w.r0 = __builtin_amdgcn_readfirstlane(w.r0);
    w.w = __builtin_amdgcn_readfirstlane(w.w);
    w.h = __builtin_amdgcn_readfirstlane(w.h);
    return w;
}

// (Eight voxels per thread spill four registers at four waves per SIMD.)
template <int ZC, int VS>
__global__ __launch_bounds__(256 * VS, VS == 1 ? 4 : 1) void mf_backproject_tiled(SfGeom g, const MfView *__restrict__ views, const float *__restrict__ sino,
                                                                     float *__restrict__ vol, int tiles_x)
{
    __shared__ double patches[VS][2][MF_PATCH];
    const int tid = threadIdx.x & 255, lane = tid & 63, group = VS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    double (*patch)[MF_PATCH] = patches[group];
    const int ty = blockIdx.x / tiles_x, tx = blockIdx.x - ty * tiles_x;
    const int i0 = tx * MF_T, j0 = ty * MF_T, k0 = blockIdx.y * ZC;
    const int i1 = i0 + MF_T < g.nx ? i0 + MF_T - 1 : g.nx - 1, j1 = j0 + MF_T < g.ny ? j0 + MF_T - 1 : g.ny - 1;
    const int k1 = k0 + ZC < g.nz ? k0 + ZC - 1 : g.nz - 1;
    const int i = i0 + (tid & (MF_T - 1)), j = j0 + tid / MF_T;
    const int ic = i < g.nx ? i : g.nx - 1, jc = j < g.ny ? j : g.ny - 1;        // threads beyond the edge shadow it
    const size_t view_stride = (size_t)g.nrows * g.ncols;

    double acc[ZC];
#pragma unroll
    for (int kk = 0; kk < ZC; ++kk) acc[kk] = 0.0;

    constexpr int NSTAGE = MF_PATCH / 256;
    float stage[NSTAGE];
    MfWindow win, next;
    auto sees = [&](const MfWindow &w) { return w.c0 < g.ncols && w.c0 + w.w > 0 && w.r0 < g.nrows && w.r0 + w.h > 0; };
    auto fetch = [&](int a, MfWindow &w) {
        w = mf_wave_window(g, views[a], i0, i1, j0, j1, k0, k1, lane);
        w.w = w.w < 1 ? 1 : (w.w > MF_PATCH ? MF_PATCH : w.w);                   // (the host checked that the window fits)
        w.h = w.h > MF_PATCH / w.w ? MF_PATCH / w.w : w.h;
        const float *__restrict__ y = sino + (size_t)a * view_stride;
#pragma unroll
        for (int s = 0; s < NSTAGE; ++s) {
            const int e = tid + 256 * s;
            stage[s] = 0.0f;
            if (256 * s < w.w * w.h) {             // uniform
                const int rr = e / w.w, r = w.r0 + rr, c = w.c0 + e - rr * w.w;
                if (rr < w.h && (unsigned)r < (unsigned)g.nrows && (unsigned)c < (unsigned)g.ncols) stage[s] = y[(size_t)r * g.ncols + c];
            }
        }
    };
    __shared__ int odd_waves[VS][2][4];        // per wave: it staged an infinity or a NaN
    int (*odd)[4] = odd_waves[group];
    auto store = [&](int a, int slot, const MfWindow &w, double *__restrict__ buf) {
        bool bad = false;
#pragma unroll
        for (int s = 0; s < NSTAGE; ++s) {
            const int e = tid + 256 * s;
            if (256 * s < w.w * w.h && e < w.w * w.h) {
                const int rr = e / w.w, r = w.r0 + rr, c = w.c0 + e - rr * w.w;
                const bool in = (unsigned)r < (unsigned)g.nrows && (unsigned)c < (unsigned)g.ncols;
                buf[e] = in ? (double)stage[s] * mf_amp(g, views[a], r, c) : 0.0;
                bad = bad || !(fabsf(stage[s]) <= 3.402823466e38f);
            }
        }
        const int any = __builtin_amdgcn_ballot_w64(bad) != 0;
        if (lane == 0) odd[slot][tid >> 6] = any;
    };
    // group v takes views v, v + VS, ...; every group makes as many steps
    if (group < g.nviews) {
        fetch(group, win);
        store(group, 0, win, patch[0]);
    }
    __syncthreads();
    for (int a = group, step = 0; a - group < g.nviews; a += VS, step ^= 1) {
        const double *__restrict__ buf = patch[step];
        if (a + VS < g.nviews) fetch(a + VS, next);               // loads in flight during the gather
        const MfView &V = views[a < g.nviews ? a : 0];
        MfWalk at = mf_walk(g, V, mf_column(g, V, ic, jc), k0);
        const bool seen = a < g.nviews && sees(win);              // uniform: a box beside the detector takes nothing from this view
        const bool finite = !(odd[step][0] | odd[step][1] | odd[step][2] | odd[step][3]);        // uniform
#pragma unroll
        for (int kk = 0; kk < ZC; ++kk) {
            if (!seen || k0 + kk >= g.nz) break;                  // uniform
            const MfFoot f = mf_next(V, at);
            const double fr0 = floor(f.e0), fc0 = floor(f.k0 + 0.5);
            const int rows = (int)(floor(f.e1) - fr0), cols = (int)(ceil(f.k3 - 0.5) - fc0);    // further rows, columns it touches
            const double *__restrict__ q = buf + ((int)fr0 - win.r0) * win.w + ((int)fc0 - win.c0);
            const double above = f.e1 - fr0;                      // upper end measured from the first row's lower edge
            const double v0 = mf_min(above, 1.0) - (f.e0 - fr0), v1 = mf_sub01(above, 1.0);
            // The common case: at most three columns and rows, nothing infinite or undefined in the window that a weight
            // of zero would spread.
            if (finite && __builtin_amdgcn_ballot_w64(cols > 2 || rows > 2) == 0) {
                double fu[3];
                mf_fu3(f, fc0 + 0.5, fu);
                const double *__restrict__ q1 = q + win.w;
                double s0 = fma(v1, q1[0], v0 * q[0]), s1 = fma(v1, q1[1], v0 * q[1]), s2 = fma(v1, q1[2], v0 * q[2]);
                if (__builtin_amdgcn_ballot_w64(rows > 1)) {
                    const double v2 = mf_sub01(above, 2.0);
                    const double *__restrict__ q2 = q1 + win.w;
                    s0 = fma(v2, q2[0], s0); s1 = fma(v2, q2[1], s1); s2 = fma(v2, q2[2], s2);
                }
                acc[kk] = fma(fu[2], s2, fma(fu[1], s1, fma(fu[0], s0, acc[kk])));
            } else {
                double below = 0.0, x = fc0 + 0.5;
                for (int m = 0; m <= cols; ++m, x += 1.0) {
                    const double upto = mf_integral_at(f, x), fu = upto - below;
                    below = upto;
                    if (!(fu > 0.0)) continue;
                    double s = v0 > 0.0 ? v0 * q[m] : 0.0;
                    for (int n = 1; n <= rows; ++n) {
                        const double fv = mf_sub01(above, (double)n);
                        if (fv > 0.0) s = fma(fv, q[n * win.w + m], s);
                    }
                    acc[kk] = fma(fu, s, acc[kk]);
                }
            }
        }
        if (a + VS < g.nviews) store(a + VS, step ^ 1, next, patch[step ^ 1]);
        win = next;
        __syncthreads();
    }
    if constexpr (VS > 1) {                                       // the groups' sums, added in the order of the groups
        static_assert(ZC * 256 <= MF_PATCH, "a group's sums fit its patch");
        if (group > 0) {
#pragma unroll
            for (int kk = 0; kk < ZC; ++kk) patch[0][kk * 256 + tid] = acc[kk];
        }
        __syncthreads();
        if (group > 0) return;
        for (int v = 1; v < VS; ++v)
#pragma unroll
            for (int kk = 0; kk < ZC; ++kk) acc[kk] += patches[v][0][kk * 256 + tid];
    }
    if (i < g.nx && j < g.ny) {
#pragma unroll
        for (int kk = 0; kk < ZC; ++kk)
            if (k0 + kk < g.nz) vol[((size_t)(k0 + kk) * g.ny + j) * g.nx + i] = (float)acc[kk];
    }
}

__device__ __forceinline__ void mf_add(double *cell, double v)
{
    __hip_atomic_fetch_add(cell, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Adds the shares of all voxels that the tile's beams can meet, layer by layer along in-plane axis `m`.
template <int m>
__device__ __forceinline__ void mf_tile_along(const SfGeom &g, const MfView &V, const float *__restrict__ vol, int c0, int c1, int r0, int r1,
                                              int lane, int first_layer, int layer_step, double *__restrict__ sums)
{
    // corner rays of the tile's rectangle, widened by how far a footprint can reach: a pyramid from the source whose section
    // with a layer holds the centres of all voxels that can touch the tile
    const double ulo = ((double)c0 - 0.5 - g.col_offd) * g.pu_d - V.pad_u, uhi = ((double)c1 + 0.5 - g.col_offd) * g.pu_d + V.pad_u;
    const double vlo = fma((double)r0 - 0.5, g.pvd, g.v0d) - V.pad_v, vhi = fma((double)r1 + 0.5, g.pvd, g.v0d) + V.pad_v;
    constexpr int p = 1 - m;                                  // the other in-plane axis
    const int n_layers = m == 0 ? g.nx : g.ny, n_p = m == 0 ? g.ny : g.nx;
    const double first[2] = {g.x0d, g.y0d};
    const double iT = 1.0 / g.Td, iTz = 1.0 / g.Tzd, zfirst = fma(0.5, g.Tzd, g.zlo0d);
    const double dm = fma(0.5 * (ulo + uhi), V.eu[m], fma(0.5 * (vlo + vhi), V.ev[m], V.C[m] - V.S[m]));
    bool narrow = true;                                       // otherwise every voxel of a layer is a candidate
    double tp[4], tz[4], im[4];                               // d_p / d_m, d_z / d_m, 1 / d_m of the corner rays
    for (int e = 0; e < 4; ++e) {
        const double u = (e & 1) ? uhi : ulo, v = (e & 2) ? vhi : vlo;
        const double d = fma(u, V.eu[m], fma(v, V.ev[m], V.C[m] - V.S[m]));
        narrow = narrow && d * dm > 0.0625 * dm * dm;
        im[e] = 1.0 / d;
        tp[e] = fma(u, V.eu[p], fma(v, V.ev[p], V.C[p] - V.S[p])) * im[e];
        tz[e] = fma(u, V.eu[2], fma(v, V.ev[2], V.C[2] - V.S[2])) * im[e];
    }
    const int kz = lane & 15, qz = lane >> 4;
    for (int layer = first_layer; layer < n_layers; layer += layer_step) {
        int qlo = 0, qhi = n_p - 1, klo = 0, khi = g.nz - 1;
        if (narrow) {
            const double s = fma((double)layer, g.Td, first[m]) - V.S[m];
            if (!(s * im[0] > 0.0)) continue;                 // the layer lies behind the source as seen along these rays
            const double pa = fmin(fmin(s * tp[0], s * tp[1]), fmin(s * tp[2], s * tp[3]));
            const double pb = fmax(fmax(s * tp[0], s * tp[1]), fmax(s * tp[2], s * tp[3]));
            const double za = fmin(fmin(s * tz[0], s * tz[1]), fmin(s * tz[2], s * tz[3]));
            const double zb = fmax(fmax(s * tz[0], s * tz[1]), fmax(s * tz[2], s * tz[3]));
            const double f1lo = ceil((pa + V.S[p] - first[p]) * iT - 1e-6), f1hi = floor((pb + V.S[p] - first[p]) * iT + 1e-6);
            const double f2lo = ceil((za + V.S[2] - zfirst) * iTz - 1e-6), f2hi = floor((zb + V.S[2] - zfirst) * iTz + 1e-6);
            if (f1hi < 0.0 || f2hi < 0.0 || f1lo > (double)qhi || f2lo > (double)khi) continue;
            qlo = f1lo < 0.0 ? 0 : (int)f1lo; qhi = f1hi > (double)qhi ? qhi : (int)f1hi;
            klo = f2lo < 0.0 ? 0 : (int)f2lo; khi = f2hi > (double)khi ? khi : (int)f2hi;
        }
        qlo = __builtin_amdgcn_readfirstlane(qlo); qhi = __builtin_amdgcn_readfirstlane(qhi);
        klo = __builtin_amdgcn_readfirstlane(klo); khi = __builtin_amdgcn_readfirstlane(khi);
        const int kc = (khi - klo + 16) >> 4, qc = (qhi - qlo + 4) >> 2;          // voxels per lane along z, columns per lane
        const int kfirst = klo + kz * kc;
        for (int qs = 0; qs < qc; ++qs) {
            const int q = qlo + qz * qc + qs;
            const bool q_ok = q <= qhi && kfirst <= khi;
            const int qq = q_ok ? q : qlo, kb = q_ok ? kfirst : klo;
            const int i = m == 0 ? layer : qq, j = m == 0 ? qq : layer;
            MfWalk at = mf_walk(g, V, mf_column(g, V, i, j), kb);
            const float *__restrict__ x0 = vol + ((size_t)kb * g.ny + j) * g.nx + i;
            const size_t kstride = (size_t)g.nx * g.ny;
            const int kn = q_ok ? (khi - kfirst + 1 < kc ? khi - kfirst + 1 : kc) : 0;
            float xv = kn > 0 ? x0[0] : 0.0f;
            for (int ks = 0; ks < kc; ++ks) {
                const double x = (double)xv;
                if (ks + 1 < kn) xv = x0[(ks + 1) * kstride];     // the next voxel's value, in flight during this one's footprint
                const MfFoot f = mf_next(V, at);
                const double fr0 = floor(f.e0), fc0 = floor(f.k0 + 0.5);
                const int rb = (int)fr0 - r0, cb = (int)fc0 - c0;                       // first row, column within the tile
                const int rows = (int)(floor(f.e1) - fr0), cols = (int)(ceil(f.k3 - 0.5) - fc0);
                const double above = f.e1 - fr0;
                const double v0 = mf_min(above, 1.0) - (f.e0 - fr0), v1 = mf_sub01(above, 1.0);
                const bool touches = ks < kn && rb + rows >= 0 && rb <= r1 - r0 && cb + cols >= 0 && cb <= c1 - c0;
                // The common case: at most three columns and rows, no infinite or undefined voxel that a weight of zero
                // would spread.  Shares beside the tile fall on the guards.
                if (__builtin_amdgcn_ballot_w64(touches && (cols > 2 || rows > 2 || !(fabsf((float)x) <= 3.402823466e38f))) == 0) {
                    const bool third = __builtin_amdgcn_ballot_w64(touches && cols > 1) != 0, tall = __builtin_amdgcn_ballot_w64(touches && rows > 1) != 0;
                    if (!touches) continue;
                    double fu[3];
                    mf_fu3(f, fc0 + 0.5, fu);
                    double *__restrict__ cell = sums + (rb + MF_TG) * MF_TS + (cb + MF_TG);
                    const double x0v = v0 * x, x1v = v1 * x;
                    mf_add(cell, fu[0] * x0v);
                    mf_add(cell + 1, fu[1] * x0v);
                    mf_add(cell + MF_TS, fu[0] * x1v);
                    mf_add(cell + MF_TS + 1, fu[1] * x1v);
                    if (third) {
                        mf_add(cell + 2, fu[2] * x0v);
                        mf_add(cell + MF_TS + 2, fu[2] * x1v);
                    }
                    if (tall) {
                        const double x2v = mf_sub01(above, 2.0) * x;
                        mf_add(cell + 2 * MF_TS, fu[0] * x2v);
                        mf_add(cell + 2 * MF_TS + 1, fu[1] * x2v);
                        mf_add(cell + 2 * MF_TS + 2, fu[2] * x2v);
                    }
                } else if (touches) {
                    double below = 0.0, xe = fc0 + 0.5;
                    for (int mm = 0; mm <= cols; ++mm, xe += 1.0) {
                        const double upto = mf_integral_at(f, xe), fu = upto - below;
                        below = upto;
                        if (cb + mm < 0 || cb + mm > c1 - c0 || !(fu > 0.0)) continue;
                        for (int n = 0; n <= rows; ++n) {
                            const double fv = n == 0 ? v0 : mf_sub01(above, (double)n);
                            if (rb + n >= 0 && rb + n <= r1 - r0 && fv > 0.0)
                                mf_add(sums + (rb + n + MF_TG) * MF_TS + (cb + mm + MF_TG), fu * (fv * x));
                        }
                    }
                }
            }
        }
    }
}

// grid: x = column tiles, one more where their number is even: workgroups go to the 8 XCDs by index in turn, and a tile at the detector's
// edge is a fraction of one in its middle, so that on a detector of eight tiles most XCDs waited for two (112^2 x 89 voxels, 720 views of 78
// x 125: 12.7 ms, 5.9 with a ninth in the grid; 128^3, 128 x 128: 14.6, now 11.2); y = bands of MF_TR rows, z = views; block: LS waves, which share the tile: each takes every LS-th layer and keeps
// sums of its own, which are added in the order of the waves.
template <int LS>
__global__ __launch_bounds__(64 * LS) void mf_project_tiles(SfGeom g, const MfView *__restrict__ views, const float *__restrict__ vol,
                                                            float *__restrict__ sino)
{
    constexpr int CELLS = (MF_TR + 2 * MF_TG) * MF_TS;
    __shared__ double tile_sums[LS][CELLS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *__restrict__ sums = tile_sums[wave];
    const int c0 = blockIdx.x * MF_TC, r0 = blockIdx.y * MF_TR, a = blockIdx.z;
    if (c0 >= g.ncols) return;                                // (a workgroup of the grid's padding, as a whole)
    const int c1 = (c0 + MF_TC < g.ncols ? c0 + MF_TC : g.ncols) - 1, r1 = (r0 + MF_TR < g.nrows ? r0 + MF_TR : g.nrows) - 1;
    for (int e = lane; e < CELLS; e += 64) sums[e] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const MfView &V = views[a];
    const double uc = (0.5 * (c0 + c1) - g.col_offd) * g.pu_d, vc = fma(0.5 * (r0 + r1), g.pvd, g.v0d);
    const double dx = fma(uc, V.eu[0], fma(vc, V.ev[0], V.C[0] - V.S[0])), dy = fma(uc, V.eu[1], fma(vc, V.ev[1], V.C[1] - V.S[1]));
    if (__builtin_amdgcn_readfirstlane((int)(fabs(dx) >= fabs(dy)))) mf_tile_along<0>(g, V, vol, c0, c1, r0, r1, lane, wave, LS, sums);
    else mf_tile_along<1>(g, V, vol, c0, c1, r0, r1, lane, wave, LS, sums);
    __syncthreads();
    for (int e = threadIdx.x; e < MF_TR * MF_TC; e += 64 * LS) {
        const int r = r0 + e / MF_TC, c = c0 + e % MF_TC, at = (e / MF_TC + MF_TG) * MF_TS + e % MF_TC + MF_TG;
        if (r > r1 || c > c1) continue;
        double sum = tile_sums[0][at];
#pragma unroll
        for (int w = 1; w < LS; ++w) sum += tile_sums[w][at];
        sino[((size_t)a * g.nrows + r) * g.ncols + c] = (float)(sum * mf_amp(g, V, r, c));
    }
}

#endif
