// Tiled back projection (A^T): voxel-driven gather, no atomics, bitwise reproducible.
//
// A workgroup of 256 threads owns a 16 x 16 tile of voxel columns and BP_ZC voxels along z; a thread
// owns one column of BP_ZC voxels and keeps their sums in registers while the workgroup walks all views.
// Per view the workgroup stages the detector window its tile can touch into LDS, already multiplied by
// the ray amplitude (so the weight left per sample is F_u * F_v), double-buffered: the loads of view
// a+1 are in flight while view a is gathered.  Everything outside the detector is staged as zero, which
// is the truncation rule for footprints that leave the detector.
//
// Static limits (checked on the host before this kernel is chosen): a voxel touches at most NC detector
// columns and NV detector rows; the window of any (view, tile, chunk) fits BP_PW x BP_PH.
#pragma once

#include "sf_footprint.h"

constexpr int BP_T = 16;        // tile edge in voxels (x and y)

// LDS row stride = window width + BP_ROW_PAD floats.  Lanes of a wave read windows that differ by a row or two
// and a few columns; a stride of 12 mod 32 banks measured fewest conflicts (1: 52.5 ms, 12: 48.3 ms on 512^3).
#ifndef BP_ROW_PAD
#define BP_ROW_PAD 12
#endif

// Shapes the kernel is instantiated for: voxels along z per thread, staged window columns x rows.
struct SfBpShape {
    int zc, pw, ph;
};
// The last one keeps 64 voxels per thread for footprints up to two rows tall (its 96 rows hold what 64 voxels of up to
// about 1.3 rows each project to); it is instantiated for NV <= 3 only, shape 0 for NV == 2 only (the general gather of
// taller footprints would spill registers).
constexpr SfBpShape BP_SHAPES[] = {{64, 32, 76}, {32, 32, 44}, {32, 32, 56}, {16, 32, 44}, {16, 64, 48}, {64, 32, 96}, {32, 42, 56}};
constexpr int BP_NSHAPES = sizeof(BP_SHAPES) / sizeof(BP_SHAPES[0]);
constexpr int BP_FIRST_SHORT_SHAPE = 1;      // first shape with fewer than 64 voxels per thread
constexpr int BP_LAST_SHORT_SHAPE = 4;       // last one
constexpr int BP_TALL_SHAPE = 5;
// 32 voxels per thread under a window wider than 32 columns (two- and three-row footprints, three or four columns wide): a
// view's set-up (window, knots, transaxial weights: about 150 instructions) is paid once for 32 voxels instead of 16.  42
// columns are what 252 threads stage six rows of at a time.  Instantiated for the footprint model only.  121 views of 211 x 187
// x 149 voxels on 163 x 257 pixels: 0.81 -> 0.71 ms.  (A window of 51 x 80 for voxels of up to two rows and three columns measured
// no better than 16 voxels under 64 x 48, 7.8 against 7.7 ms on eight 256^3 volumes of 60 views: eight samples per voxel from LDS are
// the limit there.)
constexpr int BP_WIDE_SHAPE = 6;

// Two volumes per thread (see sf_backproject_tiled): voxels per thread of either, window.  Tried in this order.
constexpr SfBpShape BP_PAIR_SHAPES[] = {{32, 32, 44}, {32, 32, 56}, {16, 32, 44}, {16, 51, 48}};
constexpr int BP_NPAIR_SHAPES = sizeof(BP_PAIR_SHAPES) / sizeof(BP_PAIR_SHAPES[0]);

// ... and which footprints they are instantiated for: narrow windows up to four columns, wide ones from three on.
constexpr bool bp_pair_instance_exists(int nc, int nv, int shape)
{
    return nv <= 3 && (BP_PAIR_SHAPES[shape].pw <= 32 ? nc <= 4 : nc >= 3);
}

// Four groups of threads that share the views (VS == 4): voxels per thread of either volume, window; the last for windows wider than
// 32 columns.
constexpr int BP_SPLIT = 4;
constexpr SfBpShape BP_SPLIT_SHAPES[] = {{32, 32, 44}, {16, 32, 44}, {8, 64, 32}};
constexpr int BP_NSPLIT_SHAPES = 3;
constexpr bool bp_split_instance_exists(int nc, int nv, int shape)
{
    return nv <= 3 && (BP_SPLIT_SHAPES[shape].pw <= 32 ? nc <= 4 : nc >= 3);
}

// Is the footprint kernel instantiated for NC columns, NV rows and this shape?
constexpr bool bp_instance_exists(int nc, int nv, int shape)
{
    if (shape == 0) return nv == 2;
    if (shape == BP_TALL_SHAPE) return nv <= 3;
    if (shape == BP_WIDE_SHAPE) return nv <= 3 && (nc == 3 || nc == 4);
    return true;
}

// Window of the detector that one (view, tile, z-chunk) can touch.  Evaluated identically on the host
// (limit check) and in the kernel; everything here is uniform over the workgroup.
struct SfWindow {
    int c0, r0;       // first staged column / row
    int need_w, need_h;
};

// Largest detector coordinate at which float bounds of a window stand: their rounding, half of 2^-7 pixels, stays below the
// hundredth of a pixel by which every window function widens them.
constexpr float BP_MAX_COORDINATE = 131072.0f;

// Staging role of a thread under a window of pw columns and ph rows: it stages column sc of rows sr + (256 / pw) s, those
// below ph.  Threads left over where pw does not divide 256 stage nothing: given the next step's first row, they would
// write its cells without an order to the threads that own them, and not the same values either (the row's detector
// coordinate comes from another number of float additions).  (Functions of constants: as one function of the window's sizes,
// inlined later, they cost the three-row instances a tenth of their time through other waits.)
template <int PW>
SF_HD int sf_stage_column(int tid) { return tid % PW; }
template <int PW, int PH>
SF_HD int sf_stage_row(int tid)
{
    if constexpr (256 % PW == 0) return tid / PW;
    else return tid < 256 / PW * PW ? tid / PW : PH;
}

// Cylindrical detector: column-coordinate range [xi_lo, xi_hi] and the range [ilo, ihi] of 1 / (in-plane distance from
// the source) over the square of half extent hx around (xc, yc).  The fan angle of a convex set is extreme at a
// corner; the distance is bounded by the centre's distance -+ the half diagonal.
SF_HD void sf_curved_tile_bounds(const SfGeom &g, const SfView &v, float xc, float yc, float hx, float &xi_lo, float &xi_hi,
                                 float &ilo, float &ihi)
{
    const float tc = fmaf(yc, v.c, -xc * v.s), dc = g.sod - fmaf(xc, v.c, yc * v.s);
    const float a = hx * (v.c - v.s), b = hx * (v.c + v.s);      // corner (+hx, +hx): (dt, dl) = (a, b); (+hx, -hx): (-b, a)
    const float g0 = atan2f(tc + a, dc - b), g1 = atan2f(tc - a, dc + b);
    const float g2 = atan2f(tc - b, dc - a), g3 = atan2f(tc + b, dc + a);
    xi_lo = fmaf(g.ku, fminf(fminf(g0, g1), fminf(g2, g3)), g.col_off);
    xi_hi = fmaf(g.ku, fmaxf(fmaxf(g0, g1), fmaxf(g2, g3)), g.col_off);
    const float dist = sf_sqrt(fmaf(tc, tc, dc * dc)), rad = 1.4143f * hx;
    ilo = sf_rcp(dist + rad);
    ihi = sf_rcp(fmaxf(dist - rad, 1e-3f * dist));
}

// xc, yc: tile centre (mm); hx: half extent of the voxel centres in x and y (mm); z0, z1: lower / upper face
// of the chunk (mm); wh: half of the widest transaxial footprint (pixels); nc, nv: columns / rows a thread reads
// per voxel (starting at the first one its footprint touches).
// Cylinder: what depends on (tile, view) only, worked out once per geometry on the host: the fan angle of the tile's
// centre in double and sf_curved_tile_bounds of the tile.  Stored [tile][view].
struct SfCurvedBounds {
    double gref;
    float xi_lo, xi_hi, ilo, ihi;
};

// Column-coordinate range and range of 1 / den of a tile in a view: what a window takes from the plane.
struct SfTileBounds {
    float xi_lo, xi_hi, ilo, ihi;
};

template <int GT = -1>
SF_HD SfTileBounds sf_bp_tile_bounds(const SfGeom &g, const SfView &v, float xc, float yc, float hx, const SfCurvedBounds *pre = nullptr)
{
    SfTileBounds b;
    b.ilo = b.ihi = 1.0f;               // smallest / largest 1/den over the tile
    if (sf_is_curved<GT>(g)) {
        if (pre) {
            b.xi_lo = pre->xi_lo; b.xi_hi = pre->xi_hi; b.ilo = pre->ilo; b.ihi = pre->ihi;
        } else {
            sf_curved_tile_bounds(g, v, xc, yc, hx, b.xi_lo, b.xi_hi, b.ilo, b.ihi);
        }
        return b;
    }
    const float tc = fmaf(yc, v.c, -xc * v.s);
    const float rho = hx * (fabsf(v.c) + fabsf(v.s));
    const float tlo = tc - rho, thi = tc + rho;
    if (g.type != SF_PARALLEL) {
        const float lc = fmaf(xc, v.c, yc * v.s);
        // a ragged edge tile's padding voxels may reach the source plane: keep the distance positive (the window then
        // comes out huge and the host rejects the kernel)
        b.ilo = sf_rcp(g.sod - lc + rho);
        b.ihi = sf_rcp(fmaxf(g.sod - lc - rho, 1e-6f * g.sod));
    }
    b.xi_lo = fmaf(g.ku * tlo, tlo >= 0.0f ? b.ilo : b.ihi, g.col_off);
    b.xi_hi = fmaf(g.ku * thi, thi >= 0.0f ? b.ihi : b.ilo, g.col_off);
    return b;
}

// Columns of the window of a tile with those bounds; rows for a chunk between the heights z0 and z1.
SF_HD void sf_bp_window_columns(const SfTileBounds &b, float wh, int nc, int &c0, int &need_w)
{
    c0 = sf_f2i(floorf(b.xi_lo - wh + 0.48f));
    need_w = sf_f2i(floorf(b.xi_hi + 0.52f)) + nc - c0;    // a thread reads nc columns from its first one
}

SF_HD void sf_bp_window_rows(const SfGeom &g, const SfTileBounds &b, float z0, float z1, int nv, int &r0, int &need_h)
{
    const float kv = (float)g.kvd, row_off = (float)g.row_offd;
    const float eta_lo = fmaf(kv * z0, z0 >= 0.0f ? b.ilo : b.ihi, row_off);
    const float eta_hi = fmaf(kv * z1, z1 >= 0.0f ? b.ihi : b.ilo, row_off);
    r0 = sf_f2i(floorf(eta_lo - 0.02f));
    need_h = sf_f2i(floorf(eta_hi + 0.02f)) + nv - r0;     // and nv rows from the first row of each voxel
}

template <int GT = -1>
SF_HD SfWindow sf_bp_window(const SfGeom &g, const SfView &v, float xc, float yc, float hx, float z0, float z1, float wh,
                            int nc, int nv, const SfCurvedBounds *pre = nullptr)
{
    SfWindow w;
    const SfTileBounds b = sf_bp_tile_bounds<GT>(g, v, xc, yc, hx, pre);
    sf_bp_window_columns(b, wh, nc, w.c0, w.need_w);
    sf_bp_window_rows(g, b, z0, z1, nv, w.r0, w.need_h);
    return w;
}

// Two volumes per workgroup (NS == 2).  All weights, placements and window bounds are the same for both, and a sample of either
// lies beside the other's in LDS, one 8-byte read (which the LDS serves as fast as a 4-byte one).  They are two items of a batch
// or, where the detector and the volume are symmetric about the source plane, the volume's upper half and the mirror image of its
// lower half: voxel k's partner is voxel nz - 1 - k, row r's row nrows - 1 - r, and the chunks start at voxel nz / 2.
struct SfBpSets {
    int mirror;
    int kfirst;       // first voxel of the first chunk
    int parts = 1;    // VS > 1: workgroups that share the views of a tile and chunk, each with sums of its own in a volume of its own
};
SF_HD int sf_mirror_first_voxel_above(int nz) { return nz / 2; }

// The tile of a workgroup.  Workgroups go to the 8 XCDs by index in turn, so by the grid's order every XCD has every eighth tile of a row, and its
// tiles at work at one time see windows all over a view.  Here an XCD takes a run of an eighth of the tiles, down bands of eight rows of
// tiles, and another run for every layer of chunks (y), so that each has tiles of the volume's edge and of its middle.  Windows come from L2 then
// where a view is as large as one: 1024^3, 1440 views, A and A^T 1153 -> 1122 ms (40 % of the loads hit L2, before 8 %, 1.04 TB beyond it, before 1.58);
// 8 x 256^3, 60 views and 512^3, 720 views (1 MiB) fetch half as much and take as long, within what two runs differ by.  Every tile once, whatever their numbers; the same bits.
SF_HD unsigned sf_bp_tile(unsigned x, unsigned y, unsigned tiles, unsigned tiles_x)
{
    const unsigned run = (x + (tiles % 8 == 0 ? y : 0)) % 8, each = tiles / 8, more = tiles % 8;
    const unsigned n = run * each + (run < more ? run : more) + x / 8;
    const unsigned band = n / (8 * tiles_x), in_band = n - band * 8 * tiles_x, left = tiles / tiles_x - band * 8, rows = left < 8 ? left : 8;
    return (band * 8 + in_band % rows) * tiles_x + in_band / rows;
}

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

// LDS row stride in samples.  Two volumes' samples are eight bytes: 12 and 8 more than the window are alike within a per cent, and
// under the 51-column window 8 leave room for a third workgroup (5.59 against 5.78 ms, eight 256^3 volumes of 60 views).
template <int NS>
constexpr int bp_row_stride(int pw) { return pw + (NS == 2 && pw > 32 ? 8 : BP_ROW_PAD); }

template <int NS>
struct alignas(4 * NS) SfBpSample {
    float v[NS];
};

// Staging, first half: fetch this thread's share of the window of one view into registers.  ya points at the view, y2 at the
// same view of the second volume, which it takes from the same places or, mirrored, from as far from the detector's other end.
template <int NC, int NV, int PW, int PH, int NSTAGE, int GT, int NS>
__device__ __forceinline__ void bp_load_view(const SfGeom &g, const SfView v, const float *__restrict__ ya, float xc, float yc,
                                             float hx, float z0, float z1, float wh, int sc, int sr, SfWindow &w,
                                             SfBpSample<NS> (&stage)[NSTAGE], const SfCurvedBounds *pre, const char *__restrict__ y2,
                                             bool mirror)
{
    constexpr int RSTEP = 256 / PW;
    w = sf_bp_window<GT>(g, v, xc, yc, hx, z0, z1, wh, NC, NV, pre);
    const int c = w.c0 + sc;
    const bool cin = (unsigned)c < (unsigned)g.ncols;
    // 32-bit byte offsets from the view's first element (a view has fewer than 2^30 pixels where this kernel is
    // chosen): one add per row instead of a 64-bit multiply; offsets of rows off the detector are never used
    const char *__restrict__ yb = reinterpret_cast<const char *>(ya);
    // (unsigned arithmetic: offsets of rows off the detector wrap around harmlessly)
    unsigned off = ((unsigned)(w.r0 + sr) * (unsigned)g.ncols + (unsigned)(cin ? c : 0)) * 4u;
    const unsigned step = (unsigned)RSTEP * (unsigned)g.ncols * 4u;
    // the partner's: the same offsets, or from the other end of the detector downwards
    unsigned off2 = mirror ? ((unsigned)(g.nrows - 1 - w.r0 - sr) * (unsigned)g.ncols + (unsigned)(cin ? c : 0)) * 4u : off;
    const unsigned step2 = mirror ? 0u - step : step;
#pragma unroll
    for (int s = 0; s < NSTAGE; ++s) {
        const int r = w.r0 + sr + RSTEP * s;
        // (rows from need_h on are never read: whole steps beyond it are left out, here and in bp_store_view)
        const bool in = cin && (unsigned)r < (unsigned)g.nrows && (sr + RSTEP * s) < PH && RSTEP * s < w.need_h;
        stage[s].v[0] = in ? *reinterpret_cast<const float *>(yb + off) : 0.0f;
        if constexpr (NS == 2) {
            stage[s].v[1] = in ? *reinterpret_cast<const float *>(y2 + off2) : 0.0f;
        }
        off += step;
        off2 += step2;
    }
}

// Staging, second half: scale by the ray amplitude and write to LDS.
template <int PW, int PH, int NSTAGE, int GT, int NS>
__device__ __forceinline__ void bp_store_view(const SfGeom &g, const SfView v, int sc, int sr, const SfWindow &w,
                                              const SfBpSample<NS> (&stage)[NSTAGE], SfBpSample<NS> *__restrict__ buf,
                                              const float2 *__restrict__ colcs = nullptr)
{
    constexpr int RSTEP = 256 / PW, PS = bp_row_stride<NS>(PW);
    SfAmpCol ac;
    if (GT == 1 && colcs) {      // cylinder: cosine and sine of the column's fan angle from the per-column table
        int c = w.c0 + sc;
        c = c < 0 ? 0 : (c > g.ncols - 1 ? g.ncols - 1 : c);    // columns off the detector were staged as zeros
        const float2 cs = colcs[c];
        ac = sf_amp_col_curved(g, v, cs.x, cs.y);
    } else {
        ac = sf_amp_col<GT>(g, v, w.c0 + sc);
    }
    // this thread's first row; RSTEP rows further per element (whole numbers, so that a row's v does not depend on the window it is
    // staged in: one volume and two may take different ones)
    float rf = (float)(w.r0 + sr);
#pragma unroll
    for (int s = 0; s < NSTAGE; ++s) {
        const int row = sr + RSTEP * s;
        if (RSTEP * s < w.need_h) {        // uniform over the workgroup
            if (row < PH) {
                const float amp = sf_amp_at(g, v, ac, fmaf(rf, g.pv, g.v0));
                SfBpSample<NS> q;
#pragma unroll
                for (int e = 0; e < NS; ++e) q.v[e] = stage[s].v[e] * amp;
                buf[row * PS + sc] = q;
            }
        }
        rf += (float)RSTEP;
    }
}

// Where a workgroup's tile and z-chunk lie in the scene a view sees (mm): tile centre, chunk faces.
struct SfBpScene {
    float xc, yc, z0, z1;
    double zlo_k0;
};

template <int BP_ZC>
SF_HD SfBpScene sf_bp_scene(const SfGeom &g, int i0, int j0, int k0)
{
    SfBpScene s;
    s.zlo_k0 = fma((double)k0, g.Tzd, g.zlo0d);
    s.z0 = (float)s.zlo_k0;
    s.z1 = s.z0 + (float)BP_ZC * g.Tz;
    s.xc = (float)(g.x0d + ((double)i0 + 0.5 * (BP_T - 1)) * g.Td);
    s.yc = (float)(g.y0d + ((double)j0 + 0.5 * (BP_T - 1)) * g.Td);
    return s;
}

// The parts' volumes summed in the order of the parts: item n of `per` to a workgroup at [n / per][part][n % per].  grid.y: items.
static __global__ __launch_bounds__(256) void sf_sum_parts(const float *__restrict__ from, float *__restrict__ vol, unsigned nvol, int parts, int per)
{
    const unsigned e = blockIdx.x * 256u + threadIdx.x;
    if (e >= nvol) return;
    const unsigned item = blockIdx.y;
    from += (size_t)(item / per * parts * per + item % per) * nvol + e;
    float sum = from[0];
    for (int p = 1; p < parts; ++p) sum += from[(size_t)p * per * nvol];
    vol[(size_t)item * nvol + e] = sum;
}

// GT: 0 flat or parallel, 1 cylindrical detector, 2 modular geometry with upright modules (every view brings its own
// parameter block geoms[a]: the scene translated so that the view is a circular cone-beam view; g holds the sizes).
// NS: volumes per workgroup.  VS: groups of 256 threads that share a tile's views, group q taking views q, q + VS, ...: a step from
// one view to the next takes a microsecond and a half and more however few voxels a thread has (the window's loads, two barriers'
// worth of waiting), so a volume too small to fill the chip is as slow as its views are many.  The groups' sums are added in order.
// Registers spilled at the bounds below (waves of 64 or 128 registers): four to six by the cylinder's two volumes of 32 voxels in parts, one to three by
// single volumes of 16 voxels and voxels three rows tall.
template <int NC, int NV, int BP_ZC, int BP_PW, int BP_PH, int GT, int NS, int VS = 1, bool PARTS = false>
__global__ __launch_bounds__(256 * VS, VS > 1 ? (NS == 1 && BP_ZC <= 16 && GT != 1 ? 8 : 4) : (GT == 1 && NV > 2 && BP_ZC * NS > 32) ? 3 : (NS == 2 && BP_PW > 42 && BP_ZC > 8 ? 3 : 4)) void sf_backproject_tiled(SfGeom g, const SfView *__restrict__ views,
                                                            const float *__restrict__ sino, float *__restrict__ vol,
                                                            int tiles_x, float wh, const void *__restrict__ aux, SfBpSets sets)
{
    // aux: GT == 2: the per-view parameter blocks; GT == 1: cosine and sine of every detector column's fan angle
    // (ncols pairs of floats), followed by the per-(tile, view) table
    const SfGeom *__restrict__ geoms = GT == 2 ? static_cast<const SfGeom *>(aux) : nullptr;
    const unsigned tile = VS > 1 ? blockIdx.x : (unsigned)__builtin_amdgcn_readfirstlane((int)sf_bp_tile(blockIdx.x, blockIdx.y, gridDim.x, (unsigned)tiles_x));
    const float2 *__restrict__ colcs = GT == 1 ? static_cast<const float2 *>(aux) : nullptr;
    const SfCurvedBounds *__restrict__ cvt =
        GT == 1 ? reinterpret_cast<const SfCurvedBounds *>(static_cast<const float2 *>(aux) + g.ncols) + (size_t)tile * g.nviews
                : nullptr;
    constexpr int BP_PS = bp_row_stride<NS>(BP_PW);      // LDS row stride (samples)
    using Sample = SfBpSample<NS>;
    __shared__ Sample patch[2 * VS][BP_PH * BP_PS];
    // blockIdx.z: item of a batch, or pair of items; PARTS: times the parts of its views, the volumes of an item's parts side by side (a template:
    // bounds of the views that are worked out in the kernel cost scans whose views stay whole 2.5 %, 102 x 97 x 74, 425 views 495 / 507 us)
    const bool mirror = NS == 2 && sets.mirror;
    const unsigned block = PARTS ? blockIdx.z / (unsigned)sets.parts : blockIdx.z;
    const int part = PARTS ? (int)(blockIdx.z - block * (unsigned)sets.parts) : 0;
    const int a_first = PARTS ? (int)((long long)g.nviews * part / sets.parts) : 0;
    const int a_end = PARTS ? (int)((long long)g.nviews * (part + 1) / sets.parts) : g.nviews;
    sino += (size_t)block * (mirror ? 1 : NS) * g.nviews * g.nrows * g.ncols;
    vol += (size_t)blockIdx.z * (mirror ? 1 : NS) * g.nx * g.ny * g.nz;
    const size_t to_second = mirror ? 0 : (size_t)g.nviews * g.nrows * g.ncols;

    const int tid = VS == 1 ? threadIdx.x : threadIdx.x & 255;
    const int group = VS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
    const int ti = tid & (BP_T - 1), tj = tid >> 4;
    const int tx = tile % tiles_x, ty = tile / tiles_x;
    const int i0 = tx * BP_T, j0 = ty * BP_T;
    const int k0 = (NS == 2 ? sets.kfirst : 0) + blockIdx.y * BP_ZC;
    const int i = i0 + ti, j = j0 + tj;
    const int ic = i < g.nx ? i : g.nx - 1, jc = j < g.ny ? j : g.ny - 1;   // out-of-volume threads shadow the edge

    const float hx = 0.5f * (float)(BP_T - 1) * g.T;
    auto geom_of = [&](int a) -> const SfGeom & {
        if constexpr (GT == 2) return geoms[a];
        else return g;
    };
    const SfBpScene scene0 = sf_bp_scene<BP_ZC>(geom_of(VS == 1 || a_first + group < a_end ? a_first + group : 0), i0, j0, k0);     // of the group's first view

    const int sc = sf_stage_column<BP_PW>(tid), sr = sf_stage_row<BP_PW, BP_PH>(tid);
    constexpr int NSTAGE = (BP_PH + 256 / BP_PW - 1) / (256 / BP_PW);
    const size_t view_stride = (size_t)g.nrows * g.ncols;

    float acc[BP_ZC][NS];
#pragma unroll
    for (int kk = 0; kk < BP_ZC; ++kk)
#pragma unroll
        for (int e = 0; e < NS; ++e) acc[kk][e] = 0.0f;

    Sample stage[NSTAGE];
    SfWindow win_next;

    // tile centre in double (cylinder only)
    const double xcd = g.x0d + ((double)i0 + 0.5 * (BP_T - 1)) * g.Td, ycd = g.y0d + ((double)j0 + 0.5 * (BP_T - 1)) * g.Td;
    auto cv_pre = [&](int a) -> const SfCurvedBounds * {
        if constexpr (GT == 1) return cvt + a;
        else return nullptr;
    };

    SfWindow win = {};
    if (VS == 1 || a_first + group < a_end) {
        const int a = a_first + group;
        const float *ya = sino + (size_t)a * view_stride;
        bp_load_view<NC, NV, BP_PW, BP_PH, NSTAGE, GT, NS>(geom_of(a), views[a], ya, scene0.xc, scene0.yc, hx, scene0.z0, scene0.z1, wh,
                                                           sc, sr, win, stage, cv_pre(a), reinterpret_cast<const char *>(ya + to_second), mirror);
        bp_store_view<BP_PW, BP_PH, NSTAGE, GT, NS>(geom_of(a), views[a], sc, sr, win, stage, patch[2 * group], colcs);
    }
    win_next = win;
    __syncthreads();

    for (int a = a_first + group; a - group < a_end; a += VS) {
        const int buffer = 2 * group + (((a - a_first - group) / VS) & 1);
        const Sample *buf = patch[buffer];
        if (VS == 1 || a < a_end) {
        double gref = 0.0;
        if constexpr (GT == 1) gref = cvt[a].gref;
        if (a + VS < a_end) {    // global loads in flight during the gather
            const SfBpScene sn = GT == 2 ? sf_bp_scene<BP_ZC>(geom_of(a + VS), i0, j0, k0) : scene0;
            const float *ya = sino + (size_t)(a + VS) * view_stride;
            bp_load_view<NC, NV, BP_PW, BP_PH, NSTAGE, GT, NS>(geom_of(a + VS), views[a + VS], ya, sn.xc, sn.yc, hx, sn.z0, sn.z1, wh, sc, sr,
                                                               win_next, stage, cv_pre(a + VS), reinterpret_cast<const char *>(ya + to_second), mirror);
        }
        const SfGeom &gv = geom_of(a);
        const double zlo_k0 = GT == 2 ? fma((double)k0, gv.Tzd, gv.zlo0d) : scene0.zlo_k0;

        const SfView v = views[a];
        SfColumn f;
        if constexpr (GT == 1)
            f = sf_column_curved_ref(gv, v, ic, jc, fma(ycd, v.cd, -xcd * v.sd), gv.sodd - fma(xcd, v.cd, ycd * v.sd), gref);
        else
            f = sf_column<GT>(gv, v, ic, jc);
        int cf, cl;
        sf_col_range(f, cf, cl);
        float fu[NC];
        {
            float e = sf_pixel_edge(f, cf);
            float g0 = sf_trap_integral(f, e);
#pragma unroll
            for (int m = 0; m < NC; ++m) {
                e += 1.0f;
                const float g1 = sf_trap_integral(f, e);
                fu[m] = fmaxf(g1 - g0, 0.0f);
                g0 = g1;
            }
        }
        const SfRowsOfVoxels ax = sf_rows_of_voxels(gv, f, zlo_k0);
        unsigned ofs = (unsigned)((ax.rb - win.r0) * BP_PS + (cf - win.c0));

        // Where no voxel of the wave is taller than a detector row in this view, consecutive voxels share rows and the
        // cheaper running scheme applies; tiles far from the source qualify even when the nearest voxels of the volume do
        // not (the instance is built for the tallest footprint).  The choice is uniform over the wave, so it costs one
        // ballot per view.
        // NV == 3 is chosen on the host only when no voxel is taller than two rows (with a margin): every lane takes one
        // of the two running schemes below, whichever fits its voxel column in this view.  Tiles far from the source hold
        // short voxels even when the nearest voxels of the volume are tall; a wave that holds both kinds (rare: the line
        // where a voxel is exactly one row tall crosses its 16 x 4 columns) runs the two schemes one after the other.
        const bool shared_rows = NV == 2 || (NV == 3 ? ax.av <= 1.0f : __builtin_amdgcn_ballot_w64(ax.av > 1.0f) == 0);
        // The voxel's first row is carried as a byte offset into the patch array (both buffers), so that every LDS read is
        // that register plus an immediate and a row crossing costs one select and one add.
        constexpr unsigned ROW = (unsigned)(BP_PS * sizeof(Sample));
        const char *const lds0 = reinterpret_cast<const char *>(&patch[0][0]);
        const unsigned lds_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) Sample *)&patch[0][0];
        unsigned pb = (unsigned)(buffer * (BP_PH * BP_PS) + (int)ofs) * (unsigned)sizeof(Sample);
        struct Sum {
            float v[NS];
        };
        auto sample = [&](unsigned byte_ofs) {
            if constexpr (NS == 1) {
                return *reinterpret_cast<const Sample *>(lds0 + byte_ofs);
            } else {
                // (volatile: two merged into one 16-byte access at 8-byte alignment cost twice their time apart)
                typedef const volatile __attribute__((address_space(3))) unsigned long long Lds;
                const unsigned long long q = *(Lds *)(uintptr_t)(lds_at + byte_ofs);
                Sample r;
                __builtin_memcpy(&r, &q, 8);
                return r;
            }
        };
        auto row_sum = [&](unsigned byte_ofs) {
            Sum s;
            Sample q[NC];
#pragma unroll
            for (int m = 0; m < NC; ++m) q[m] = sample(byte_ofs + m * (unsigned)sizeof(Sample));
#pragma unroll
            for (int e = 0; e < NS; ++e) {
                s.v[e] = fu[0] * q[0].v[e];
#pragma unroll
                for (int m = 1; m < NC; ++m) s.v[e] = fmaf(fu[m], q[m].v[e], s.v[e]);
            }
            return s;
        };
        // An opaque dependency every few voxels: the LDS reads of the next group need `pb` / `ofs`, which is only available once
        // this group's sums exist.  Without it the compiler issues all reads of the unrolled loop first and spills them.
        auto hold = [&](int kk, unsigned &reg) {
            if constexpr (NS == 1) {
                if ((kk & 3) == 3)
                    asm volatile("" : "+v"(reg), "+v"(acc[kk - 3][0]), "+v"(acc[kk - 2][0]), "+v"(acc[kk - 1][0]), "+v"(acc[kk][0]));
            } else {
                if ((kk & 1) == 1)
                    asm volatile("" : "+v"(reg), "+v"(acc[kk - 1][0]), "+v"(acc[kk - 1][1]), "+v"(acc[kk][0]), "+v"(acc[kk][1]));
            }
        };
        if (shared_rows) {
            // A voxel is at most one row tall, so consecutive voxels share a row: keep the u-combined samples of the
            // current and the next row in registers and fetch one new row per voxel (half the LDS traffic).
            // f: where the voxel's lower face lies inside its first row, in [0,1); the face moves up by av per voxel.
            float f = ax.phi0;
            Sum s_cur = row_sum(pb), s_next = row_sum(pb + ROW);
#pragma unroll
            for (int kk = 0; kk < BP_ZC; ++kk) {
                const float t = f + ax.av;                        // upper face, still measured from the first row
                const float w1 = sf_clamp(t - 1.0f, 0.0f, 1.0f);  // part of the voxel in the next row
                const float w0 = ax.av - w1;
#pragma unroll
                for (int e = 0; e < NS; ++e) acc[kk][e] = fmaf(w1, s_next.v[e], fmaf(w0, s_cur.v[e], acc[kk][e]));
                if (kk + 1 < BP_ZC) {
                    const bool cross = t >= 1.0f;                 // the next voxel starts in the next row
                    pb += cross ? ROW : 0u;
                    const Sum s_new = row_sum(pb + ROW);          // equals s_next when no row was crossed
#pragma unroll
                    for (int e = 0; e < NS; ++e) s_cur.v[e] = cross ? s_next.v[e] : s_cur.v[e];
                    s_next = s_new;
                    f = cross ? w1 : t;                           // t - 1 where a row was crossed
                }
                hold(kk, pb);
            }
        } else if constexpr (NV == 3) {
            // Between one and two rows tall: a voxel covers the rest of its first row, then up to one whole row, then
            // part of a third, and the next voxel starts one or two rows further: the u-combined sum of that row is
            // carried over (one select), the two rows after it are fetched fresh.
            float f = ax.phi0;
            Sum s0 = row_sum(pb), s1 = row_sum(pb + ROW), s2 = row_sum(pb + 2u * ROW);
#pragma unroll
            for (int kk = 0; kk < BP_ZC; ++kk) {
                const float t = f + ax.av;                        // upper face from the first row's lower edge: in (1, 3)
                const float w2 = sf_clamp(t - 2.0f, 0.0f, 1.0f);  // part in the third row
                const float w0 = 1.0f - f;                        // the rest of the first row
                const float w1 = (ax.av - w0) - w2;
#pragma unroll
                for (int e = 0; e < NS; ++e) acc[kk][e] = fmaf(w2, s2.v[e], fmaf(w1, s1.v[e], fmaf(w0, s0.v[e], acc[kk][e])));
                if (kk + 1 < BP_ZC) {
                    const bool two = t >= 2.0f;                   // the next voxel starts two rows further
                    pb += two ? 2u * ROW : ROW;
#pragma unroll
                    for (int e = 0; e < NS; ++e) s0.v[e] = two ? s2.v[e] : s1.v[e];
                    s1 = row_sum(pb + ROW);
                    s2 = row_sum(pb + 2u * ROW);
                    f = two ? w2 : t - 1.0f;                      // t - 2 where two rows were crossed
                }
                hold(kk, pb);
            }
        } else if constexpr (NV > 3) {
            static_assert(NS == 1, "taller footprints are back projected one volume at a time");
            const float *bufs = reinterpret_cast<const float *>(buf);
            float lo = ax.phi0;
#pragma unroll
            for (int kk = 0; kk < BP_ZC; ++kk) {
                const float hi = fmaf(ax.av, (float)(kk + 1), ax.phi0);
                const float fl = floorf(lo);
                const float *q = bufs + (ofs + __umul24((unsigned)(int)fl, (unsigned)BP_PS));   // 24-bit multiply: one full-rate op
                float edge = fl + 1.0f;                                   // upper edge of the first row the voxel touches
                float w = fminf(edge, hi) - lo;
                float sum = acc[kk][0];
#pragma unroll
                for (int jj = 0; jj < NV; ++jj) {
                    float s = fu[0] * q[jj * BP_PS];
#pragma unroll
                    for (int m = 1; m < NC; ++m) s = fmaf(fu[m], q[jj * BP_PS + m], s);
                    sum = fmaf(w, s, sum);
                    w = sf_clamp(hi - edge, 0.0f, 1.0f);                  // overlap with the next row
                    edge += 1.0f;
                }
                acc[kk][0] = sum;
                lo = hi;
                hold(kk, ofs);
            }
        }

        if (a + VS < a_end)
            bp_store_view<BP_PW, BP_PH, NSTAGE, GT, NS>(geom_of(a + VS), views[a + VS], sc, sr, win_next, stage, patch[buffer ^ 1], colcs);
        }
        win = win_next;
        __syncthreads();
    }

    if constexpr (VS > 1) {
        // the groups' sums, a few voxels at a time through the windows' place
        constexpr int FIT = (int)(sizeof(patch) / VS / (256 * NS * sizeof(float))), SLICE = FIT >= BP_ZC ? BP_ZC : (FIT >= 16 ? 16 : (FIT >= 8 ? 8 : 4));
        static_assert(FIT >= 4 && BP_ZC % SLICE == 0, "a slice of every group's sums fits the windows' place");
        float *const sums = reinterpret_cast<float *>(&patch[0][0]);
#pragma unroll
        for (int s0 = 0; s0 < BP_ZC; s0 += SLICE) {
            if (group > 0) {
#pragma unroll
                for (int kk = 0; kk < SLICE; ++kk)
#pragma unroll
                    for (int e = 0; e < NS; ++e) sums[((group * SLICE + kk) * NS + e) * 256 + tid] = acc[s0 + kk][e];
            }
            __syncthreads();
            if (group == 0) {
#pragma unroll
                for (int q = 1; q < VS; ++q)
#pragma unroll
                    for (int kk = 0; kk < SLICE; ++kk)
#pragma unroll
                        for (int e = 0; e < NS; ++e) acc[s0 + kk][e] += sums[((q * SLICE + kk) * NS + e) * 256 + tid];
            }
            __syncthreads();
        }
        if (group > 0) return;
    }

    if (i < g.nx && j < g.ny) {
#pragma unroll
        for (int kk = 0; kk < BP_ZC; ++kk)
            if (k0 + kk < g.nz) {
                const int k = k0 + kk;
                vol[((size_t)k * g.ny + j) * g.nx + i] = acc[kk][0];
                if constexpr (NS == 2) {
                    const int k2 = mirror ? g.nz - 1 - k : k + g.nz;      // (an odd volume's middle layer is its own mirror image)
                    if (k2 != k) vol[((size_t)k2 * g.ny + j) * g.nx + i] = acc[kk][1];
                }
            }
    }
}

#endif
