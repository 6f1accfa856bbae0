// Host geometry module: validates the CT parameter set ("PyTorch Interfaces and CT Parameters") and turns
// it into the constant tables the kernels read.  All derivations run in double; the tables are rounded to
// float once, here.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <cstring>
#include <exception>
#include <new>
#include <thread>

#include "leap_internal.h"
#define SF_NO_KERNELS   // this file needs the kernels' host-side limit functions only
#include "sf_backproject_tiled.h"
#include "sf_project_columns.h"
#include "md_backproject_tiled.h"
#include "sf_flat.h"
#include "md_footprint_tiled.h"
#include "sd_backproject_tiled.h"

static thread_local std::string g_last_error;

void leap_set_error(const std::string &msg) { g_last_error = msg; }

int leap_hip_fail(hipError_t e, const char *what)
{
    g_last_error = std::string(what) + ": " + hipGetErrorString(e);
    return LEAP_HIP_ERROR;
}

extern "C" const char *leap_last_error(void) { return g_last_error.c_str(); }

extern "C" const char *leap_status_string(int status)
{
    switch (status) {
    case LEAP_OK: return "ok";
    case LEAP_INVALID_ARG: return "invalid argument";
    case LEAP_BAD_GEOMETRY: return "geometry not supported: source must lie strictly outside the volume";
    case LEAP_HIP_ERROR: return "HIP runtime error";
    case LEAP_UNSUPPORTED: return "size not supported";
    default: return "unknown status";
    }
}

static int invalid(const char *why)
{
    leap_set_error(why);
    return LEAP_INVALID_ARG;
}

static void add_note(leap_geometry *G, const char *what)
{
    if (!G->note.empty()) G->note += "; ";
    G->note += what;
}

static bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

// Siddon model: constants of the line of every (view, detector column), in double ("sd_ray.h" states the formulation).
static void build_ray_table(leap_geometry *G)
{
    const leap_geometry_desc &d = G->desc;
    const double T = d.voxel_xy, Tz = d.voxel_z;
    G->raycols.resize((size_t)d.nviews * d.ncols);
    double max_slope = 0.0, min_h = 1e300, max_h = 0.0;
    G->sd_max_z = 0.0;
    for (int a = 0; a < d.nviews; ++a) {
        // modular scans with upright modules bring one parameter block per view: a circular cone-beam view of the
        // translated scene, with its own source distance, detector distance and column offset
        const bool per_view = !G->geoms.empty();
        const SfGeom &g = per_view ? G->geoms[a] : G->g;
        const int type = per_view ? (int)LEAP_CONE : d.type;
        const double sod = per_view ? g.sodd : d.sod, sdd = per_view ? g.kud * d.pixel_u : d.sdd;
        const double xlo = g.x0d - 0.5 * T, ylo = g.y0d - 0.5 * T;      // lower faces of voxel (0, 0)
        const double c = G->views[a].cd, s = G->views[a].sd;
        double max_dh = 0.0;
        for (int col = 0; col < d.ncols; ++col) {
            const double u = ((double)col - g.col_offd) * d.pixel_u;
            double ox, oy, dx, dy;
            if (type == LEAP_PARALLEL) {
                ox = -u * s; oy = u * c; dx = c; dy = s;
            } else if (type == LEAP_CONE_CURVED) {    // pixel at fan angle u / sdd on the cylinder
                const double cg = std::cos(u / sdd), sg = std::sin(u / sdd);
                ox = sod * c; oy = sod * s;
                dx = -sdd * (cg * c + sg * s); dy = sdd * (sg * c - cg * s);
            } else {
                ox = sod * c; oy = sod * s;
                dx = -sdd * c - u * s; dy = -sdd * s + u * c;
            }
            SdRayCol R;
            R.xmajor = std::fabs(dx) >= std::fabs(dy) ? 1 : 0;
            const double dmaj = R.xmajor ? dx : dy, dmin = R.xmajor ? dy : dx;
            const double omaj = R.xmajor ? ox : oy, omin = R.xmajor ? oy : ox;
            const double lomaj = R.xmajor ? xlo : ylo, lomin = R.xmajor ? ylo : xlo;
            R.m = dmin / dmaj;
            R.b = (omin - lomin) / T - R.m * (omaj - lomaj) / T;
            const double inv_m = R.m != 0.0 ? 1.0 / R.m : 1e30;
            R.inv_m = (float)std::fmin(std::fmax(inv_m, -1e30), 1e30);
            R.lxy = (float)(T * std::sqrt(dx * dx + dy * dy) / std::fabs(dmaj));
            if (type == LEAP_CONE || type == LEAP_CONE_CURVED) {
                R.h0 = (lomaj - omaj) / (dmaj * Tz);
                R.dh = T / (dmaj * Tz);
                R.vscale = (float)(T / std::fabs(dmaj));
            } else if (type == LEAP_PARALLEL) {
                R.h0 = 1.0 / Tz; R.dh = 0.0; R.vscale = 0.0f;
            } else {
                R.h0 = 0.0; R.dh = 0.0; R.vscale = 0.0f;
            }
            max_dh = std::fmax(max_dh, std::fabs(R.dh));
            // h over the slabs in which the line meets the volume (a slab and a cell to spare)
            const double n_major = R.xmajor ? d.nx : d.ny, n_minor = R.xmajor ? d.ny : d.nx;
            double x_in = 0.0, x_out = n_major;
            if (R.m != 0.0) {
                const double xa = (-1.0 - R.b) / R.m, xb = (n_minor + 1.0 - R.b) / R.m;
                x_in = std::fmax(x_in, std::fmin(xa, xb) - 1.0);
                x_out = std::fmin(x_out, std::fmax(xa, xb) + 1.0);
            } else if (R.b < -1.0 || R.b > n_minor + 1.0) {
                x_out = -1.0;
            }
            if (x_in <= x_out) {
                const double ha = R.h0 + R.dh * x_in, hb = R.h0 + R.dh * x_out;
                min_h = std::fmin(min_h, std::fmin(ha, hb));
                max_h = std::fmax(max_h, std::fmax(ha, hb));
            }
            G->raycols[(size_t)a * d.ncols + col] = R;
        }
        const double vmax = std::fmax(std::fabs(g.v0d), std::fabs(g.v0d + (d.nrows - 1) * g.pvd));
        max_slope = std::fmax(max_slope, max_dh * vmax);
        G->sd_max_z = std::fmax(G->sd_max_z, std::fabs(g.zk0d) + (vmax + 1024.0 * d.pixel_v) * max_h);
    }
    G->sd_min_row_step = min_h * d.pixel_v;
    G->sd_max_row_step = max_h * d.pixel_v;
    G->sd_max_axial_slope = max_slope;
}

// ---- debugging aid ---------------------------------------------------------------------------------------------------
// One environment variable, LEAP_DEBUG, read when a handle is created: comma-separated key=value pairs that override
// what the selection below would pick (include/leap.h lists the keys).  Unknown keys are ignored.
static bool debug_option(const char *key, long &value)
{
    const char *env = std::getenv("LEAP_DEBUG");
    if (!env) return false;
    const size_t klen = std::strlen(key);
    for (const char *p = env; *p;) {
        const char *end = std::strchr(p, ',');
        const size_t len = end ? (size_t)(end - p) : std::strlen(p);
        if (len > klen + 1 && std::strncmp(p, key, klen) == 0 && p[klen] == '=') {
            value = std::atol(p + klen + 1);
            return true;
        }
        if (!end) break;
        p = end + 1;
    }
    return false;
}

// bp_pair, bp_split: the shape asked for, -1 none, -2 the selection's own.  A back-projection shape asked for by bp_shape is one of the kernels
// of one volume without shared views, so it leaves none of the others unless they are named too.
static long back_option(const char *key)
{
    long shape, only = -2;
    if (!debug_option(key, only) && debug_option("bp_shape", shape)) only = -1;
    return only;
}

// The parameter block view a is projected with: its own (modular scans with upright modules) or the shared one.
static const SfGeom &view_geom(const leap_geometry *G, int a) { return G->geoms.empty() ? G->g : G->geoms[a]; }

// Footprint bounds over the whole volume and all views, in double.  Magnification is extreme at the corner of the
// volume's bounding circle; a flat detector stretches a footprint seen at fan angle gamma by 1 / cos(gamma).
// Returns false when some view's source does not clear the bounding circle (then no fast kernel applies).
static bool footprint_bounds(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    const double T = d->voxel_xy, half_x = 0.5 * d->nx * T, half_y = 0.5 * d->ny * T;
    const int blocks = G->geoms.empty() ? 1 : d->nviews;
    double cols = 0.0, rows = 0.0, vpr = 0.0, slope = 1.0;
    for (int a = 0; a < blocks; ++a) {
        const SfGeom &ga = view_geom(G, a);
        const double cx = ga.x0d + 0.5 * (d->nx - 1) * T, cy = ga.y0d + 0.5 * (d->ny - 1) * T;
        const double rx = std::fabs(cx) + half_x, ry = std::fabs(cy) + half_y;
        const double reach = std::sqrt(rx * rx + ry * ry) + T;
        double mag_max = 1.0, mag_min = 1.0, stretch = 1.0;
        if (ga.type != SF_PARALLEL) {
            const double sdd = ga.kud * d->pixel_u, sod = ga.sodd;
            if (!(sod > reach) && !G->geoms.empty()) return false;
            mag_max = sdd / std::fmax(sod - reach, 1e-9 * sod);
            mag_min = sdd / (sod + reach);
            const double umax = std::fmax(std::fabs(-2.0 - ga.col_offd), std::fabs(d->ncols + 1.0 - ga.col_offd)) * d->pixel_u;
            const bool curved = ga.type == SF_CONE_CURVED;
            const double gam = curved ? std::fmin(umax / sdd, 1.57) : std::atan(umax / sdd);
            stretch = curved ? 1.02 : 1.02 / std::cos(gam);       // no stretch on the cylinder
            slope = std::fmax(slope, gam < 0.78 ? std::tan(0.7853981633974483 + gam) : 1e30);
        }
        const bool fan = ga.type == SF_FAN;
        cols = std::fmax(cols, mag_max * T * std::sqrt(2.0) / d->pixel_u * stretch);
        rows = std::fmax(rows, fan ? 1.0 : mag_max * d->voxel_z / d->pixel_v);
        vpr = std::fmax(vpr, fan ? 1.0 : d->pixel_v / (mag_min * d->voxel_z));
    }
    G->max_cols_per_voxel = cols; G->max_rows_per_voxel = rows; G->max_voxels_per_row = vpr; G->max_minor_slope = slope;
    return true;
}

// Runs share(0) .. share(workers - 1) on that many threads, the caller's among them; the caller takes over the shares of threads
// that cannot be started.  What a share throws reaches the caller once all threads have ended.
template <class Share>
static void run_shares(int workers, Share share)
{
    std::vector<std::exception_ptr> thrown(workers);
    std::vector<std::thread> pool;
    pool.reserve(workers);
    auto run = [&](int t) {
        try {
            share(t);
        } catch (...) {
            thrown[t] = std::current_exception();
        }
    };
    int t = 1;
    try {
        for (; t < workers; ++t) pool.emplace_back(run, t);
    } catch (...) {          // no further thread to be had
    }
    for (; t < workers; ++t) run(t);
    run(0);
    for (auto &th : pool) th.join();
    for (auto &e : thrown)
        if (e) std::rethrow_exception(e);
}

// Chunks of zc voxels from voxel kfirst on, and the largest staged window any (view, tile, chunk) of theirs asks for.
struct WindowNeed {
    int zc, kfirst;
    int w = 0, h = 0;
};

// Largest staged windows of a tiled back projection for several heights of chunk at once, evaluated with the kernel's own window
// functions on the view's own parameter block.  tile(ga, view, xc, yc, window): what the windows of a tile have in common, their columns
// among it; rows(ga, that, z0, z1, window): the rows of one.
template <class TileFn, class RowsFn>
static void staged_window_needs(const leap_geometry *G, std::vector<WindowNeed> &needs, TileFn tile, RowsFn rows)
{
    const leap_geometry_desc *d = &G->desc;
    const int tiles_x = (d->nx + BP_T - 1) / BP_T, tiles_y = (d->ny + BP_T - 1) / BP_T;
    // the views are shared out among a few threads (a thousand views of a few thousand tiles each)
    const int workers = (int)std::max(1, std::min(8, d->nviews / 32));
    std::vector<std::vector<WindowNeed>> found(workers, needs);
    auto scan = [&](int t) {
        std::vector<WindowNeed> mine = needs;       // kept local: the workers' results share cache lines
        for (int a = t; a < d->nviews; a += workers) {
            const SfGeom &ga = view_geom(G, a);
            for (int ty = 0; ty < tiles_y; ++ty)
                for (int tx = 0; tx < tiles_x; ++tx) {
                    const float xc = (float)(ga.x0d + ((double)(tx * BP_T) + 0.5 * (BP_T - 1)) * ga.Td);
                    const float yc = (float)(ga.y0d + ((double)(ty * BP_T) + 0.5 * (BP_T - 1)) * ga.Td);
                    SfWindow win;
                    const auto bounds = tile(ga, G->views[a], xc, yc, win);
                    for (WindowNeed &n : mine) {
                        const int chunks = (d->nz - n.kfirst + n.zc - 1) / n.zc;
                        for (int ch = 0; ch < chunks; ch += (chunks > 1 ? chunks - 1 : 1)) {   // extremes: first and last chunk
                            const float z0 = (float)(ga.zlo0d + (double)(n.kfirst + ch * n.zc) * ga.Tzd), z1 = z0 + (float)n.zc * ga.Tz;
                            rows(ga, bounds, z0, z1, win);
                            const bool near = std::abs((float)win.c0) < BP_MAX_COORDINATE - 1024.0f && std::abs((float)win.r0) < BP_MAX_COORDINATE - 1024.0f;
                            n.w = std::max(n.w, near ? win.need_w : 1 << 30);
                            n.h = std::max(n.h, near ? win.need_h : 1 << 30);
                        }
                    }
                }
        }
        found[t] = mine;
    };
    run_shares(workers, scan);
    for (const auto &mine : found)
        for (size_t n = 0; n < needs.size(); ++n) {
            needs[n].w = std::max(needs[n].w, mine[n].w);
            needs[n].h = std::max(needs[n].h, mine[n].h);
        }
}

// one spare row and column: host and device floats may round apart
static bool window_fits(const WindowNeed &n, const SfBpShape &S) { return n.w <= S.pw - 1 && n.h <= S.ph - 1; }

// Detector and volume symmetric about the source plane: the weight of voxel k for row r is that of voxel nz - 1 - k for row
// nrows - 1 - r, in every view.
static bool mirrored_about_source_plane(const leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    return (d->type == LEAP_CONE || d->type == LEAP_CONE_CURVED || d->type == LEAP_PARALLEL) && d->shift_v == 0.0 && d->center_z == 0.0;
}

// What a launch of the tiled back projections takes per view, for footprints in units of 32 voxels per thread under a narrow window on an
// idle chip (2.8 us): `idle` while its workgroups have a compute unit each, `full` per round of 256 workgroups once the compute units are
// full and for `late` rounds more (the last of several workgroups per compute unit run beside fewer); a launch takes as long as `views`
// further views whatever it holds (the window's first loads, the sums of groups of threads that share the views).
struct LaunchTime {
    double idle, full, views, late = 0.0;
};
static double launch_time(const LaunchTime &t, double workgroups, int views)
{
    const double rounds = std::ceil(workgroups / 256.0);
    return std::max(t.idle * (1.0 + 0.07 * (rounds - 1.0)), t.full * (rounds + t.late)) * (views + t.views);
}

// Footprint model: one volume and two volumes per workgroup by shape; views shared, one volume and two (one volume of 16 voxels or fewer: two
// workgroups of 1024 threads per compute unit, but not on a cylinder).
static const LaunchTime BP_TIMES[BP_NSHAPES] = {{1.35, 0.46, 0.5, 1.0}, {1.0, 0.30, 0.5, 1.0}, {1.15, 0.35, 0.5, 1.0}, {0.7, 0.21, 0.5, 1.0},
                                                {1.18, 0.33, 0.5, 1.0}, {1.85, 0.62, 0.5, 1.0}, {1.35, 0.42, 0.5, 1.0}};
static const LaunchTime BP_PAIR_TIMES[BP_NPAIR_SHAPES] = {{1.35, 0.55, 1.0}, {1.4, 0.58, 1.0}, {0.9, 0.27, 1.0}, {1.35, 0.59, 1.0}};
static const LaunchTime BP_SPLIT_TIMES[2][BP_NSPLIT_SHAPES] = {{{0.42, 0.43, 4.0}, {0.29, 0.24, 4.0}, {0.24, 0.20, 4.0}},
                                                               {{0.56, 0.56, 4.0}, {0.34, 0.34, 4.0}, {0.29, 0.29, 4.0}}};
constexpr double BACK_MOST_FLOATS = 16777216.0;      // room for the volumes of parts, at most 64 MiB
constexpr int BP_FEW_VIEWS = 4;        // fewer leave a launch little but its start and end: 10 to 12 us whichever the kernel

static int tile_chunks(const leap_geometry *G, int zc, int kfirst = 0)
{
    return ((G->g.nx + BP_T - 1) / BP_T) * ((G->g.ny + BP_T - 1) / BP_T) * ((G->g.nz - kfirst + zc - 1) / zc);
}

// Two items per workgroup where there are workgroups enough (the bits are the same): eight volumes, 60 views, one by one / in twos, us: 32
// voxels per thread 64^3 (128 workgroups of two) 145 / 195, 96^3 (432) 209 / 193; wide windows 64^3 (256) 202 / 230, 96^3 (864) 419 / 434,
// 128^3 (2048) 890 / 742.
int leap_back_pairs(const leap_geometry *G, int items)
{
    if (G->bp_pair_shape < 0) return 0;
    if (G->bp_mirror) return items;
    if (G->bp_pair_forced) return items / 2;
    const SfBpShape S = BP_PAIR_SHAPES[G->bp_pair_shape];
    const int chunks = tile_chunks(G, S.zc), views = G->g.nviews;
    if (chunks * (items / 2) < (S.pw > 32 ? 1200 : 400) || views < BP_FEW_VIEWS) return 0;
    // (an odd last item is a launch of its own: one more than the two would save where a launch is a few rounds of workgroups)
    const double twos = launch_time(BP_PAIR_TIMES[G->bp_pair_shape], (double)chunks * (items / 2), views);
    if (items % 2 && twos + launch_time(BP_TIMES[G->bp_shape], chunks, views) > 0.93 * launch_time(BP_TIMES[G->bp_shape], (double)chunks * items, views)) return 0;
    return items / 2;
}

// Launches that leave the chip idle: four groups of threads share the views.  A step from view to view takes a workgroup of 256 threads
// much the same time until there are two or three per compute unit, so four groups beside each other save up to three quarters of it;
// but a workgroup of 1024 threads fills a compute unit, and short chunks stage more rows per voxel.  One volume takes the shape of least
// time by its workgroups and views; a batch takes that one too (its items then come out the same bits as alone) as long as it is a gain,
// then another that is, then none.  60 views, us, unsplit / 8 / 16 / 32 voxels: mirror image 64^3 138 / 41 / 53 / 79, four of them 138 / 44 /
// 54 / 79, sixteen 175 / 161 / 119 / 105; off centre 96^3 138 / 55 / 46 / 61, sixteen 373 / 583 / 370 / 308; 16 items of one view 96^3 26 /
// 66 / 60 / 57.  (Lines by the workgroups of one volume alone, whatever the batch and the views, had 580 of 4260 launches of 24^3 to
// 192^3, 1 to 16 items, 1 to 180 views above 1.035 times the unsplit time, up to 2.6.)
static double back_unsplit_time(const leap_geometry *G, int items)
{
    const int views = G->g.nviews, kfirst = G->bp_mirror ? sf_mirror_first_voxel_above(G->g.nz) : 0;
    const int pairs = leap_back_pairs(G, items), left = G->bp_mirror && pairs ? 0 : items - 2 * pairs;
    double unsplit = 0.0;
    if (pairs) unsplit += launch_time(BP_PAIR_TIMES[G->bp_pair_shape], (double)tile_chunks(G, BP_PAIR_SHAPES[G->bp_pair_shape].zc, kfirst) * pairs, views);
    if (left) unsplit += launch_time(BP_TIMES[G->bp_shape], (double)tile_chunks(G, BP_SHAPES[G->bp_shape].zc) * left, views);
    return unsplit;
}

static double back_split_time(const leap_geometry *G, int sh, int items, int parts)
{
    const int views = (G->g.nviews + parts - 1) / parts, kfirst = G->bp_mirror ? sf_mirror_first_voxel_above(G->g.nz) : 0;
    const int twos = leap_back_split_pairs(G, items), ones = G->bp_mirror ? 0 : items - 2 * twos;
    const double chunks = (double)tile_chunks(G, BP_SPLIT_SHAPES[sh].zc, kfirst) * parts, wider = BP_SPLIT_SHAPES[sh].pw > 32 && G->bp_need_w > 31 ? 1.25 : 1.0;
    return wider * ((twos ? launch_time(BP_SPLIT_TIMES[1][sh], chunks * twos, views) : 0.0) +
                    (ones ? launch_time(BP_SPLIT_TIMES[G->g.type == SF_CONE_CURVED][sh], chunks * ones, views) : 0.0));
}

int leap_back_split_shape(const leap_geometry *G, int items)
{
    if (!G->bp_split_fits || (G->g.nviews < BP_FEW_VIEWS && !G->bp_split_forced)) return -1;
    const double unsplit = 0.93 * back_unsplit_time(G, items);       // (a clear gain: the times are good to some five per cent)
    auto time_of = [&](int sh) { return back_split_time(G, sh, items, 1); };
    if (G->bp_split_shape >= 0 && (G->bp_split_forced || time_of(G->bp_split_shape) < unsplit)) return G->bp_split_shape;
    if (G->bp_split_shape < 0 && items > 1) return -1;
    int best = -1;
    double least = unsplit;
    for (int sh = 0; sh < BP_NSPLIT_SHAPES; ++sh)
        if ((G->bp_split_fits >> sh & 1u) && time_of(sh) < least) {
            least = time_of(sh);
            best = sh;
        }
    return best;
}

// Workgroups that share the views, each with sums of its own: a volume of a few tiles leaves most compute units without a workgroup however
// its views are shared within one, and has views enough for all of them.  The parts' volumes are added by a kernel of their own, which costs
// a launch and their traffic.  The same estimate decides, by shapes and up to 32 parts of at least eight views each; a batch takes what one
// volume takes as long as that is a gain.  us, before / in parts: 57 x 65 x 37, 310 views 274 / 79; 58 x 57 x 28, 626 views 533 / 78; 142 x 148 x
// 108, 677 parallel views 1265 / 1083; 81 x 66 x 67, 53 views 45 / 36.
// without: the time of the launch as it is else; split_time(shape, items, parts); both in units of `unit` us.
template <class SplitTime>
static LeapBackParts choose_parts(const leap_geometry *G, int items, int nshapes, double without, double unit, SplitTime split_time)
{
    const size_t nvol = (size_t)G->g.nx * G->g.ny * G->g.nz;
    const LeapBackParts none = {-1, 1, items};
    auto time_of = [&](int sh, int parts, int at_once) {
        const double launches = std::ceil((double)items / at_once);
        return launches * (split_time(sh, std::min(items, at_once), parts) + 5.0 / unit) + (parts + 1.0) * items * 4.0 * (double)nvol / (2.5e6 * unit);
    };
    if (items > 1) {
        if (G->bp_parts == 1) return none;
        const int at_once = (int)std::min<size_t>(items, G->back_floats / (nvol * G->bp_parts));
        return at_once >= 1 && time_of(G->bp_parts_shape, G->bp_parts, at_once) < 0.93 * without ? LeapBackParts{G->bp_parts_shape, G->bp_parts, at_once} : none;
    }
    if (G->bp_parts > 1) return {G->bp_parts_shape, G->bp_parts, 1};
    LeapBackParts best = none;
    double least = 0.85 * without;
    for (int sh = 0; sh < nshapes; ++sh)
        for (const int parts : {2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32})
            if ((G->bp_parts_fits >> sh & 1u) && G->g.nviews >= 8 * parts && (double)nvol * parts <= BACK_MOST_FLOATS && time_of(sh, parts, 1) < least) {
                least = time_of(sh, parts, 1);
                best = {sh, parts, 1};
            }
    return best;
}

LeapBackParts leap_back_parts(const leap_geometry *G, int items)
{
    if (!G->bp_parts_fits || G->bp_split_forced) return {-1, 1, items};
    const int split = leap_back_split_shape(G, items);
    return choose_parts(G, items, BP_NSPLIT_SHAPES, split >= 0 ? back_split_time(G, split, items, 1) : back_unsplit_time(G, items), 2.8,
                        [&](int sh, int n, int parts) { return back_split_time(G, sh, n, parts); });
}

// Tiled back projection, two volumes per workgroup: the shapes that leave the chip enough workgroups.
static std::vector<int> backproject_pair_shapes(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    std::vector<int> shapes;
    if (G->bp_nv > 3 || d->type == LEAP_MODULAR) return shapes;
    G->bp_mirror = mirrored_about_source_plane(G);
    const long only = back_option("bp_pair");
    if (only == -1) return shapes;
    const int kfirst = G->bp_mirror ? sf_mirror_first_voxel_above(d->nz) : 0;
    const int tiles = ((d->nx + BP_T - 1) / BP_T) * ((d->ny + BP_T - 1) / BP_T);
    for (int sh = 0; sh < BP_NPAIR_SHAPES; ++sh) {
        const SfBpShape S = BP_PAIR_SHAPES[sh];
        if ((only >= 0 && sh != only) || !bp_pair_instance_exists(G->bp_nc, G->bp_nv, sh)) continue;
        // Mirror image, parallel beams, 120 views, one volume / 32 + 32 / 16 + 16 voxels per thread: 256^3 (1024 workgroups of the
        // larger) 693 / 552 / 648 us, 224^3 (784) 689 / 537 / 534, 192^3 (432) 479 / 375 / 358, 160^3 (300; 500 of the smaller) 476 /
        // 372 / 257, 128^3 (256 of the smaller) 465 / 378 / 262, 112^3 280 / 379 / 261, 64^3 267 / 369 / 247.
        // Wide windows leave room for 768 workgroups: 60 views, one volume under 64 columns and 16 voxels / 51 columns and 16 + 16 voxels, us:
        // 128^3 (256 workgroups) 196 / 229, 160^3 (500) 260 / 243; a second round nearly empty is none (192^3, 864 workgroups).
        const int workgroups = tiles * ((d->nz - kfirst + S.zc - 1) / S.zc);
        const bool enough = S.pw <= 32 ? workgroups >= (S.zc == 32 ? 800 : 250) : 10 * workgroups >= 6 * 768 * ((workgroups + 767) / 768);
        if (G->bp_mirror && only < 0 && !enough) continue;
        shapes.push_back(sh);
    }
    return shapes;
}

// The general kernel instead, and none of the choices that go with the tiled ones.
static void no_tiled_back_projection(leap_geometry *G)
{
    G->bp_tiled = G->bp_mirror = G->bp_pair_forced = G->bp_split_forced = false;
    G->bp_pair_shape = G->bp_split_shape = G->bp_parts_shape = -1;
    G->bp_parts = 1;
    G->bp_split_fits = G->bp_parts_fits = 0;
}

// Footprint model, tiled back projection: pick the template instance and verify its staged window.
static void select_footprint_tiled(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    if (d->type == LEAP_FAN || d->nz < 8 || !std::isfinite(G->max_cols_per_voxel) || G->max_cols_per_voxel > 4.0 ||
        G->max_rows_per_voxel > 3.0 || !((double)d->nrows * d->ncols < 1073741824.0))     // 32-bit byte offsets within a view
        return;
    // Cylinder: the tiled kernel takes the angle between a voxel's centre and its corners from a short series,
    // good to 3e-9 rad below 0.08 rad.
    if (d->type == LEAP_CONE_CURVED) {
        const double rx = std::fabs(d->center_x) + 0.5 * d->nx * d->voxel_xy, ry = std::fabs(d->center_y) + 0.5 * d->ny * d->voxel_xy;
        const double nearest = d->sod - std::sqrt(rx * rx + ry * ry);
        if (!(0.7072 * d->voxel_xy <= 0.08 * nearest)) return;
    }
    G->bp_nc = std::max(2, (int)std::ceil(G->max_cols_per_voxel) + 1);
    // rows a voxel can touch; the three-row instance runs schemes that need every voxel at most two rows tall, so a
    // bound that close to two rows takes the four-row instance
    const double mr = G->max_rows_per_voxel;
    G->bp_nv = mr <= 1.0 + 1e-6 ? 2 : (mr <= 1.999 ? 3 : std::max(4, (int)std::ceil(mr - 1e-6) + 1));
    G->bp_wh = (float)(0.5 * G->max_cols_per_voxel);
    const float hx = 0.5f * (float)(BP_T - 1) * G->g.T;
    // 64-voxel chunks only pay off on tall volumes; the two-row instances keep 64 sums in registers in either 64-voxel
    // shape, the three-row instances in the tall one only
    int order[BP_NSHAPES], norder = 0;
    if (d->nz >= 128 && G->bp_nv == 2) order[norder++] = 0;
    if (d->nz >= 128 && G->bp_nv <= 3) order[norder++] = BP_TALL_SHAPE;
    // The wide window's 32 voxels per thread: for voxels of up to a row and a half (taller ones are limited by LDS reads), where
    // it leaves the chip's 256 compute units 700 workgroups and no more than a fifth of the layers as padding.  60 views, 16 voxels'
    // time over 32's: 500 to 605 workgroups 0.87 to 1.13 (below 1 on flat detectors), 720 to 845 1.12 to 1.35, 1092 0.98 to 1.12, 1280 to
    // 2048 1.04 to 1.34.
    const int tiles = ((d->nx + BP_T - 1) / BP_T) * ((d->ny + BP_T - 1) / BP_T), chunks32 = (d->nz + 31) / 32;
    const bool wide = G->bp_nv <= 3 && mr <= 1.5 && (G->bp_nc == 3 || G->bp_nc == 4) && tiles * chunks32 >= 700 && 160 * chunks32 <= 6 * d->nz;
    for (int sh = BP_FIRST_SHORT_SHAPE; sh <= BP_LAST_SHORT_SHAPE; ++sh) {
        if (wide && sh == 3) order[norder++] = BP_WIDE_SHAPE;        // before the 16-voxel shapes
        order[norder++] = sh;
    }
    long forced;
    if (debug_option("bp_shape", forced)) {        // start at a given shape, then the short ones after it
        forced = ((forced % BP_NSHAPES) + BP_NSHAPES) % BP_NSHAPES;
        norder = 0;
        if (bp_instance_exists(G->bp_nc, G->bp_nv, (int)forced)) order[norder++] = (int)forced;
        for (int sh = std::max((int)forced + 1, BP_FIRST_SHORT_SHAPE); sh <= BP_LAST_SHORT_SHAPE; ++sh) order[norder++] = sh;
    }
    // One volume per workgroup and two: the first shape of either kind that fits, a pair of shapes per pass over the tiles.  Two items of a
    // batch take chunks of the same height as one, so that going in twos changes no item's bits: known when one's shape is.
    const std::vector<int> pair_shapes = backproject_pair_shapes(G);
    const int kfirst = G->bp_mirror ? sf_mirror_first_voxel_above(d->nz) : 0;
    std::vector<WindowNeed> known;               // by height and first chunk: shapes of one height share theirs
    auto need_of = [&](int zc, int from) {
        return std::find_if(known.begin(), known.end(), [&](const WindowNeed &k) { return k.zc == zc && k.kfirst == from; });
    };
    auto look_at = [&](std::vector<WindowNeed> needs) {
        if (needs.empty()) return;
        staged_window_needs(G, needs,
                            [&](const SfGeom &ga, const SfView &v, float xc, float yc, SfWindow &w) {
                                const SfTileBounds b = sf_bp_tile_bounds(ga, v, xc, yc, hx);
                                sf_bp_window_columns(b, G->bp_wh, G->bp_nc, w.c0, w.need_w);
                                return b;
                            },
                            [&](const SfGeom &ga, const SfTileBounds &b, float z0, float z1, SfWindow &w) {
                                sf_bp_window_rows(ga, b, z0, z1, G->bp_nv, w.r0, w.need_h);
                            });
        known.insert(known.end(), needs.begin(), needs.end());
    };
    for (size_t n = 0, p = 0;;) {
        std::vector<WindowNeed> needs;
        const bool single = n < (size_t)norder && !G->bp_tiled;
        if (!G->bp_mirror)
            while (!single && p < pair_shapes.size() && BP_PAIR_SHAPES[pair_shapes[p]].zc != BP_SHAPES[G->bp_shape].zc) ++p;
        const bool pair = p < pair_shapes.size() && G->bp_pair_shape < 0 && (single ? G->bp_mirror : G->bp_tiled);
        if (!single && !pair) break;
        const int single_zc = single ? BP_SHAPES[order[n]].zc : 0, pair_zc = pair ? BP_PAIR_SHAPES[pair_shapes[p]].zc : 0;
        if (single && need_of(single_zc, 0) == known.end()) needs.push_back({single_zc, 0});
        if (pair && need_of(pair_zc, kfirst) == known.end()) needs.push_back({pair_zc, kfirst});
        look_at(needs);
        if (single) {
            const WindowNeed &need = *need_of(single_zc, 0);
            G->bp_need_w = need.w;
            G->bp_need_h = need.h;
            G->bp_shape = order[n];
            G->bp_tiled = window_fits(need, BP_SHAPES[order[n]]);
            ++n;
        }
        if (pair) {
            if (window_fits(*need_of(pair_zc, kfirst), BP_PAIR_SHAPES[pair_shapes[p]])) G->bp_pair_shape = pair_shapes[p];
            ++p;
        }
    }
    G->bp_pair_forced = back_option("bp_pair") >= 0;
    // Where the 42-column window and its 32 voxels do, 16 + 16 under 51 columns are no gain.  42 columns / mirror image, 60 views, ratio, 256^3,
    // three and eight of them, 256 x 256 x 128: rows of 0.85 voxels (voxels of up to 1.4 rows) 0.98, 1.03 and 1.14, of 1.05 1.02, 1.04 and
    // 1.17, of 1.25 1.03, 1.07 and 1.18, of 1.4 1.08, 1.11 and 1.22; 224^3 0.89 to 1.00, three of them 1.01 to 1.12.
    if (G->bp_mirror && G->bp_tiled && G->bp_shape == BP_WIDE_SHAPE && !G->bp_pair_forced) G->bp_pair_shape = -1;
    // Four groups of threads that share the views: the shapes whose windows fit, where one volume would take any of them.
    const long only = back_option("bp_split");
    if (G->bp_tiled && G->bp_nv <= 3 && only != -1) {
        const int wide = known.front().w;
        auto exists = [&](int sh) { return bp_split_instance_exists(G->bp_nc, G->bp_nv, sh) && wide <= BP_SPLIT_SHAPES[sh].pw - 1 && (only < 0 || only == sh); };
        unsigned candidates = 0;
        for (int sh = 0; sh < BP_NSPLIT_SHAPES; ++sh) candidates |= exists(sh) ? 1u << sh : 0u;
        G->bp_split_fits = candidates;
        long want = -1;
        debug_option("bp_parts", want);
        G->bp_parts_fits = only < 0 && want != 1 ? candidates : 0u;
        if (only >= 0 || leap_back_split_shape(G, 1) >= 0 || leap_back_parts(G, 1).parts > 1) {
            std::vector<WindowNeed> needs;
            for (int sh = 0; sh < BP_NSPLIT_SHAPES; ++sh)
                if ((candidates >> sh & 1u) && need_of(BP_SPLIT_SHAPES[sh].zc, kfirst) == known.end()) needs.push_back({BP_SPLIT_SHAPES[sh].zc, kfirst});
            look_at(needs);
            for (int sh = 0; sh < BP_NSPLIT_SHAPES; ++sh)
                if ((candidates >> sh & 1u) && !window_fits(*need_of(BP_SPLIT_SHAPES[sh].zc, kfirst), BP_SPLIT_SHAPES[sh])) G->bp_split_fits &= ~(1u << sh);
            G->bp_parts_fits &= G->bp_split_fits;
            G->bp_split_forced = only >= 0 && G->bp_split_fits != 0;
            G->bp_split_shape = G->bp_split_forced ? (int)only : leap_back_split_shape(G, 1);
            const LeapBackParts plan = leap_back_parts(G, 1);
            G->bp_parts_shape = plan.shape;
            G->bp_parts = plan.parts;
        }
        if (G->bp_split_shape < 0) G->bp_split_fits = 0;
        if (G->bp_parts == 1) G->bp_parts_fits = 0;
    }
    if (!G->bp_tiled) no_tiled_back_projection(G);
}

// Row groups per wave of the column-wise forward kernels.  A wave pays a fixed share per candidate voxel column (its
// parameters, the transaxial record) worth about a group and a half, then one share per group whether or not the group
// holds rows of the detector; the detector needs ceil(groups / rg) bands of waves.
static int row_groups(int nrows, int rows_per_group, const int *choices, int nchoices)
{
    const int groups = (nrows + rows_per_group - 1) / rows_per_group;
    int best = choices[0];
    double best_cost = 1e300;
    for (int n = 0; n < nchoices; ++n) {
        const int rg = choices[n], bands = (groups + rg - 1) / rg;
        const double cost = bands * (1.6 + rg);
        if (cost < best_cost - 1e-9) { best_cost = cost; best = rg; }
    }
    long v;
    if (debug_option("rg", v))
        for (int n = 0; n < nchoices; ++n)
            if (choices[n] == v) best = (int)v;
    return best;
}

static void block_order_options(leap_geometry *G)
{
    long v;
    if (debug_option("vb", v) && v >= 1 && v <= 1024) G->fp_vb = (int)v;
    if (debug_option("tb", v) && v >= 1 && v <= 1024) G->fp_tb = (int)v;
}

// Two volumes to a wave halve a launch's waves and take more registers: worth it where enough workgroups are left, and the launch of
// its own that an odd last item takes must fill the chip too.  Times of two over one per wave, by workgroups of two volumes: one group
// of rows 20 to 600 1.15 to 0.92, 700 and more 0.66 to 1.02; two groups 20 to 700 1.20 to 0.94, 1000 and more 0.84 to 1.06; three groups,
// four workgroups per compute unit, 1020, 2040 and 3060 0.78 to 0.87, but 1380 and 2200 (a last round nearly empty) 1.06 to 1.08, 3000
// and more 0.83 to 0.92; cylinder 1000 and more 0.65 to 0.95.  Batches of three, by workgroups of one volume: one group 20 to 720 1.98 to
// 1.38, 900 to 1400 0.92 to 1.13, 1600 and more 0.88 to 1.00; several groups 20 to 2800 1.99 to 0.94, 4000 and more 0.94 to 1.00.  An item's
// bits are the same either way.
// Those are of a wave per bundle.  Where four waves share one (forward_parts) a launch has four times the waves, and two volumes would pay before
// these lines: by workgroups as they are counted here, one group of rows, even batches up to 100 0.84 to 1.07, 100 to 200 0.67 to 1.02, 200 to 700 0.64
// to 0.87, above 0.62 to 0.82; odd ones 1.28 to 1.64, 1.11 to 1.36, 200 to 400 0.85 to 1.20, 400 to 700 0.89 to 1.05, above 0.77 to 0.99.
int leap_forward_paired(const leap_geometry *G, int items)
{
    if (!G->fp_pair_rg || items < 2) return 0;
    if (G->fp_pair_always) return items / 2 * 2;
    const int groups = G->fp_pair_rg;
    const double blocks = (double)((G->g.ncols + FP_WAVES * G->fp_cw - 1) / (FP_WAVES * G->fp_cw)) * G->g.nviews *
                          ((G->g.nrows + groups * 128 - 1) / (groups * 128));
    const double launch = blocks * (items / 2), rounds = launch / 1024.0;
    if (launch < (groups == 1 ? 700.0 : 900.0)) return 0;
    if (groups > 2 && G->g.type != SF_CONE_CURVED && launch < 3000.0 && rounds < 0.88 * std::ceil(rounds)) return 0;
    if (items % 2 && blocks < (groups == 1 ? 1600.0 : 4000.0)) return 0;
    return items / 2 * 2;
}

// Waves of a workgroup that share a bundle's layers: where a volume has too few bundles to keep the chip's 1024 SIMDs supplied with
// waves, each waiting for its own loads most of the time.  By the waves of one volume (its views, bundles and bands of rows), us for one
// volume and for four at once, a wave per bundle -> four: cone 500 66 -> 34, 80 -> 59; 1350 200 -> 85, 267 -> 228; 2010 371 -> 177, 534 ->
// 454; 2700 82 -> 54, 124 -> 107; 4020 133 -> 96, 258 -> 245; 5400 202 -> 174, 405 -> 428; 8040 436 -> 414, 1135 -> 1340; 10700 131 -> 128,
// 309 -> 333.  Parallel beams by rows: 2040 55 -> 35, 97 -> 92; 2700 69 -> 46, 128 -> 133 (two waves 54, 127); 5400 183 -> 151, 447 -> 518.
// The sums are added in another order, so the choice depends on the scan alone: an item has the same bits in any batch.
static int forward_parts(const leap_geometry *G, int nbundles)
{
    const leap_geometry_desc *d = &G->desc;
    if (G->fp_cw < 2) return 1;
    const int band = G->fp_rows ? G->fp_row_groups * 64 * G->fp_rows : G->fp_rg * 128;
    const double waves = (double)d->nviews * nbundles * ((d->nrows + band - 1) / band);
    int parts = waves <= 4500.0 ? FP_PARTS : 1;
    if (G->fp_rows && waves > 2200.0) parts = std::min(parts, 2);
    long v;
    if (debug_option("parts", v) && (v == 1 || v == FP_PARTS || (v == 2 && G->fp_rows))) parts = (int)v;
    return parts;
}

// Footprint model, column-wise forward projection: static limits and the marching axis of every bundle.
static void select_footprint_columns(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    const double vpr = G->max_voxels_per_row;
    if (d->type == LEAP_FAN || d->nrows < FP_MIN_ROWS || !std::isfinite(vpr) || vpr > 3.0) return;
    // kappa (the axial voxel coordinate of a row's edge) must stay within +-2^19 for the kernel's placement arithmetic
    if (!((d->nrows + 1024.0) * vpr + d->nz + 64.0 < 500000.0)) return;
    long v;
    G->fp_cw = 4;
    // Short detectors (fewer than about 200 rows) have too few bundles of four to fill the chip: two columns measured
    // 5 to 12 % faster there.  The cylinder's record phase is heavier: four columns only pay off from about 450 rows on.
    if (d->nrows <= 192 || (d->type == LEAP_CONE_CURVED && d->nrows <= 448)) G->fp_cw = 2;
    const bool forced_cw = debug_option("cw", v) && (v == 1 || v == 2 || v == 4);
    if (forced_cw) G->fp_cw = (int)v;
    if (d->type != LEAP_CONE && d->type != LEAP_PARALLEL && G->fp_cw == 1) G->fp_cw = 2;   // instances of 4 and 2 columns only
    // candidate slots per slab: widest range of voxel columns any bundle of cw detector columns can see
    auto slots_needed = [&](int cw) {
        int need = 0;
        for (int a = 0; a < d->nviews && need <= 16; ++a)
            for (int c = 0; c < d->ncols; c += cw) {
                const SfRayLines L = sf_ray_lines(view_geom(G, a), G->views[a], c, cw);
                const int n_major = L.xmajor ? d->nx : d->ny;
                const float d0 = std::fabs(L.b0 - L.b1);
                const float d1 = std::fabs(fmaf(L.m0 - L.m1, (float)(n_major - 1), L.b0 - L.b1));
                const float dm = d0 > d1 ? d0 : d1;
                if (!(dm < 1e6f)) return 1 << 20;
                need = std::max(need, (int)std::floor(dm + 2.0f * L.spread + 1e-3f) + 2);
            }
        return need;
    };
    int need = slots_needed(G->fp_cw);
    const int cw_min = (d->type == LEAP_CONE || d->type == LEAP_PARALLEL) ? 1 : 2;
    while (need > 16 && G->fp_cw > cw_min) {
        G->fp_cw /= 2;
        need = slots_needed(G->fp_cw);
    }
    // cylinder: a candidate's fan angle is taken from its bundle's middle ray (detectors of a few dozen columns can be too coarse for that)
    if (d->type == LEAP_CONE_CURVED) {
        while (G->fp_cw > cw_min && sf_bundle_reach(G->fp_cw, G->max_cols_per_voxel) / G->g.kud >= std::atan(SF_ATAN_MAX)) need = slots_needed(G->fp_cw /= 2);
        if (!(sf_bundle_reach(G->fp_cw, G->max_cols_per_voxel) / G->g.kud < std::atan(SF_ATAN_MAX))) return;
    }
    G->fp_need_q = need;
    G->fp_nq = need <= 4 ? 4 : (need <= 8 ? 8 : 16);
    G->fp_nkp = std::min(FP_MAX_P, std::max(2, (int)std::ceil(2.0 * vpr - 1e-6) + 1));
    static const int pair_groups[] = {1, 2, 3, 4};
    G->fp_rg = row_groups(d->nrows, 128, pair_groups, 4);
    G->fp_columns = need <= 16;
    block_order_options(G);
    if (!G->fp_columns) return;
    v = -1;
    debug_option("pairs", v);
    const int pair_rg = G->fp_rg == 4 ? 2 : G->fp_rg;
    if (v != 0 && fp_instance_exists(fp_height_class(G->fp_nkp), pair_rg, G->fp_cw, d->type == LEAP_CONE_CURVED ? 1 : (d->type == LEAP_MODULAR ? 2 : 0), 2))
        G->fp_pair_rg = pair_rg;
    G->fp_pair_always = v > 0;
    // Parallel beams: the axial overlaps go into the slab copy and a wave's lanes own adjacent rows, as many as it takes for
    // one wave to hold the detector's height, up to 512 rows.  Only where the copy by rows of the whole volume fits either
    // scratch (up to 256^3): a detector of many more rows than the volume has layers would otherwise take narrower slabs.
    const double n_side = std::max(d->nx, d->ny);
    if (d->type == LEAP_PARALLEL && G->fp_cw >= 2 &&
        4.0 * (n_side * n_side + 1.0) * ((d->nrows + 3) / 4 * 4 + 2 * FP_PAD) <= (double)LEAP_STATIC_SCRATCH_BYTES) {
        G->fp_rows = d->nrows <= 64 ? 1 : (d->nrows <= 128 ? 2 : 4);
        G->fp_row_groups = d->nrows > 256 ? 2 : 1;
    }
    const int nbundles = (d->ncols + G->fp_cw - 1) / G->fp_cw;
    G->fp_parts = forward_parts(G, nbundles);
    G->major.resize((size_t)d->nviews * nbundles);
    for (int a = 0; a < d->nviews; ++a)
        for (int b = 0; b < nbundles; ++b)
            G->major[(size_t)a * nbundles + b] = (unsigned char)sf_ray_lines(view_geom(G, a), G->views[a], b * G->fp_cw, G->fp_cw).xmajor;
}

// Footprint model, scans of one detector row and one voxel layer: limits of the flat kernels (sf_flat.h) in both
// directions.  Wider footprints, coarser detectors and beams that fan out too far stay with the general kernels.
static void select_footprint_flat(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    const SfGeom &g = G->g;
    if (!(d->type == LEAP_FAN || (d->type == LEAP_PARALLEL && d->nrows == 1 && d->nz == 1))) return;
    // a launch holds fewer than 2^32 threads, and the forward kernel needs a wave per view and tile of 64 columns
    if (!((double)flat_tiles(d->ncols, d->nviews) * d->nviews * 64.0 < 4294967296.0)) return;
    // widest footprint of any voxel, on the detector or beside it (footprint_bounds looks at the detector's fan only)
    const double rx = std::fabs(d->center_x) + 0.5 * d->nx * d->voxel_xy, ry = std::fabs(d->center_y) + 0.5 * d->ny * d->voxel_xy;
    const double reach = std::sqrt(rx * rx + ry * ry);
    double widest = d->voxel_xy * std::sqrt(2.0) / d->pixel_u;
    if (d->type == LEAP_FAN) widest *= d->sdd / (d->sod - reach) / std::sqrt(1.0 - (reach / d->sod) * (reach / d->sod));
    if (!(widest <= FLAT_MAX_COLS) || !((double)d->nx * d->ny < 268435456.0)) return;       // 32-bit offsets within a slice
    int span = 0;
    for (int a = 0; a < d->nviews; ++a)
        for (int c0 = 0; c0 < d->ncols; c0 += FLAT_RAYS) {
            const int c1 = std::min(c0 + FLAT_RAYS, d->ncols) - 1;
            const int xmajor = sf_flat_xmajor(g, G->views[a], c0);
            const SfRayLines L0 = sf_ray_lines<0>(g, G->views[a], c0, 1, xmajor), L1 = sf_ray_lines<0>(g, G->views[a], c1, 1, xmajor);
            // nearly parallel beams: slopes of at most 2 and no column between the two that leaves their span
            if (!(L0.spread <= 1.0f && L1.spread <= 1.0f && std::fabs(L0.b0) < 1e6f && std::fabs(L1.b0) < 1e6f)) return;
            const int ends[2] = {0, (xmajor ? d->nx : d->ny) - 1};
            for (int n : ends) {
                int f0, l0, f1, l1;
                sf_candidates(L0, n, f0, l0);
                sf_candidates(L1, n, f1, l1);
                span = std::max(span, std::max(l0, l1) - std::min(f0, f1) + 1);
            }
        }
    span += 4;                                       // host and device floats may round apart
    if (span > FLAT_MAX_SPAN) return;
    G->flat = true;
    G->flat_span = (span + 63) / 64 * 64;
    if (d->type == LEAP_PARALLEL) {                  // the layer's overlap with the row
        const double lo = g.kvd * g.zlo0d + g.row_offd, hi = lo + g.kvd * g.Tzd;
        G->flat_fv = (float)std::fmax(std::fmin(1.0, hi) - std::fmax(0.0, lo), 0.0);
    }
}

// Siddon model, launches that leave the chip idle: four groups of threads share the views (two under 64 columns on tilted modules), by the
// launch's workgroups and views as for footprints (leap_back_split_shape); here the times are in us per view, and a round of the split
// kernels is dearer where the window of the unsplit shape is larger (more pixels per voxel).  us, unsplit / 16 / 8 voxels per thread, 60
// views: parallel beams 64^3 330 / 87 / 66, four of them 335 / 92 / 134, sixteen 358 / 351 / 524; 96^3 325 / 89 / 132, sixteen 1051 / 1215 /
// 1764; 128^3 328 / 176 / 264, sixteen 2158 / 2765 / 4165; eight views of 128^3 43 / 29 / 44, sixteen 280 / 430 / 666.  Tilted modules, unsplit /
// four groups: 64^3 437 / 111, sixteen 868 / 885, 128^3 460 / 432, four 1360 / 1700; 62 x 63 x 43 x 207 views 1796 / 422; where the window
// leaves a compute unit one workgroup of 256 threads, 135 x 140 x 148 x 156 views 5598 / 1986, or two groups of threads 165 x 164 x 79 x 58 2440
// / 1216, 234 x 196 x 225 x 206 22998 / 13630.
static const LaunchTime SD_BP_TIMES[BP_LAST_SHORT_SHAPE + 1] = {{}, {4.8, 1.95, 0.5}, {6.2, 3.25, 0.5}, {5.2, 2.05, 0.5}, {5.1, 2.05, 0.5}};
static const double SD_BP_SPLIT_TIMES[BP_LAST_SHORT_SHAPE + 1][SD_BP_NSPLIT_SHAPES] = {{}, {1.3, 1.07}, {1.7, 1.45}, {1.95, 1.68}, {2.0, 1.45}};
static const LaunchTime MD_BP_TIMES[MD_BP_NSHAPES] = {{6.9, 2.35, 0.5}, {8.5, 2.95, 0.5}, {14.0, 9.0, 0.5}, {10.0, 5.0, 0.5}, {18.0, 17.0, 0.5}, {12.4, 12.0, 0.5}};
static const double MD_BP_SPLIT_TIMES[MD_BP_NSHAPES][MD_BP_NSPLIT_SHAPES] = {{1.65, 2.5, 2.7}, {1.9, 2.9, 3.1}, {2.2, 3.4, 3.6}, {2.2, 3.4, 3.6}, {2.2, 3.4, 3.6}, {2.2, 3.4, 3.6}};

static double siddon_unsplit_time(const leap_geometry *G, int items)
{
    const bool tilted = G->g.type == SF_MODULAR && G->geoms.empty();
    const SfBpShape &S = tilted ? MD_BP_SHAPES[G->bp_shape] : BP_SHAPES[G->bp_shape];
    return launch_time(tilted ? MD_BP_TIMES[G->bp_shape] : SD_BP_TIMES[G->bp_shape], (double)tile_chunks(G, S.zc) * items, G->g.nviews);
}

static double siddon_split_time(const leap_geometry *G, int sh, int items, int parts)
{
    const bool tilted = G->g.type == SF_MODULAR && G->geoms.empty();
    const SfBpShape &S = tilted ? MD_BP_SPLIT_SHAPES[sh] : SD_BP_SPLIT_SHAPES[sh];
    const double round = tilted ? MD_BP_SPLIT_TIMES[G->bp_shape][sh] : SD_BP_SPLIT_TIMES[G->bp_shape][sh];
    return launch_time({round, round, 3.0}, (double)tile_chunks(G, S.zc) * items * parts, (G->g.nviews + parts - 1) / parts);
}

int leap_siddon_split_shape(const leap_geometry *G, int items)
{
    if (!G->bp_split_fits) return -1;
    if (G->bp_split_shape >= 0 && G->bp_split_forced) return G->bp_split_shape;
    if (G->g.nviews < 2 || (G->bp_split_shape < 0 && items > 1)) return -1;
    const bool tilted = G->g.type == SF_MODULAR && G->geoms.empty();
    const double unsplit = 0.93 * siddon_unsplit_time(G, items);
    auto time_of = [&](int sh) { return siddon_split_time(G, sh, items, 1); };
    if (G->bp_split_shape >= 0 && time_of(G->bp_split_shape) < unsplit) return G->bp_split_shape;
    int best = -1;
    double least = unsplit;
    for (int sh = 0; sh < (tilted ? MD_BP_NSPLIT_SHAPES : SD_BP_NSPLIT_SHAPES); ++sh)
        if ((G->bp_split_fits >> sh & 1u) && time_of(sh) < least) {
            least = time_of(sh);
            best = sh;
        }
    return best;
}

// The views shared among workgroups, as for footprints; times in us.  us, before / in parts: cone 62 x 51 x 44, 455 views 604 / 281; parallel 70 x
// 76 x 37, 389 views 415 / 179; tilted modules 50 x 40 x 23, 248 views 521 / 114, and where an unsplit workgroup's window fills a compute unit,
// 190 x 172 x 92, 206 views 11030 / 5780.
LeapBackParts leap_siddon_parts(const leap_geometry *G, int items)
{
    if (!G->bp_parts_fits || G->bp_split_forced) return {-1, 1, items};
    const int split = leap_siddon_split_shape(G, items);
    return choose_parts(G, items, G->g.type == SF_MODULAR && G->geoms.empty() ? MD_BP_NSPLIT_SHAPES : SD_BP_NSPLIT_SHAPES,
                        split >= 0 ? siddon_split_time(G, split, items, 1) : siddon_unsplit_time(G, items), 1.0,
                        [&](int sh, int n, int parts) { return siddon_split_time(G, sh, n, parts); });
}

// The shapes that fit (fits(shape): their windows do) and the one a single volume takes.
template <class FitsFn>
static void choose_siddon_split(leap_geometry *G, int nshapes, FitsFn fits)
{
    const long only = back_option("bp_split");
    if (only == -1) return;
    for (int sh = 0; sh < nshapes; ++sh)
        if (only < 0 || only == sh) G->bp_split_fits |= 1u << sh;
    long want = -1;
    debug_option("bp_parts", want);
    G->bp_parts_fits = only < 0 && want != 1 ? G->bp_split_fits : 0u;
    const bool parts = leap_siddon_parts(G, 1).parts > 1;
    if (!parts) G->bp_parts_fits = 0;
    if (only < 0 && !parts && leap_siddon_split_shape(G, 1) < 0) G->bp_split_fits = 0;
    for (int sh = 0; sh < nshapes; ++sh)
        if ((G->bp_split_fits >> sh & 1u) && !fits(sh)) G->bp_split_fits &= ~(1u << sh);
    G->bp_parts_fits &= G->bp_split_fits;
    G->bp_split_forced = only >= 0 && G->bp_split_fits;
    G->bp_split_shape = G->bp_split_forced ? (int)only : leap_siddon_split_shape(G, 1);
    const LeapBackParts plan = leap_siddon_parts(G, 1);
    G->bp_parts_shape = plan.shape;
    G->bp_parts = plan.parts;
    if (plan.parts == 1) G->bp_parts_fits = 0;
    if (G->bp_split_shape < 0) G->bp_split_fits = 0;
}

// Siddon model, detectors of fewer than 32 rows: does the column-wise forward projection gain on one thread per ray, which reads only the voxels the
// rays cross and copies nothing?  On circular scanners with one copy of the whole volume, at any number of views; with slabs of the volume (copied
// once for either axis) where every voxel is crossed often enough.  Modules need more rows, crossings and views: their thread-per-ray kernel
// is faster on few rays.  By a voxel's crossings (rays times slabs over voxels), column-wise over thread-per-ray: one copy, 16 to 31 rows, cone and cylinder
// of 16^3 to 256^2 x 400 voxels 0.35 to 0.9, parallel beams from 22 rows 0.4 to 0.9; slabs, cone 16 rows 2.6 (0.2 crossings), 1.3 (2), 1.08 (6), 0.98
// (18), 0.92 (22), 28 rows 2.6 (0.05), 1.1 (1.6), 0.6 (10), parallel 22 rows 3.3 (0.3), 1.3 (4), 1.05 (12), 0.87 (25); modules, one copy, 16 to 21 rows 0.7 to
// 1.5, 22 rows and more 1.5 (0.1), 1.07 (4.4), 0.6 to 0.85 from 16 on, but 1.44 with four views of 16^2 x 7 voxels; slabs 5.6 (0.1), 1.16 (4), 1.0 (12).
static bool siddon_columns_gain(const leap_geometry_desc *d)
{
    if (d->nrows >= 32) return true;
    const bool modules = d->type == LEAP_MODULAR;
    if (d->nrows < (d->type == LEAP_PARALLEL || modules ? 22 : 16)) return false;
    const double n_side = std::max(d->nx, d->ny);
    const bool whole = 4.0 * (n_side * n_side + 1.0) * (d->nz + 2.0 * FP_PAD) <= 128.0 * 1048576.0;
    if (whole && !modules) return true;
    const double crossings = (double)d->nviews * d->nrows * d->ncols * n_side / ((double)d->nx * d->ny * d->nz);
    return crossings >= 16.0 && (!modules || d->nviews >= 15);
}

// Siddon model: static limits of the two fast kernels.
static void select_siddon_fast_kernels(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    if (d->type == LEAP_FAN || !(G->sd_max_axial_slope <= 0.999)) return;

    // wave-per-column forward projection: no ray may cross more than one z-face per slab
    // (short detectors leave most lanes idle; column-wise over one thread per ray, 30 / 720 views: 256^2 x 20 voxels, 22 rows, cone 0.54 / 0.64,
    // parallel 0.79 / 0.86; 128^2 x 15, 16 rows, 0.48 / 0.72 and 0.64 / 1.07; 256^2, 8 rows 0.85 / 1.64 and 1.02 / 2.16; tilted modules at 22
    // rows 0.96 / 1.24: those from 32 rows on)
    if (siddon_columns_gain(d)) {
        G->sd_columns = true;
        static const int single_groups[] = {1, 2, 4, 8};
        G->fp_rg = row_groups(d->nrows, 64, single_groups, 4);
        // Two rows per lane where adjacent rows lie less than two voxels apart (their cells then fit one 16-byte load) and Z
        // fits the placement's fixed point.  Detectors of up to 64 rows would leave half the lanes idle: one row each.
        if (G->fp_rg >= 2 && G->sd_min_row_step > 0.0 && G->sd_max_row_step < 2.0 - 1e-6 && G->sd_max_z < 500000.0)
            G->sd_pairs = G->sd_min_row_step > 1.0 + 1e-6 ? 2 : 1;
        block_order_options(G);
    }

    // tiled back projection: at most 4 pixel centres inside a voxel's footprint, and the staged window of every
    // (view, tile, z-chunk) must fit the instance (checked with the kernel's own function)
    if (d->nz >= 8 && std::isfinite(G->max_cols_per_voxel) && G->max_cols_per_voxel > 0.0 && G->max_cols_per_voxel < 3.9 &&
        (double)d->nrows * d->ncols < 1073741824.0) {      // the staging loads use 32-bit byte offsets within a view
        G->bp_nc = std::max(2, (int)std::floor(G->max_cols_per_voxel + 0.01) + 1);
        const float hx = 0.5f * (float)BP_T * G->g.T;
        long first_shape = BP_FIRST_SHORT_SHAPE;       // the 64-voxel shapes do not fit: the sums live in LDS
        if (debug_option("bp_shape", first_shape))
            first_shape = std::min((long)BP_LAST_SHORT_SHAPE, std::max((long)BP_FIRST_SHORT_SHAPE, first_shape % BP_NSHAPES));
        struct Tile {
            const SfView *v;
            float xc, yc;
        };
        auto window_of = [&](int zc) {
            std::vector<WindowNeed> need = {{zc, 0}};
            staged_window_needs(G, need, [&](const SfGeom &, const SfView &v, float xc, float yc, SfWindow &) { return Tile{&v, xc, yc}; },
                                [&](const SfGeom &ga, const Tile &t, float z0, float z1, SfWindow &w) { w = sd_bp_window(ga, *t.v, t.xc, t.yc, hx, z0, z1); });
            return need[0];
        };
        for (int sh = (int)first_shape; sh <= BP_LAST_SHORT_SHAPE && !G->bp_tiled; ++sh) {
            const WindowNeed need = window_of(BP_SHAPES[sh].zc);
            G->bp_need_w = need.w;
            G->bp_need_h = need.h;
            G->bp_shape = sh;
            G->bp_tiled = window_fits(need, BP_SHAPES[sh]);
        }
        if (!G->bp_tiled) return;
        // Groups of threads that share the views: the shapes whose windows fit, where one volume would take any of them.
        auto fits = [&](int sh) { return G->bp_need_w <= SD_BP_SPLIT_SHAPES[sh].pw - 1 && window_fits(window_of(SD_BP_SPLIT_SHAPES[sh].zc), SD_BP_SPLIT_SHAPES[sh]); };
        choose_siddon_split(G, SD_BP_NSPLIT_SHAPES, fits);
    }
}

// Is the convex polygon {rect} cut by the half-planes a u + b v + c >= 0 non-empty?  (Sutherland-Hodgman; a polygon
// that shrinks to a point or a segment still counts.)
static bool rectangle_meets(double u0, double u1, double v0, double v1, const double (*planes)[3], int nplanes)
{
    std::vector<std::pair<double, double>> poly = {{u0, v0}, {u1, v0}, {u1, v1}, {u0, v1}}, next;
    for (int p = 0; p < nplanes && !poly.empty(); ++p) {
        next.clear();
        const double a = planes[p][0], b = planes[p][1], c = planes[p][2];
        for (size_t q = 0; q < poly.size(); ++q) {
            const auto &A = poly[q], &B = poly[(q + 1) % poly.size()];
            const double fa = a * A.first + b * A.second + c, fb = a * B.first + b * B.second + c;
            if (fa >= 0.0) next.push_back(A);
            if ((fa >= 0.0) != (fb >= 0.0)) {
                const double t = fa / (fa - fb);
                next.push_back({A.first + t * (B.first - A.first), A.second + t * (B.second - A.second)});
            }
        }
        poly.swap(next);
    }
    return !poly.empty();
}

// Siddon model on tilted modules: can the per-lane slab kernels serve the scan?  They need every ray to rise by less
// than one axial cell per slab along its faster in-plane axis (kappa |Dz| <= limit * max(|Dx|, |Dy|), kappa = T / Tz;
// D is affine in the detector coordinates, so the rays that break it fill a convex polygon of the detector per sign of
// Dz), and every source more than a voxel away from the volume's box.
static bool tilted_rays_stay_flat(const leap_geometry *G, double limit)
{
    const leap_geometry_desc *d = &G->desc;
    const SfGeom &g = G->g;
    const double kappa = d->voxel_xy / d->voxel_z;
    const double u0 = (0.0 - g.col_offd) * g.pu_d, u1 = ((double)(d->ncols - 1) - g.col_offd) * g.pu_d;
    const double v0 = g.v0d, v1 = g.v0d + (double)(d->nrows - 1) * g.pvd;
    const double half[3] = {0.5 * d->nx * d->voxel_xy + d->voxel_xy, 0.5 * d->ny * d->voxel_xy + d->voxel_xy,
                            0.5 * d->nz * d->voxel_z + d->voxel_z};
    const double ctr[3] = {d->center_x, d->center_y, d->center_z};
    for (const MdPose &P : G->poses) {
        bool clear = false;
        for (int q = 0; q < 3; ++q) clear = clear || std::fabs(P.S[q] - ctr[q]) > half[q];
        if (!clear) return false;
        for (int sign = -1; sign <= 1; sign += 2) {
            double planes[4][3];
            for (int h = 0; h < 4; ++h) {
                const int axis = h >> 1;                       // 0: x, 1: y
                const double w = (h & 1) ? limit : -limit;     // sign kappa Dz -+ limit D_axis >= 0
                planes[h][0] = sign * kappa * P.ucol[2] + w * P.ucol[axis];
                planes[h][1] = sign * kappa * P.vrow[2] + w * P.vrow[axis];
                planes[h][2] = sign * kappa * (P.C[2] - P.S[2]) + w * (P.C[axis] - P.S[axis]);
            }
            if (rectangle_meets(u0, u1, v0, v1, planes, 4)) return false;
        }
    }
    return true;
}

// Siddon model on tilted modules, tiled back projection: largest window any (view, tile, z-chunk) asks for (every chunk
// counts: a tilted module's windows are not extreme at the ends of the volume only).  The corners of all those boxes are
// the points of one lattice, so each view projects the lattice once and every window takes the extremes of its eight
// corners; the kernel's own function forms the same corners by increments and may round apart in the last place, which
// the spare row and column of the fit test absorb.  The views are shared out among a few threads.
static void tilted_window_need(const leap_geometry *G, const std::vector<MdBpView> &views, int zc, int &need_w, int &need_h)
{
    const leap_geometry_desc *d = &G->desc;
    const SfGeom &g = G->g;
    const int tiles_x = (d->nx + BP_T - 1) / BP_T, tiles_y = (d->ny + BP_T - 1) / BP_T, chunks = (d->nz + zc - 1) / zc;
    const int lx = tiles_x + 1, ly = tiles_y + 1, lz = chunks + 1;
    const int workers = (int)std::max<size_t>(1, std::min<size_t>(8, views.size() / 8));
    std::vector<int> w(workers, 0), h(workers, 0);
    auto scan = [&](int t) {
        std::vector<float> xi((size_t)lx * ly * lz), eta(xi.size());
        float ew = 0.0f, eh = 0.0f;             // widest and tallest shadow; a window holds at most that many pixel centres + 1.04
        for (size_t a = t; a < views.size(); a += workers) {
            const MdBpView &V = views[a];
            for (int iz = 0; iz < lz; ++iz)
                for (int iy = 0; iy < ly; ++iy)
                    for (int ix = 0; ix < lx; ++ix) {
                        const float dx = fmaf((float)(ix * BP_T), g.T, V.dlo[0]), dy = fmaf((float)(iy * BP_T), g.T, V.dlo[1]);
                        const float dz = fmaf((float)(iz * zc), g.Tz, V.dlo[2]);
                        const float inv = 1.0f / fmaf(dx, V.nrm[0], fmaf(dy, V.nrm[1], dz * V.nrm[2]));
                        const size_t o = ((size_t)iz * ly + iy) * lx + ix;
                        xi[o] = fmaf(fmaf(dx, V.euP[0], fmaf(dy, V.euP[1], dz * V.euP[2])), inv, V.xi0);
                        eta[o] = fmaf(fmaf(dx, V.evP[0], fmaf(dy, V.evP[1], dz * V.evP[2])), inv, V.eta0);
                    }
            for (int iz = 0; iz < chunks; ++iz)
                for (int iy = 0; iy < tiles_y; ++iy)
                    for (int ix = 0; ix < tiles_x; ++ix) {
                        float a0 = 3.0e38f, a1 = -3.0e38f, b0 = 3.0e38f, b1 = -3.0e38f;
                        for (int q = 0; q < 8; ++q) {
                            const size_t o = ((size_t)(iz + (q >> 2)) * ly + iy + ((q >> 1) & 1)) * lx + ix + (q & 1);
                            const float u = xi[o], v = eta[o];
                            a0 = u < a0 ? u : a0; a1 = u > a1 ? u : a1;
                            b0 = v < b0 ? v : b0; b1 = v > b1 ? v : b1;
                        }
                        ew = a1 - a0 > ew ? a1 - a0 : ew;
                        eh = b1 - b0 > eh ? b1 - b0 : eh;
                        if (!(std::fmax(-a0, a1) < BP_MAX_COORDINATE && std::fmax(-b0, b1) < BP_MAX_COORDINATE)) ew = eh = 1.0e6f;   // NaN or too far out: no instance fits
                    }
        }
        w[t] = sf_f2i(floorf(ew + 1.04f));
        h[t] = sf_f2i(floorf(eh + 1.04f));
    };
    run_shares(workers, scan);
    need_w = *std::max_element(w.begin(), w.end());
    need_h = *std::max_element(h.begin(), h.end());
}

// Siddon model, scans with tilted modules: the per-lane variants of the two fast kernels.
static void select_tilted_siddon_kernels(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    long v;
    if (debug_option("general", v) && v == 1) return;
    if (d->nrows >= 32 && tilted_rays_stay_flat(G, 0.999)) {        // forward projection on the slab scratch
        G->md_tilted = true;
        G->sd_columns = true;
        static const int single_groups[] = {1, 2, 4};
        G->fp_rg = row_groups(d->nrows, 64, single_groups, 3);
        block_order_options(G);
    }
    // Tiled back projection.  Its rays are marched along the TILE's faster in-plane axis: a ray through a tile whose
    // centre lies c_maj from the source along that axis has |d_maj| >= c_maj - 8 T and max(|dx|, |dy|) <= c_maj + 8 T, so
    // a rise of at most 0.8 cells per slab along the ray's own axis stays below one cell along the tile's if
    // c_maj >= 72 T, which an in-plane distance of 102 T between source and volume guarantees.
    if (d->nz < 8 || !((double)d->nrows * d->ncols < 1073741824.0) || !tilted_rays_stay_flat(G, 0.8)) return;
    const double half[3] = {0.5 * d->nx * d->voxel_xy, 0.5 * d->ny * d->voxel_xy, 0.5 * d->nz * d->voxel_z};
    const double ctr[3] = {d->center_x, d->center_y, d->center_z};
    for (const MdPose &P : G->poses) {
        const double ox = std::fmax(std::fabs(P.S[0] - ctr[0]) - half[0], 0.0), oy = std::fmax(std::fabs(P.S[1] - ctr[1]) - half[1], 0.0);
        if (!(std::hypot(ox, oy) >= 102.0 * d->voxel_xy)) return;
        const double n[3] = {P.ucol[1] * P.vrow[2] - P.ucol[2] * P.vrow[1], P.ucol[2] * P.vrow[0] - P.ucol[0] * P.vrow[2],
                             P.ucol[0] * P.vrow[1] - P.ucol[1] * P.vrow[0]};
        const double gap = (P.C[0] - P.S[0]) * n[0] + (P.C[1] - P.S[1]) * n[1] + (P.C[2] - P.S[2]) * n[2];
        for (int corner = 0; corner < 8; ++corner) {                // the whole volume in front of the source
            double along = 0.0;
            for (int q = 0; q < 3; ++q) along += (ctr[q] + ((corner >> q) & 1 ? half[q] : -half[q]) - P.S[q]) * n[q];
            if (!(along * gap > 0.0) || !(std::fabs(along) > 1e-3 * std::fabs(gap))) return;
        }
    }
    std::vector<MdBpView> views;
    views.reserve(G->poses.size());
    for (const MdPose &P : G->poses) views.push_back(md_bp_view(G->g, P));
    long first_shape = 0;
    if (debug_option("bp_shape", first_shape)) first_shape = ((first_shape % MD_BP_NSHAPES) + MD_BP_NSHAPES) % MD_BP_NSHAPES;
    bool fits = false;
    for (int sh = (int)first_shape; sh < MD_BP_NSHAPES && !fits; ++sh) {
        tilted_window_need(G, views, MD_BP_SHAPES[sh].zc, G->bp_need_w, G->bp_need_h);
        G->bp_shape = sh;
        fits = G->bp_need_w <= MD_BP_SHAPES[sh].pw - 1 && G->bp_need_h <= MD_BP_SHAPES[sh].ph - 1;
    }
    if (!fits) return;
    auto split_fits = [&](int sh) {
        const SfBpShape S = MD_BP_SPLIT_SHAPES[sh];
        int w, h;
        if (G->bp_need_w > S.pw - 1) return false;
        tilted_window_need(G, views, S.zc, w, h);
        return w <= S.pw - 1 && h <= S.ph - 1;
    };
    choose_siddon_split(G, MD_BP_NSPLIT_SHAPES, split_fits);
    hipError_t e = hipMalloc((void **)&G->d_mdbp, sizeof(MdBpView) * views.size());
    if (e == hipSuccess) e = hipMemcpy(G->d_mdbp, views.data(), sizeof(MdBpView) * views.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (G->d_mdbp) (void)hipFree(G->d_mdbp);
        G->d_mdbp = nullptr;
        (void)hipGetLastError();
        no_tiled_back_projection(G);
        add_note(G, "table allocation failed: back projection runs on the general kernel");
        return;
    }
    G->bp_tiled = true;
}

// Footprint model, scans with tilted modules: the fast kernels of md_footprint_tiled.h.
static void select_tilted_footprint_kernels(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    const SfGeom &g = G->g;
    long v;
    if (debug_option("general", v) && v == 1) return;
    // Forward: layers are walked along x or y, whichever a tile's central ray advances faster on.  Modules seen from above,
    // whose rays advance fastest along z, have beams that cross such a layer in long strips: they stay with the general
    // kernel, which can walk along z.
    for (const MfView &V : G->mfviews) {
        G->max_cols_per_voxel = std::max(G->max_cols_per_voxel, 2.0 * V.pad_u * V.ipu);
        G->max_rows_per_voxel = std::max(G->max_rows_per_voxel, 2.0 * V.pad_v * V.ipv);
    }
    // A voxel that covers many pixels makes as many LDS additions in each of the tiles it reaches, where the general kernel's
    // threads share its footprint between eight rows.  32^3 x 40 views, general / tiles: voxels of up to 13 x 9 pixels 798 / 602 us,
    // 16 x 11 897 / 1021, 21 x 15 999 / 1737; 6 x 15 816 / 581, 2 x 19 638 / 715, 21 x 5 943 / 911.
    G->mf_tiles = G->max_cols_per_voxel * G->max_rows_per_voxel <= 120.0 && G->max_rows_per_voxel <= 16.0 &&
                  tilted_rays_stay_flat(G, d->voxel_xy / d->voxel_z);
    // Back: the staged window of every (view, tile, chunk) must fit.  The boxes' corners are the points of one lattice; the
    // views are shared out among a few threads.
    const int tiles_x = (d->nx + MF_T - 1) / MF_T, tiles_y = (d->ny + MF_T - 1) / MF_T, chunks = (d->nz + MF_ZC - 1) / MF_ZC;
    const int lx = tiles_x + 1, ly = tiles_y + 1, lz = chunks + 1;
    const int workers = (int)std::max<size_t>(1, std::min<size_t>(8, G->mfviews.size() / 8));
    std::vector<int> need(workers, 0);
    auto scan = [&](int t) {
        std::vector<float> xi((size_t)lx * ly * lz), eta(xi.size());
        int worst = 0;
        for (size_t a = t; a < G->mfviews.size(); a += workers) {
            const MfView &V = G->mfviews[a];
            for (int z = 0; z < lz; ++z)
                for (int y = 0; y < ly; ++y)
                    for (int x = 0; x < lx; ++x) {
                        const size_t o = ((size_t)z * ly + y) * lx + x;
                        // corner 0 of the box that starts here: the lattice point itself
                        mf_box_corner(g, V, std::min(x * MF_T, d->nx), 0, std::min(y * MF_T, d->ny), 0, std::min(z * MF_ZC, d->nz), 0, 0, xi[o], eta[o]);
                    }
            for (int z = 0; z < chunks; ++z)
                for (int y = 0; y < tiles_y; ++y)
                    for (int x = 0; x < tiles_x; ++x) {
                        float a0 = 3.0e38f, a1 = -3.0e38f, b0 = 3.0e38f, b1 = -3.0e38f;
                        for (int q = 0; q < 8; ++q) {
                            const size_t o = ((size_t)(z + (q >> 2)) * ly + y + ((q >> 1) & 1)) * lx + x + (q & 1);
                            a0 = std::min(a0, xi[o]); a1 = std::max(a1, xi[o]);
                            b0 = std::min(b0, eta[o]); b1 = std::max(b1, eta[o]);
                        }
                        const MfWindow w = mf_window(a0, a1, b0, b1);
                        // one spare row and column: host and device may round apart
                        const bool near = std::fmax(-a0, a1) < BP_MAX_COORDINATE && std::fmax(-b0, b1) < BP_MAX_COORDINATE;
                        worst = std::max(worst, near && a1 - a0 < 4096.0f && b1 - b0 < 4096.0f ? (w.w + 1) * (w.h + 1) : 1 << 30);
                    }
        }
        need[t] = worst;
    };
    run_shares(workers, scan);
    G->mf_tiled = *std::max_element(need.begin(), need.end()) <= MF_PATCH;
}

// Picks the kernels of a validated scan (circular scanners, or modular scans made of upright modules).
static void select_fast_kernels(leap_geometry *G)
{
    if (!footprint_bounds(G)) return;
    long v;
    if (debug_option("general", v) && v == 1) return;       // testing aid: every call on the general kernels
    if (G->desc.model == LEAP_MODEL_SF) {
        select_footprint_tiled(G);
        select_footprint_columns(G);
        select_footprint_flat(G);
    } else {
        select_siddon_fast_kernels(G);
    }
}

// Slab width and items per launch that a scratch of `floats` floats affords for a batch of `batch` volumes: as many
// items at once as the batch has (16 at most) while a slab stays at least 32 voxel layers wide, the whole volume per
// copy if it fits.  Returns false if not even four layers fit.
bool leap_plan_scratch(const leap_geometry *G, size_t floats, int batch, int &width, int &items)
{
    const leap_geometry_desc *d = &G->desc;
    const int n_side = std::max(d->nx, d->ny);                  // a slab holds up to width * n_side voxel columns
    const double nzp = G->nzp;
    auto width_for = [&](int it) {
        const double w = std::floor(((double)floats / it - nzp) / (nzp * n_side));
        return w >= n_side ? n_side : (w < 4 ? 0 : ((int)w & ~3));
    };
    items = std::max(1, std::min(batch, 16));
    // (a slab whose layers four waves share: as wide as for one item)
    const int least = G->fp_parts > 1 ? width_for(1) : std::min(32, n_side);
    while (items > 1 && width_for(items) < least) items = (items + 1) / 2;
    width = width_for(items);
    if (G->dbg_items > 0) items = std::min(G->dbg_items, std::max(1, batch));
    if (G->dbg_slab > 0) width = std::min(G->dbg_slab, n_side);
    if (G->dbg_items > 0 || G->dbg_slab > 0) {                  // overrides must still fit
        while (items > 1 && ((double)width * n_side + 1.0) * nzp * items > (double)floats) --items;
        if (((double)width * n_side + 1.0) * nzp * items > (double)floats) width = width_for(items);
    }
    // the copy kernel puts (voxel rows of a slab) x (items) into one grid dimension
    items = std::max(1, std::min(items, 65535 / std::max(std::max(d->ny, width), 1)));
    return width >= 4 && ((double)width * n_side + 1.0) * nzp < 4294967296.0;     // slab columns are indexed with 32 bits
}

// The scratch of the column-wise forward kernels: z-fastest copies of one slab of the volume (plus a spare zero column
// each).  Large volumes: an eighth of one volume (a quarter for the Siddon kernel, whose waves own a single detector
// column and lose more to narrow slabs); volumes under 512 MiB: 128 MiB, which lets a batch of small training volumes
// go through together.  On failure the handle falls back to the general kernel and says so (leap_last_error, and the
// note shown by leap_geometry_describe).
static void allocate_forward_scratch(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    if (!G->fp_columns && !G->sd_columns) return;
    G->nzp = (G->fp_rows ? (d->nrows + 3) / 4 * 4 : d->nz) + 2 * FP_PAD;      // floats per voxel column of the copy
    if (4.0 * d->nx * d->ny * (double)G->nzp <= FP_TURN_BYTES) G->fp_turn = 3;
    const double volume_bytes = 4.0 * d->nx * d->ny * (double)d->nz;
    const double share = volume_bytes / (d->model == LEAP_MODEL_SIDDON ? 4.0 : 8.0);
    double budget = volume_bytes / 8.0 >= 64.0 * 1048576.0 ? share : 128.0 * 1048576.0;
    long v;
    if (debug_option("scratch_mib", v) && v >= 1) budget = 1048576.0 * (double)v;
    if (debug_option("slab", v) && v >= 4) G->dbg_slab = (int)(v & ~3L);
    if (debug_option("items", v) && v >= 1 && v <= 16) G->dbg_items = (int)v;
    // no more than 16 whole copies
    const double whole = 4.0 * ((double)d->nx * d->ny + 1.0) * G->nzp;
    budget = std::fmin(budget, 16.0 * whole);
    hipError_t e = hipErrorOutOfMemory;
    int width = 0, items = 0;
    for (int attempt = 0; attempt < 6; ++attempt, budget *= 0.5) {
        G->scratch_bytes = (size_t)budget & ~(size_t)255;
        if (!leap_plan_scratch(G, G->scratch_bytes / sizeof(float), 1, width, items)) break;
        e = hipMalloc((void **)&G->d_volz, G->scratch_bytes);
        if (e == hipSuccess) e = hipMemset(G->d_volz, 0, G->scratch_bytes);   // the pads stay zero for the handle's life
        if (e == hipSuccess) e = hipDeviceSynchronize();
        if (e == hipSuccess) break;
        if (G->d_volz) (void)hipFree(G->d_volz);
        G->d_volz = nullptr;
        (void)hipGetLastError();
    }
    if (e == hipSuccess && !G->major.empty()) {
        e = hipMalloc((void **)&G->d_major, G->major.size());
        if (e == hipSuccess) e = hipMemcpy(G->d_major, G->major.data(), G->major.size(), hipMemcpyHostToDevice);
    }
    // Short detectors, which share no scratch under capture: a slot per copy of the whole volume.
    const double n_side = std::max(d->nx, d->ny), copy = (n_side * n_side + 1.0) * G->nzp;
    const int slots = d->nrows < FP_FREE_ROWS ? std::max(1, (int)std::min((double)LeapRoom::MOST_SLOTS, std::floor((double)(G->scratch_bytes / sizeof(float)) / copy))) : 1;
    G->scratch_slot_floats = G->scratch_bytes / sizeof(float) / G->nzp / slots * G->nzp;       // (whole columns: the pads lie alike)
    if (e == hipSuccess) e = G->scratch.create(slots);
    if (e != hipSuccess) {
        if (G->d_volz) (void)hipFree(G->d_volz);
        if (G->d_major) (void)hipFree(G->d_major);
        G->d_volz = nullptr; G->d_major = nullptr;
        G->fp_columns = G->sd_columns = false;
        G->scratch_bytes = 0;
        const char *const what = "scratch allocation failed: forward projection runs on the general kernel";
        add_note(G, what);
        leap_set_error(std::string("leap_geometry_create: ") + what + " (" + hipGetErrorString(e) + ")");
        (void)hipGetLastError();
        return;
    }
    G->slab_width = width;
}

// Flat scans: room for the batch-fastest copies, by rows and turned, of up to 16 slices, 256 MiB at most; of half as many, and so on
// down to two, where that cannot be had.  Without it every item of a batch is projected by itself.
static void allocate_flat_scratch(leap_geometry *G)
{
    const double slice = 4.0 * G->desc.nx * (double)G->desc.ny;
    double items = std::fmin(16.0, std::floor(128.0 * 1048576.0 / slice));
    if (!(items >= 2.0)) return;
    hipError_t e = hipErrorOutOfMemory;
    for (; e != hipSuccess && items >= 2.0; items = std::floor(0.5 * items)) {
        G->scratch_bytes = (size_t)(2.0 * items * slice);
        e = hipMalloc((void **)&G->d_volz, G->scratch_bytes);
        if (e != hipSuccess) (void)hipGetLastError();
    }
    if (e == hipSuccess) e = G->scratch.create(1);
    if (e == hipSuccess) return;
    if (G->d_volz) (void)hipFree(G->d_volz);
    G->d_volz = nullptr;
    G->scratch_bytes = 0;
    add_note(G, "scratch allocation failed: the items of a batch are projected one by one");
    (void)hipGetLastError();
}

// Room for the volumes of the parts in which a back projection's views are shared among workgroups: for as many items at once as
// fit 64 MiB, in slots for calls on several streams.  Without it the views stay with one workgroup.
static void allocate_back_room(leap_geometry *G)
{
    const size_t one = (size_t)G->g.nx * G->g.ny * G->g.nz * G->bp_parts;
    const int items = (int)std::max<size_t>(1, std::min<size_t>(16, (size_t)BACK_MOST_FLOATS / one)), slots = std::min(items, LeapRoom::MOST_SLOTS);
    G->back_floats = one * items;
    G->back_slot_items = items / slots;
    hipError_t e = hipMalloc((void **)&G->d_back, G->back_floats * sizeof(float));
    if (e == hipSuccess) e = G->back.create(slots);
    if (e == hipSuccess) return;
    if (G->d_back) (void)hipFree(G->d_back);
    G->d_back = nullptr;
    G->back_floats = 0;
    G->bp_parts = 1;
    G->bp_parts_fits = 0;
    add_note(G, "no room for the back projection's parts: its views stay with one workgroup");
    (void)hipGetLastError();
}

static void free_handle(leap_geometry *G)
{
    if (!G) return;
    leap_host_stage_free(G);
    if (G->d_views) (void)hipFree(G->d_views);
    if (G->d_volz) (void)hipFree(G->d_volz);
    if (G->d_major) (void)hipFree(G->d_major);
    if (G->d_raycols) (void)hipFree(G->d_raycols);
    if (G->d_poses) (void)hipFree(G->d_poses);
    if (G->d_geoms) (void)hipFree(G->d_geoms);
    if (G->d_mfviews) (void)hipFree(G->d_mfviews);
    if (G->d_mdbp) (void)hipFree(G->d_mdbp);
    if (G->d_colcs) (void)hipFree(G->d_colcs);
    if (G->d_back) (void)hipFree(G->d_back);
    delete G;
}

// Cylindrical detector, tiled back projection: cosine and sine of every detector column's fan angle (ray amplitudes),
// then per (tile, view) the tile centre's fan angle and the tile's window bounds.  No room for the tables: the general
// kernel needs none.
static void upload_curved_tables(leap_geometry *G)
{
    const leap_geometry_desc *d = &G->desc;
    const SfGeom &g = G->g;
    const int tiles_x = (d->nx + BP_T - 1) / BP_T, tiles_y = (d->ny + BP_T - 1) / BP_T;
    const size_t head = 2 * sizeof(float) * (size_t)d->ncols;
    const size_t bytes = head + sizeof(SfCurvedBounds) * (size_t)tiles_x * tiles_y * d->nviews;
    std::vector<unsigned char> blob(bytes);
    float *cs = reinterpret_cast<float *>(blob.data());
    for (int c = 0; c < d->ncols; ++c) {
        const double gam = ((double)c - g.col_offd) * d->pixel_u / d->sdd;
        cs[2 * (size_t)c] = (float)std::cos(gam);
        cs[2 * (size_t)c + 1] = (float)std::sin(gam);
    }
    SfCurvedBounds *tab = reinterpret_cast<SfCurvedBounds *>(blob.data() + head);
    const float hx = 0.5f * (float)(BP_T - 1) * g.T;
    for (int ty = 0; ty < tiles_y; ++ty)
        for (int tx = 0; tx < tiles_x; ++tx) {
            const double xcd = g.x0d + ((double)(tx * BP_T) + 0.5 * (BP_T - 1)) * g.Td;
            const double ycd = g.y0d + ((double)(ty * BP_T) + 0.5 * (BP_T - 1)) * g.Td;
            SfCurvedBounds *row = tab + ((size_t)ty * tiles_x + tx) * d->nviews;
            for (int a = 0; a < d->nviews; ++a) {
                const SfView &v = G->views[a];
                row[a].gref = std::atan2(std::fma(ycd, v.cd, -xcd * v.sd), g.sodd - std::fma(xcd, v.cd, ycd * v.sd));
                sf_curved_tile_bounds(g, v, (float)xcd, (float)ycd, hx, row[a].xi_lo, row[a].xi_hi, row[a].ilo, row[a].ihi);
            }
        }
    hipError_t et = hipMalloc((void **)&G->d_colcs, bytes);
    if (et == hipSuccess) et = hipMemcpy(G->d_colcs, blob.data(), bytes, hipMemcpyHostToDevice);
    if (et != hipSuccess) {
        if (G->d_colcs) (void)hipFree(G->d_colcs);
        G->d_colcs = nullptr;
        no_tiled_back_projection(G);
        add_note(G, "no room for the cylinder's tile tables: back projection runs on the general kernel");
        (void)hipGetLastError();
    }
}

// Uploads every table the chosen kernels read to the current device and allocates the forward scratch; on failure
// frees the handle.
static int finish_handle(leap_geometry *G, leap_geometry **out)
{
    const leap_geometry_desc *d = &G->desc;
    auto upload = [](void **dst, const void *src, size_t bytes) {
        hipError_t e = hipMalloc(dst, bytes);
        if (e == hipSuccess) e = hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice);
        return e;
    };
    long kib;
    if (debug_option("stage_kib", kib) && kib >= 4) G->stage_chunk = (size_t)kib << 10;
    hipError_t e = hipGetDevice(&G->device);
    if (e == hipSuccess) (void)leap_static_scratch_init(G->device);   // set-up for leap_project_static_scratch; it reports a failure itself
    if (e == hipSuccess && !G->views.empty()) e = upload((void **)&G->d_views, G->views.data(), sizeof(SfView) * G->views.size());
    if (e == hipSuccess) allocate_forward_scratch(G);
    if (e == hipSuccess && G->flat) allocate_flat_scratch(G);
    if (e == hipSuccess && !G->raycols.empty()) e = upload((void **)&G->d_raycols, G->raycols.data(), sizeof(SdRayCol) * G->raycols.size());
    if (e == hipSuccess && !G->geoms.empty()) e = upload((void **)&G->d_geoms, G->geoms.data(), sizeof(SfGeom) * G->geoms.size());
    if (e == hipSuccess && !G->poses.empty()) e = upload((void **)&G->d_poses, G->poses.data(), sizeof(MdPose) * G->poses.size());
    if (e == hipSuccess && !G->mfviews.empty())
        e = upload((void **)&G->d_mfviews, G->mfviews.data(), sizeof(MfView) * G->mfviews.size());
    if (e == hipSuccess && d->type == LEAP_CONE_CURVED && d->model == LEAP_MODEL_SF && G->bp_tiled) upload_curved_tables(G);
    if (e == hipSuccess && G->bp_parts > 1) allocate_back_room(G);         // (after what may still leave the general kernel)
    if (e != hipSuccess) {
        const int rc = leap_hip_fail(e, "uploading the geometry tables");       // (may throw: the handle is freed after it)
        free_handle(G);
        return rc;
    }
    *out = G;
    return LEAP_OK;
}

// Modular geometry: per-view poses instead of the angle list; only the fields the modular kernels read are filled.
static int create_modular(const leap_geometry_desc *d, leap_geometry **out, leap_geometry *&G)
{
    if (!d->poses) return invalid("poses is null");
    if (d->nviews > 65535 || (double)d->nx * d->ny * d->nz >= 4294967296.0 ||
        (double)d->nviews * d->nrows * d->ncols >= 4294967296.0 || d->ny > 262140 || d->nz > 65535 || d->nrows > 262140) {
        leap_set_error("sizes beyond what one launch covers");
        return LEAP_UNSUPPORTED;
    }
    const double half[3] = {0.5 * d->nx * d->voxel_xy, 0.5 * d->ny * d->voxel_xy, 0.5 * d->nz * d->voxel_z};
    const double ctr[3] = {d->center_x, d->center_y, d->center_z};
    for (int a = 0; a < d->nviews; ++a) {
        const double *p = d->poses + 12 * (size_t)a;
        for (int q = 0; q < 12; ++q)
            if (!std::isfinite(p[q])) return invalid("poses must be finite");
        const double uu = p[6] * p[6] + p[7] * p[7] + p[8] * p[8], vv = p[9] * p[9] + p[10] * p[10] + p[11] * p[11];
        const double uv = p[6] * p[9] + p[7] * p[10] + p[8] * p[11];
        if (std::fabs(uu - 1.0) > 1e-9 || std::fabs(vv - 1.0) > 1e-9 || std::fabs(uv) > 1e-9)
            return invalid("detector axes must be orthonormal");
        bool inside = true;
        for (int q = 0; q < 3; ++q) inside = inside && std::fabs(p[q] - ctr[q]) <= half[q];
        if (inside) {
            leap_set_error("a source lies inside the volume");
            return LEAP_BAD_GEOMETRY;
        }
    }
    // Upright modules (column axis horizontal, row axis +z, detector behind the volume as seen from the source, source
    // clear of the volume's bounding circle in the module's frame) are circular cone-beam views of a translated scene:
    // both models have fast kernels for scans made of them.  A scan with any other module goes through the general
    // kernels of its model.
    bool tilted = false, upright = true;
    for (int a = 0; a < d->nviews; ++a) {
        const double *p = d->poses + 12 * (size_t)a;
        if (std::fabs(p[8]) > 1e-9 || std::fabs(p[9]) > 1e-9 || std::fabs(p[10]) > 1e-9 || std::fabs(p[11] - 1.0) > 1e-9) {
            tilted = true;
            upright = false;
        }
    }
    for (int a = 0; a < d->nviews && !tilted && upright; ++a) {
        const double *p = d->poses + 12 * (size_t)a;
        const double c = p[7], s = -p[6];
        const double lS = p[0] * c + p[1] * s, lD = p[3] * c + p[4] * s, tS = -p[0] * s + p[1] * c;
        // the volume as this view sees it: moved by -tS along the column axis
        const double mx = std::fabs(d->center_x - tS * p[6]) + half[0], my = std::fabs(d->center_y - tS * p[7]) + half[1];
        const double reach_a = std::sqrt(mx * mx + my * my);
        if (!(lS - lD > 0.0) || !(lS > reach_a) || !(d->pixel_u < 0.25 * (lS - lD))) upright = false;
    }
    if (d->model == LEAP_MODEL_SF && !upright && !tilted) {
        leap_set_error("module does not face its source across the volume");
        return LEAP_BAD_GEOMETRY;
    }
    G = new (std::nothrow) leap_geometry;
    if (!G) return invalid("out of host memory");
    G->desc = *d;
    G->desc.angles_rad = nullptr;
    SfGeom &g = G->g;
    std::memset(&g, 0, sizeof(g));
    g.type = d->type; g.model = d->model;
    g.nviews = d->nviews; g.nrows = d->nrows; g.ncols = d->ncols;
    g.nx = d->nx; g.ny = d->ny; g.nz = d->nz;
    g.Td = d->voxel_xy; g.Tzd = d->voxel_z;
    g.x0d = d->center_x - 0.5 * (d->nx - 1) * d->voxel_xy;
    g.y0d = d->center_y - 0.5 * (d->ny - 1) * d->voxel_xy;
    g.zlo0d = d->center_z - 0.5 * d->nz * d->voxel_z;
    g.col_offd = 0.5 * (d->ncols - 1) - d->shift_u;
    g.row_offd = 0.5 * (d->nrows - 1) - d->shift_v + 0.5;
    g.v0d = (-0.5 * (d->nrows - 1) + d->shift_v) * d->pixel_v;
    g.pvd = d->pixel_v;
    g.pu_d = d->pixel_u;
    g.T = (float)d->voxel_xy; g.Tz = (float)d->voxel_z; g.pu = (float)d->pixel_u; g.pv = (float)d->pixel_v;
    G->poses.resize(d->nviews);
    std::memcpy(G->poses.data(), d->poses, sizeof(MdPose) * (size_t)d->nviews);
    G->desc.poses = reinterpret_cast<const double *>(G->poses.data());
    if (upright) {
        // per view: the same scene translated so that the source sits on the frame's axis at height 0
        g.iTzd = 1.0 / d->voxel_z;
        G->views.resize(d->nviews);
        G->geoms.resize(d->nviews);
        const double h = 0.5 * d->voxel_xy;
        for (int a = 0; a < d->nviews; ++a) {
            const MdPose &P = G->poses[a];
            const double c = P.ucol[1], s = -P.ucol[0];
            const double lS = P.S[0] * c + P.S[1] * s, tS = -P.S[0] * s + P.S[1] * c, zS = P.S[2];
            const double sdd = lS - (P.C[0] * c + P.C[1] * s), tC = -P.C[0] * s + P.C[1] * c, zC = P.C[2];
            SfView &v = G->views[a];
            std::memset(&v, 0, sizeof(v));
            v.cd = c; v.sd = s; v.c = (float)c; v.s = (float)s;
            v.p = (float)(h * c); v.q = (float)(h * s);
            v.xmajor = std::fabs(c) >= std::fabs(s) ? 1 : 0;
            SfGeom &ga = G->geoms[a];
            ga = g;
            ga.type = SF_CONE;
            ga.x0d = g.x0d - tS * P.ucol[0];
            ga.y0d = g.y0d - tS * P.ucol[1];
            ga.zlo0d = g.zlo0d - zS;
            ga.sodd = lS;
            ga.kud = sdd / d->pixel_u; ga.kvd = sdd / d->pixel_v; ga.ikvd = 1.0 / ga.kvd;
            ga.col_offd = g.col_offd - (tC - tS) / d->pixel_u;
            ga.row_offd = g.row_offd - (zC - zS) / d->pixel_v;
            ga.v0d = g.v0d + (zC - zS);
            ga.zk0d = -ga.zlo0d / d->voxel_z;
            ga.sod = (float)lS; ga.sdd = (float)sdd; ga.ku = (float)ga.kud;
            ga.col_off = (float)ga.col_offd; ga.v0 = (float)ga.v0d;
        }
    }
    if (upright) {
        if (d->model == LEAP_MODEL_SIDDON) build_ray_table(G);
        select_fast_kernels(G);
    } else if (d->model == LEAP_MODEL_SIDDON) {
        select_tilted_siddon_kernels(G);
        // The general back projection bounds a voxel's pixel search by its projected corners; a voxel that reaches behind
        // a source's plane (the plane through the source parallel to its module) has no such bound and tests every pixel
        // of that view.  On large scans that is not a slow call but one that never ends: refuse it.
        if (!G->bp_tiled) {
            double behind = 0.0;
            for (const MdPose &P : G->poses) {
                const double n[3] = {P.ucol[1] * P.vrow[2] - P.ucol[2] * P.vrow[1], P.ucol[2] * P.vrow[0] - P.ucol[0] * P.vrow[2],
                                     P.ucol[0] * P.vrow[1] - P.ucol[1] * P.vrow[0]};
                const double gap = (P.C[0] - P.S[0]) * n[0] + (P.C[1] - P.S[1]) * n[1] + (P.C[2] - P.S[2]) * n[2];
                bool all_in_front = true;
                for (int corner = 0; corner < 8; ++corner) {
                    double along = 0.0;
                    for (int q = 0; q < 3; ++q) along += (ctr[q] + ((corner >> q) & 1 ? half[q] : -half[q]) - P.S[q]) * n[q];
                    all_in_front = all_in_front && along * gap > 0.0;
                }
                behind += all_in_front ? 0.0 : 1.0;
            }
            if (behind * d->nrows * d->ncols * ((double)d->nx * d->ny * d->nz) > 5.0e11) {
                leap_set_error("in " + std::to_string((long)behind) + " views the volume reaches behind the source's plane (the plane "
                               "through the source parallel to its module); on a scan of this size the back projection of such "
                               "views is not supported");
                free_handle(G);
                return LEAP_UNSUPPORTED;
            }
        }
    }
    if (!upright && d->model == LEAP_MODEL_SF) {
        G->mfviews.resize(d->nviews);
        for (int a = 0; a < d->nviews; ++a) {
            const MdPose &P = G->poses[a];
            MfView &V = G->mfviews[a];
            for (int q = 0; q < 3; ++q) { V.S[q] = P.S[q]; V.C[q] = P.C[q]; V.eu[q] = P.ucol[q]; V.ev[q] = P.vrow[q]; }
            if (!mf_prepare_view(g, V)) {
                leap_set_error("view " + std::to_string(a) + " has no footprints: the whole volume must lie in front of the "
                               "source (on the module's side) and no pixel's ray may run along z");
                free_handle(G);
                return LEAP_BAD_GEOMETRY;
            }
            // the forward kernel looks for a pixel's voxels within the footprint's reach around its ray: a source so close
            // to the volume that the nearest voxel's footprint spans dozens of pixels makes that search the whole volume
            if (V.pad_u * V.ipu > 32.0 || V.pad_v * V.ipv > 32.0) {
                leap_set_error("view " + std::to_string(a) + ": the source is so close to the volume that a voxel's footprint on "
                               "this tilted module spans more than 64 pixels; not supported by the footprint kernels for "
                               "tilted modules");
                free_handle(G);
                return LEAP_UNSUPPORTED;
            }
        }
        select_tilted_footprint_kernels(G);
    }
    return finish_handle(G, out);
}

// G: the handle under construction (the caller frees it if anything throws).
static int create_handle(const leap_geometry_desc *d, leap_geometry **out, leap_geometry *&G)
{
    if (d->type != LEAP_PARALLEL && d->type != LEAP_FAN && d->type != LEAP_CONE && d->type != LEAP_CONE_CURVED &&
        d->type != LEAP_MODULAR)
        return invalid("unknown geometry type");
    if (d->model != LEAP_MODEL_SF && d->model != LEAP_MODEL_SIDDON) return invalid("unknown projector model");
    if (d->nviews <= 0 || d->nrows <= 0 || d->ncols <= 0) return invalid("nviews, nrows and ncols must be positive");
    if (d->nx <= 0 || d->ny <= 0 || d->nz <= 0) return invalid("nx, ny and nz must be positive");
    if (!finite_pos(d->pixel_u) || !finite_pos(d->pixel_v)) return invalid("pixel sizes must be positive");
    if (!finite_pos(d->voxel_xy) || !finite_pos(d->voxel_z)) return invalid("voxel sizes must be positive");
    if (!std::isfinite(d->shift_u) || !std::isfinite(d->shift_v)) return invalid("detector shifts must be finite");
    if (!std::isfinite(d->center_x) || !std::isfinite(d->center_y) || !std::isfinite(d->center_z))
        return invalid("volume centre must be finite");
    if (d->type == LEAP_MODULAR) return create_modular(d, out, G);
    if (!d->angles_rad) return invalid("angles_rad is null");
    for (int a = 0; a < d->nviews; ++a)
        if (!std::isfinite(d->angles_rad[a])) return invalid("view angles must be finite");
    if (d->type == LEAP_FAN && (d->nrows != 1 || d->nz != 1)) return invalid("fan-beam needs nrows == 1 and nz == 1");
    if (d->nviews > 65535) {
        leap_set_error("more than 65535 views in one geometry");
        return LEAP_UNSUPPORTED;
    }
    if ((double)d->nx * d->ny * d->nz >= 2147483648.0 * 2.0 || (double)d->nviews * d->nrows * d->ncols >= 2147483648.0 * 2.0) {
        leap_set_error("array of more than 2^32 elements");
        return LEAP_UNSUPPORTED;
    }

    const double T = d->voxel_xy, h = 0.5 * T;
    const double half_x = 0.5 * d->nx * T, half_y = 0.5 * d->ny * T;
    if (d->type != LEAP_PARALLEL) {
        if (!finite_pos(d->sdd) || !finite_pos(d->sod)) {
            leap_set_error("sod and sdd must be positive");
            return LEAP_BAD_GEOMETRY;
        }
        // farthest in-plane corner of the volume from the rotation axis
        const double rx = std::fabs(d->center_x) + half_x, ry = std::fabs(d->center_y) + half_y;
        const double reach = std::sqrt(rx * rx + ry * ry);
        if (!(d->sod > reach)) {
            leap_set_error("source orbit radius (sod) does not clear the volume's bounding circle");
            return LEAP_BAD_GEOMETRY;
        }
        if (!(d->pixel_u < 0.25 * d->sdd)) {
            leap_set_error("detector pixel wider than a quarter of sdd");
            return LEAP_BAD_GEOMETRY;
        }
        if (d->type == LEAP_CONE_CURVED && !((0.5 * d->ncols + std::fabs(d->shift_u) + 1.0) * d->pixel_u < 1.5 * d->sdd)) {
            leap_set_error("curved detector spans a fan of more than +-1.5 rad");
            return LEAP_BAD_GEOMETRY;
        }
    }

    G = new (std::nothrow) leap_geometry;
    if (!G) return invalid("out of host memory");
    G->desc = *d;
    G->angles.assign(d->angles_rad, d->angles_rad + d->nviews);
    G->desc.angles_rad = G->angles.data();

    SfGeom &g = G->g;
    std::memset(&g, 0, sizeof(g));
    const bool par = d->type == LEAP_PARALLEL;
    g.type = d->type;
    g.nviews = d->nviews; g.nrows = d->nrows; g.ncols = d->ncols;
    g.nx = d->nx; g.ny = d->ny; g.nz = d->nz;
    g.Td = T; g.Tzd = d->voxel_z;
    g.x0d = d->center_x - 0.5 * (d->nx - 1) * T;
    g.y0d = d->center_y - 0.5 * (d->ny - 1) * T;
    g.zlo0d = d->center_z - 0.5 * d->nz * d->voxel_z;
    g.sodd = par ? 0.0 : d->sod;
    g.kud = par ? 1.0 / d->pixel_u : d->sdd / d->pixel_u;
    g.kvd = par ? 1.0 / d->pixel_v : d->sdd / d->pixel_v;
    g.ikvd = 1.0 / g.kvd;
    g.iTzd = 1.0 / d->voxel_z;
    g.col_offd = 0.5 * (d->ncols - 1) - d->shift_u;
    g.row_offd = 0.5 * (d->nrows - 1) - d->shift_v + 0.5;
    g.T = (float)T; g.Tz = (float)d->voxel_z;
    g.sod = (float)g.sodd; g.sdd = par ? 0.0f : (float)d->sdd;
    g.pu = (float)d->pixel_u; g.pv = (float)d->pixel_v;
    g.ku = (float)g.kud;
    g.col_off = (float)g.col_offd;
    g.v0 = (float)((-0.5 * (d->nrows - 1) + d->shift_v) * d->pixel_v);
    g.model = d->model;
    g.v0d = (-0.5 * (d->nrows - 1) + d->shift_v) * d->pixel_v;
    g.pvd = d->pixel_v;
    g.pu_d = d->pixel_u;
    g.zk0d = d->type == LEAP_FAN ? 0.5 : -g.zlo0d / d->voxel_z;

    G->views.resize(d->nviews);
    for (int a = 0; a < d->nviews; ++a) {
        const double c = std::cos(G->angles[a]), s = std::sin(G->angles[a]);
        SfView &v = G->views[a];
        v.cd = c; v.sd = s;
        v.c = (float)c; v.s = (float)s;
        v.p = (float)(h * c); v.q = (float)(h * s);
        v.par_out = (float)(h * (std::fabs(c) + std::fabs(s)) / d->pixel_u);
        v.par_in = (float)(h * std::fabs(std::fabs(c) - std::fabs(s)) / d->pixel_u);
        v.par_amp = (float)(T / std::fmax(std::fabs(c), std::fabs(s)));
        v.xmajor = std::fabs(c) >= std::fabs(s) ? 1 : 0;
    }

    if (d->model == LEAP_MODEL_SIDDON) build_ray_table(G);
    select_fast_kernels(G);
    return finish_handle(G, out);
}

extern "C" int leap_geometry_create(const leap_geometry_desc *d, leap_geometry **out)
{
    if (out) *out = nullptr;
    if (!d || !out) return invalid("null descriptor or output pointer");
    leap_geometry *G = nullptr;
    try {
        return create_handle(d, out, G);
    } catch (...) {          // std::bad_alloc from the tables
        free_handle(G);
        return invalid("out of host memory");
    }
}

extern "C" void leap_geometry_destroy(leap_geometry *G) { free_handle(G); }

extern "C" int leap_geometry_describe(const leap_geometry *G, char *buf, int32_t cap)
{
    if (!G || !buf || cap <= 0) return invalid("null handle or buffer");
    char fwd[160], back[160];
    const bool siddon = G->g.model == SF_MODEL_SIDDON;
    if (siddon && G->sd_columns)
        std::snprintf(fwd, sizeof fwd, "columns(rg=%d,slab=%d%s)", G->fp_rg, G->slab_width, G->sd_pairs == 2 ? ",pairs apart" : (G->sd_pairs ? ",pairs" : ""));
    else if (!siddon && G->fp_columns)
        std::snprintf(fwd, sizeof fwd, G->fp_parts > 1 ? "columns(nq=%d/%d,nkp=%d,rg=%d,cw=%d,slab=%d,parts=%d%s)" : "columns(nq=%d/%d,nkp=%d,rg=%d,cw=%d,slab=%d%.0d%s)",
                      G->fp_need_q, G->fp_nq, G->fp_nkp, G->fp_rg, G->fp_cw, G->slab_width, G->fp_parts > 1 ? G->fp_parts : 0, G->fp_rows ? ",rows" : "");
    else
        std::snprintf(fwd, sizeof fwd, G->flat ? "general(flat,span=%d)" : (G->mf_tiles ? "general(tiles)" : "general"), G->flat_span);
    if (G->bp_tiled && G->d_mdbp)
        std::snprintf(back, sizeof back, "tiled(zc=%d,window=%dx%d)", MD_BP_SHAPES[G->bp_shape].zc, G->bp_need_w, G->bp_need_h);
    else if (G->bp_tiled && siddon)
        std::snprintf(back, sizeof back, "tiled(nc=%d,zc=%d,window=%dx%d)", G->bp_nc, BP_SHAPES[G->bp_shape].zc, G->bp_need_w, G->bp_need_h);
    else if (G->bp_tiled)
        std::snprintf(back, sizeof back, "tiled(nc=%d,nv=%d,zc=%d%s,window=%dx%d)", G->bp_nc, G->bp_nv, BP_SHAPES[G->bp_shape].zc,
                      G->bp_shape == BP_WIDE_SHAPE ? ",wide" : "", G->bp_need_w, G->bp_need_h);
    else
        std::snprintf(back, sizeof back, G->flat ? "general(flat)" : (G->mf_tiled ? "general(tiled)" : "general"));
    if (G->bp_pair_shape >= 0) {
        const SfBpShape &S = BP_PAIR_SHAPES[G->bp_pair_shape];
        const size_t n = std::strlen(back);
        std::snprintf(back + n, sizeof back - n, "+%s(zc=%d,%dx%d)", G->bp_mirror ? "mirror" : "pairs", S.zc, S.pw, S.ph);
    }
    if (G->bp_split_shape >= 0) {
        const SfBpShape &S = (G->d_mdbp ? MD_BP_SPLIT_SHAPES : (siddon ? SD_BP_SPLIT_SHAPES : BP_SPLIT_SHAPES))[G->bp_split_shape];
        const size_t n = std::strlen(back);
        std::snprintf(back + n, sizeof back - n, "+split(%szc=%d,%dx%d)", G->bp_mirror ? "mirror," : "", S.zc, S.pw, S.ph);
    }
    if (G->bp_parts > 1) {
        const SfBpShape &S = (G->d_mdbp ? MD_BP_SPLIT_SHAPES : (siddon ? SD_BP_SPLIT_SHAPES : BP_SPLIT_SHAPES))[G->bp_parts_shape];
        const size_t n = std::strlen(back);
        std::snprintf(back + n, sizeof back - n, "+parts(%d,zc=%d,%dx%d)", G->bp_parts, S.zc, S.pw, S.ph);
    }
    const char *modules = G->g.type != SF_MODULAR ? "" : (G->geoms.empty() ? " (tilted modules)" : " (upright modules)");
    std::snprintf(buf, (size_t)cap, "type=%d model=%s A=%s AT=%s scratch=%zu%s cols/voxel<=%.2f rows/voxel<=%.2f voxels/row<=%.2f%s%s",
                  G->g.type, siddon ? "siddon" : "sf", fwd, back, G->scratch_bytes + G->back_floats * sizeof(float), modules, G->max_cols_per_voxel,
                  G->max_rows_per_voxel, G->max_voxels_per_row, G->note.empty() ? "" : " note=", G->note.c_str());
    return LEAP_OK;
}

static int check_call(const leap_geometry *G, const void *in, const void *out, int32_t batch)
{
    if (!G || !in || !out) return invalid("null handle or data pointer");
    if (batch <= 0) return invalid("batch must be positive");
    if (in == out) return invalid("input and output must not alias");
    return LEAP_OK;
}

extern "C" int leap_project(const leap_geometry *G, const float *d_vol, float *d_sino, int32_t batch, void *hip_stream)
{
    const int rc = check_call(G, d_vol, d_sino, batch);
    if (rc != LEAP_OK) return rc;
    return leap_launch_project_batch(G, d_vol, d_sino, batch, (hipStream_t)hip_stream);
}

extern "C" int leap_backproject(const leap_geometry *G, const float *d_sino, float *d_vol, int32_t batch, void *hip_stream)
{
    const int rc = check_call(G, d_sino, d_vol, batch);
    if (rc != LEAP_OK) return rc;
    return leap_launch_backproject_batch(G, d_sino, d_vol, batch, (hipStream_t)hip_stream);
}
