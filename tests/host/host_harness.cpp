// Host-side harness for the HIP library's host/device code (test infrastructure; built with g++, no GPU).
//
// It links the library's real host geometry module against stubs of the few HIP runtime calls that module makes,
// and supplies CPU versions of the two launchers that step the general kernel bodies thread by thread.  On top of
// that it re-enacts, on the CPU, the index arithmetic of the tiled back projection (does every LDS access of every
// thread of every workgroup stay inside the staged window?) and the arithmetic of the column-wise forward kernel
// (candidate slots, padded z-columns, axial overlap cascade), so that mistakes in them show up without a GPU.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../paper_2307_05801_amd/csrc/leap_internal.h"
#include "../../paper_2307_05801_amd/csrc/sf_general.h"
#define SF_NO_KERNELS
#include "../../paper_2307_05801_amd/csrc/sf_backproject_tiled.h"
#include "../../paper_2307_05801_amd/csrc/sf_project_columns.h"
#include "../../paper_2307_05801_amd/csrc/sf_project_rows.h"
#include "../../paper_2307_05801_amd/csrc/sf_flat.h"
#include "../../paper_2307_05801_amd/csrc/md_project_columns.h"
#include "../../paper_2307_05801_amd/csrc/md_backproject_tiled.h"
#include "../../paper_2307_05801_amd/csrc/md_footprint_tiled.h"
#include "../../paper_2307_05801_amd/csrc/sd_backproject_tiled.h"

// ---- stubs of the HIP runtime calls made by leap_geometry.cpp: "device" memory is host memory ---------------
extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
static long g_device_fail_at = -1;
static size_t g_device_limit = ~(size_t)0;
hipError_t hipMalloc(void **p, size_t n)
{
    *p = (g_device_fail_at >= 0 && g_device_fail_at-- == 0) || n > g_device_limit ? nullptr : std::malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
void host_fail_device_allocation(long n) { g_device_fail_at = n; }   // the n-th device allocation from now on fails (n < 0: none does)
void host_limit_device_allocations(size_t bytes) { g_device_limit = bytes ? bytes : ~(size_t)0; }         // larger ones fail from now on (0: none does)
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)std::malloc(1); return *e ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
// the host-memory entry points (leap_host.cpp): every asynchronous call happens at once, so the pipeline's buffer
// rotation and chunk arithmetic are checked, not its overlap
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
static long long g_capture = 0;                             // the capture every stream is in (0: none, below: the runtime will not say)
static std::vector<std::pair<char, hipEvent_t>> g_order;    // waits 'w' and records 'r', in order
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned) { g_order.push_back({'w', e}); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { g_order.push_back({'r', e}); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = g_capture > 0 ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return g_capture < 0 ? hipErrorStreamCaptureImplicit : hipSuccess;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t, hipStreamCaptureStatus *s, unsigned long long *id)
{
    *id = (unsigned long long)g_capture;
    return hipStreamIsCapturing(nullptr, s);
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
}

// The n-th allocation of this library from now on fails (n < 0: none does); returns how many the last setting has counted.
static std::atomic<long> g_fail_at{-1}, g_allocations{0};
static void *harness_new(size_t n)
{
    const long k = g_allocations++;
    void *p = g_fail_at >= 0 && k == g_fail_at ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n) { return harness_new(n); }
void *operator new[](size_t n) { return harness_new(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }
extern "C" long host_fail_allocation(long n)
{
    g_fail_at = n;
    return g_allocations.exchange(0);
}

// n turns at one shared memory, on streams[k] in capture captures[k]; turn `abandoned` is not ended by its call.  out: per turn the event waited for
// and the one recorded (0: none, 1: the eager turns', 2: the captured turns'), and what leap_capturing says of its stream.
extern "C" void host_shared_turns(const int64_t *streams, const int64_t *captures, int n, int abandoned, int64_t (*out)[3])
{
    LeapShared shared;
    (void)shared.create();
    auto name = [&](hipEvent_t e) { return e == shared.done ? 1 : (e == shared.captured ? 2 : -1); };
    for (int k = 0; k < n; ++k) {
        g_capture = captures[k];
        g_order.clear();
        out[k][2] = leap_capturing((hipStream_t)streams[k]);
        {
            LeapTurn turn(shared, (hipStream_t)streams[k]);
            (void)turn.begin();
            if (k != abandoned) (void)turn.end();
        }
        out[k][0] = out[k][1] = 0;
        for (const auto &call : g_order) out[k][call.first == 'r'] = name(call.second);
    }
    g_capture = 0;
}

// The slots that n calls on streams[k] take of a room of `slots`; a call on a stream below 0 takes them all.  out: the slot (-1: all), and how many
// waits the call's turn makes.
extern "C" void host_room_slots(const int64_t *streams, int n, int slots, int64_t (*out)[2])
{
    LeapRoom room;
    (void)room.create(slots);
    for (int k = 0; k < n; ++k) {
        const bool all = streams[k] < 0;
        const int slot = all ? 0 : room.pick((hipStream_t)streams[k]);
        g_order.clear();
        LeapTurn turn = all ? room.turn_at_all((hipStream_t)streams[k]) : room.turn(slot, (hipStream_t)streams[k]);
        (void)turn.begin();
        out[k][0] = all ? -1 : slot;
        out[k][1] = (int64_t)g_order.size();
        (void)turn.end();
    }
}

int leap_static_scratch_init(int) { return LEAP_OK; }   // the fixed device array exists on a GPU only

// ---- CPU launchers: the general kernel bodies, one "thread" at a time ----------------------------------------
int leap_launch_project(const leap_geometry *G, const float *vol, float *sino, hipStream_t)
{
    const SfGeom &g = G->g;
    constexpr int RC = 8;
    if (g.type == SF_MODULAR && g.model == SF_MODEL_SIDDON) {
#pragma omp parallel for collapse(2)
        for (int a = 0; a < g.nviews; ++a)
            for (int r = 0; r < g.nrows; ++r)
                for (int c = 0; c < g.ncols; ++c)
                    sino[((size_t)a * g.nrows + r) * g.ncols + c] = md_project_ray(g, G->d_poses[a], vol, r, c);
        return LEAP_OK;
    }
    if (G->d_mfviews) {
#pragma omp parallel for collapse(2)
        for (int a = 0; a < g.nviews; ++a)
            for (int r0 = 0; r0 < g.nrows; r0 += RC)
                for (int c = 0; c < g.ncols; ++c) {
                    float out[RC];
                    mf_project_rows<RC>(g, G->d_mfviews[a], vol, r0, c, out);
                    for (int rr = 0; rr < RC && r0 + rr < g.nrows; ++rr) sino[((size_t)a * g.nrows + r0 + rr) * g.ncols + c] = out[rr];
                }
        return LEAP_OK;
    }
    if (g.model == SF_MODEL_SIDDON) {
#pragma omp parallel for collapse(2)
        for (int a = 0; a < g.nviews; ++a)
            for (int r = 0; r < g.nrows; ++r)
                for (int c = 0; c < g.ncols; ++c)
                    sino[((size_t)a * g.nrows + r) * g.ncols + c] = sd_project_ray(g, G->d_raycols[(size_t)a * g.ncols + c], vol, r);
        return LEAP_OK;
    }
#pragma omp parallel for collapse(2)
    for (int a = 0; a < g.nviews; ++a)
        for (int r0 = 0; r0 < g.nrows; r0 += RC)
            for (int c = 0; c < g.ncols; ++c) {
                float out[RC];
                sf_project_ray_chunk<RC>(G->d_geoms ? G->d_geoms[a] : g, G->d_views[a], vol, c, r0, out);
                for (int rr = 0; rr < RC && r0 + rr < g.nrows; ++rr) sino[((size_t)a * g.nrows + r0 + rr) * g.ncols + c] = out[rr];
            }
    return LEAP_OK;
}

int leap_launch_project_batch(const leap_geometry *G, const float *vol, float *sino, int batch, hipStream_t st)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.nviews * g.nrows * g.ncols;
    for (int b = 0; b < batch; ++b) {
        const int rc = leap_launch_project(G, vol + b * nvol, sino + b * nsino, st);
        if (rc != LEAP_OK) return rc;
    }
    return LEAP_OK;
}

int leap_launch_backproject(const leap_geometry *G, const float *sino, float *vol, hipStream_t)
{
    const SfGeom &g = G->g;
    constexpr int ZC = 8;
    if (g.type == SF_MODULAR && g.model == SF_MODEL_SIDDON) {
#pragma omp parallel for collapse(2)
        for (int k = 0; k < g.nz; ++k)
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i) vol[((size_t)k * g.ny + j) * g.nx + i] = md_backproject_voxel(g, G->d_poses, sino, i, j, k);
        return LEAP_OK;
    }
    if (G->d_mfviews) {
#pragma omp parallel for collapse(2)
        for (int k = 0; k < g.nz; ++k)
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i) vol[((size_t)k * g.ny + j) * g.nx + i] = mf_backproject_voxel(g, G->d_mfviews, sino, i, j, k);
        return LEAP_OK;
    }
    if (g.model == SF_MODEL_SIDDON) {
#pragma omp parallel for collapse(2)
        for (int k = 0; k < g.nz; ++k)
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i)
                    vol[((size_t)k * g.ny + j) * g.nx + i] = sd_backproject_voxel(g, G->d_views, G->d_raycols, sino, i, j, k);
        return LEAP_OK;
    }
#pragma omp parallel for collapse(2)
    for (int k0 = 0; k0 < g.nz; k0 += ZC)
        for (int j = 0; j < g.ny; ++j)
            for (int i = 0; i < g.nx; ++i) {
                float acc[ZC] = {0};
                sf_backproject_column_chunk<ZC>(g, G->d_views, sino, i, j, k0, acc, G->d_geoms);
                for (int kk = 0; kk < ZC && k0 + kk < g.nz; ++kk) vol[((size_t)(k0 + kk) * g.ny + j) * g.nx + i] = acc[kk];
            }
    return LEAP_OK;
}

int leap_launch_backproject_batch(const leap_geometry *G, const float *sino, float *vol, int batch, hipStream_t st)
{
    const SfGeom &g = G->g;
    const size_t nvol = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.nviews * g.nrows * g.ncols;
    for (int b = 0; b < batch; ++b) {
        const int rc = leap_launch_backproject(G, sino + b * nsino, vol + b * nvol, st);
        if (rc != LEAP_OK) return rc;
    }
    return LEAP_OK;
}

// ---- tiled back projection: every thread's LDS reads against the staged window --------------------------------
// For one shape, chunks from voxel kfirst on: report[0..3] = {max column index read, max row index read, widest footprint in pixels,
// violations}.
static void host_check_windows(const leap_geometry *G, const SfBpShape S, int kfirst, int64_t *report)
{
    const SfGeom &g = G->g;
    const int NC = G->bp_nc, NV = G->bp_nv;
    const int tiles_x = (g.nx + BP_T - 1) / BP_T, tiles_y = (g.ny + BP_T - 1) / BP_T, chunks = (g.nz - kfirst + S.zc - 1) / S.zc;
    int maxc = -1, maxr = -1, maxspan = 0;
    long bad = 0;
#pragma omp parallel for collapse(2) reduction(max : maxc, maxr, maxspan) reduction(+ : bad)
    for (int a = 0; a < g.nviews; ++a)
        for (int ty = 0; ty < tiles_y; ++ty)
            for (int tx = 0; tx < tiles_x; ++tx)
                for (int ch = 0; ch < chunks; ++ch) {
                    const SfGeom &g = G->geoms.empty() ? G->g : G->geoms[a];      // modular: the view's own parameter block
                    const int i0 = tx * BP_T, j0 = ty * BP_T, k0 = kfirst + ch * S.zc;
                    const double zlo = fma((double)k0, g.Tzd, g.zlo0d);
                    const float z0 = (float)zlo, z1 = z0 + (float)S.zc * g.Tz;
                    const float hx = 0.5f * (float)(BP_T - 1) * g.T;
                    const float xc = (float)(g.x0d + ((double)i0 + 0.5 * (BP_T - 1)) * g.Td);
                    const float yc = (float)(g.y0d + ((double)j0 + 0.5 * (BP_T - 1)) * g.Td);
                    const SfWindow w = sf_bp_window(g, G->views[a], xc, yc, hx, z0, z1, G->bp_wh, NC, NV);
                    for (int tj = 0; tj < BP_T; ++tj)
                        for (int ti = 0; ti < BP_T; ++ti) {
                            const int i = std::min(i0 + ti, g.nx - 1), j = std::min(j0 + tj, g.ny - 1);
                            SfColumn f;
                            if (g.type == SF_CONE_CURVED) {      // as the kernel: relative to the tile centre
                                const double xcd = g.x0d + ((double)i0 + 0.5 * (BP_T - 1)) * g.Td;
                                const double ycd = g.y0d + ((double)j0 + 0.5 * (BP_T - 1)) * g.Td;
                                const SfView &v = G->views[a];
                                const double tref = fma(ycd, v.cd, -xcd * v.sd), dnref = g.sodd - fma(xcd, v.cd, ycd * v.sd);
                                f = sf_column_curved_ref(g, v, i, j, tref, dnref, atan2(tref, dnref));
                            } else {
                                f = sf_column(g, G->views[a], i, j);
                            }
                            int cf, cl;
                            sf_col_range(f, cf, cl);
                            const SfRowsOfVoxels ax = sf_rows_of_voxels(g, f, zlo);
                            const int c_lo = cf - w.c0, c_hi = c_lo + NC - 1;
                            const int r_lo = ax.rb - w.r0;
                            // last row read: first row of the last voxel plus NV-1 (the shared-row variant reads the same set)
                            const int r_hi = r_lo + (int)std::floor(fmaf(ax.av, (float)(S.zc - 1), ax.phi0)) + NV - 1;
                            maxc = std::max(maxc, c_hi);
                            maxr = std::max(maxr, r_hi);
                            maxspan = std::max(maxspan, cl - cf + 1);
                            if (c_lo < 0 || c_hi >= S.pw || r_lo < 0 || r_hi >= S.ph) ++bad;   // read outside the staged window
                            if (cl - cf + 1 > NC) ++bad;                                          // footprint wider than NC columns
                            if (ax.av > (float)(NV - 1) * 1.000001f) ++bad;                       // voxel taller than NV-1 rows
                        }
                }
    report[0] = maxc; report[1] = maxr; report[2] = maxspan; report[3] = bad;
}

// report[0..7] = {tiled?, nc, nv, zc, max column index read, max row index read, widest footprint in pixels, violations}: the kernel of one
// volume per workgroup; violations also under the windows of two volumes and of shared views, every shape a launch of the handle may take.
extern "C" int host_check_backproject_windows(const leap_geometry *G, int64_t *report)
{
    std::fill(report, report + 8, 0);
    report[0] = G->bp_tiled;
    if (!G->bp_tiled) return 0;
    const int kfirst = G->bp_mirror ? sf_mirror_first_voxel_above(G->g.nz) : 0;
    int64_t r[4];
    host_check_windows(G, BP_SHAPES[G->bp_shape], 0, report + 4);
    report[1] = G->bp_nc; report[2] = G->bp_nv; report[3] = BP_SHAPES[G->bp_shape].zc;
    if (G->bp_pair_shape >= 0) {
        host_check_windows(G, BP_PAIR_SHAPES[G->bp_pair_shape], kfirst, r);
        report[7] += r[3];
    }
    for (int sh = 0; sh < BP_NSPLIT_SHAPES; ++sh)
        if ((G->bp_split_fits | G->bp_parts_fits) >> sh & 1u) {
            host_check_windows(G, BP_SPLIT_SHAPES[sh], kfirst, r);
            report[7] += r[3];
        }
    return report[7] != 0;
}

// ---- tiled back projection: who stages what ----------------------------------------------------------------------
// Number of cells of a window that are not written by exactly one (thread, step) of a group of 256 threads: a cell without a
// writer holds another view's sample, one with two writers in different steps is written without an order between them.
template <int PW, int PH>
static long host_staging_roles()
{
    constexpr int step = 256 / PW, nstage = (PH + step - 1) / step;
    std::vector<int> writers((size_t)PH * PW, 0);
    for (int tid = 0; tid < 256; ++tid)
        for (int s = 0; s < nstage; ++s) {
            const int row = sf_stage_row<PW, PH>(tid) + step * s;
            if (row < PH) ++writers[(size_t)row * PW + sf_stage_column<PW>(tid)];
        }
    long bad = 0;
    for (int w : writers) bad += w != 1;
    return bad;
}

extern "C" long host_check_staging_roles()
{
    static_assert(BP_NSHAPES == 7 && BP_NPAIR_SHAPES == 4 && BP_NSPLIT_SHAPES == 3, "every shape is checked");
#define ROLES(S) host_staging_roles<S.pw, S.ph>()
    return ROLES(BP_SHAPES[0]) + ROLES(BP_SHAPES[1]) + ROLES(BP_SHAPES[2]) + ROLES(BP_SHAPES[3]) + ROLES(BP_SHAPES[4]) + ROLES(BP_SHAPES[5]) +
           ROLES(BP_SHAPES[6]) + ROLES(BP_PAIR_SHAPES[0]) + ROLES(BP_PAIR_SHAPES[1]) + ROLES(BP_PAIR_SHAPES[2]) + ROLES(BP_PAIR_SHAPES[3]) +
           ROLES(BP_SPLIT_SHAPES[0]) + ROLES(BP_SPLIT_SHAPES[1]) + ROLES(BP_SPLIT_SHAPES[2]);
#undef ROLES
}

// ---- cylinder: the tile-relative column function of the tiled kernel against the general one ------------------------
// out[0] = largest |difference| of the column coordinate (pixels), out[1] = of the four knot offsets, over every view,
// tile and voxel column; out[2] = largest corner angle met (rad).
extern "C" int host_curved_column_deviation(const leap_geometry *G, double *out)
{
    const SfGeom &g = G->g;
    out[0] = out[1] = out[2] = 0.0;
    if (g.type != SF_CONE_CURVED) return -1;
    const int tiles_x = (g.nx + BP_T - 1) / BP_T, tiles_y = (g.ny + BP_T - 1) / BP_T;
    double dxi = 0.0, dof = 0.0, ang = 0.0;
#pragma omp parallel for collapse(2) reduction(max : dxi, dof, ang)
    for (int a = 0; a < g.nviews; ++a)
        for (int ty = 0; ty < tiles_y; ++ty)
            for (int tx = 0; tx < tiles_x; ++tx) {
                const SfView &v = G->views[a];
                const double xcd = g.x0d + ((double)(tx * BP_T) + 0.5 * (BP_T - 1)) * g.Td;
                const double ycd = g.y0d + ((double)(ty * BP_T) + 0.5 * (BP_T - 1)) * g.Td;
                const double tref = fma(ycd, v.cd, -xcd * v.sd), dnref = g.sodd - fma(xcd, v.cd, ycd * v.sd);
                const double gref = atan2(tref, dnref);
                for (int tj = 0; tj < BP_T; ++tj)
                    for (int ti = 0; ti < BP_T; ++ti) {
                        const int i = std::min(tx * BP_T + ti, g.nx - 1), j = std::min(ty * BP_T + tj, g.ny - 1);
                        const SfColumn p = sf_column(g, v, i, j), q = sf_column_curved_ref(g, v, i, j, tref, dnref, gref);
                        dxi = std::max(dxi, std::fabs(p.xi - q.xi));
                        dof = std::max(dof, (double)std::max(std::max(std::fabs(p.o0 - q.o0), std::fabs(p.o1 - q.o1)),
                                                             std::max(std::fabs(p.o2 - q.o2), std::fabs(p.o3 - q.o3))));
                        ang = std::max(ang, (double)std::max(std::fabs(p.o0), std::fabs(p.o3)) / g.ku);
                    }
            }
    out[0] = dxi; out[1] = dof; out[2] = ang;
    return 0;
}

// ---- cylinder: the bundle-relative column function of the column-wise forward kernel against the general one ---------
// Over every view, bundle of cw columns and voxel column that touches one of them: out[0] = largest |difference| of the column coordinate
// (pixels), out[1] = of the knot offsets, out[2] = of the distance from the source (relative); out[3] = largest tangent fed to the
// arc-tangent polynomials, out[4] = the number of voxel columns compared.
extern "C" int host_curved_bundle_deviation(const leap_geometry *G, double *out)
{
    const SfGeom &g = G->g;
    if (g.type != SF_CONE_CURVED || !G->fp_columns) return -1;
    const int cw = G->fp_cw, nbundles = (g.ncols + cw - 1) / cw;
    double dxi = 0.0, dof = 0.0, dden = 0.0, tangent = 0.0, count = 0.0;
#pragma omp parallel for collapse(2) reduction(max : dxi, dof, dden, tangent) reduction(+ : count)
    for (int a = 0; a < g.nviews; ++a)
        for (int b = 0; b < nbundles; ++b) {
            const SfView &v = G->views[a];
            const SfNearRay ray = sf_near_ray(g, sf_bundle_middle(b * cw, cw));
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i) {
                    const SfColumn p = sf_column(g, v, i, j);
                    if (p.xi + p.o3 < b * cw - 0.5 || p.xi + p.o0 > b * cw + cw - 0.5) continue;
                    const SfColumn q = sf_column_curved_near(g, v, i, j, ray);
                    dxi = std::max(dxi, std::fabs(p.xi - q.xi));
                    dof = std::max(dof, (double)std::max(std::max(std::fabs(p.o0 - q.o0), std::fabs(p.o1 - q.o1)),
                                                         std::max(std::fabs(p.o2 - q.o2), std::fabs(p.o3 - q.o3))));
                    dden = std::max(dden, std::max(std::fabs(q.den / p.den - 1.0), std::fabs(q.inv * p.den - 1.0)));
                    tangent = std::max(tangent, std::tan(std::max(std::fabs(p.xi - ray.xi0), (double)std::max(std::fabs(p.o0), std::fabs(p.o3))) / g.kud));
                    count += 1.0;
                }
        }
    out[0] = dxi; out[1] = dof; out[2] = dden; out[3] = tangent; out[4] = count;
    return 0;
}

// ---- column-wise forward projection: the kernel's own per-lane functions, stepped serially ------------------------------
// One (view, bundle of CW detector columns) at a time, the way a wavefront of sf_project_columns works through it: the
// host's marching axis for the bundle, candidate slots per slab, sf_candidate_record for every candidate, then for every
// pair of adjacent rows sf_place_row, a window of P voxels read from the z-fastest copy (zero outside the padded
// column, as the kernel's buffer loads return) and the axial sums in the body of the candidate's height class, from the four numbers its lane
// leaves in LDS.  The whole volume stands in for one slab.
template <int CW, int HC, int CLS>
static void host_pairs_of_candidate(const SfGeom &g, const float *col, int nzp, double mu, double zkp, const float (&fa)[CW],
                                    std::vector<float> &acc)
{
    using C = SfPairClass<CLS>;
    SfPairOffsets k;
    sf_unpack_offsets<CLS>(sf_pack_offsets<HC>(HC > 1 ? sf_pair_class((float)mu) : HC, sf_pair_offsets((float)mu)), k);
    for (int r = 0; r < g.nrows; r += 2) {
        float fr1;
        unsigned hi;
        sf_place_row((double)r - g.row_offd, mu, zkp, fr1, hi);
        const int kf = (int)(hi - FP_KAP_HI);
        float x[C::P];
        for (int t = 0; t < C::P; ++t) x[t] = (kf + t >= 0 && kf + t < nzp) ? col[kf + t] : 0.0f;
        float sa, sb;
        sf_pair_apply<C::LO2, C::HI2>(x, sf_pair_weights<C::LO2, C::HI2>(fr1, k), sa, sb);
        for (int cw = 0; cw < CW; ++cw) {
            acc[(size_t)r * CW + cw] = fmaf(fa[cw], sa, acc[(size_t)r * CW + cw]);
            if (r + 1 < g.nrows) acc[(size_t)(r + 1) * CW + cw] = fmaf(fa[cw], sb, acc[(size_t)(r + 1) * CW + cw]);
        }
    }
}

// The class whose body a candidate of a scan of highest class HC is walked in.
template <int CW, int HC>
static void host_pairs_of_scan(const SfGeom &g, const float *col, int nzp, double mu, double zkp, const float (&fa)[CW], std::vector<float> &acc)
{
    switch (HC > 1 ? std::min(sf_pair_class((float)mu), HC) : HC) {
    case 0: host_pairs_of_candidate<CW, HC, 0>(g, col, nzp, mu, zkp, fa, acc); break;
    case 1: host_pairs_of_candidate<CW, HC, 1>(g, col, nzp, mu, zkp, fa, acc); break;
    case 2: host_pairs_of_candidate<CW, HC, 2>(g, col, nzp, mu, zkp, fa, acc); break;
    case 3: host_pairs_of_candidate<CW, HC, 3>(g, col, nzp, mu, zkp, fa, acc); break;
    default: host_pairs_of_candidate<CW, HC, 4>(g, col, nzp, mu, zkp, fa, acc); break;
    }
}

// The layers of a bundle as the waves that share it take them: layer(n, sums) for every layer of every part, the parts' sums added in order.  Returns
// how many layers were not taken once.
template <class Layer>
static long host_layers(const leap_geometry *G, const SfSlab &slab, std::vector<float> &acc, Layer layer)
{
    int nq_log2 = 2;
    while ((1 << nq_log2) < G->fp_nq) ++nq_log2;
    std::vector<int> taken(slab.n1 - slab.n0, 0);
    for (int part = 0; part < G->fp_parts; ++part) {
        std::vector<float> sums(acc.size(), 0.f);
        int n_first = slab.n0, n_end = slab.n1;
        if (G->fp_parts > 1) fp_part_of(slab, 64 >> nq_log2, part, G->fp_parts, n_first, n_end);
        for (int n = n_first; n < n_end; ++n) {
            if (n >= slab.n0 && n < slab.n1) ++taken[n - slab.n0];
            layer(n, sums);
        }
        for (size_t e = 0; e < acc.size(); ++e) acc[e] = part ? acc[e] + sums[e] : sums[e];
    }
    return (long)taken.size() - (long)std::count(taken.begin(), taken.end(), 1);
}

template <int CW>
static long host_project_bundles(const leap_geometry *G, const std::vector<float> (&volz)[2], int nzp, float *sino)
{
    const int NQ = G->fp_nq;
    const int nbundles = (G->g.ncols + CW - 1) / CW;
    long uncovered = 0;
#pragma omp parallel for collapse(2) reduction(+ : uncovered)
    for (int a = 0; a < G->g.nviews; ++a)
        for (int b = 0; b < nbundles; ++b) {
            const int c0 = b * CW;
            const SfGeom &g = G->geoms.empty() ? G->g : G->geoms[a];      // modular: the view's own parameter block
            const double zkp = sf_kappa_const(g);
            const SfView v = G->views[a];
            const int xmajor = G->major[(size_t)a * nbundles + b];
            const SfRayLines L = sf_ray_lines(g, v, c0, CW, xmajor);
            const int n_major = xmajor ? g.nx : g.ny, n_minor = xmajor ? g.ny : g.nx;
            const SfSlab slab = {0, n_major, xmajor, 1, n_major};
            std::vector<float> total((size_t)g.nrows * CW, 0.f);
            const bool curved = g.type == SF_CONE_CURVED;
            SfNearRay ray = {};
            if (curved) ray = sf_near_ray(g, sf_bundle_middle(c0, CW));
            uncovered += host_layers(G, slab, total, [&](int n, std::vector<float> &acc) {
                int qf, ql;
                sf_candidates(L, n, qf, ql);
                if (ql - qf + 1 > NQ) ++uncovered;
                for (int s = 0; s < NQ; ++s) {
                    const int q = qf + s;
                    if (q < 0 || q >= n_minor || q > ql) continue;
                    const int i = xmajor ? n : q, j = xmajor ? q : n;
                    float fa[CW];
                    double mu;
                    if (!sf_footprint_record<CW>(g, curved ? sf_column_curved_near(g, v, i, j, ray) : sf_column(g, v, i, j), c0, true, fa, mu)) continue;
                    const float *col = &volz[xmajor][(size_t)sf_slab_column(slab, g.nx, i, j) * nzp];
                    switch (fp_height_class(G->fp_nkp)) {
                    case 0: host_pairs_of_scan<CW, 0>(g, col, nzp, mu, zkp, fa, acc); break;
                    case 1: host_pairs_of_scan<CW, 1>(g, col, nzp, mu, zkp, fa, acc); break;
                    case 2: host_pairs_of_scan<CW, 2>(g, col, nzp, mu, zkp, fa, acc); break;
                    case 3: host_pairs_of_scan<CW, 3>(g, col, nzp, mu, zkp, fa, acc); break;
                    default: host_pairs_of_scan<CW, 4>(g, col, nzp, mu, zkp, fa, acc); break;
                    }
                }
            });
            for (int cw = 0; cw < CW && c0 + cw < g.ncols; ++cw) {
                const SfAmpCol ac = sf_amp_col(g, v, c0 + cw);
                for (int r = 0; r < g.nrows; ++r)
                    sino[((size_t)a * g.nrows + r) * g.ncols + c0 + cw] = sf_amp(g, v, ac, r) * total[(size_t)r * CW + cw];
            }
        }
    return uncovered;
}

// Returns -1 when the handle does not use the column kernel, else the number of (view, bundle, slab) cases in which the
// candidate slots do not cover the candidate range (must be 0).
extern "C" long host_project_columns(const leap_geometry *G, const float *vol, float *sino)
{
    const SfGeom &g = G->g;
    if (!G->fp_columns) return -1;
    const int nzp = g.nz + 2 * FP_PAD;
    // the z-fastest copy in both slab layouts (a slab across x is laid out differently from one across y)
    std::vector<float> volz[2];
    for (int xmajor = 0; xmajor < 2; ++xmajor) {
        const SfSlab slab = {0, xmajor ? g.nx : g.ny, xmajor, 1, xmajor ? g.nx : g.ny};
        volz[xmajor].assign((size_t)g.nx * g.ny * nzp, 0.f);
        for (int k = 0; k < g.nz; ++k)
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i)
                    volz[xmajor][(size_t)sf_slab_column(slab, g.nx, i, j) * nzp + FP_PAD + k] = vol[((size_t)k * g.ny + j) * g.nx + i];
    }
    switch (G->fp_cw) {
    case 1: return host_project_bundles<1>(G, volz, nzp, sino);
    case 2: return host_project_bundles<2>(G, volz, nzp, sino);
    default: return host_project_bundles<4>(G, volz, nzp, sino);
    }
}

// Tiles that the back projection's order of workgroups leaves out or names twice, in one layer of chunks.
extern "C" long host_check_tile_order(unsigned tiles_x, unsigned tiles_y, unsigned y)
{
    const unsigned tiles = tiles_x * tiles_y;
    std::vector<int> seen(tiles, 0);
    long wrong = 0;
    for (unsigned x = 0; x < tiles; ++x) {
        const unsigned tile = sf_bp_tile(x, y, tiles, tiles_x);
        if (tile >= tiles || seen[tile]++) ++wrong;
    }
    return wrong;
}

// How many of a launch's items go two to a wave.
// Blocks of a slab by the waves that fp_waves_for leaves: the groups that are added must be those of all the parts, in their order (empty ones aside).
extern "C" long host_check_waves_for()
{
    long bad = 0;
    auto groups = [](int n, int block, int parts) {
        std::vector<std::pair<int, int>> out;
        for (int p = 0; p < parts; ++p) {
            int first = 0, end = n;
            if (parts > 1) fp_part_of({0, n, 1, 1, n}, block, p, parts, first, end);
            if (end > first) out.push_back({first, end});
        }
        return out;
    };
    for (int block : {4, 8, 16})
        for (int n = 1; n <= 200; ++n)
            for (int parts : {1, 2, 4})
                for (int rows = parts == 2; rows < 2; ++rows) {
                    const int waves = fp_waves_for(n, block, parts, rows);
                    if (!(waves == 1 || waves == FP_PARTS || (waves == 2 && rows)) || waves > parts || groups(n, block, waves) != groups(n, block, parts)) ++bad;
                }
    return bad;
}

// The slab width and the items per launch of a batch on the handle's scratch.
extern "C" void host_plan_scratch(const leap_geometry *G, int batch, int64_t out[2])
{
    int width = 0, items = 0;
    (void)leap_plan_scratch(G, G->scratch_bytes / sizeof(float), batch, width, items);
    out[0] = width;
    out[1] = items;
}

extern "C" int host_forward_paired(const leap_geometry *G, int items) { return leap_forward_paired(G, items); }

// Back projection of a launch's items: the shape whose groups of threads share the views (-1: none), pairs of items per workgroup.
extern "C" int host_back_split_shape(const leap_geometry *G, int items) { return leap_back_split_shape(G, items); }
extern "C" int host_siddon_split_shape(const leap_geometry *G, int items) { return leap_siddon_split_shape(G, items); }
extern "C" int host_back_pairs(const leap_geometry *G, int items) { return leap_back_pairs(G, items); }

// Voxels a pair of adjacent rows reads in the scan's highest height class.
extern "C" int host_voxels_of_pair(const leap_geometry *G)
{
    static constexpr int voxels[] = {SfPairClass<0>::P, SfPairClass<1>::P, SfPairClass<2>::P, SfPairClass<3>::P, SfPairClass<4>::P};
    return voxels[fp_height_class(G->fp_nkp)];
}

// ---- Siddon column-wise forward projection: the kernel's own functions, serially, with every read of the padded copy
// checked ----
// Returns -1 when the handle does not use that kernel, else the number of reads that would leave the scratch array.
extern "C" long host_sd_project_columns(const leap_geometry *G, const float *vol, float *sino)
{
    const SfGeom &gk = G->g;
    const SfGeom &g = gk;
    if (!G->sd_columns) return -1;
    const int nzp = g.nz + 2 * FP_PAD, kmax = nzp - 2;
    const size_t total = ((size_t)g.nx * g.ny + 1) * nzp;
    const unsigned zero_col = (unsigned)g.nx * (unsigned)g.ny * (unsigned)nzp;
    std::vector<float> volz(total, 0.f);
    for (int k = 0; k < g.nz; ++k)
        for (int j = 0; j < g.ny; ++j)
            for (int i = 0; i < g.nx; ++i) volz[((size_t)j * g.nx + i) * nzp + FP_PAD + k] = vol[((size_t)k * g.ny + j) * g.nx + i];
    long bad = 0;
#pragma omp parallel for collapse(2) reduction(+ : bad)
    for (int a = 0; a < g.nviews; ++a)
        for (int c = 0; c < g.ncols; ++c) {
            const SfGeom &g = G->geoms.empty() ? gk : G->geoms[a];        // modular: the view's own parameter block
            const SdRayCol R = G->raycols[(size_t)a * g.ncols + c];
            const int n_major = R.xmajor ? g.nx : g.ny, n_minor = R.xmajor ? g.ny : g.nx;
            for (int r = 0; r < g.nrows; ++r) {
                const SdAxial A = sd_axial(g, R, r);
                float acc = 0.f;
                for (int n = 0; n < n_major; ++n) {
                    const SdSplit s = sd_slab_split(R, n);
                    const bool a_ok = s.qa >= 0 && s.qa < n_minor, b_ok = s.qa != s.qb && s.qb >= 0 && s.qb < n_minor;
                    const unsigned base_a = a_ok ? (unsigned)(R.xmajor ? s.qa * g.nx + n : n * g.nx + s.qa) * (unsigned)nzp : zero_col;
                    const unsigned base_b = b_ok ? (unsigned)(R.xmajor ? s.qb * g.nx + n : n * g.nx + s.qb) * (unsigned)nzp : zero_col;
                    int kf;
                    float tlow;
                    sd_axial_place(A, fma((double)n, R.dh, R.h0), kmax, kf, tlow);
                    if (kf < 0 || (size_t)base_a + kf + 1 >= total || (size_t)base_b + kf + 1 >= total) { ++bad; continue; }
                    const float *xa = &volz[(size_t)base_a + kf], *xb = &volz[(size_t)base_b + kf];
                    acc = s.qa != s.qb ? sd_gather_two(xa, xb, A.inc, s.f, 1.0f - s.f, tlow, acc) : sd_gather_one(xa, tlow, acc);
                }
                sino[((size_t)a * g.nrows + r) * g.ncols + c] = sd_ray_length(R, A.vr) * acc;
            }
        }
    return bad;
}

// The same for the kernel with two adjacent rows per lane: one load of four voxels per pair and in-plane cell, zero outside the
// padded column, as the kernel's buffer loads return.  Returns -1 when the handle does not use that kernel, else the number of
// pairs whose cells do not fit the load.
template <bool SPREAD>
static long host_sd_pairs(const leap_geometry *G, const float *vol, float *sino)
{
    const int nx = G->g.nx, ny = G->g.ny, nz = G->g.nz, nzp = nz + 2 * FP_PAD;
    std::vector<float> volz((size_t)nx * ny * nzp, 0.f);
    for (int k = 0; k < nz; ++k)
        for (int j = 0; j < ny; ++j)
            for (int i = 0; i < nx; ++i) volz[((size_t)j * nx + i) * nzp + FP_PAD + k] = vol[((size_t)k * ny + j) * nx + i];
    long bad = 0;
#pragma omp parallel for collapse(2) reduction(+ : bad)
    for (int a = 0; a < G->g.nviews; ++a)
        for (int c = 0; c < G->g.ncols; ++c) {
            const SfGeom &g = G->geoms.empty() ? G->g : G->geoms[a];
            const SdRayCol R = G->raycols[(size_t)a * g.ncols + c];
            const int n_major = R.xmajor ? nx : ny, n_minor = R.xmajor ? ny : nx;
            for (int r = 0; r < g.nrows; r += 2) {
                const SdPairRow A[2] = {sd_pair_row(g, R, r), sd_pair_row(g, R, r + 1)};
                float acc[2] = {0.f, 0.f};
                for (int n = 0; n < n_major; ++n) {
                    const SdSplit s = sd_slab_split(R, n);
                    float f, omf;
                    sd_pair_crossing(s.f, f, omf);
                    const bool two = s.qa != s.qb, a_ok = s.qa >= 0 && s.qa < n_minor, b_ok = two && s.qb >= 0 && s.qb < n_minor;
                    if (!a_ok && !b_ok) continue;
                    unsigned hi[2];
                    float low[2], x[2][4];
                    for (int p = 0; p < 2; ++p) sd_pair_place(A[p], fma((double)n, R.dh, R.h0), hi[p], low[p]);
                    const unsigned d = hi[1] - hi[0];
                    if (d > 2u || (SPREAD && d == 0u)) ++bad;
                    const long k0 = (long)(int)(hi[0] - FP_KAP_HI) - 1;
                    for (int t = 0; t < 4; ++t)
                        for (int p = 0; p < 2; ++p) {
                            const int q = p ? s.qb : s.qa;
                            const size_t col = (size_t)(R.xmajor ? q * nx + n : n * nx + q) * nzp;
                            x[p][t] = (p ? b_ok : a_ok) && k0 + t >= 0 && k0 + t < nzp ? volz[col + k0 + t] : 0.f;
                        }
                    float lo[2], up[2];
                    for (int p = 0; p < 2; ++p) sd_pair_upper_row<SPREAD>(x[p], d, lo[p], up[p]);
                    if (two) {
                        acc[0] = sd_pair_two(x[0][0], x[0][1], x[1][0], x[1][1], A[0].inc, f, omf, low[0], acc[0]);
                        acc[1] = sd_pair_two(lo[0], up[0], lo[1], up[1], A[1].inc, f, omf, low[1], acc[1]);
                    } else {
                        acc[0] = sd_pair_one(x[0][0], x[0][1], low[0], acc[0]);
                        acc[1] = sd_pair_one(lo[0], up[0], low[1], acc[1]);
                    }
                }
                for (int p = 0; p < 2 && r + p < g.nrows; ++p)
                    sino[((size_t)a * g.nrows + r + p) * g.ncols + c] = sd_ray_length(R, A[p].vr) * acc[p];
            }
        }
    return bad;
}

// One slab's value for given cells, in-plane crossing f and share `low` of the slab in the lower axial cells.
extern "C" float host_sd_pair_slab(float alo, float aup, float blo, float bup, int two, int inc, float at, float low)
{
    float f, omf;
    sd_pair_crossing(at, f, omf);
    return two ? sd_pair_two(alo, aup, blo, bup, inc != 0, f, omf, low, 0.0f) : sd_pair_one(alo, aup, low, 0.0f);
}

extern "C" long host_sd_project_pairs(const leap_geometry *G, const float *vol, float *sino)
{
    if (!G->sd_pairs) return -1;
    return G->sd_pairs == 2 ? host_sd_pairs<true>(G, vol, sino) : host_sd_pairs<false>(G, vol, sino);
}

// ---- Siddon model, tiled back projection: tile by tile, with the kernel's own functions -------------------------------------
// report[0]: (view, tile, chunk) windows beyond what the instance stages; report[1]: reads outside the staged window;
// report[2]: slots outside the per-thread sums; report[3]: rows walked in pairs of which both add to the same voxel.
// Returns -1 when the handle does not use that kernel, else the sum of the four.
template <int ZC, int PW, int PH>
static void host_sd_bp_shape(const leap_geometry *G, const float *sino, float *vol, int64_t *report)
{
    const SfGeom &g = G->g;
    constexpr int NSLOT = ZC + 4;
    const bool apart = G->sd_min_row_step > 1.0 + 1e-6;
    const int tiles_x = (g.nx + BP_T - 1) / BP_T, tiles_y = (g.ny + BP_T - 1) / BP_T, chunks = (g.nz + ZC - 1) / ZC;
    int64_t wide = 0, outside = 0, badslot = 0, shared = 0;
#pragma omp parallel for collapse(2) reduction(+ : wide, outside, badslot, shared)
    for (int ch = 0; ch < chunks; ++ch)
        for (int tile = 0; tile < tiles_x * tiles_y; ++tile) {
            const int i0 = (tile % tiles_x) * BP_T, j0 = (tile / tiles_x) * BP_T, k0 = ch * ZC;
            std::vector<float> sums((size_t)NSLOT * 256, 0.f), buf((size_t)PH * PW), rinv(PH);
            for (int a = 0; a < g.nviews; ++a) {
                const SfGeom &gv = G->geoms.empty() ? G->g : G->geoms[a];
                const SdBpScene scene = sd_bp_scene<ZC>(gv, i0, j0, k0);
                const SfWindow win = sd_bp_window(gv, G->views[a], scene.xc, scene.yc, 0.5f * (float)BP_T * gv.T, scene.z0, scene.z1);
                wide += win.need_w > PW || win.need_h > PH;
                for (int row = 0; row < PH; ++row)
                    for (int sc = 0; sc < PW; ++sc) {
                        const int c = win.c0 + sc, r = win.r0 + row, cc = std::min(std::max(c, 0), g.ncols - 1);
                        const bool in = c >= 0 && c < g.ncols && r >= 0 && r < g.nrows;
                        const SdRayCol &R = G->raycols[(size_t)a * g.ncols + cc];
                        const float vr = (float)sd_row_v(gv, r), t = R.vscale * vr;
                        buf[(size_t)row * PW + sc] = in ? sino[((size_t)a * g.nrows + r) * g.ncols + c] * sf_sqrt(fmaf(t, t, R.lxy * R.lxy)) : 0.f;
                        rinv[row] = sd_bp_inverse(fabsf(vr));
                    }
                for (int tid = 0; tid < 256; ++tid) {
                    const int ic = std::min(i0 + (tid & (BP_T - 1)), g.nx - 1), jc = std::min(j0 + (tid >> 4), g.ny - 1);
                    const SfColumn f = sf_column(gv, G->views[a], ic, jc);
                    const int cfirst = (int)ceil(f.xi + (double)f.o0 - 1e-3), clast = (int)floor(f.xi + (double)f.o3 + 1e-3);
                    for (int m = 0; m < G->bp_nc; ++m) {
                        const int c = cfirst + m, wc = c - win.c0;
                        if (c > clast || c < 0 || c >= g.ncols || wc < 0 || wc >= PW) continue;
                        const SdRayCol R = G->raycols[(size_t)a * g.ncols + c];
                        const int n = R.xmajor ? ic : jc, q = R.xmajor ? jc : ic;
                        const SdSplit s = sd_slab_split(R, n);
                        const float t0 = q == s.qa ? 0.0f : s.f, t1 = q == s.qa ? s.f : 1.0f;
                        if ((q != s.qa && q != s.qb) || !(t1 - t0 > 0.0f)) continue;
                        const float dt = t1 - t0;
                        const double ha = fma((double)n + (double)t0, R.dh, R.h0), hb = fma((double)n + (double)t1, R.dh, R.h0);
                        const double hmin = fmin(ha, hb), hmax = fmax(ha, hb);
                        const float scale = dt * sd_bp_inverse((float)(hmax - hmin)) * 2.3283064365386963e-10f;
                        const int H = std::min(win.need_h, PH);
                        const int rz = sd_bp_plane_row(gv, win.r0, H);
                        for (int run = 0; run < 2; ++run) {
                            const int rs = run ? rz : 0, re = run ? H : rz;
                            const double h = run ? hmin : hmax, dq = sd_bp_advance(gv.pvd, h);
                            double at = sd_bp_position<ZC>(sd_row_v(gv, win.r0 + rs), h, scene.zrel0, !((float)(hmax - hmin) > 0.0f));
                            std::vector<unsigned> slots;
                            for (int row = rs; row < re; ++row, at -= dq) {
                                if (row < 0 || row >= PH) { ++outside; continue; }
                                unsigned slot;
                                float wl;
                                sd_bp_place<ZC>(at, scale * rinv[row], dt, slot, wl);
                                slot -= SD_BP_HI;
                                slots.push_back(slot);
                                if (slot + 1 >= (unsigned)NSLOT) { ++badslot; continue; }
                                const float y = buf[(size_t)row * PW + wc];
                                sums[(size_t)slot * 256 + tid] = fmaf(dt - wl, y, sums[(size_t)slot * 256 + tid]);
                                sums[(size_t)(slot + 1) * 256 + tid] = fmaf(wl, y, sums[(size_t)(slot + 1) * 256 + tid]);
                            }
                            for (size_t p = 0; apart && p + 2 < slots.size(); ++p)          // any row and the next but one
                                for (unsigned cell = 2; cell < (unsigned)ZC + 2; ++cell)
                                    shared += (slots[p] == cell || slots[p] + 1 == cell) && (slots[p + 2] == cell || slots[p + 2] + 1 == cell);
                        }
                    }
                }
            }
            for (int tid = 0; tid < 256; ++tid) {
                const int i = i0 + (tid & (BP_T - 1)), j = j0 + (tid >> 4);
                if (i >= g.nx || j >= g.ny) continue;
                for (int kk = 0; kk < ZC && k0 + kk < g.nz; ++kk)
                    vol[((size_t)(k0 + kk) * g.ny + j) * g.nx + i] = sums[(size_t)(ZC + 1 - kk) * 256 + tid];
            }
        }
    report[0] = wide; report[1] = outside; report[2] = badslot; report[3] = shared;
}

// The shape with shared views that one volume takes, -1: none (each group of threads, and each part, takes some of the views: the same windows and slots).
static int host_shared_views_shape(const leap_geometry *G) { return G->bp_parts > 1 ? G->bp_parts_shape : G->bp_split_shape; }

extern "C" long host_sd_backproject_tiled(const leap_geometry *G, const float *sino, float *vol, int64_t *report)
{
    if (G->g.model != SF_MODEL_SIDDON || G->d_mdbp || !G->bp_tiled) return -1;
    static_assert(SD_BP_NSPLIT_SHAPES == 2, "every shape has a case");
    const int split = host_shared_views_shape(G);
    if (split >= 0) {
        if (split == 0) host_sd_bp_shape<SD_BP_SPLIT_SHAPES[0].zc, SD_BP_SPLIT_SHAPES[0].pw, SD_BP_SPLIT_SHAPES[0].ph>(G, sino, vol, report);
        else host_sd_bp_shape<SD_BP_SPLIT_SHAPES[1].zc, SD_BP_SPLIT_SHAPES[1].pw, SD_BP_SPLIT_SHAPES[1].ph>(G, sino, vol, report);
        return report[0] + report[1] + report[2] + report[3];
    }
    switch (G->bp_shape) {
    case 1: host_sd_bp_shape<BP_SHAPES[1].zc, BP_SHAPES[1].pw, BP_SHAPES[1].ph>(G, sino, vol, report); break;
    case 2: host_sd_bp_shape<BP_SHAPES[2].zc, BP_SHAPES[2].pw, BP_SHAPES[2].ph>(G, sino, vol, report); break;
    case 3: host_sd_bp_shape<BP_SHAPES[3].zc, BP_SHAPES[3].pw, BP_SHAPES[3].ph>(G, sino, vol, report); break;
    case 4: host_sd_bp_shape<BP_SHAPES[4].zc, BP_SHAPES[4].pw, BP_SHAPES[4].ph>(G, sino, vol, report); break;
    default: return -1;
    }
    return report[0] + report[1] + report[2] + report[3];
}

// ---- Siddon model on tilted modules: the per-lane forward kernel, slab by slab, with the kernel's own functions ---------
// Returns -1 when the handle does not use that kernel, else the number of samples that came out non-finite (the slab
// copies sit between guard bands of NaN, so a gather outside a copy shows).
extern "C" long host_md_project_columns(const leap_geometry *G, const float *vol, float *sino, int width)
{
    const SfGeom &g = G->g;
    if (!G->md_tilted) return -1;
    const int nzp = g.nz + 2 * FP_PAD;
    const size_t guard = 4096;
    std::vector<float> acc((size_t)g.nviews * g.nrows * g.ncols, 0.f);
    for (int xmajor = 1; xmajor >= 0; --xmajor) {
        const int n_major = xmajor ? g.nx : g.ny, n_side = xmajor ? g.ny : g.nx;
        for (int n0 = 0; n0 < n_major; n0 += width) {
            const int n1 = std::min(n0 + width, n_major);
            const SfSlab slab = {n0, n1, xmajor, n0 == 0 ? 1 : 0, width};
            const size_t columns = (size_t)width * n_side;
            std::vector<float> buf(2 * guard + (columns + 1) * nzp, NAN);
            float *volz = buf.data() + guard;
            std::fill(volz, volz + (columns + 1) * nzp, 0.f);
            for (int n = n0; n < n1; ++n)
                for (int q = 0; q < n_side; ++q) {
                    const int i = xmajor ? n : q, j = xmajor ? q : n;
                    float *col = volz + (size_t)sf_slab_column(slab, g.nx, i, j) * nzp + FP_PAD;
                    for (int k = 0; k < g.nz; ++k) col[k] = vol[((size_t)k * g.ny + j) * g.nx + i];
                }
            const unsigned zero_col = (unsigned)(columns * nzp);
#pragma omp parallel for collapse(2)
            for (int a = 0; a < g.nviews; ++a)
                for (int r = 0; r < g.nrows; ++r)
                    for (int c = 0; c < g.ncols; ++c) {
                        const MdSlabRay M = md_slab_ray(g, G->poses[a], r, c);
                        const MdAxial A = md_axial(M);
                        const bool mine = M.R.xmajor == xmajor;
                        float t = 0.f;
                        const MdPitch pitch = md_pitch(slab, xmajor != 0, g.nx, nzp);
                        unsigned base = 0;
                        for (int n = n0; n < n1; ++n, base += pitch.n) {
                            const SdSplit s = sd_slab_split(M.R, n);
                            bool a_ok, b_ok;
                            md_slab_meets(M, s, n, xmajor ? g.ny : g.nx, mine, a_ok, b_ok);
                            if (!a_ok && !b_ok) continue;
                            unsigned k;
                            float tlow;
                            md_axial_place(M, A, n, nzp, k, tlow);
                            const unsigned at_a = md_cell_a(s, pitch, base);
                            const float *xa = volz + (a_ok ? at_a : zero_col) + k, *xb = volz + (b_ok ? md_cell_b(s, pitch, at_a) : zero_col) + k;
                            const float one = md_gather_one(xa[0], xa[1], tlow, t);
                            t = sd_gather_two(xa, xb, A.inc, s.f, 1.0f - s.f, tlow, t);
                            if (s.qa == s.qb && one != t) t = NAN;          // (a wave in which no ray crosses takes the short form)
                        }
                        if (mine) acc[((size_t)a * g.nrows + r) * g.ncols + c] += M.len * t;
                    }
        }
    }
    long bad = 0;
    for (size_t q = 0; q < acc.size(); ++q) {
        sino[q] = acc[q];
        bad += !std::isfinite(acc[q]);
    }
    return bad;
}

// ---- Siddon model on tilted modules: the tiled back projection, tile by tile, with the kernel's own functions ------------
// report[0]: (view, tile, chunk) windows wider or taller than the instance stages; report[1]: reads outside the staged
// window; report[2]: slots outside the per-thread sums.  Returns -1 when the handle does not use that kernel.
template <int ZC, int PW, int PH>
static void host_md_bp_shape(const leap_geometry *G, const float *sino, float *vol, int64_t *report)
{
    const SfGeom &g = G->g;
    constexpr int PS = PW + 1, NSLOT = ZC + 4;
    const int tiles_x = (g.nx + BP_T - 1) / BP_T, tiles_y = (g.ny + BP_T - 1) / BP_T, chunks = (g.nz + ZC - 1) / ZC;
    int64_t wide = 0, outside = 0, badslot = 0;
#pragma omp parallel for collapse(2) reduction(+ : wide, outside, badslot)
    for (int ch = 0; ch < chunks; ++ch)
        for (int tile = 0; tile < tiles_x * tiles_y; ++tile) {
            const int i0 = (tile % tiles_x) * BP_T, j0 = (tile / tiles_x) * BP_T, k0 = ch * ZC;
            std::vector<float> sums((size_t)NSLOT * 256, 0.f);
            std::vector<MdBpPixel> px((size_t)PH * PS);
            for (int a = 0; a < g.nviews; ++a) {
                const MdBpView &V = G->d_mdbp[a];
                const SfWindow win = md_bp_window(g, V, i0, j0, k0, ZC);
                wide += win.need_w > PW || win.need_h > PH;
                const bool xmajor = md_bp_tile_xmajor(g, V, i0, j0);
                for (int sc = 0; sc < PW; ++sc) {
                    const int c = win.c0 + sc;
                    for (int row = 0; row < PH; ++row) {
                        const int r = win.r0 + row;
                        const bool in = c >= 0 && c < g.ncols && r >= 0 && r < g.nrows;
                        const float y = in ? sino[((size_t)a * g.nrows + r) * g.ncols + c] : 0.f;
                        px[(size_t)row * PS + sc] = md_bp_pixel(md_bp_slopes(g, V, xmajor, r, c), y);
                    }
                }
                const int H = std::min(win.need_h, PH);
                for (int tid = 0; tid < 256; ++tid) {
                    const int i = i0 + (tid & (BP_T - 1)), j = j0 + (tid >> 4);
                    const int ic = std::min(i, g.nx - 1), jc = std::min(j, g.ny - 1);
                    const MdBpColumn C = md_bp_column<ZC>(g, V, xmajor, ic, jc, k0);
                    const int cbeg = std::max(C.cfirst, win.c0), cend = std::min(C.clast, win.c0 + PW - 1);
                    for (int c = cbeg; c <= cend; ++c) {
                        const int wc = c - win.c0;
                        if (c < 0 || c >= g.ncols) continue;
                        int rs, re;
                        md_bp_rows(C, c, win.r0, H, rs, re);
                        for (int row = rs; row < re; ++row) {
                            if (row < 0 || row >= PH) { ++outside; continue; }
                            const MdBpPixel &p = px[(size_t)row * PS + wc];
                            float t0, t1, w_above, w_below;
                            if (!(md_bp_piece(C, p, t0, t1) > 0.0f)) continue;
                            unsigned slot;
                            md_bp_shares<ZC>(C, p, t0, t1, slot, w_above, w_below);
                            slot -= SD_BP_HI;
                            if (slot + 1 >= (unsigned)NSLOT) { ++badslot; continue; }
                            sums[(size_t)slot * 256 + tid] += w_above;
                            sums[(size_t)(slot + 1) * 256 + tid] += w_below;
                        }
                    }
                }
            }
            for (int tid = 0; tid < 256; ++tid) {
                const int i = i0 + (tid & (BP_T - 1)), j = j0 + (tid >> 4);
                if (i >= g.nx || j >= g.ny) continue;
                for (int kk = 0; kk < ZC && k0 + kk < g.nz; ++kk)
                    vol[((size_t)(k0 + kk) * g.ny + j) * g.nx + i] = sums[(size_t)(ZC + 1 - kk) * 256 + tid];
            }
        }
    report[0] = wide; report[1] = outside; report[2] = badslot;
}

extern "C" long host_md_backproject_tiled(const leap_geometry *G, const float *sino, float *vol, int64_t *report)
{
    if (!G->d_mdbp || !G->bp_tiled) return -1;
    static_assert(MD_BP_NSPLIT_SHAPES == 3, "every shape has a case");
    const int split = host_shared_views_shape(G);
    if (split >= 0) {
        if (split == 2) host_md_bp_shape<MD_BP_SPLIT_SHAPES[2].zc, MD_BP_SPLIT_SHAPES[2].pw, MD_BP_SPLIT_SHAPES[2].ph>(G, sino, vol, report);
        else if (split == 0) host_md_bp_shape<MD_BP_SPLIT_SHAPES[0].zc, MD_BP_SPLIT_SHAPES[0].pw, MD_BP_SPLIT_SHAPES[0].ph>(G, sino, vol, report);
        else host_md_bp_shape<MD_BP_SPLIT_SHAPES[1].zc, MD_BP_SPLIT_SHAPES[1].pw, MD_BP_SPLIT_SHAPES[1].ph>(G, sino, vol, report);
        return report[0] + report[1] + report[2];
    }
    switch (G->bp_shape) {
    case 0: host_md_bp_shape<MD_BP_SHAPES[0].zc, MD_BP_SHAPES[0].pw, MD_BP_SHAPES[0].ph>(G, sino, vol, report); break;
    case 1: host_md_bp_shape<MD_BP_SHAPES[1].zc, MD_BP_SHAPES[1].pw, MD_BP_SHAPES[1].ph>(G, sino, vol, report); break;
    case 2: host_md_bp_shape<MD_BP_SHAPES[2].zc, MD_BP_SHAPES[2].pw, MD_BP_SHAPES[2].ph>(G, sino, vol, report); break;
    case 3: host_md_bp_shape<MD_BP_SHAPES[3].zc, MD_BP_SHAPES[3].pw, MD_BP_SHAPES[3].ph>(G, sino, vol, report); break;
    case 4: host_md_bp_shape<MD_BP_SHAPES[4].zc, MD_BP_SHAPES[4].pw, MD_BP_SHAPES[4].ph>(G, sino, vol, report); break;
    case 5: host_md_bp_shape<MD_BP_SHAPES[5].zc, MD_BP_SHAPES[5].pw, MD_BP_SHAPES[5].ph>(G, sino, vol, report); break;
    default: return -1;
    }
    return report[0] + report[1] + report[2];
}

// ---- footprints on tilted modules: the tiled kernels, with their own functions ------------------------------------------------
// Back: voxel by voxel on the staged window of its workgroup's box; report[0]: windows larger than the staging buffer, report[1]: reads
// of the common case (three rows of three columns) outside the window.  Returns -1 when the handle does not use that kernel.
extern "C" long host_mf_backproject_tiled(const leap_geometry *G, const float *sino, float *vol, int64_t *report)
{
    const SfGeom &g = G->g;
    if (!G->mf_tiled) return -1;
    const int tiles_x = (g.nx + MF_T - 1) / MF_T, tiles_y = (g.ny + MF_T - 1) / MF_T, chunks = (g.nz + MF_ZC - 1) / MF_ZC;
    int64_t large = 0, outside = 0;
#pragma omp parallel for collapse(2) reduction(+ : large, outside)
    for (int ch = 0; ch < chunks; ++ch)
        for (int tile = 0; tile < tiles_x * tiles_y; ++tile) {
            const int i0 = (tile % tiles_x) * MF_T, j0 = (tile / tiles_x) * MF_T, k0 = ch * MF_ZC;
            const int i1 = std::min(i0 + MF_T, g.nx) - 1, j1 = std::min(j0 + MF_T, g.ny) - 1, k1 = std::min(k0 + MF_ZC, g.nz) - 1;
            std::vector<double> acc((size_t)MF_T * MF_T * MF_ZC, 0.0);
            for (int a = 0; a < g.nviews; ++a) {
                const MfView &V = G->d_mfviews[a];
                float x[4] = {3e38f, -3e38f, 3e38f, -3e38f};
                for (int q = 0; q < 8; ++q) {
                    float xi, eta;
                    mf_box_corner(g, V, i0, i1, j0, j1, k0, k1, q, xi, eta);
                    x[0] = std::min(x[0], xi); x[1] = std::max(x[1], xi); x[2] = std::min(x[2], eta); x[3] = std::max(x[3], eta);
                }
                const MfWindow w = mf_window(x[0], x[1], x[2], x[3]);
                if ((int64_t)w.w * w.h > MF_PATCH || w.w < 1 || w.h < 1) { ++large; continue; }
                std::vector<double> patch((size_t)w.w * w.h);
                for (int rr = 0; rr < w.h; ++rr)
                    for (int cc = 0; cc < w.w; ++cc) {
                        const int r = w.r0 + rr, c = w.c0 + cc;
                        const bool in = r >= 0 && r < g.nrows && c >= 0 && c < g.ncols;
                        patch[(size_t)rr * w.w + cc] = in ? (double)sino[((size_t)a * g.nrows + r) * g.ncols + c] * mf_amp(g, V, r, c) : 0.0;
                    }
                for (int j = j0; j <= j1; ++j)
                    for (int i = i0; i <= i1; ++i) {
                        MfWalk at = mf_walk(g, V, mf_column(g, V, i, j), k0);
                        for (int k = k0; k <= k1; ++k) {
                            const MfFoot f = mf_next(V, at);
                            const double fr0 = floor(f.e0), fc0 = floor(f.k0 + 0.5), above = f.e1 - fr0;
                            const int rows = (int)(floor(f.e1) - fr0), cols = (int)(ceil(f.k3 - 0.5) - fc0);
                            const int rr = (int)fr0 - w.r0, cc = (int)fc0 - w.c0;
                            if (rr < 0 || cc < 0 || rr + std::max(rows, 2) >= w.h || cc + std::max(cols, 2) >= w.w) { ++outside; continue; }
                            double fu[3], &sum = acc[((size_t)(k - k0) * MF_T + (j - j0)) * MF_T + (i - i0)];
                            double x_edge = fc0 + 0.5, below = 0.0;
                            mf_fu3(f, x_edge, fu);
                            for (int m = 0; m <= std::max(cols, 2); ++m, x_edge += 1.0) {
                                const double upto = mf_integral_at(f, x_edge), share = cols > 2 ? upto - below : fu[m];
                                below = upto;
                                for (int n = 0; n <= std::max(rows, 1); ++n) {
                                    const double fv = n == 0 ? mf_min(above, 1.0) - (f.e0 - fr0) : mf_sub01(above, (double)n);
                                    sum = fma(share * fv, patch[(size_t)(rr + n) * w.w + cc + m], sum);
                                }
                            }
                        }
                    }
            }
            for (int k = k0; k <= k1; ++k)
                for (int j = j0; j <= j1; ++j)
                    for (int i = i0; i <= i1; ++i)
                        vol[((size_t)k * g.ny + j) * g.nx + i] = (float)acc[((size_t)(k - k0) * MF_T + (j - j0)) * MF_T + (i - i0)];
        }
    report[0] = large; report[1] = outside;
    return large + outside;
}

// Forward: every voxel's shares on every detector tile (the kernel visits a subset: those its beams can meet).  Returns -1 when the
// handle does not use that kernel, else the number of shares of the common case beside the tile's guarded sums.
extern "C" long host_mf_project_tiles(const leap_geometry *G, const float *vol, float *sino)
{
    const SfGeom &g = G->g;
    if (!G->mf_tiles) return -1;
    long beside = 0;
    const int tiles_c = (g.ncols + MF_TC - 1) / MF_TC, tiles_r = (g.nrows + MF_TR - 1) / MF_TR;
#pragma omp parallel for collapse(2) reduction(+ : beside)
    for (int a = 0; a < g.nviews; ++a)
        for (int tile = 0; tile < tiles_c * tiles_r; ++tile) {
            const MfView &V = G->d_mfviews[a];
            const int c0 = (tile % tiles_c) * MF_TC, r0 = (tile / tiles_c) * MF_TR;
            const int c1 = std::min(c0 + MF_TC, g.ncols) - 1, r1 = std::min(r0 + MF_TR, g.nrows) - 1;
            std::vector<double> sums((size_t)(MF_TR + 2 * MF_TG) * MF_TS, 0.0);
            auto add = [&](int r, int c, double v) {
                const long cell = (long)(r + MF_TG) * MF_TS + c + MF_TG;
                if (cell < 0 || cell >= (long)sums.size() || c + MF_TG < 0 || c + MF_TG >= MF_TS) ++beside;
                else sums[cell] += v;
            };
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i) {
                    MfWalk at = mf_walk(g, V, mf_column(g, V, i, j), 0);
                    for (int k = 0; k < g.nz; ++k) {
                        const MfFoot f = mf_next(V, at);
                        const double x = vol[((size_t)k * g.ny + j) * g.nx + i], fr0 = floor(f.e0), fc0 = floor(f.k0 + 0.5), above = f.e1 - fr0;
                        const int rb = (int)fr0 - r0, cb = (int)fc0 - c0;
                        const int rows = (int)(floor(f.e1) - fr0), cols = (int)(ceil(f.k3 - 0.5) - fc0);
                        if (!(rb + rows >= 0 && rb <= r1 - r0 && cb + cols >= 0 && cb <= c1 - c0)) continue;
                        const bool common = cols <= 2 && rows <= 2;
                        double fu[3], below = 0.0, edge = fc0 + 0.5;
                        mf_fu3(f, edge, fu);
                        for (int m = 0; m <= (common ? 2 : cols); ++m, edge += 1.0) {
                            const double upto = mf_integral_at(f, edge), share = common ? fu[m] : upto - below;
                            below = upto;
                            for (int n = 0; n <= (common ? 2 : rows); ++n) {
                                const double fv = n == 0 ? mf_min(above, 1.0) - (f.e0 - fr0) : mf_sub01(above, (double)n);
                                if (common || (rb + n >= 0 && rb + n <= r1 - r0 && cb + m >= 0 && cb + m <= c1 - c0)) add(rb + n, cb + m, share * (fv * x));
                            }
                        }
                    }
                }
            for (int r = r0; r <= r1; ++r)
                for (int c = c0; c <= c1; ++c)
                    sino[((size_t)a * g.nrows + r) * g.ncols + c] = (float)(sums[(size_t)(r - r0 + MF_TG) * MF_TS + c - c0 + MF_TG] * mf_amp(g, V, r, c));
        }
    return beside;
}

// ---- parallel beams by detector rows: the copy's row overlaps, then the candidates' transaxial weights -------------------------
// Returns -1 when the handle does not use that kernel, else the number of (view, bundle, slab) cases in which the candidate slots do
// not cover the candidate range.
template <int CW>
static long host_rows(const leap_geometry *G, const std::vector<float> &rows, float *sino)
{
    const SfGeom &g = G->g;
    const int nbundles = (g.ncols + CW - 1) / CW;
    long uncovered = 0;
#pragma omp parallel for collapse(2) reduction(+ : uncovered)
    for (int a = 0; a < g.nviews; ++a)
        for (int b = 0; b < nbundles; ++b) {
            const SfView v = G->views[a];
            const int c0 = b * CW, xmajor = G->major[(size_t)a * nbundles + b];
            const SfRayLines L = sf_ray_lines<0>(g, v, c0, CW, xmajor);
            const int n_major = xmajor ? g.nx : g.ny, n_minor = xmajor ? g.ny : g.nx;
            const SfSlab slab = {0, n_major, xmajor, 1, n_major};
            std::vector<float> total((size_t)g.nrows * CW, 0.f);
            uncovered += host_layers(G, slab, total, [&](int n, std::vector<float> &acc) {
                int qf, ql;
                sf_candidates(L, n, qf, ql);
                if (ql - qf + 1 > G->fp_nq) ++uncovered;
                for (int q = std::max(qf, 0); q <= std::min(std::min(ql, qf + G->fp_nq - 1), n_minor - 1); ++q) {
                    const int i = xmajor ? n : q, j = xmajor ? q : n;
                    float fa[CW];
                    double mu;
                    if (!sf_candidate_record<CW, 0>(g, v, i, j, c0, true, fa, mu)) continue;
                    const float *x = &rows[((size_t)j * g.nx + i) * g.nrows];
                    for (int r = 0; r < g.nrows; ++r)
                        for (int cw = 0; cw < CW; ++cw)
                            if (fa[cw] != 0.0f) acc[(size_t)r * CW + cw] = fmaf(fa[cw], x[r], acc[(size_t)r * CW + cw]);
                }
            });
            for (int cw = 0; cw < CW && c0 + cw < g.ncols; ++cw)
                for (int r = 0; r < g.nrows; ++r) sino[((size_t)a * g.nrows + r) * g.ncols + c0 + cw] = v.par_amp * total[(size_t)r * CW + cw];
        }
    return uncovered;
}

extern "C" long host_project_rows(const leap_geometry *G, const float *vol, float *sino)
{
    const SfGeom &g = G->g;
    if (!G->fp_rows) return -1;
    std::vector<float> rows((size_t)g.nx * g.ny * g.nrows, 0.f);
    for (int r = 0; r < g.nrows; ++r) {
        const SfRowOverlap o = sf_row_overlap(g, r);
        for (int t = 0; t < o.n; ++t) {
            const int k = o.kb + t;
            const float w = sf_row_weight(o, t);
            if (k < 0 || k >= g.nz || !(w > 0.0f)) continue;
            for (size_t ij = 0; ij < (size_t)g.nx * g.ny; ++ij) rows[ij * g.nrows + r] = fmaf(w, vol[(size_t)k * g.nx * g.ny + ij], rows[ij * g.nrows + r]);
        }
    }
    return G->fp_cw == 2 ? host_rows<2>(G, rows, sino) : host_rows<4>(G, rows, sino);
}

// Back projection of a launch's items with the views shared among workgroups: out = {parts, shape, items at a time, shape one volume takes without parts}.
extern "C" void host_back_parts(const leap_geometry *G, int items, int32_t *out)
{
    const bool siddon = G->g.model == SF_MODEL_SIDDON;
    const LeapBackParts p = siddon ? leap_siddon_parts(G, items) : leap_back_parts(G, items);
    out[0] = p.parts; out[1] = p.shape; out[2] = p.items; out[3] = G->bp_split_shape;
}

// ---- flat scans: a wave's records per slab (parallel beams: the footprints stepped along it), a thread's columns in the staged window -----------
// report[0]: candidate voxels that the wave's outermost columns do not bound or the records do not hold; report[1]: columns read
// outside the staged ones, for the tiles of one, two and four views at a time.  Returns -1 when the handle does not use these kernels.
extern "C" int host_flat_tiles(int ncols, int nviews) { return flat_tiles(ncols, nviews); }

// Slabs that the waves of a workgroup do not take once, in order.
extern "C" long host_check_flat_shares(int n_major, int nwaves)
{
    long wrong = 0;
    int at = 0;
    for (int w = 0; w < nwaves; ++w) {
        int begin, end;
        sf_flat_share(n_major, w, nwaves, begin, end);
        wrong += begin != at || end < begin;
        at = end;
    }
    return wrong + (at != n_major);
}

template <int SUB>
static bool host_flat_outside(const SfGeom &g, const SfView &v, int i, int j, int cf)
{
    typedef FlatTile<SUB> Tile;
    const int ic = i / Tile::TX * Tile::TX + Tile::TX / 2, jc = j / Tile::TY * Tile::TY + Tile::TY / 2;      // the tile's middle voxel
    const int first = (int)floor(sf_column<0>(g, v, std::min(ic, g.nx - 1), std::min(jc, g.ny - 1)).xi) - Tile::COLS / 2;
    return cf < first || cf + FLAT_NC - 1 >= first + Tile::COLS;
}

extern "C" long host_flat(const leap_geometry *G, const float *vol, float *sino, const float *sino_in, float *vol_out, int64_t *report)
{
    const SfGeom &g = G->g;
    if (!G->flat) return -1;
    int64_t beyond = 0, outside = 0;
    const int tiles = (g.ncols + FLAT_RAYS - 1) / FLAT_RAYS;
    const bool parallel = g.type == SF_PARALLEL;
#pragma omp parallel for collapse(2) reduction(+ : beyond)
    for (int a = 0; a < g.nviews; ++a)
        for (int t = 0; t < tiles; ++t) {
            const SfView &v = G->views[a];
            const int c0 = t * FLAT_RAYS, c1 = std::min(c0 + FLAT_RAYS, g.ncols) - 1, xmajor = sf_flat_xmajor(g, v, c0);
            const int n_major = xmajor ? g.nx : g.ny, n_minor = xmajor ? g.ny : g.nx;
            for (int c = c0; c <= c1; ++c) {
                const SfRayLines L = sf_ray_lines<0>(g, v, c, 1, xmajor), L0 = sf_ray_lines<0>(g, v, c0, 1, xmajor), L1 = sf_ray_lines<0>(g, v, c1, 1, xmajor);
                float acc = 0.f;
                for (int n = 0; n < n_major; ++n) {
                    int qf, ql, f0, l0, f1, l1;
                    sf_candidates(L, n, qf, ql);
                    sf_candidates(L0, n, f0, l0);
                    sf_candidates(L1, n, f1, l1);
                    const int q_lo = std::max(std::min(f0, f1), 0), q_hi = std::min(std::max(l0, l1), n_minor - 1);
                    if (q_hi - q_lo + 1 > G->flat_span) ++beyond;
                    qf = std::max(qf, q_lo);
                    SfColumn stepped = {};
                    double edge = 0.0;
                    if (parallel) {
                        stepped = sf_flat_parallel_column(g, v, xmajor ? n : qf, xmajor ? qf : n);
                        edge = ((double)c - 0.5) - stepped.xi;
                    }
                    for (int q = qf; q <= std::min(ql, n_minor - 1); ++q) {
                        const int i = xmajor ? n : q, j = xmajor ? q : n;
                        const float fu = parallel ? sf_flat_stepped_fu(stepped, edge, sf_flat_step(g, v, xmajor), q - qf)
                                                  : sf_flat_fu(sf_flat_record(sf_column<0>(g, v, i, j)), c);
                        if (!(fu > 0.0f)) continue;
                        if (q < q_lo || q > q_hi) ++beyond;
                        acc = fmaf(fu, vol[(size_t)j * g.nx + i], acc);
                    }
                }
                sino[(size_t)a * g.ncols + c] = sf_amp(g, v, sf_amp_col<0>(g, v, c), 0) * G->flat_fv * acc;
            }
        }
#pragma omp parallel for collapse(2) reduction(+ : outside)
    for (int j = 0; j < g.ny; ++j)
        for (int i = 0; i < g.nx; ++i) {
            float acc = 0.f;
            for (int a = 0; a < g.nviews; ++a) {
                const SfView &v = G->views[a];
                const SfColumn f = sf_column<0>(g, v, i, j);
                int cf, cl;
                sf_col_range(f, cf, cl);
                if (host_flat_outside<1>(g, v, i, j, cf) || host_flat_outside<2>(g, v, i, j, cf) || host_flat_outside<4>(g, v, i, j, cf) || cl - cf >= FLAT_NC) ++outside;
                for (int c = std::max(cf, 0); c <= std::min(cl, g.ncols - 1); ++c)
                    acc = fmaf(sf_fu(f, c), sino_in[(size_t)a * g.ncols + c] * (sf_amp(g, v, sf_amp_col<0>(g, v, c), 0) * G->flat_fv), acc);
            }
            vol_out[(size_t)j * g.nx + i] = acc;
        }
    report[0] = beyond; report[1] = outside;
    return beyond + outside;
}
