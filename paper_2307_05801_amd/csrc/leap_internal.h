// Library-private definitions shared by the host geometry module and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>
#include <string>
#include <vector>

#include "../../include/leap.h"
#include "sf_types.h"
#include "sd_ray.h"
#include "md_siddon.h"
#include "md_footprint.h"

struct MdBpView;                       // per-view table of the tiled Siddon back projection on tilted modules (md_backproject_tiled.h)
struct LeapHostStage;                  // streams, events, staging and device buffers of the host-memory entry points (leap_host.cpp)

// Device memory of a handle that its calls use in turn, from any stream and thread.  The turns are ordered on the device: each waits for the
// event that the last one recorded, whatever its stream, because equal stream handles need not be one stream (hipStreamPerThread is one handle
// for a stream of every thread; a destroyed stream's handle is given out again).  Under capture an eager event says nothing about the graph's launches:
// captured turns are ordered among those of their own capture, and eager ones among the eager ones.
struct LeapShared {
    std::mutex mutex;
    hipEvent_t done = nullptr, captured = nullptr;     // its last eager turn's end; the last captured one's, in capture `capture`
    hipEvent_t latest = nullptr;                       // the last eager turn's event, of this memory's or of a turn at several (null: there was none)
    bool captured_used = false;
    unsigned long long capture = 0;

    hipError_t create()
    {
        hipError_t e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
        return e == hipSuccess ? hipEventCreateWithFlags(&captured, hipEventDisableTiming) : e;
    }
    ~LeapShared()
    {
        if (done) (void)hipEventDestroy(done);
        if (captured) (void)hipEventDestroy(captured);
    }
};

// Is work on the stream being captured?  (Also where the runtime will not say: such a call takes the kernels that share nothing.)
inline bool leap_capturing(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// One call's turn at a handle's shared memory, or at n of them at once, from begin() to end(); a call that returns early, some of its kernels perhaps
// launched, ends it too.
class LeapTurn {
public:
    LeapTurn(LeapShared &memory, hipStream_t s) : LeapTurn(&memory, 1, memory.done, s) {}
    // done: the event that the turn records, and the next ones at any of the n wait for
    LeapTurn(LeapShared *memory, int n, hipEvent_t event, hipStream_t s) : shared(memory), count(n), done(event), stream(s)
    {
        for (int i = 0; i < count; ++i) shared[i].mutex.lock();
    }
    ~LeapTurn()
    {
        if (begun) (void)record();
        for (int i = 0; i < count; ++i) shared[i].mutex.unlock();
    }
    LeapTurn(const LeapTurn &) = delete;
    LeapTurn &operator=(const LeapTurn &) = delete;
    hipError_t begin()
    {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &status) != hipSuccess) (void)hipGetLastError();
        hipError_t e = hipSuccess;
        capturing = status == hipStreamCaptureStatusActive;
        if (capturing) e = hipStreamGetCaptureInfo(stream, &status, &capture);
        for (int i = 0; i < count && e == hipSuccess; ++i) {
            const LeapShared &s = shared[i];
            if (capturing && s.captured_used && s.capture == capture) e = hipStreamWaitEvent(stream, s.captured, 0);
            bool waits = !capturing && s.latest;
            for (int k = 0; k < i; ++k) waits = waits && shared[k].latest != s.latest;
            if (waits) e = hipStreamWaitEvent(stream, s.latest, 0);
        }
        begun = e == hipSuccess;
        return e;
    }
    hipError_t end()
    {
        begun = false;
        return record();
    }

private:
    hipError_t record()
    {
        hipError_t failed = capturing ? hipSuccess : hipEventRecord(done, stream);
        for (int i = 0; i < count; ++i) {
            LeapShared &s = shared[i];
            if (capturing) {
                const hipError_t e = hipEventRecord(s.captured, stream);
                s.captured_used = e == hipSuccess;
                s.capture = capture;
                if (e != hipSuccess) failed = e;
            } else if (failed == hipSuccess) {
                s.latest = done;
            }
        }
        return failed;
    }
    LeapShared *shared;
    int count;
    hipEvent_t done;
    hipStream_t stream;
    bool capturing = false, begun = false;
    unsigned long long capture = 0;
};

// Shared memory in up to four equal slots, a turn each for the calls that one holds, so that they run beside each other on as many streams; a call that needs
// more takes all of them.  Four, as many as the hardware queues that HIP spreads streams over.  us per call on 1 / 2 / 4 streams, kernels that share nothing; one
// slot; four: footprint A^T 57^2 x 37, 310 views 316 / 159 / 81; 72 / 77 / 75; 72 / 60 / 48; 81^2 x 67, 53 views 59 / 38 / 36; 52 / 58 / 59; 52 / 33 / 30; 128^2 x 20, 60
// views 60 / 32 / 28; 35 / 40 / 40; 34 / 25 / 21; Siddon A, 20 rows, 64^2 x 20, 30 views 63 / 35 / 23; 34 / 41 / 42; 34 / 20 / 17.
struct LeapRoom {
    static constexpr int MOST_SLOTS = 4;
    LeapShared slot[MOST_SLOTS];
    hipEvent_t whole = nullptr;                            // the end of the last turn at all of them
    int slots = 1;

    hipError_t create(int n)
    {
        slots = n;
        hipError_t e = hipEventCreateWithFlags(&whole, hipEventDisableTiming);
        for (int i = 0; i < slots && e == hipSuccess; ++i) e = slot[i].create();
        return e;
    }
    ~LeapRoom()
    {
        if (whole) (void)hipEventDestroy(whole);
    }
    LeapTurn turn(int i, hipStream_t stream) { return LeapTurn(&slot[i], 1, slot[i].done, stream); }
    LeapTurn turn_at_all(hipStream_t stream) { return LeapTurn(&slot[0], slots, whole, stream); }
    // A stream's calls stay with the slot it took first, where their order is the stream's own, until more streams have come than there are slots.
    int pick(hipStream_t stream)
    {
        std::lock_guard<std::mutex> lock(picking);
        for (int i = 0; i < slots; ++i)
            if (taken[i] && last[i] == stream && stream != hipStreamPerThread) return i;
        const int i = next;
        next = (next + 1) % slots;
        taken[i] = true;
        last[i] = stream;
        return i;
    }

private:
    std::mutex picking;
    bool taken[MOST_SLOTS] = {};
    hipStream_t last[MOST_SLOTS] = {};
    int next = 0;
};

struct leap_geometry {
    leap_geometry_desc desc;            // caller's parameters (angles_rad re-pointed at `angles`)
    std::vector<double> angles;
    SfGeom g;                           // float parameter block handed to every kernel by value
    std::vector<SfView> views;          // host copy of the per-view table
    SfView *d_views = nullptr;          // device copy
    int device = -1;
    // static bounds of the footprints, derived in double at creation; they select the kernel family
    double max_cols_per_voxel = 0;      // widest transaxial footprint, in detector pixels
    double max_rows_per_voxel = 0;      // tallest axial footprint, in detector pixels
    double max_voxels_per_row = 0;      // tallest pixel, in voxels (at the smallest magnification)
    double max_minor_slope = 0;         // largest |d minor / d major| of any ray in its marching frame
    // tiled back projection: columns / rows read per voxel, half footprint width, and whether its limits hold
    int bp_nc = 0, bp_nv = 0, bp_shape = 0;   // bp_shape indexes BP_SHAPES
    float bp_wh = 0.f;
    bool bp_tiled = false;
    int bp_need_w = 0, bp_need_h = 0;   // largest staged window any (view, tile, chunk) asks for
    int bp_pair_shape = -1;             // two volumes per workgroup: index into BP_PAIR_SHAPES (-1: one volume)
    bool bp_pair_forced = false;        // (debugging: two items per workgroup in every batch)
    bool bp_mirror = false;             // ... the volume's upper half and its lower half's mirror image, whatever the batch
    // Groups of threads that share the views: the shape one volume takes, an index into BP_SPLIT_SHAPES (Siddon: SD_BP_SPLIT_SHAPES,
    // tilted modules: MD_BP_SPLIT_SHAPES), -1: none.  A batch may take another of those that fit, one bit each, or none
    // (leap_back_split_shape, leap_siddon_split_shape).
    int bp_split_shape = -1;
    unsigned bp_split_fits = 0;
    // ... and workgroups of them, each with a volume of its own: what one volume takes (parts 1: none), the shapes that fit, the room for the
    // parts' volumes (floats)
    int bp_parts_shape = -1, bp_parts = 1;
    unsigned bp_parts_fits = 0;
    float *d_back = nullptr;
    size_t back_floats = 0;
    int back_slot_items = 0;            // items whose parts a slot of the room holds
    mutable LeapRoom back;
    bool bp_split_forced = false;       // (debugging: bp_split_shape, whatever the launch)
    // column-wise forward projection (footprint and Siddon models): the volume goes through a z-fastest scratch copy
    // slab by slab (sf_project_columns.h)
    int fp_nq = 0, fp_need_q = 0;       // candidate slots per slab: instance / needed
    int fp_nkp = 0;                     // voxels a pair of adjacent detector rows can overlap
    int fp_rg = 0;                      // row groups per wave (footprints: groups of 128 rows; Siddon: of 64)
    int fp_cw = 4, fp_vb = 128, fp_tb = 1;   // detector columns per wave; block order: views per run, tiles per chunk
    int fp_turn = 31;                   // ... and log2 of the views after which tiles change XCD (31: never)
    int fp_parts = 1;                   // waves of a workgroup that share a bundle's layers (1: none, each has a bundle of its own)
    bool fp_columns = false;
    int fp_pair_rg = 0;                 // row groups per wave with two volumes per wave (0: one volume per wave only)
    bool fp_pair_always = false;        // (debugging: two volumes per wave in every batch, however few its waves)
    int fp_rows = 0;                    // parallel beams: rows per lane of sf_project_rows (0: not used); fp_row_groups groups of 64 of them
    int fp_row_groups = 1;
    bool flat = false;                  // one row, one layer: the kernels of sf_flat.h in both directions
    int flat_span = 0;                  // voxels of a slab that the beams of 64 adjacent columns cover, rounded up to 64
    float flat_fv = 1.0f;               // the scan's one axial weight
    float *d_volz = nullptr;            // the scratch: scratch_items copies of one slab
    size_t scratch_bytes = 0;           // bytes allocated at d_volz
    int slab_width = 0;                 // voxel layers across the marching axis per slab when one volume is projected
    int dbg_slab = 0, dbg_items = 0;    // debugging overrides of the slab width and the items per launch (0: none)
    int nzp = 0;                        // floats per padded z-column
    std::vector<unsigned char> major;   // footprints: [view][bundle of fp_cw columns] 1 if the bundle advances fastest along x
    unsigned char *d_major = nullptr;
    std::string note;                   // what went differently from the plan at creation (shown by leap_geometry_describe)
    mutable LeapRoom scratch;           // the turns of its calls at d_volz
    size_t scratch_slot_floats = 0;     // ... of which each of its slots has so many (where it has more than one)
    // Siddon model: per-(view, detector column) ray constants, host copy and device copy
    std::vector<SdRayCol> raycols;
    SdRayCol *d_raycols = nullptr;
    double sd_max_axial_slope = 0;      // largest |dZ/dX| of any ray: voxels of z crossed per slab
    double sd_min_row_step = 0, sd_max_row_step = 0, sd_max_z = 0;   // voxels of z between adjacent rows; largest |Z| of any ray
    int sd_pairs = 0;                   // two rows per lane (sd_project_pairs): 0 no, 1 rows closer than a voxel somewhere, 2 nowhere
    // modular geometry: per-view poses, host copy and device copy
    std::vector<MdPose> poses;
    MdPose *d_poses = nullptr;
    // footprint model on upright modules: every view is a cone-beam view with its own parameter block
    std::vector<SfGeom> geoms;
    SfGeom *d_geoms = nullptr;
    // footprint model on tilted modules: per-view table of the general kernels (md_footprint.h)
    std::vector<MfView> mfviews;
    MfView *d_mfviews = nullptr;
    bool mf_tiles = false, mf_tiled = false;   // the fast kernels of md_footprint_tiled.h, forward / back
    void *d_colcs = nullptr;            // cylinder, tiled back projection: (cos, sin) of every column's fan angle, then the (tile, view) table
    // leap_project_host / leap_backproject_host: created by the first such call, freed with the handle
    mutable LeapHostStage *host_stage = nullptr;
    mutable std::mutex host_mutex;
    size_t stage_chunk = (size_t)32 << 20;   // bytes per pinned staging buffer
    MdBpView *d_mdbp = nullptr;         // Siddon model on tilted modules, tiled back projection: its per-view table
    bool md_tilted = false;             // Siddon model on tilted modules: the per-lane variants of the two fast kernels
    bool sd_columns = false;            // wave-per-column forward kernel (needs the scratch copy and slope <= 1)
};

void leap_set_error(const std::string &msg);
int leap_hip_fail(hipError_t e, const char *what);

#define LEAP_HIP_CHECK(expr)                                   \
    do {                                                       \
        hipError_t e__ = (expr);                               \
        if (e__ != hipSuccess) return leap_hip_fail(e__, #expr); \
    } while (0)

// Size of the file-scope device array behind leap_project_static_scratch (one per GPU the library runs on).
constexpr size_t LEAP_STATIC_SCRATCH_BYTES = (size_t)72 << 20;
// Looks up the array's address on `device` (which must be current) once; called from leap_geometry_create.
int leap_static_scratch_init(int device);

// Slab width and batch items per launch that a scratch of `floats` floats affords (leap_geometry.cpp).
bool leap_plan_scratch(const leap_geometry *G, size_t floats, int batch, int &width, int &items);

// Tiled footprint back projection of `items` volumes: pairs of items that go two per workgroup (mirror images: all items), and the shape of
// BP_SPLIT_SHAPES that all of them take instead, -1: none (leap_geometry.cpp).
int leap_back_pairs(const leap_geometry *G, int items);
inline int leap_back_split_pairs(const leap_geometry *G, int items) { return G->bp_mirror ? items : (G->g.type != SF_MODULAR ? items / 2 : 0); }
int leap_back_split_shape(const leap_geometry *G, int items);
// ... or the shape and the number of workgroups that share the views, items of the batch at a time (parts 1: as above).
struct LeapBackParts {
    int shape, parts, items;
};
LeapBackParts leap_back_parts(const leap_geometry *G, int items);
LeapBackParts leap_siddon_parts(const leap_geometry *G, int items);
// The same of the tiled Siddon back projection: a shape of SD_BP_SPLIT_SHAPES or, on tilted modules, MD_BP_SPLIT_SHAPES.
int leap_siddon_split_shape(const leap_geometry *G, int items);

// Footprint forward projection: how many of a launch's `items` volumes go two to a wave (leap_geometry.cpp).
int leap_forward_paired(const leap_geometry *G, int items);

// Frees what the host-memory entry points created on the handle (leap_host.cpp).
void leap_host_stage_free(leap_geometry *G);

// Where the column-wise forward kernels find their z-fastest copy of a slab: the handle's own scratch, or the library's
// fixed array (leap_project_static_scratch).
struct FwdScratch {
    float *volz;
    size_t item_floats;     // floats per copy (one per item of a batch in flight): (columns of a slab + 1) * nzp
    int width;              // voxel layers across the marching axis per slab
    int items;              // copies
};

inline unsigned cdiv(unsigned a, unsigned b) { return (a + b - 1) / b; }

// kernel launchers (leap_kernels.hip); one batch item per call
int leap_launch_project_batch(const leap_geometry *geom, const float *d_vol, float *d_sino, int batch, hipStream_t stream);
int leap_launch_backproject(const leap_geometry *geom, const float *d_sino, float *d_vol, hipStream_t stream);
struct SfSlab;
bool leap_launch_footprint_slab(const leap_geometry *geom, const FwdScratch &S, const SfSlab &slab, float *d_sino, hipStream_t stream, int items);   // leap_footprint_forward.hip
bool leap_launch_footprint_slab_parts(const leap_geometry *geom, const FwdScratch &S, const SfSlab &slab, int waves, float *d_sino, hipStream_t stream, int items);   // leap_footprint_forward_parts.hip
int leap_launch_footprint_back(const leap_geometry *geom, const float *d_sino, float *d_vol, int items, hipStream_t stream);                         // leap_footprint_back.hip
bool leap_launch_backproject_split(const leap_geometry *geom, int shape, int parts, const float *d_sino, float *room, float *d_vol, int items, hipStream_t stream);          // leap_footprint_back_split.hip
bool leap_launch_siddon_back_split(const leap_geometry *geom, int shape, int parts, const float *d_sino, float *d_vol, int items, hipStream_t stream);          // leap_siddon_back_split.hip
bool leap_launch_backproject_pairs(const leap_geometry *geom, const float *d_sino, float *d_vol, int blocks, hipStream_t stream);                     // leap_footprint_back_pairs.hip
int leap_launch_backproject_batch(const leap_geometry *geom, const float *d_sino, float *d_vol, int batch, hipStream_t stream);
