// Footprint pair of flat scans: one detector row, one voxel layer (fan-beam, and parallel-beam with nrows = nz = 1).  The
// axial factor of a weight is then one number for the whole scan, w = amp(view, c) * F_u(view, c; i, j) * F_v, and the batch
// (the slices of a mini-batch) is the only dimension left to share a weight over: a weight is formed once and applied to up
// to eight items.
//
// Both kernels are bound by vector-ALU issue on forming the footprints (about 65 instructions for a voxel's knots, half of
// them double precision), so the splits below are chosen to form each (view, voxel) pair's knots once per wave.
//
// Forward (sf_project_flat): a wave owns 64 adjacent detector columns of one view and walks its share of the slabs.  In a
// slab the wave's beams cover a run of consecutive voxels; lane q works out the footprint of the q-th of them and leaves it
// in LDS, then every lane reads back the two or three its pixel can touch.  Small scans split the slabs over up to 16
// waves of a workgroup (partial sums added through LDS in wave order, so the result does not depend on scheduling).
// Several items: a copy of the slices with the batch fastest puts the items of a voxel side by side, one or two 16-byte
// loads for all of them whatever the view angle.  A wave whose slabs run along y reads a cache line per lane with every load, the
// kernel's bound beside issue where there is much to do: it then has a copy of its own, whose rows run along y (FLAT_TURN_STEPS).
// Back (sf_backproject_flat): a wave owns 8 x 8 voxels and its share of the views.  Per view it loads the 64 detector
// samples around the tile's shadow, one column per lane, times the ray amplitude, into LDS (batch fastest), and every lane
// gathers its few columns.  No barrier: a wave reads only what it wrote.  Loads of the next view are in flight meanwhile.  Slices of few such
// tiles leave units idle (64 of 256 at work on 64^2): a wave then takes two or four views at a time on smaller tiles.  90 parallel views of
// 64^2 7.1 -> 5.8 us, 360 20.8 -> 9.1; 90 fan views 9.2 -> 5.2; 16 slices, 360 fan views 37.9 -> 27.6.
//
// Measured, A + A^T, against the general kernels (one thread per ray and item, three quarters of a block idle on one row):
// 8 slices of 512^2, 720 views of 736 columns 40.7 -> 3.0 ms; one slice of 64^2, 90 views 237 -> 23 us.  A since then (an odd number of
// tiles per view where there are many, voxels fetched ahead, the turned copy, no records for parallel beams): the 8 slices 1.95 -> 1.73 ms;
// one slice of 361 x 379, 577 parallel views of 409 columns 636 -> 415 us; 223 x 246, 271 fan views 159 -> 131 us; one slice of 64^2, 90
// parallel views, the kernel alone 10.5 -> 7.8 us.
#pragma once

#include "sf_footprint.h"
#include "sf_project_columns.h"

constexpr int FLAT_RAYS = 64;        // detector columns per wave (forward), staged columns per view (back)
constexpr int FLAT_MAX_SPAN = 256;   // most voxels of a slab that a wave's beams may cover
constexpr int FLAT_MAX_WAVES = 16;   // waves of a workgroup that share its slabs / its views
// Candidates of a pixel in a slab whose voxels are fetched before the slab's records are formed, under eight items and from eight on.  One
// item, none / 1 / 2 / 3 / 4 ahead: fan 223 x 246, 271 views of 295 160 / 136 / 132 / 129 / 132 us; eight: 450 x 373, 553 views of 408 816 /
// 752 (none, without the grid's idle tiles) / 727 / 708 (2) us.
constexpr int FLAT_AHEAD = 3, FLAT_AHEAD_8 = 2;
// Fewest wave steps (views, tiles of 64 columns, slabs, groups of items) for which a launch of several items makes the turned copy as well,
// fan / parallel beams.  With over without: fan 36000 to 148000 steps 1.04 to 1.13, 226000 0.83, 282000 1.00, 1400000 and 4400000 0.96 and
// 0.95; parallel 32000 1.05, 46000 0.90, 950000 0.77.  One item gains nothing.
constexpr double FLAT_TURN_STEPS = 2e5, FLAT_TURN_STEPS_PARALLEL = 4e4;
// Tiles of 64 columns per view: an odd number (see sf_project_flat) where there are more than two and more than two workgroups per CU, and
// one launch (fewer than 2^32 threads) holds it.  Odd over the number as it is: 4 tiles of 200 views 0.91 to 0.98, of 60 views 1.15; 2 tiles, 90 to 2000
// views 1.02 to 1.40.
SF_HD int flat_tiles(int ncols, int nviews)
{
    const int tiles = ncols / FLAT_RAYS + (ncols % FLAT_RAYS != 0);
    return tiles > 2 && (double)tiles * nviews > 512.0 && (double)(tiles | 1) * nviews * 64.0 < 4294967296.0 ? tiles | 1 : tiles;
}

constexpr int FLAT_T = 8;            // tile edge of the back projection, voxels
// Widest footprint of any voxel, in detector columns, and the columns a voxel can then touch.  A tile's voxel lies at most
// 4 sqrt(2) T from the voxel the window is centred on, and a displacement of sqrt(2) T moves the shadow by at most the
// widest footprint: the columns a lane reads lie within 4 * 5 + 5 / 2 + 6 < 32 of the centre.
constexpr double FLAT_MAX_COLS = 5.0;
constexpr int FLAT_NC = 6;

// A voxel's transaxial footprint as the forward kernel keeps it in LDS.
struct alignas(16) SfFlatRec {
    double xi;
    float o0, o1, o2, o3, h01, h23;
};

SF_HD SfFlatRec sf_flat_record(const SfColumn &f) { return SfFlatRec{f.xi, f.o0, f.o1, f.o2, f.o3, f.h01, f.h23}; }

SF_HD float sf_flat_fu(const SfFlatRec &r, int c)
{
    SfColumn f;
    f.xi = r.xi;
    f.o0 = r.o0; f.o1 = r.o1; f.o2 = r.o2; f.o3 = r.o3;
    f.h01 = r.h01; f.h23 = r.h23;
    return sf_fu(f, c);
}

// Parallel beams: all footprints of a view have one shape, only their place differs.  (The same numbers as sf_column's.)
SF_HD SfColumn sf_flat_parallel_column(const SfGeom &g, const SfView &v, int i, int j)
{
    SfColumn f;
    const double x = fma((double)i, g.Td, g.x0d), y = fma((double)j, g.Td, g.y0d);
    f.xi = fma(fma(y, v.cd, -x * v.sd), g.kud, g.col_offd);
    f.den = f.inv = 1.0;
    f.o0 = -v.par_out; f.o1 = -v.par_in; f.o2 = v.par_in; f.o3 = v.par_out;
    f.h01 = 0.5f * sf_rcp(fmaxf(f.o1 - f.o0, 1e-20f));
    f.h23 = 0.5f * sf_rcp(fmaxf(f.o3 - f.o2, 1e-20f));
    return f;
}

// ... and how far it moves on the detector from one voxel of a slab to the next.
SF_HD double sf_flat_step(const SfGeom &g, const SfView &v, int xmajor) { return xmajor ? g.Td * v.cd * g.kud : -g.Td * v.sd * g.kud; }

// F_u of a voxel whole steps beyond the footprint `first`, `edge` the pixel's lower edge from that one's centre.
SF_HD float sf_flat_stepped_fu(const SfColumn &first, double edge, double step, int steps) { return sf_fu_at(first, (float)fma((double)-steps, step, edge)); }

// Slabs [begin, end) of a wave: n_major * wave / nwaves on, nwaves a power of two (64-bit divisions cost the smallest calls a microsecond).
SF_HD void sf_flat_share(int n_major, int wave, int nwaves, int &begin, int &end)
{
    const int share = 31 - __builtin_clz(nwaves), whole = n_major >> share, rest = n_major - (whole << share);
    begin = whole * wave + (rest * wave >> share);
    end = begin + whole + ((rest * (wave + 1) >> share) - (rest * wave >> share));
}

// Marching axis of the wave whose first column is c0: that of its middle beam.
SF_HD int sf_flat_xmajor(const SfGeom &g, const SfView &v, int c0)
{
    const int mid = c0 + FLAT_RAYS / 2 < g.ncols ? c0 + FLAT_RAYS / 2 : g.ncols - 1;
    return sf_ray_lines<0>(g, v, mid, 1).xmajor;
}

// Tile and staged columns of the back projection by the number of views a wave takes at a time (SUB: 1, 2 or 4; 64 / SUB lanes each).  The
// lanes beside the tile's middle voxel lie at most 4 sqrt(2), sqrt(20), 2 sqrt(2) voxels from it, so the columns they read lie within
// 29, 25, 19 of its own (see FLAT_MAX_COLS).
template <int SUB>
struct FlatTile {
    static constexpr int TX = SUB == 4 ? 4 : 8, TY = SUB == 1 ? 8 : 4, LANES = 64 / SUB, COLS = SUB == 4 ? 48 : 64, LOADS = COLS / LANES;
};

#if defined(__HIPCC__) && !defined(SF_NO_KERNELS)

// [nvol] slices of `items` items, nvol apart, to [group][nvol][NB]; the last group's missing items become zeros.
template <int NB>
__global__ __launch_bounds__(256) void sf_interleave(const float *__restrict__ vol, float *__restrict__ dst, unsigned nvol, int items)
{
    const unsigned e = blockIdx.x * 256u + threadIdx.x;
    if (e >= nvol) return;
    const int b0 = blockIdx.y * NB;
    float x[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) x[b] = b0 + b < items ? vol[(size_t)(b0 + b) * nvol + e] : 0.0f;
    float *__restrict__ d = dst + ((size_t)blockIdx.y * nvol + e) * NB;
#pragma unroll
    for (int b = 0; b < NB; ++b) d[b] = x[b];
}

// The same with the slices' rows running along y: [ny][nx] to [group][nx][ny][NB].  Block 32 x 8 threads, tile 32 x 32 voxels; blockIdx.z: group.
template <int NB>
__global__ __launch_bounds__(256) void sf_interleave_turned(const float *__restrict__ vol, float *__restrict__ turned, int nx, int ny, int items)
{
    __shared__ float tile[32][33 * NB];
    const size_t nvol = (size_t)nx * ny;
    const int b0 = blockIdx.z * NB, i0 = blockIdx.x * 32, j0 = blockIdx.y * 32, tx = threadIdx.x, ty = threadIdx.y;
    turned += (size_t)b0 * nvol;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int i = i0 + tx, j = j0 + ty + 8 * s;
        const bool in = i < nx && j < ny;
#pragma unroll
        for (int b = 0; b < NB; ++b) tile[ty + 8 * s][tx * NB + b] = in && b0 + b < items ? vol[(size_t)(b0 + b) * nvol + (size_t)j * nx + i] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int i = i0 + ty + 8 * s, j = j0 + tx;
        if (i >= nx || j >= ny) continue;
#pragma unroll
        for (int b = 0; b < NB; ++b) turned[((size_t)i * ny + j) * NB + b] = tile[tx][(ty + 8 * s) * NB + b];
    }
}

// Sums the waves' partial results of a workgroup in wave order; the total is valid in wave 0.  red: NB * 64 floats per wave.
template <int NB>
__device__ __forceinline__ void flat_reduce(float (&acc)[NB], float *__restrict__ red, int wave, int lane, int nwaves)
{
    if (nwaves == 1) return;
    __syncthreads();                    // every wave has read what it keeps in this LDS
    if (wave > 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) red[(wave * NB + b) * 64 + lane] = acc[b];
    }
    __syncthreads();
    if (wave == 0) {
        for (int w = 1; w < nwaves; ++w)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] += red[(w * NB + b) * 64 + lane];
    }
}

// Orders a wave's LDS writes before its own later reads (and the other way round); no other wave is involved.
__device__ __forceinline__ void flat_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// grid.x = views * tiles of 64 columns, tiles rounded up to an odd number where there are many: workgroups go to the 8 XCDs by index in turn, and an XCD that gets
// the same tile of every view finishes early if it is one at the detector's edge.  grid.y: groups of NB items (NB == 1: items).  Block: waves
// that share the slabs.  src: NB == 1 the slices themselves, otherwise the batch-fastest copy of this launch's items; turned: the copy whose
// rows run along y, for waves whose slabs do (nullptr: they read src across its rows).  span: records per wave
// (PAR, parallel beams: none, every lane works out where its few voxels' footprints lie).
template <int NB, bool PAR>
__global__ __launch_bounds__(FLAT_MAX_WAVES * 64) void sf_project_flat(SfGeom g, const SfView *__restrict__ views,
                                                                       const float *__restrict__ src, const float *__restrict__ turned,
                                                                       float *__restrict__ sino, int tiles, int span, int items, float fv)
{
    extern __shared__ float4 flat_lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    // a record's halves lie in arrays of their own: neighbouring lanes read neighbouring 16 bytes of either
    float4 *__restrict__ rec_lo = flat_lds + (size_t)wave * span * 2, *__restrict__ rec_hi = rec_lo + span;
    const int a = blockIdx.x / tiles, c0 = (blockIdx.x - a * tiles) * FLAT_RAYS;
    if (c0 >= g.ncols) return;                   // the grid's padding (whole workgroups)
    const unsigned nvol = (unsigned)g.nx * (unsigned)g.ny;

    const SfView v = views[a];
    const int c = c0 + lane < g.ncols ? c0 + lane : g.ncols - 1;
    const int xmajor = __builtin_amdgcn_readfirstlane(sf_flat_xmajor(g, v, c0));
    const SfRayLines L = sf_ray_lines<0>(g, v, c, 1, xmajor);
    const int n_major = xmajor ? g.nx : g.ny, n_minor = xmajor ? g.ny : g.nx;
    const bool across = xmajor && !turned;
    src = (xmajor && turned ? turned : src) + (size_t)blockIdx.y * nvol * NB;
    const unsigned n_stride = across ? 1u : (unsigned)n_minor, q_stride = across ? (unsigned)g.nx : 1u;
    int n_begin, n_end;
    sf_flat_share(n_major, wave, nwaves, n_begin, n_end);
    const double step = sf_flat_step(g, v, xmajor);         // (PAR)

    float acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = 0.0f;
    for (int n = n_begin; n < n_end; ++n) {
        int qf, ql;
        sf_candidates(L, n, qf, ql);
        // the beams of the outermost columns bound the run of voxels
        const int f0 = __builtin_amdgcn_readlane(qf, 0), f1 = __builtin_amdgcn_readlane(qf, 63);
        const int l0 = __builtin_amdgcn_readlane(ql, 0), l1 = __builtin_amdgcn_readlane(ql, 63);
        int q_lo = f0 < f1 ? f0 : f1, q_hi = l0 > l1 ? l0 : l1;
        q_lo = q_lo < 0 ? 0 : q_lo;
        q_hi = q_hi > n_minor - 1 ? n_minor - 1 : q_hi;
        q_hi = q_hi > q_lo + span - 1 ? q_lo + span - 1 : q_hi;        // (never: the host sized the span)
        if (q_lo > q_hi) continue;
        qf = qf < q_lo ? q_lo : qf;
        ql = ql > q_hi ? q_hi : ql;
        // the first candidates' voxels, in flight while the records are formed (a lane without candidates reads another's)
        const float *__restrict__ col = src + (size_t)((unsigned)n * n_stride) * NB;
        constexpr int AHEAD = NB < 8 ? FLAT_AHEAD : FLAT_AHEAD_8;
        float ahead[AHEAD > 0 ? AHEAD : 1][NB];
#pragma unroll
        for (int m = 0; m < AHEAD; ++m) {
            const int q = qf + m < q_hi ? qf + m : q_hi;
            const float *__restrict__ x = col + (size_t)((unsigned)q * q_stride) * NB;
#pragma unroll
            for (int b = 0; b < NB; ++b) ahead[m][b] = x[b];
        }
        for (int q0 = q_lo; !PAR && q0 <= q_hi; q0 += 64) {
            const int q = q0 + lane;
            if (q <= q_hi) {
                const SfFlatRec r = sf_flat_record(sf_column<0>(g, v, xmajor ? n : q, xmajor ? q : n));
                rec_lo[q - q_lo] = reinterpret_cast<const float4 *>(&r)[0];
                rec_hi[q - q_lo] = reinterpret_cast<const float4 *>(&r)[1];
            }
        }
        if constexpr (!PAR) flat_wave_sync();
        // PAR: the footprint of the lane's first candidate and the pixel's lower edge from its centre; the others' lie whole steps on
        SfColumn first;
        double edge = 0.0;
        if constexpr (PAR) {
            first = sf_flat_parallel_column(g, v, xmajor ? n : qf, xmajor ? qf : n);
            edge = ((double)c - 0.5) - first.xi;
        }
        auto weight = [&](int q) {
            if constexpr (PAR) return sf_flat_stepped_fu(first, edge, step, q - qf);
            SfFlatRec r;
            reinterpret_cast<float4 *>(&r)[0] = rec_lo[q - q_lo];
            reinterpret_cast<float4 *>(&r)[1] = rec_hi[q - q_lo];
            return sf_flat_fu(r, c);
        };
        // (a voxel beside the beam does not touch it, whatever it holds)
#pragma unroll
        for (int m = 0; m < AHEAD; ++m) {
            if (qf + m <= ql) {
                const float fu = weight(qf + m);
                if (fu > 0.0f) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = fmaf(fu, ahead[m][b], acc[b]);
                }
            }
        }
        for (int q = qf + AHEAD; q <= ql; ++q) {
            const float fu = weight(q);
            if (!(fu > 0.0f)) continue;
            const float *__restrict__ x = col + (size_t)((unsigned)q * q_stride) * NB;
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = fmaf(fu, x[b], acc[b]);
        }
        if constexpr (!PAR) flat_wave_sync();
    }
    flat_reduce<NB>(acc, reinterpret_cast<float *>(flat_lds), wave, lane, nwaves);
    if (wave == 0 && c0 + lane < g.ncols) {
        const float amp = sf_amp(g, v, sf_amp_col<0>(g, v, c), 0) * fv;
        const size_t nsino = (size_t)g.nviews * g.ncols;
        float *__restrict__ y = sino + (size_t)blockIdx.y * NB * nsino + (size_t)a * g.ncols + c;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if ((int)blockIdx.y * NB + b < items) y[b * nsino] = amp * acc[b];
    }
}

// grid.x = tiles of TX x TY voxels; grid.y: groups of NB items.  Block: waves that share the views; wave w takes runs of `shares` adjacent
// views, shares w on, a run of every wave apart, and sums the first of every run, then the second, ...  SUB > 1 (16 waves, shares a multiple of SUB):
// SUB views of a run at a time, so that slices whose 8 x 8 tiles are fewer than the compute units give every unit a workgroup.  The order of
// the sums depends on shares alone: however many views a wave takes at a time, the bits are the same.
// RUNS: shares may be above 1 (a template, for one item: the loop over runs costs it up to 4 % where a run is one view, 313 x 334 voxels, 135
// parallel views 40.0 -> 41.2 us, and two to eight items take up to 7 % less time with it, 16 x 210 x 239, 100 views 66.1 -> 61.9).
template <int NB, int SUB, bool RUNS>
__global__ __launch_bounds__(FLAT_MAX_WAVES * 64) void sf_backproject_flat(SfGeom g, const SfView *__restrict__ views,
                                                                           const float *__restrict__ sino, float *__restrict__ vol,
                                                                           int tiles_x, int items, int run_views, float fv)
{
    static_assert(SUB == 1 || RUNS, "several views at a time are views of a run");
    const int shares = RUNS ? run_views : 1;
    typedef FlatTile<SUB> Tile;
    constexpr int LOADS = Tile::LOADS;
    float *lds;
    if constexpr (SUB > 1) {
        __shared__ float room[FLAT_MAX_WAVES * SUB * Tile::COLS * NB];
        lds = room;
    } else {
        extern __shared__ float4 flat_lds[];
        lds = reinterpret_cast<float *>(flat_lds);
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int sub = SUB == 1 ? 0 : lane / Tile::LANES, l = SUB == 1 ? lane : lane % Tile::LANES;
    float *__restrict__ buf = lds + (wave * SUB + sub) * (Tile::COLS * NB);       // [column][item]
    const int ty = blockIdx.x / tiles_x, tx = blockIdx.x - ty * tiles_x;
    const int i = tx * Tile::TX + l % Tile::TX, j = ty * Tile::TY + l / Tile::TX;
    const int ic = i < g.nx ? i : g.nx - 1, jc = j < g.ny ? j : g.ny - 1;    // lanes beyond the edge shadow it
    const size_t nsino = (size_t)g.nviews * g.ncols;
    const int b0 = blockIdx.y * NB;
    sino += (size_t)b0 * nsino;

    float total[NB], acc[NB], stage[LOADS][NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) total[b] = 0.0f;
    SfColumn f;
    int first = 0;                              // first staged column
    // a: the first of the SUB views; one beyond the last is read as zeros
    auto view_of = [&](int a) { return SUB == 1 ? a : (a + sub < g.nviews ? a + sub : g.nviews - 1); };
    auto fetch = [&](int a) {
        f = sf_column<0>(g, views[view_of(a)], ic, jc);
        const int centre = (int)floor(f.xi);
        constexpr int MIDDLE = (Tile::TY / 2) * Tile::TX + Tile::TX / 2;
        if constexpr (SUB == 1) first = __builtin_amdgcn_readlane(centre, MIDDLE) - Tile::COLS / 2;
        else first = __shfl(centre, sub * Tile::LANES + MIDDLE) - Tile::COLS / 2;
#pragma unroll
        for (int k = 0; k < LOADS; ++k) {
            const int c = first + l + k * Tile::LANES;
            const bool in = (unsigned)c < (unsigned)g.ncols && (SUB == 1 || a + sub < g.nviews);
            const float *__restrict__ y = sino + (size_t)view_of(a) * g.ncols + (in ? c : 0);
#pragma unroll
            for (int b = 0; b < NB; ++b) stage[k][b] = in && b0 + b < items ? y[b * nsino] : 0.0f;
        }
    };
    const int run = wave * shares;
    if (run < g.nviews) fetch(run);
    for (int s = 0; s < shares && run + s < g.nviews; s += SUB) {
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = 0.0f;
        for (int a = run + s; a < g.nviews; a += nwaves * shares) {
            const SfView &v = views[view_of(a)];
#pragma unroll
            for (int k = 0; k < LOADS; ++k) {
                const float amp = sf_amp(g, v, sf_amp_col<0>(g, v, first + l + k * Tile::LANES), 0) * fv;
#pragma unroll
                for (int b = 0; b < NB; ++b) buf[(l + k * Tile::LANES) * NB + b] = stage[k][b] * amp;
            }
            flat_wave_sync();
            int cf, cl;
            sf_col_range(f, cf, cl);
            const float *__restrict__ q = buf + (cf - first) * NB;
            float e = sf_pixel_edge(f, cf);
            const SfColumn now = f;
            // the next views, in flight during the gather
            const int next = !RUNS || a + nwaves * shares < g.nviews ? a + nwaves * shares : run + s + SUB;
            if (next < g.nviews && (!RUNS || next > a || s + SUB < shares)) fetch(next);
            float g0 = sf_trap_integral(now, e);
#pragma unroll
            for (int m = 0; m < FLAT_NC; ++m) {
                if (m > 1 && __builtin_amdgcn_ballot_w64(cf + m <= cl) == 0) break;      // no lane's footprint reaches this far
                e += 1.0f;
                const float g1 = sf_trap_integral(now, e), fu = fmaxf(g1 - g0, 0.0f);
                g0 = g1;
                if (fu > 0.0f) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = fmaf(fu, q[m * NB + b], acc[b]);
                }
            }
            flat_wave_sync();
        }
#pragma unroll
        for (int k = 0; k < SUB; ++k)
#pragma unroll
            for (int b = 0; b < NB; ++b) total[b] += SUB == 1 ? acc[b] : __shfl(acc[b], k * Tile::LANES + l);
    }
    flat_reduce<NB>(total, lds, wave, lane, nwaves);
    if (wave == 0 && sub == 0 && i < g.nx && j < g.ny) {
        const size_t nvol = (size_t)g.nx * g.ny;
        float *__restrict__ x = vol + (size_t)b0 * nvol + (size_t)j * g.nx + i;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (b0 + b < items) x[b * nvol] = total[b];
    }
}

#endif
