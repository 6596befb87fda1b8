// Internal types shared by the host runtime and the gfx950 kernels. The tile
// list and queue split they consume are described in plan_logic.h.
#pragma once

#include <stdint.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "plan_logic.h"

namespace dg {

constexpr int kSupportUV = 8;   // G_uv support per axis (Section 2)
constexpr int kSupportW = 4;    // G_w support (Section 2)
constexpr int kWave = 64;       // CDNA wavefront
constexpr int kBlockThreads = 256;
constexpr int kWavesPerBlock = kBlockThreads / kWave;
// The table-gradient kernel runs one workgroup of eight wavefronts per CU
// (its registers allow two wavefronts per SIMD), so that eight wavefronts
// share one LDS copy of dL/dG_uv and half as many copies are added to the
// output at the end as with two workgroups of four.
constexpr int kTableGradThreads = 512;

// Invalid-offset sentinel for hardware bounds-checked (buffer) loads: any
// offset at or above a resource's size returns zero. Subgrids and tables are
// limited to less than this many bytes.
constexpr uint32_t kOutOfRange = 0x40000000u;

// Everything a kernel needs to know about one problem.
struct Problem {
    const void* subgrids;   // [S][n_v][n_u][n_w] in the grid dtype
    const void* g_uv;       // [os_uv][os_uv][8][8] in the gcf dtype
    const void* g_w;        // [os_w][4] in the gcf dtype
    const double* uvw;      // [N][3]
    void* vis;              // complex float32 [N]: degrid output / adjoint input
    void* grid_out;         // complex float32 [S][n_v][n_u][n_w]: adjoint output
    const uint32_t* perm;   // work order: tile position -> visibility index; nullptr = identity
    int64_t cells_per_sub;  // n_v * n_u * n_w
    int32_t n_v, n_u, n_w;
    int32_t log2_os_uv, log2_os_w;   // log2 of the oversampling, or -1 if not a power of two
    uint32_t guv_bytes;     // size of G_uv in bytes
    uint32_t sub_bytes;     // size of one subgrid in bytes (grid dtype)
    int32_t os_uv, os_w;    // oversampling factors
    int32_t pad_;
    double hi_u, hi_v, hi_w;  // exclusive upper bounds of in-range coordinates
};

// Device control block of a plan or batch: queue cursors (one 128-byte line
// each, so atomics from different XCDs do not share a line), the count of
// finished workgroups, and the out-of-range counters. The last workgroup of
// every launch resets the cursors and the counters, so a launch needs no
// separate reset and can be replayed from a graph. Atomics on one counter
// take about 20 ns apiece when they queue, so with one counter the end of a
// launch whose workgroups all finish together waits on a chain as long as
// the grid. Such a kernel (the adjoint's record pass), on a grid of more than
// kDoneFlat workgroups, counts their ends in two levels: into one of
// kDoneGroups group counters (workgroup b into b mod kDoneGroups), and the
// last of each group into `done`. Other kernels, and small grids, count into
// `done` directly, which saves the second, dependent atomic.
constexpr int kDoneGroups = 8;
constexpr int kDoneFlat = 64;
struct alignas(128) CtlLine { uint32_t v[32]; };
struct Ctl {
    CtlLine cursor[kMaxQueues];   // v[0]: tiles claimed; v[1]: queues known to have run dry (degrid kernel)
    CtlLine done;
    CtlLine oob;   // v[0..1]: running count (u64), v[2..3]: count of the last launch
    CtlLine group[kDoneGroups];
    CtlLine moved;   // owner-computes adjoint: visibilities whose first tap moved; v[0] running, v[1] of the last call
};

struct LaunchParams {
    Problem prob;               // used when probs == nullptr
    const Problem* probs;       // per-problem table of a batch
    const Tile* tiles;
    const uint32_t* tile_vis;   // [n_tiles][kMaxNb]: visibility index of each work item
    Ctl* ctl;
    QueueSpec q;
    StaticDeal deal;            // filled by launch_degrid for its grid size
    // Residual mode (one problem only; v_obs == nullptr: plain degrid). The
    // output becomes v_obs - degrid and each tile stores the float64 sum of
    // |residual|^2 of its visibilities in tile_loss[t] (summed afterwards by
    // launch_loss_sum).
    const float2* v_obs;
    double* tile_loss;
};

// The owner-computes adjoint of a sorted plan. The output is cut into bands
// of kOwnerBand rows, segments of columns and slabs of kSupportW w planes. The
// visibilities that reach a band, ordered by first column, are one run of the
// owner order; a visibility has a place in each of the one or two bands its
// window reaches.
constexpr int kOwnerBand = 16;            // rows of a band
constexpr int kOwnerMaxSegment = 112;     // columns of a segment, at most
// w planes of a subgrid, at most: every slab's task walks the visibilities of its
// band and segment, and writes 32 bytes of each cell, so deeper stacks scatter
// instead (owners and scattered, us: 100 000 visibilities on 4 subgrids of 64 x 64 x
// 3000 384 and 2721, x 8000 994 and 2958; 1000 on 64 x 64 x 2000 42 and 53, x 8000
// 126 and 85).
constexpr int kOwnerMaxPlanes = 3072;
constexpr uint32_t kNoPlace = 0xFFFFFFFFu;
// visibilities, at most: the positions of their two places each, and a batch past
// the last of them, are 32-bit
constexpr int64_t kOwnerMaxVis = 0x7FFFFF00;
static_assert(2 * kOwnerMaxVis + kWave <= (int64_t)kNoPlace, "a run's last batch ends within 32 bits");

struct OwnerPlaces {
    uint32_t first, second;   // positions in the owner order, or kNoPlace
};

// What the sums need of one visibility, per position of the owner order.
struct alignas(16) OwnerRecord {
    uint32_t start;   // first tap (y0 << 16 | x0), or kNoStart: skipped
    uint32_t rows;    // G_uv block, G_w row and first w plane
    float re, im;
};
static_assert(sizeof(OwnerRecord) == 16, "one 16-byte load");

// One segment of a band (and slab of planes): what one wavefront writes.
struct OwnerTask {
    uint32_t begin, end;   // positions of the owner order
    int32_t band;          // subgrid * nby + band
    int32_t place;         // segment * n_slabs + slab
};
static_assert(sizeof(OwnerTask) == 16, "OwnerTask must stay 16 bytes");

// A task's run takes one wavefront about 0.1 us per visibility, so on plans whose
// longest run is much longer than an even share, runs are cut into slices, one
// wavefront each. A slice writes the columns it reaches to a workspace
// ([kOwnerBand rows][width][4 w values] complex64), and the join pass adds a task's
// slices in their order and writes the segment.
//
// With W = places times slabs: runs are cut where the longest exceeds W /
// kOwnerEven + kOwnerJoin. W / 2844 is a wavefront's even share of all runs at 16
// per CU, where a visibility takes 0.23 us, and kOwnerJoin (22 us) stands for the
// workspace and the join, a launch more on the host. Whole and cut (us): 8 subgrids
// of 283 x 266 with 400 000 visibilities (longest about 450) 72 and 96, 4 of 256 x
// 256 with 64 000 (190) 32 and 38, with 128 000 (330) 52 and 45 (not enough where the
// host sets the pace); 4 of 512 x 512 with 16 000 at their centres 49 and 32, 3 of
// 430 x 176 with 400 000 (1150) 136 and 81, 3 of 188 x 162 with 100 000 (700) 87 and 37.
// Longest slice: the larger of kOwnerMinSlice and W / kOwnerSlices, whole batches of
// 64 (60 000 visibilities on one spot 40 us, with 64 52 and with 256 50; 1.0 M dense
// at the centres of 16 subgrids 157 us, with W / 1024 216 and with W / 4096 167). At
// most kOwnerMaxSlices can come of that: the runs are together at most 2 W (a window
// reaches two segments at most), and cutting adds at most one slice per run longer
// than a slice.
constexpr int kOwnerMinSlice = 128;
constexpr int kOwnerSlices = 2048;
constexpr int kOwnerMaxSlices = 4 * kOwnerSlices;
constexpr int kOwnerEven = 1280;
constexpr int kOwnerJoin = 220;
constexpr int kOwnerShared = 16;   // slices that one wavefront of the join pass adds by itself
struct alignas(16) OwnerSlice {
    uint32_t begin, end;   // positions of the owner order
    int32_t band;          // subgrid * nby + band
    int32_t slab;
    int32_t x_lo, width;   // columns (x_lo a multiple of 8)
    uint32_t column;       // columns of the slices before it
    int32_t task;          // index of its task
};
static_assert(sizeof(OwnerSlice) == 32, "OwnerSlice must stay 32 bytes");
constexpr size_t kOwnerColumnBytes = (size_t)kOwnerBand * kSupportW * 8;   // of a slice's workspace

// What the tasks of a plan came to.
struct OwnerCounts {
    int64_t n_items;      // places of the owner order
    int64_t columns;      // of all slices
    int32_t n_split;      // tasks cut into slices: the first of the list
    int32_t n_slices;
    int32_t n_shared;     // of the split tasks, the first: more than kOwnerShared slices
};

// Plans of at most this many visibilities have no records: the owner pass reads the
// visibilities themselves, and the fix-up pass checks every one. That is one launch
// less, on the host too, and more scattered reads (records and direct): 2 subgrids
// with 8000 visibilities 20.7 and 14.8 us, 16 with 32 000 36.8 and 33.2, with
// 128 000 47.9 and 45.0, with 256 000 62.5 and 64.1, with 512 000 88.3 and 95.5.
// Every slab reads them again: at most kOwnerDirectWork visibilities times slabs
// (100 000 visibilities on 4 subgrids of 64 x 64 x 256: 352 and 398 us).
constexpr int64_t kOwnerDirect = 3 << 16;
constexpr int64_t kOwnerDirectWork = 1 << 18;

struct OwnerParams {
    Problem prob;                  // g_uv, g_w, vis (input), grid_out; uvw without records
    const OwnerRecord* records;    // from the record pass, or nullptr: the two below
    const uint32_t* items;         // visibility at each position of the owner order
    const uint32_t* plan_start;    // first tap of each visibility at the sort
    const OwnerTask* tasks;        // heaviest first, n_split of them in slices
    const OwnerSlice* slices;      // by task and position
    const uint32_t* first_slice;   // per split task, and the end
    char* partials;                // the slices' workspace
    int64_t n_tasks;
    int32_t n_split, n_slices;
    Ctl* ctl;
    int32_t accumulate;            // 1: add to grid_out, 0: overwrite
    int32_t nby;                   // bands per subgrid
    int32_t segment;               // columns of a segment
    int32_t n_slabs;               // slabs of w planes
    int32_t n_shared;              // OwnerCounts
};

// Table-gradient pass: dL/dG_uv and dL/dG_w from dL/dV over the tiles of a
// plan (prob.vis holds dL/dV, complex float32 [N]).
struct TableGradParams {
    Problem prob;
    const Tile* tiles;
    const uint32_t* tile_vis;
    int64_t n_tiles;
    float* grad_uv;   // [os_uv][os_uv][8][8], or nullptr
    float* grad_w;    // [os_w][4], or nullptr
};

enum GridKind : int32_t { kGridC64 = 0, kGridCBF16 = 1, kGridCF16 = 2 };
enum GcfKind : int32_t { kGcfF32 = 0, kGcfF16 = 1, kGcfBF16 = 2 };

// Kernel launchers (defined in degrid_kernels.hip, grid_kernels.hip and
// table_grad_kernels.hip).
hipError_t launch_degrid(const LaunchParams& p, int grid_kind, int gcf_kind, int variant,
                         int blocks, hipStream_t stream);
hipError_t launch_grid_adjoint(const LaunchParams& p, int gcf_kind, int variant, int blocks,
                               hipStream_t stream);
hipError_t launch_zero(void* ptr, int64_t bytes, hipStream_t stream);
// Index of the degrid kernel variant for subgrids deeper than the w support
// (no staging).
constexpr int kDeepVariant = 5;
// Index of the variant with the lane mapping of the paper's kernel D1 (two
// visibilities per wavefront, lanes over (t_u, t_w), accumulation along v).
constexpr int kD1Variant = 6;
// *loss = sum of tile_loss[0 .. n_tiles) in a fixed order (same bits every time).
hipError_t launch_loss_sum(const double* tile_loss, int64_t n_tiles, double* loss, hipStream_t stream);
// *p = v (one float64 written by a kernel, so that graphs may capture it).
hipError_t launch_set_f64(double* p, double v, hipStream_t stream);
// Owner-computes adjoint: every output cell written once (a second launch joins
// the slices, if there are any). n_cu and max_lds: the device's compute units and
// LDS bytes per workgroup.
hipError_t launch_grid_owner(const OwnerParams& p, int gcf_kind, int n_cu, size_t max_lds, hipStream_t stream);
// Record pass of the adjoint: the records of every visibility, the
// out-of-range count into ctl, and the number whose first tap differs from
// plan_start (their records are skipped ones) into own_ctl. At most max_blocks
// workgroups (each one's end is an atomic on the control block, so the grid is
// kept near the device's resident capacity).
hipError_t launch_grid_record(const Problem& pr, int64_t n_vis, const uint32_t* plan_start, const OwnerPlaces* place,
                              OwnerRecord* records, Ctl* ctl, Ctl* own_ctl, int max_blocks, hipStream_t stream);
// Adds, with atomics, the visibilities whose first tap differs from the
// plan's; nothing when the record pass counted none (own_ctl; nullptr: there was
// none, and every visibility is checked and the out-of-range count goes to ctl).
// n_vis visibilities of one problem; vis_offsets on the device.
hipError_t launch_grid_fixup(const Problem& pr, const int64_t* vis_offsets, int64_t n_sub, int64_t n_vis,
                             const uint32_t* plan_start, const Ctl* own_ctl, Ctl* ctl, int gcf_kind, int max_blocks,
                             hipStream_t stream);
// tile_vis[t * kMaxNb + j] = visibility index of item j of tile t: through
// perms[tile.problem] (a work-order permutation, or nullptr for input order)
// at position tile.begin + j; items past the tile's count repeat its first.
hipError_t launch_expand_tiles(const Tile* tiles, int64_t n_tiles, const uint32_t* const* perms,
                               uint32_t* tile_vis, hipStream_t stream);

// Device memory for the length of a plan-building call; grows on demand.
struct DeviceTemp {
    void* p = nullptr;
    size_t bytes = 0;
    DeviceTemp() = default;
    DeviceTemp(const DeviceTemp&) = delete;
    DeviceTemp& operator=(const DeviceTemp&) = delete;
    ~DeviceTemp() {
        if (p) (void)hipFree(p);
    }
    hipError_t ensure(size_t need) {
        if (need <= bytes) return hipSuccess;
        if (p) (void)hipFree(p);
        p = nullptr;
        bytes = 0;
        const hipError_t e = hipMalloc(&p, need);
        if (e == hipSuccess) bytes = need;
        else p = nullptr;
        return e;
    }
};

// Cutting of tiles that fit a staging box, on the device, by one wavefront for
// each chunk of up to kFitChunk positions (a tile does not cross the end of a
// chunk): a tile is the longest run of at most nb visibilities whose box holds
// at most cap_cells cells; where that is fewer than min_fit, min_fit
// visibilities that are gathered without staging.
constexpr int kFitChunk = 2048;
struct FitChunk {
    int64_t begin;    // first position of the work order
    int32_t count;    // positions, at most kFitChunk
    int32_t sub;      // subgrid
};
struct FitRule {
    int32_t nb, support, cap_cells, min_fit;
};
// first_tile[k] = tiles of the chunks before k, for k = 0 .. n_chunks.
hipError_t launch_count_tiles(const FitChunk* chunks, int64_t n_chunks, const uint32_t* start, const FitRule& rule,
                              uint32_t* first_tile, hipStream_t stream);
// The tiles and their visibility indices, and the queues of about equal numbers
// of visibilities that split_queues makes of such a list (n_vis in all).
hipError_t launch_write_tiles(const FitChunk* chunks, int64_t n_chunks, const uint32_t* start, const uint32_t* perm,
                              const FitRule& rule, const uint32_t* first_tile, int64_t n_tiles, int64_t n_vis,
                              Tile* tiles, uint32_t* tile_vis, QueueSpec* q, hipStream_t stream);

// Stable sort of each subgrid's visibilities by the Hilbert-curve position of
// their first tap (defined in plan_sort.hip); pr names the coordinates and the
// subgrid geometry. Writes perm[n_vis], the visibility index at each position
// of the work order; plan_start[n_vis], the first tap of each visibility
// (kNoStart when out of range), and start[n_vis], the same per position of the
// work order. offsets: device copy of offsets_host. Uses 'temp' on 'stream'.
hipError_t sort_visibilities(const Problem& pr, const int64_t* offsets_host, const int64_t* offsets, int64_t n_sub,
                             uint32_t* perm, uint32_t* plan_start, uint32_t* start, DeviceTemp& temp,
                             hipStream_t stream);
// The owner order of the adjoint and its tasks, from the first taps: places
// [n_vis] and tasks[shape.tasks()], heaviest first; the slices [shape.slices()]
// of the heavy ones and first_slice [shape.slices() + 1]. *counts receives what
// there is of them. shape.direct: 'places' receives the visibility at each position
// instead ([2 n_vis] uint32). Uses 'temp'; synchronises 'stream'.
struct OwnerShape {
    int64_t n_sub, n_vis;
    int32_t nby, n_u, segment, n_seg, n_slabs;
    bool direct;   // no records (kOwnerDirect)
    int64_t tasks() const { return n_sub * nby * n_seg * n_slabs; }
    // room for slices (a visibility has two places, each reaches two segments)
    int64_t slices() const { return std::min<int64_t>(kOwnerMaxSlices, 8 * n_vis * n_slabs / kOwnerMinSlice + 1); }
};
hipError_t build_owner_order(const OwnerShape& shape, const int64_t* offsets, const uint32_t* plan_start,
                             OwnerPlaces* places, OwnerTask* tasks, OwnerSlice* slices, uint32_t* first_slice,
                             OwnerCounts* counts, DeviceTemp& temp, hipStream_t stream);
hipError_t degrid_kernel_occupancy(int grid_kind, int gcf_kind, int variant, int* blocks_per_cu);
hipError_t adjoint_kernel_occupancy(int gcf_kind, int variant, int* blocks_per_cu);
int degrid_variant_count();
int adjoint_variant_count();
int degrid_variant_box_bytes(int variant);   // LDS staging bytes per wavefront (0: none)
int degrid_variant_max_nb(int variant);      // largest tile the variant accepts
bool degrid_variant_any_depth(int variant);  // reads subgrids with n_w > 4
constexpr int kMaxVariants = 8;
// Adds dL/dG_uv and dL/dG_w of every in-range visibility to p.grad_uv and
// p.grad_w (float atomics). deep: subgrids with more w planes than the support.
// max_lds: the device's LDS bytes per workgroup.
hipError_t launch_table_grad(const TableGradParams& p, int grid_kind, int gcf_kind, bool deep, int blocks,
                             size_t max_lds, hipStream_t stream);
// Dynamic LDS bytes of that kernel, and whether it accumulates dL/dG_uv in LDS.
void table_grad_shape(int os_uv, int os_w, bool want_uv, bool want_w, size_t max_lds, bool* lds_uv,
                      size_t* lds_bytes);
// p[0 .. n) = 0.0f (a kernel, so that graphs may capture it).
hipError_t launch_zero_f32(float* p, int64_t n, hipStream_t stream);

// Degridding without a plan (defined in noalloc.hip): its scratch is a
// file-scope device array of kNoAllocBytes per GPU (control blocks, the
// staged offsets and the tile offsets of at most kNoAllocMaxSubgrids
// subgrids). Input-order tiles of nb visibilities; n_tiles = sum over
// subgrids of ceil(N_s / nb). offsets_host [n_sub + 1] is copied into the
// scratch on 'stream', or travels with the launch. oob_out (device, may be null) receives the launch's
// out-of-range count. Allocates nothing.
constexpr int64_t kNoAllocMaxSubgrids = 16384;
constexpr size_t kNoAllocBytes = 235776;
// Resident workgroups of the kernel that call would launch on the current device.
hipError_t noalloc_resident(int grid_kind, int gcf_kind, int* resident);
hipError_t launch_degrid_noalloc(const Problem& pr, int grid_kind, int gcf_kind,
                                 const int64_t* offsets_host, int64_t n_sub, int nb, int64_t n_tiles,
                                 unsigned long long* oob_out, hipStream_t stream);

}  // namespace dg
