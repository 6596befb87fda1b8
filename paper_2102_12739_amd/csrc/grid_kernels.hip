// gfx950 kernels for gridding, the adjoint of 3D degridding (the transpose
// of the sum in Section 2): the tile kernel with an LDS staging box, the
// owner-computes kernel over plan-time output blocks, and its fix-up pass.
#include "dg_device.h"

#include <algorithm>
#include <type_traits>

namespace dg {
namespace {

// ---------------------------------------------------------------------------
// Adjoint (gridding) kernel
// ---------------------------------------------------------------------------
//
// The transpose of degridding: every in-range visibility V adds
// G_w[o_w][t_w] * G_uv[o_v][o_u][t_v][t_u] * V to the cell (y + t_v, x + t_u,
// z + t_w). Lanes map onto the 8 x 8 (t_v, t_u) taps as in the gather. When
// the tile's cells fit the wavefront's LDS box, contributions are summed
// there first (plain read-modify-write: a visibility's taps are distinct
// cells and LDS operations of one wavefront run in order) and the box is added to the output once
// with global float atomics; otherwise each contribution is a global atomic.

// V times the four G_w taps of one visibility, interleaved (re, im).
struct WeightedVis {
    float c[8];
};

template <int F, int BOX, int NB>
__global__ __launch_bounds__(kBlockThreads) void grid_adjoint_kernel(LaunchParams P) {
    static_assert(NB % 8 == 0 && NB <= kMaxNb, "tile size");
    constexpr int kBoxBytes = BOX > 0 ? BOX : 16;
    constexpr uint32_t kCell = kSupportW * 8;   // complex64 cell of 4 w values
    __shared__ __attribute__((aligned(16))) char s_box[kWavesPerBlock][kBoxBytes];

    const int lane = lane_id();
    const int wv = (int)(threadIdx.x / kWave);
    QueueState st{xcc_id() % P.q.n_queues, 0};
    uint32_t wave_oob = 0;

    int t = pop_tile(P.q, P.ctl, st);
    while (t >= 0) {
        const Tile tc = load_tile(P.tiles, t);
        const int t_next = pop_tile(P.q, P.ctl, st);
        const Problem pr = P.probs ? load_problem(P.probs, tc.problem) : P.prob;
        const int count = tc.count;

        // Coordinate stage; lane j also forms G_w * V of visibility j.
        int32_t x0 = 0, y0 = 0, cell = 0, tab = 0, ow = 0;
        bool in_range = false;
        WeightedVis cw;
#pragma unroll
        for (int q = 0; q < 8; ++q) cw.c[q] = 0.0f;
        if (lane < count) {
            const int64_t i = P.tile_vis[(int64_t)t * kMaxNb + lane];
            in_range = vis_coords(pr, i, cell, tab, ow, x0, y0);
            if (in_range) {
                const float2 vv = static_cast<const float2*>(pr.vis)[i];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float gw = load_gcf<F>(pr.g_w, ow * kSupportW + k);
                    cw.c[2 * k] = gw * vv.x;
                    cw.c[2 * k + 1] = gw * vv.y;
                }
            }
        }
        wave_oob += (uint32_t)__popcll(__ballot(lane < count && !in_range));

        // G_uv weights of the whole tile (zero for out-of-range visibilities).
        const __amdgpu_buffer_rsrc_t rg = make_rsrc(pr.g_uv, pr.guv_bytes);
        const uint32_t lane_g = (uint32_t)lane * GcfTraits<F>::kBytes;
        const int g_off = in_range ? tab * (int)GcfTraits<F>::kBytes : (int)kOutOfRange;
        float gv[NB];
#pragma unroll
        for (int g0 = 0; g0 < NB; g0 += 8) {
            if (g0 < count) {
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    gv[g0 + k] = load_gcf_rsrc<F>(rg, (uint32_t)__builtin_amdgcn_readlane(g_off, g0 + k) + lane_g);
            }
        }

        bool staged = false;
        int bx0 = 0, by0 = 0, bw = 0, bh = 0, bp = 0;
        if (BOX > 0 && pr.n_w == kSupportW) {   // the box holds w 0..3 of each cell
            int bx1 = -1, by1 = -1;
            wave_bbox(in_range, x0, y0, bx0, by0, bx1, by1);
            if (bx1 >= 0) {
                bw = bx1 - bx0 + kSupportUV;
                bh = by1 - by0 + kSupportUV;
                bp = scatter_box_pitch(bw, bh, (int)((uint32_t)BOX / kCell));
                staged = (uint32_t)(bp * bh) * kCell <= (uint32_t)BOX;
            }
        }

        float* out = static_cast<float*>(pr.grid_out) + 2 * (int64_t)tc.sub * pr.n_v * pr.n_u * pr.n_w;
        const int tv = lane >> 3, tu = lane & 7;
        if (staged) {
            char* box = s_box[wv];
            const int n_chunks = bp * bh * (int)(kCell / 16);
            for (int c = lane; c < n_chunks; c += kWave)
                *reinterpret_cast<uint4*>(box + (uint32_t)c * 16u) = make_uint4(0u, 0u, 0u, 0u);
            wave_lds_sync();
            const int rel = in_range ? ((y0 - by0) * bp + (x0 - bx0)) : 0;
            const uint32_t lane_box = ((uint32_t)tv * bp + tu) * kCell;
#pragma unroll
            for (int g0 = 0; g0 < NB; g0 += 8) {
                if (g0 < count) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int j = g0 + k;
                        const uint32_t base = lane_box + (uint32_t)__builtin_amdgcn_readlane(rel, j) * kCell;
                        // distinct cells per visibility, in-order LDS: plain
                        // read-modify-write is exact
                        float4* dst = reinterpret_cast<float4*>(box + base);
                        float c[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            c[q] = gv[j] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cw.c[q]), j));
                        float4 a = dst[0], b = dst[1];
                        a.x += c[0]; a.y += c[1]; a.z += c[2]; a.w += c[3];
                        b.x += c[4]; b.y += c[5]; b.z += c[6]; b.w += c[7];
                        dst[0] = a;
                        dst[1] = b;
                    }
                }
            }
            wave_lds_sync();
            // Add the box to the output row by row: a box row is bw * 8
            // consecutive floats both in LDS and in the subgrid, so lane l of
            // a step adds float l and one atomic instruction covers 256
            // contiguous bytes.
            const int row_floats = bw * (int)(kCell / 4);
            const float* lds_rows = reinterpret_cast<const float*>(box);
            for (int row = 0; row < bh; ++row) {
                float* dst = out + 2 * ((int64_t)((by0 + row) * pr.n_u + bx0) * pr.n_w);
                const float* src = lds_rows + (uint32_t)row * bp * (kCell / 4);
                for (int f = lane; f < row_floats; f += kWave) {
                    const float v = src[f];
                    if (v != 0.0f) unsafeAtomicAdd(dst + f, v);
                }
            }
            wave_lds_sync();
        } else {
            const int64_t lane_cell = (int64_t)(tv * pr.n_u + tu) * pr.n_w;
#pragma unroll
            for (int g0 = 0; g0 < NB; g0 += 8) {
                if (g0 < count) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int j = g0 + k;
                        const int cj = __builtin_amdgcn_readlane(in_range ? cell : -1, j);
                        if (cj >= 0) {
                            float* dst = out + 2 * ((int64_t)cj + lane_cell);
#pragma unroll
                            for (int q = 0; q < 8; ++q) {
                                const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cw.c[q]), j));
                                unsafeAtomicAdd(dst + q, gv[j] * c);
                            }
                        }
                    }
                }
            }
        }
        t = t_next;
    }
    finish_launch(P.ctl, wave_oob);
}

// ---------------------------------------------------------------------------
// Owner-computes adjoint
// ---------------------------------------------------------------------------
//
// Three launches, or four; on small plans two, or three. The record pass (not on
// small plans: kOwnerDirect) reads the visibilities in input order and
// writes what the sums need of each (first tap, table rows, value: 16 bytes)
// at its places in the owner order. The owner pass sums and writes every
// output cell once with plain stores: no global atomics, and the sums do not
// depend on timing. Where visibilities crowd a few segments, a segment's are shared
// by several wavefronts (slices), and the join pass adds what they wrote. A
// visibility whose first tap at run time differs from the plan's is skipped there;
// the fix-up pass adds those with atomics and ends at once when there are none.
//
// Owner pass. The output is cut into bands of kOwnerBand rows (and up to four
// w planes), and bands into segments of columns. A wavefront takes a segment
// and adds the records that reach it in the order of their first column, one
// contiguous run of the owner order. Eight columns of the band are in
// registers, one cell per lane in each of two groups of 8 rows: column x
// sits in the lanes with lane mod 8 = x mod 8. The window of a visibility is
// eight columns wide, so it covers all lanes whatever its first column. When
// the first column advances, the columns left behind go to LDS, and every
// fourth column four are stored, 128 contiguous bytes per row (each column
// stored from its lanes, 32 bytes per row, took as long as all the sums). So
// a visibility takes 1.3 groups of 64 cells per band, where fixed blocks of
// 16 x 16 cells took 1.7 per block and met more blocks.
//
// The sum is an outer product per visibility, (cells) x (4 w values, real and
// imaginary), so it runs on the matrix cores: v_mfma_f32_4x4x1_16b_f32 adds
// c[i] * b[lane] to accumulator i of every lane, for four values c. b is the
// lane's G_uv weight (0 outside the window's rows) and c is G_w * V, value i
// in the lanes with lane mod 4 = i. In float32 it does twice the
// multiply-adds per clock of the vector ALU.
//
// Measured on 16 subgrids of 512 x 512 with 65536 uniform visibilities each:
// 105 us for the owner pass and 26 us for the records, where one wavefront per
// 16 x 16 block, adding each visibility's taps to an LDS copy of the block,
// took 180 us and 9 us. What bounds it now is vector issue (17 instructions
// per visibility and band, the 2.6 matrix ones among them).
//
// Weight of lane (ly, lx) in row group g for a window that starts dy rows
// into the band and at column x0: entry (8 g + ly - dy) * 8 + ((lx - x0) mod
// 8) of its G_uv block. With LDS_TAB the workgroup keeps the whole table in
// LDS; otherwise the wavefront loads the visibility's block (lane l, entry l)
// and lanes exchange entries.
//
// A batch with a value c that is not finite (0 * inf would reach cells
// outside its window) is added by vector instructions under the windows'
// masks; for DEEP also one with a weight that is not (0 * inf would reach
// planes outside its taps).
//
// DEEP: subgrids with more than four w planes; a segment covers planes 4 slab
// .. 4 slab + 3, and c is 0 for planes outside the visibility's four taps. A
// visibility reaches one or two slabs, so of each 64 those that reach this one are
// brought together first (320 000 on 8 subgrids of 256 x 256 x 16: 132 us without
// that, with it 105; 100 000 on 4 of 64 x 64 x 256 346 and 78).

typedef float F32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) OwnerTask* ConstOwnerTaskPtr;
typedef const __attribute__((address_space(4))) OwnerSlice* ConstOwnerSlicePtr;

constexpr int kOwnerMaxWaves = 16;                 // one workgroup per CU, four wavefronts per SIMD
constexpr int kOwnerRec = kSupportW * 2;           // values of c per visibility
constexpr int kOwnerStage = 4;                     // columns stored together
// per wavefront: c of 64 visibilities, and four finished columns
constexpr size_t kOwnerWaveBytes = (size_t)(kWave + kOwnerBand * kOwnerStage) * kOwnerRec * sizeof(float);
// entries a masked lane may read past the end of the table (before its start
// it reads the wavefronts' own LDS)
constexpr int kOwnerTablePad = 128;
constexpr size_t kOwnerStaticLds = 512;   // (the workgroup-wide OR of the DEEP kernels)
// table blocks and w rows of a record: 12 bits (os_uv^2 <= 4096) and 6 bits
// (os_w <= 64), then the first w plane
constexpr int kRecBlockBits = 12, kRecRowBits = 6, kRecPlaneShift = kRecBlockBits + kRecRowBits;
static_assert(kOwnerMaxPlanes <= 1 << (32 - kRecPlaneShift), "first w plane of a record");

// One visibility of a batch as the wavefront reads it, in two words. Scalar
// instructions per visibility set the pace (one per SIMD and 4 clocks), so
// the fields are where an instruction takes them without unpacking.
//   flags: bits 0-5 8 b, where the window starts 8 a + b rows into the band (b
//   < 8): its rows b .. 7 fall in group a and 0 .. b - 1 in group a + 1; bits
//   6-7 the groups its rows reach; bit 8 set unless a = 0; from bit 9 its first
//   column less that of the segment's first possible window. 0: not in this
//   segment's planes, or moved.
//   at: bits 0-4 its first column mod 8 in entries; from bit 5 the offset of
//   its table block, less 8 dy entries.
constexpr int kOwnerGroup0 = 1 << 6, kOwnerGroup1 = 1 << 7, kOwnerOther = 1 << 8;
constexpr int kOwnerColShift = 9;
static_assert(kOwnerMaxSegment % 8 == 0, "segments of whole groups of columns");

template <int F, bool LDS_TAB>
struct OwnerTable {
    static constexpr uint32_t kB = GcfTraits<F>::kBytes;
    const char* lds;               // LDS_TAB: the table
    __amdgpu_buffer_rsrc_t rg;
    uint32_t lane_b;               // lane * kB
    int row_b;                     // ly * 8 * entry bytes
    int col_b;                     // lx * entry bytes

    static constexpr int kEntry = LDS_TAB ? (int)kB : 4;   // bytes of one entry where lanes pick it
    static __device__ __forceinline__ int pack_at(int x0, int dy, int blk) {
        // (exchanged between lanes: the entry is taken mod 64)
        const int e = LDS_TAB ? blk * 64 - 8 * dy : blk * 64 + ((-8 * dy) & 63);
        return (int)((uint32_t)(e * kEntry) << 5) | ((x0 & 7) * kEntry);
    }

    // Weights of the two row groups (at is wave-uniform). Whether one is not
    // finite (not looked at for LDS_TAB).
    __device__ __forceinline__ bool load(int at, float (&w)[2]) const {
        const int tu = (col_b - at) & (7 * kEntry);
        if constexpr (LDS_TAB) {
            const char* a = lds + ((at >> 5) + tu + row_b);
            if constexpr (F == kGcfF32) {
                w[0] = *reinterpret_cast<const float*>(a);
                w[1] = *reinterpret_cast<const float*>(a + 64 * kEntry);
            } else {
                w[0] = widen_gcf16<F>(*reinterpret_cast<const unsigned short*>(a));
                w[1] = widen_gcf16<F>(*reinterpret_cast<const unsigned short*>(a + 64 * kEntry));
            }
            return false;
        } else {
            const float x = load_gcf_rsrc<F>(rg, lane_b, (uint32_t)(at >> 13) * (64u * kB));
            w[0] = w[1] = __int_as_float(__builtin_amdgcn_ds_bpermute((at >> 5) + tu + row_b, __float_as_int(x)));
            return __any(!isfinite(x));
        }
    }
};

// x where the lane's bit of the wave-uniform mask is set, else y.
__device__ __forceinline__ float lane_select(uint64_t mask, float x, float y) {
    return __builtin_amdgcn_inverse_ballot_w64(mask) ? x : y;
}

// Adds one visibility to the cells of its window.
__device__ __forceinline__ void owner_item(F32x4 (&acc)[2][2], float c0, float c1, int flags, const float (&w)[2]) {
    // lanes of group 0's rows, and of the rows of group 1 that are not its:
    // rows b .. 7 (a = 0) or 0 .. b - 1
    const uint32_t flip = (uint32_t)((flags << 23) >> 31);
    const uint64_t mask = (~0ull << (flags & 63)) ^ (((uint64_t)flip << 32) | flip);
    if (flags & kOwnerGroup0) {
        const float b = lane_select(mask, w[0], 0.0f);
        acc[0][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(c0, b, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(c1, b, acc[0][1], 0, 0, 0);
    }
    if (flags & kOwnerGroup1) {
        const float b = lane_select(mask, 0.0f, w[1]);
        acc[1][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(c0, b, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(c1, b, acc[1][1], 0, 0, 0);
    }
}

// What the sums need of a visibility at coordinates (u, v, w), or a record that is
// skipped where it is out of range or starts elsewhere than at the sort.
__device__ __forceinline__ uint4 owner_record(const Problem& pr, double u, double v, double w, uint32_t plan_start,
                                              float2 vis, bool& in_range, bool& moved) {
    int32_t cell = 0, tab = 0, ow = 0, x0 = 0, y0 = 0;
    in_range = coords_from(pr, u, v, w, cell, tab, ow, x0, y0);
    const uint32_t f = ((uint32_t)y0 << 16) | (uint32_t)x0;
    moved = in_range && f != plan_start;
    const uint32_t z0 = (uint32_t)(cell - (y0 * pr.n_u + x0) * pr.n_w);
    return make_uint4(in_range && !moved ? f : kNoStart,
                      (uint32_t)(tab / (kSupportUV * kSupportUV)) | ((uint32_t)ow << kRecBlockBits) | (z0 << kRecPlaneShift),
                      __float_as_uint(vis.x), __float_as_uint(vis.y));
}

// One visibility's inputs, in flight.
struct OwnerInputs {
    double u, v, w;
    float2 vis;
    uint32_t plan_start;
};

// DIRECT: no records; the visibilities are read through P.items.
template <int F, bool LDS_TAB, bool DEEP, bool DIRECT>
__global__ __launch_bounds__(kOwnerMaxWaves* kWave) void grid_owner_kernel(OwnerParams P) {
    extern __shared__ __attribute__((aligned(16))) char s_mem[];
    const int lane = lane_id();
    const int ly = lane >> 3, lx = lane & 7;
    const int waves = (int)(blockDim.x / kWave);
    const int wv = uniform((int)(threadIdx.x / kWave));
    float* rec = reinterpret_cast<float*>(s_mem + (uint32_t)wv * (uint32_t)kOwnerWaveBytes);
    float4* stage = reinterpret_cast<float4*>(rec + kWave * kOwnerRec);   // [row][column mod 4][half]
    char* s_shared = s_mem + (uint32_t)waves * (uint32_t)kOwnerWaveBytes;
    float4* s_gw = reinterpret_cast<float4*>(s_shared);   // [os_w] G_w rows
    const Problem& pr = P.prob;
    for (int o = (int)threadIdx.x; o < pr.os_w; o += (int)blockDim.x)
        s_gw[o] = make_float4(load_gcf<F>(pr.g_w, o * kSupportW), load_gcf<F>(pr.g_w, o * kSupportW + 1),
                              load_gcf<F>(pr.g_w, o * kSupportW + 2), load_gcf<F>(pr.g_w, o * kSupportW + 3));

    OwnerTable<F, LDS_TAB> table;
    table.rg = make_rsrc(pr.g_uv, pr.guv_bytes);
    table.lane_b = (uint32_t)lane * GcfTraits<F>::kBytes;
    table.row_b = ly * kSupportUV * OwnerTable<F, LDS_TAB>::kEntry;
    table.col_b = lx * OwnerTable<F, LDS_TAB>::kEntry;
    table.lds = s_shared + pr.os_w * (int)sizeof(float4);
    bool bad_table = false;   // DEEP && LDS_TAB: some entry is not finite
    if constexpr (LDS_TAB) {
        char* t = s_shared + pr.os_w * (int)sizeof(float4);
        bool bad = false;
        for (uint32_t o = threadIdx.x * 16u; o < pr.guv_bytes; o += blockDim.x * 16u) {
            uint32_t x[4];
            if constexpr (F == kGcfF32) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(table.rg, o, 0, 0);
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = v[k];
            } else {   // (a 16-bit table may start on any element)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    x[k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(table.rg, o + 4u * k, 0, 0) |
                           ((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(table.rg, o + 4u * k + 2u, 0, 0) << 16);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (F == kGcfF32)
                    bad = bad || !isfinite(__uint_as_float(x[k]));
                else
                    bad = bad || !isfinite(widen_gcf16<F>(x[k] & 0xFFFFu)) || !isfinite(widen_gcf16<F>(x[k] >> 16));
            }
            *reinterpret_cast<uint4*>(t + o) = make_uint4(x[0], x[1], x[2], x[3]);
        }
        if constexpr (DEEP) bad_table = __syncthreads_or(bad) != 0;
    }
    __syncthreads();

    // Slices come first, then the other tasks, heaviest first, and are dealt to the
    // launch's wavefronts back and forth, those of one workgroup far apart: no
    // atomic. (Claimed one by one from the queues' cursors, they waited up to 30 us
    // for the atomics.)
    const int64_t n_waves = (int64_t)gridDim.x * waves;
    const int64_t me = (int64_t)wv * gridDim.x + blockIdx.x;
    const int64_t n_runs = P.n_tasks - P.n_split + P.n_slices;
    for (int64_t r0 = 0; r0 < n_runs; r0 += n_waves) {
        const int64_t t = uniform((int)((r0 / n_waves) & 1)) ? r0 + n_waves - 1 - me : r0 + me;
        if (t >= n_runs) continue;
        const bool slice = t < P.n_slices;
        uint32_t begin, end;
        int band, slab = 0, x_lo, width;   // the columns
        int planes = kSupportW, n_u = pr.n_u, row_out = 0;
        uint32_t cell_bytes, out_bytes;
        char* out;
        int accumulate = 0;
        if (slice) {
            const ConstOwnerSlicePtr sp = (ConstOwnerSlicePtr)uniform_u64((uint64_t)P.slices) + t;
            begin = sp->begin;
            end = sp->end;
            band = sp->band;
            if (DEEP) slab = sp->slab;
            x_lo = sp->x_lo;
            width = sp->width;
            n_u = width;
            cell_bytes = kSupportW * 8u;
            out = P.partials + (int64_t)sp->column * (int64_t)kOwnerColumnBytes;
            out_bytes = (uint32_t)width * (uint32_t)kOwnerColumnBytes;
        } else {
            const ConstOwnerTaskPtr tp = (ConstOwnerTaskPtr)uniform_u64((uint64_t)P.tasks) + (t - P.n_slices + P.n_split);
            begin = tp->begin;
            end = tp->end;
            band = tp->band;
            const int seg = DEEP ? tp->place / P.n_slabs : tp->place;
            if (DEEP) {
                slab = tp->place - seg * P.n_slabs;
                planes = min(kSupportW, pr.n_w - kSupportW * slab);
            }
            x_lo = seg * P.segment;
            width = min(P.segment, pr.n_u - x_lo);
            cell_bytes = (uint32_t)pr.n_w * 8u;
            // the subgrid's output; rows past its end fall outside the resource
            const int s = band / P.nby;
            out = static_cast<char*>(pr.grid_out) + 8 * (int64_t)s * pr.cells_per_sub;
            out_bytes = (uint32_t)(pr.cells_per_sub * 8);
            row_out = (band - s * P.nby) * kOwnerBand;
            accumulate = P.accumulate;
        }
        const int row0 = band % P.nby * kOwnerBand;
        const __amdgpu_buffer_rsrc_t ro = make_rsrc(out, out_bytes);
        // of four staged columns, lane l stores 16 bytes of rows l / 8 and
        // l / 8 + 8: half l mod 2 of column l / 2 mod 4
        const int st_col = (lane >> 1) & 3, st_half = lane & 1;
        const uint32_t lane_off = (uint32_t)((row_out + ly) * n_u + (slice ? 0 : x_lo) + st_col) * cell_bytes +
                                  (uint32_t)((slice ? 0 : slab * kSupportW * 8) + st_half * 16);
        const uint32_t group_rows = (uint32_t)(8 * n_u) * cell_bytes;

        F32x4 acc[2][2];
#pragma unroll
        for (int g = 0; g < 2; ++g) acc[g][0] = acc[g][1] = F32x4{0.f, 0.f, 0.f, 0.f};
        // columns from the segment's first: the first in work (ahead: from the
        // first possible one), and this lane's
        int ahead = 0;
        int lane_col = lx == 0 ? 0 : lx - kSupportUV;
        // (a lane's columns are 8 apart, so its place among the four is fixed)
        float4* leaving = stage + (ly * kOwnerStage + (lx & (kOwnerStage - 1))) * 2;

        // Makes 'to' the first column in work.
        auto advance = [&](int to) {
            int cur = ahead - (kSupportUV - 1);
            do {
                cur = min(to, (cur & ~(kOwnerStage - 1)) + kOwnerStage);
                const bool leave = lane_col < cur;
                if (leave) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        leaving[(k >> 1) * 64 + (k & 1)] = __builtin_bit_cast(float4, acc[k >> 1][k & 1]);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[k >> 1][k & 1][q] = leave ? 0.0f : acc[k >> 1][k & 1][q];
                lane_col += leave ? kSupportUV : 0;
                const int first = cur - kOwnerStage;   // of the columns in LDS
                if ((cur & (kOwnerStage - 1)) == 0 && first >= 0) {
                    wave_lds_sync();
                    if (st_col < width - first) {
                        const uint32_t off = lane_off + (uint32_t)first * cell_bytes;
#pragma unroll
                        for (int g = 0; g < 2; ++g) {
                            float4 v = stage[g * 64 + lane];
                            const uint32_t rows = g == 0 ? 0 : group_rows;
                            if constexpr (DEEP) {
                                const bool p0 = 2 * st_half < planes, p1 = 2 * st_half + 1 < planes;
                                if (accumulate) {
                                    const auto a = __builtin_amdgcn_raw_buffer_load_b64(ro, p0 ? off : kOutOfRange, rows, 0);
                                    const auto b = __builtin_amdgcn_raw_buffer_load_b64(ro, p1 ? off + 8u : kOutOfRange, rows, 0);
                                    v = make_float4(v.x + __uint_as_float(a[0]), v.y + __uint_as_float(a[1]),
                                                    v.z + __uint_as_float(b[0]), v.w + __uint_as_float(b[1]));
                                }
                                if (p0) __builtin_amdgcn_raw_buffer_store_b64(U32x2{__float_as_uint(v.x), __float_as_uint(v.y)}, ro, off, rows, 0);
                                if (p1) __builtin_amdgcn_raw_buffer_store_b64(U32x2{__float_as_uint(v.z), __float_as_uint(v.w)}, ro, off + 8u, rows, 0);
                            } else {
                                if (accumulate) {
                                    const auto a = __builtin_amdgcn_raw_buffer_load_b128(ro, off, rows, 0);
                                    v = make_float4(v.x + __uint_as_float(a[0]), v.y + __uint_as_float(a[1]),
                                                    v.z + __uint_as_float(a[2]), v.w + __uint_as_float(a[3]));
                                }
                                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U32x4, v), ro, off, rows, 0);
                            }
                        }
                    }
                    wave_lds_sync();
                }
            } while (cur < to);
            ahead = to + kSupportUV - 1;
        };

        auto fetch = [&](uint32_t pos) {
            const uint32_t p = min(pos + (uint32_t)lane, end - 1);
            if constexpr (DIRECT) {
                const int64_t i = P.items[p];
                const double* c = pr.uvw + 3 * i;
                return OwnerInputs{c[0], c[1], c[2], static_cast<const float2*>(pr.vis)[i], P.plan_start[i]};
            } else {
                return reinterpret_cast<const uint4*>(P.records)[p];
            }
        };
        decltype(fetch(0)) nxt{};
        if (begin < end) nxt = fetch(begin);
        for (uint32_t pos = begin; pos < end; pos += kWave) {
            // Lane j prepares record j; the next 64 are requested before.
            uint4 x;
            if constexpr (DIRECT) {
                bool in_range, moved;
                x = owner_record(pr, nxt.u, nxt.v, nxt.w, nxt.plan_start, nxt.vis, in_range, moved);
            } else {
                x = nxt;
            }
            int n = (int)min((uint32_t)kWave, end - pos);
            if (pos + kWave < end) nxt = fetch(pos + kWave);
            int flags = 0, at = 0, dz = 0;
            float c[kOwnerRec];
#pragma unroll
            for (int q = 0; q < kOwnerRec; ++q) c[q] = 0.0f;
            if constexpr (DEEP) dz = (int)(x.y >> kRecPlaneShift) - kSupportW * slab;
            if (lane < n && x.x != kNoStart && (!DEEP || (dz > -kSupportW && dz < kSupportW))) {
                const int dy = (int)(x.x >> 16) - row0;
                const int x0 = (int)(x.x & 0xFFFFu);
                flags = ((dy & 7) << 3) | (dy < 8 ? kOwnerGroup0 : 0) | (dy > 0 ? kOwnerGroup1 : 0) |
                        ((unsigned)dy < 8u ? 0 : kOwnerOther) |
                        ((x0 - x_lo + kSupportUV - 1) << kOwnerColShift);
                at = OwnerTable<F, LDS_TAB>::pack_at(x0, dy, (int)(x.y & ((1u << kRecBlockBits) - 1u)));
                const float4 row = s_gw[(x.y >> kRecBlockBits) & ((1u << kRecRowBits) - 1u)];
                const float gw[kSupportW] = {row.x, row.y, row.z, row.w};
                const float re_v = __uint_as_float(x.z), im_v = __uint_as_float(x.w);
#pragma unroll
                for (int k = 0; k < kSupportW; ++k) {
                    float g = gw[k];
                    bool in = true;
                    if constexpr (DEEP) {
                        in = (unsigned)(k - dz) < (unsigned)kSupportW;
#pragma unroll
                        for (int tw = 0; tw < kSupportW; ++tw)
                            if (tw == k - dz) g = gw[tw];
                    }
                    c[2 * k] = in ? g * re_v : 0.0f;
                    c[2 * k + 1] = in ? g * im_v : 0.0f;
                }
            }
            bool odd = bad_table;
#pragma unroll
            for (int q = 0; q < kOwnerRec; ++q) odd = odd || !isfinite(c[q]);
            int slot = lane;
            if constexpr (DEEP) {
                // those that reach this slab first, in their order
                const uint64_t mine = __ballot(flags != 0);
                const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
                n = (int)__popcll(mine);
                slot = flags != 0 ? before : n + lane - before;
                flags = __builtin_amdgcn_ds_permute(slot * 4, flags);
                at = __builtin_amdgcn_ds_permute(slot * 4, at);
                dz = __builtin_amdgcn_ds_permute(slot * 4, dz);
            }
            *reinterpret_cast<float4*>(rec + slot * kOwnerRec) = make_float4(c[0], c[1], c[2], c[3]);
            *reinterpret_cast<float4*>(rec + slot * kOwnerRec + 4) = make_float4(c[4], c[5], c[6], c[7]);
            wave_lds_sync();

            // one visibility under its window's mask (values not finite)
            auto masked = [&](int j) {
                const int fl = __builtin_amdgcn_readlane(flags, j);
                if (!(fl & (kOwnerGroup0 | kOwnerGroup1))) return;
                if ((fl >> kOwnerColShift) > ahead) advance((fl >> kOwnerColShift) - (kSupportUV - 1));
                float w[2];
                (void)table.load(__builtin_amdgcn_readlane(at, j), w);
                const int a = !(fl & kOwnerOther) ? 0 : ((fl & kOwnerGroup0) ? -1 : 1);
                const int dy = 8 * a + ((fl >> 3) & 7);
                const int dzj = DEEP ? __builtin_amdgcn_readlane(dz, j) : 0;
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    if ((unsigned)(8 * g + ly - dy) < (unsigned)kSupportUV) {
#pragma unroll
                        for (int q = 0; q < kOwnerRec; ++q)
                            if (!DEEP || (unsigned)(q / 2 - dzj) < (unsigned)kSupportW)
                                acc[g][q >> 2][q & 3] += w[g] * rec[j * kOwnerRec + q];
                    }
            };
            if (__any(odd)) {
                for (int j = 0; j < n; ++j) masked(j);
            } else {
                for (int j0 = 0; j0 < n; j0 += 4) {
                    int fl[4];
                    float w[4][2], c0[4], c1[4];
                    bool bad = false;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {   // (past n: no group)
                        fl[k] = __builtin_amdgcn_readlane(flags, j0 + k);
                        bad = table.load(__builtin_amdgcn_readlane(at, j0 + k), w[k]) || bad;
                        c0[k] = rec[(j0 + k) * kOwnerRec + (lane & 3)];
                        c1[k] = rec[(j0 + k) * kOwnerRec + 4 + (lane & 3)];
                    }
                    if (DEEP && bad) {
                        for (int k = 0; k < 4; ++k) masked(j0 + k);
                        continue;
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int col = fl[k] >> kOwnerColShift;
                        if (col > ahead) advance(col - (kSupportUV - 1));
                        owner_item(acc, c0[k], c1[k], fl[k], w[k]);
                    }
                }
            }
            wave_lds_sync();
        }
        advance((width + kOwnerStage - 1) & ~(kOwnerStage - 1));
    }
    // the last workgroup publishes the moved visibilities the record pass
    // counted, for the fix-up pass, and clears the count for the next call
    if (!DIRECT && finish_launch(P.ctl, 0u)) atomicExch(&P.ctl->moved.v[1], atomicExch(&P.ctl->moved.v[0], 0u));
}

// Join pass: adds the slices of each split task, in their order (so the sums are
// the same on every run), and writes the segment. A wavefront takes 64 consecutive
// halves of cells (16 bytes). The wavefronts of a workgroup take a set of 64 each;
// for the first n_shared tasks, those with many slices, they share the slices of
// one set, and their sums meet in LDS. (All tasks so: 4 subgrids of 256 x 256 with
// 128 000 visibilities, three slices each, 58 us instead of 45; 1.0 M dense at the
// centres of 16 subgrids 168 instead of 157.)
constexpr int kJoinWaves = 8;
constexpr int kJoinAhead = 8;    // loads in flight

__global__ __launch_bounds__(kJoinWaves* kWave) void grid_join_kernel(OwnerParams P, int n_chunks) {
    __shared__ float4 s_sum[kJoinWaves][kWave];
    const Problem& pr = P.prob;
    const int lane = lane_id(), wv = uniform((int)(threadIdx.x / kWave));
    const int n_groups = (n_chunks + kJoinWaves - 1) / kJoinWaves;
    const int group = (int)blockIdx.x - P.n_shared * n_chunks;
    const bool alone = group >= 0;
    const int task = alone ? P.n_shared + group / n_groups : (int)blockIdx.x / n_chunks;
    const int chunk = alone ? group % n_groups * kJoinWaves + wv : (int)blockIdx.x % n_chunks;
    const int k0 = (int)P.first_slice[task], n = (int)P.first_slice[task + 1] - k0;
    const ConstOwnerTaskPtr tp = (ConstOwnerTaskPtr)uniform_u64((uint64_t)P.tasks) + task;
    const int s = tp->band / P.nby, seg = tp->place / P.n_slabs, slab = tp->place - seg * P.n_slabs;
    const int row0 = (tp->band - s * P.nby) * kOwnerBand, x_lo = seg * P.segment;
    const int width = min(P.segment, pr.n_u - x_lo);
    const int e = chunk * kWave + lane;   // of [kOwnerBand rows][width][2 halves]
    const int row = e / (2 * width), col = (e - row * 2 * width) >> 1, half = e & 1;
    const bool cell = row < kOwnerBand && row0 + row < pr.n_v;
    const int k_begin = alone ? k0 : k0 + (int)((int64_t)n * wv / kJoinWaves);
    const int k_end = alone ? k0 + n : k0 + (int)((int64_t)n * (wv + 1) / kJoinWaves);
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](float4 v) {
        sum.x += v.x;
        sum.y += v.y;
        sum.z += v.z;
        sum.w += v.w;
    };
    for (int k = k_begin; k < k_end; k += kJoinAhead) {
        float4 v[kJoinAhead];
#pragma unroll
        for (int j = 0; j < kJoinAhead; ++j) {
            const OwnerSlice* x = P.slices + min(k + j, k_end - 1);
            const int c = x_lo + col - x->x_lo;
            const bool in = k + j < k_end && cell && c >= 0 && c < x->width;
            const char* at = P.partials + (int64_t)x->column * (int64_t)kOwnerColumnBytes;
            v[j] = in ? *reinterpret_cast<const float4*>(at + ((row * x->width + c) * 2 + half) * 16)
                      : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int j = 0; j < kJoinAhead; ++j) add(v[j]);
    }
    if (!alone) {
        s_sum[wv][lane] = sum;
        __syncthreads();
        if (wv != 0) return;
#pragma unroll
        for (int k = 1; k < kJoinWaves; ++k) add(s_sum[k][lane]);
    }
    if (!cell) return;
    const int plane = slab * kSupportW + 2 * half;
    float2* to = static_cast<float2*>(pr.grid_out) + (int64_t)s * pr.cells_per_sub +
                 ((int64_t)(row0 + row) * pr.n_u + x_lo + col) * pr.n_w + plane;
    const float2 a = make_float2(sum.x, sum.y), b = make_float2(sum.z, sum.w);
    if (plane < pr.n_w) to[0] = P.accumulate ? make_float2(to[0].x + a.x, to[0].y + a.y) : a;
    if (plane + 1 < pr.n_w) to[1] = P.accumulate ? make_float2(to[1].x + b.x, to[1].y + b.y) : b;
}

// Record pass: lane by lane in input order, kRecordPerLane visibilities 64
// apart, all their loads in flight before any is used. Counts the
// visibilities out of range (ctl) and those whose first tap moved since the
// sort (own_ctl), which leave a record that no block takes.
constexpr int kRecordPerLane = 4;

__global__ __launch_bounds__(kBlockThreads) void grid_record_kernel(Problem pr, int64_t n_vis,
                                                                    const uint32_t* plan_start,
                                                                    const uint2* place, uint4* records, Ctl* ctl,
                                                                    Ctl* own_ctl) {
    const int lane = lane_id();
    uint32_t wave_oob = 0, wave_moved = 0;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t first = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
    constexpr int64_t kSpan = (int64_t)kWave * kRecordPerLane;
    for (int64_t w0 = first * kSpan; w0 < n_vis; w0 += n_waves * kSpan) {
        double cu[kRecordPerLane], cv[kRecordPerLane], cw[kRecordPerLane];
        uint32_t ps[kRecordPerLane];
        uint2 at[kRecordPerLane];
        float2 vv[kRecordPerLane];
        // branch-free loads (a lane past the end re-reads the last
        // visibility and ignores it), so all of them are in flight at once
#pragma unroll
        for (int k = 0; k < kRecordPerLane; ++k) {
            int64_t i = w0 + k * kWave + lane;
            i = i < n_vis ? i : n_vis - 1;
            const double* uv = pr.uvw + 3 * i;
            cu[k] = uv[0];
            cv[k] = uv[1];
            cw[k] = uv[2];
            ps[k] = plan_start[i];
            at[k] = place[i];
            vv[k] = static_cast<const float2*>(pr.vis)[i];
        }
#pragma unroll
        for (int k = 0; k < kRecordPerLane; ++k) {
            const int64_t i = w0 + k * kWave + lane;
            bool in_range = false, moved = false;
            if (i < n_vis) {
                const uint4 r = owner_record(pr, cu[k], cv[k], cw[k], ps[k], vv[k], in_range, moved);
                if (at[k].x != kNoPlace) records[at[k].x] = r;
                if (at[k].y != kNoPlace) records[at[k].y] = r;
            }
            wave_oob += (uint32_t)__popcll(__ballot(i < n_vis && !in_range));
            wave_moved += (uint32_t)__popcll(__ballot(moved));
        }
    }
    if (lane == 0 && wave_moved != 0u) atomicAdd(&own_ctl->moved.v[0], wave_moved);
    finish_launch<true>(ctl, wave_oob);
}

// Visibilities the owner pass skipped (first tap differs from the plan's),
// added with atomics by whole wavefronts. Ends at once when the record pass
// found none. CHECK: without a record pass, so it counts those out of range too.
template <int F, bool CHECK>
__global__ __launch_bounds__(kBlockThreads) void grid_fixup_kernel(Problem pr, const int64_t* offsets,
                                                                   int64_t n_sub, int64_t n_vis,
                                                                   const uint32_t* plan_start, const Ctl* own_ctl,
                                                                   Ctl* ctl) {
    if (!CHECK && own_ctl->moved.v[1] == 0u) return;
    uint32_t wave_oob = 0;
    const int lane = lane_id();
    const int tv = lane >> 3, tu = lane & 7;
    const int64_t lane_cell = (int64_t)(tv * pr.n_u + tu) * pr.n_w;
    const int64_t n_waves = (int64_t)gridDim.x * kWavesPerBlock;
    const int64_t first = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
    for (int64_t w0 = first * kWave; w0 < n_vis; w0 += n_waves * kWave) {
        const int64_t i = w0 + lane;
        int32_t cell = 0, tab = 0, ow = 0, x0 = 0, y0 = 0;
        bool in_range = false, redo = false;
        if (i < n_vis) {
            in_range = vis_coords(pr, i, cell, tab, ow, x0, y0);
            redo = in_range && (((uint32_t)y0 << 16) | (uint32_t)x0) != plan_start[i];
        }
        if (CHECK) wave_oob += (uint32_t)__popcll(__ballot(i < n_vis && !in_range));
        uint64_t mask = __ballot(redo);
        if (mask == 0) continue;
        // subgrid of each visibility to redo
        int64_t sub = 0;
        float c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q] = 0.0f;
        if (redo) {
            int64_t lo = 0, hi = n_sub;
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (offsets[mid] <= i) lo = mid; else hi = mid;
            }
            sub = lo;
            const float2 vv = static_cast<const float2*>(pr.vis)[i];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float gw = load_gcf<F>(pr.g_w, ow * kSupportW + t);
                c[2 * t] = gw * vv.x;
                c[2 * t + 1] = gw * vv.y;
            }
        }
        while (mask) {
            const int j = __builtin_ctzll(mask);
            mask &= mask - 1;
            const int64_t sj = ((int64_t)__builtin_amdgcn_readlane((int)(sub >> 32), j) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)sub, j);
            const int cj = __builtin_amdgcn_readlane(cell, j);
            const int tj = __builtin_amdgcn_readlane(tab, j);
            const float g = load_gcf<F>(pr.g_uv, (int64_t)tj + lane);
            float* dst = static_cast<float*>(pr.grid_out) + 2 * (sj * pr.cells_per_sub + cj + lane_cell);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                unsafeAtomicAdd(dst + q, g * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c[q]), j)));
        }
    }
    if (CHECK) finish_launch<true>(ctl, wave_oob);
}

}  // namespace

int adjoint_variant_count() { return kNumVariants; }

template <int F, int V>
hipError_t launch_adjoint_t(const LaunchParams& p, int blocks, hipStream_t s) {
    hipLaunchKernelGGL((grid_adjoint_kernel<F, kVariants[V].box, kVariants[V].nb>), dim3(blocks), dim3(kBlockThreads),
                       0, s, p);
    return hipGetLastError();
}

template <int F, int V>
hipError_t occ_adjoint_t(int* n) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        n, grid_adjoint_kernel<F, kVariants[V].box, kVariants[V].nb>, kBlockThreads, 0);
}

template <int F>
hipError_t launch_adjoint_v(const LaunchParams& p, int variant, int blocks, hipStream_t s) {
    switch (variant) {
        case 0: return launch_adjoint_t<F, 0>(p, blocks, s);
        case 1: return launch_adjoint_t<F, 1>(p, blocks, s);
        case 2: return launch_adjoint_t<F, 2>(p, blocks, s);
        case 3: return launch_adjoint_t<F, 3>(p, blocks, s);
        case 4: return launch_adjoint_t<F, 4>(p, blocks, s);
        case 5: return launch_adjoint_t<F, 5>(p, blocks, s);
        case 6: return launch_adjoint_t<F, 6>(p, blocks, s);
        default: return hipErrorInvalidValue;
    }
}

template <int F>
hipError_t occ_adjoint_v(int variant, int* n) {
    switch (variant) {
        case 0: return occ_adjoint_t<F, 0>(n);
        case 1: return occ_adjoint_t<F, 1>(n);
        case 2: return occ_adjoint_t<F, 2>(n);
        case 3: return occ_adjoint_t<F, 3>(n);
        case 4: return occ_adjoint_t<F, 4>(n);
        case 5: return occ_adjoint_t<F, 5>(n);
        case 6: return occ_adjoint_t<F, 6>(n);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_grid_adjoint(const LaunchParams& p, int gcf_kind, int variant, int blocks,
                               hipStream_t stream) {
    if (gcf_kind == kGcfF32) return launch_adjoint_v<kGcfF32>(p, variant, blocks, stream);
    if (gcf_kind == kGcfF16) return launch_adjoint_v<kGcfF16>(p, variant, blocks, stream);
    if (gcf_kind == kGcfBF16) return launch_adjoint_v<kGcfBF16>(p, variant, blocks, stream);
    return hipErrorInvalidValue;
}

hipError_t adjoint_kernel_occupancy(int gcf_kind, int variant, int* n) {
    if (gcf_kind == kGcfF32) return occ_adjoint_v<kGcfF32>(variant, n);
    if (gcf_kind == kGcfF16) return occ_adjoint_v<kGcfF16>(variant, n);
    if (gcf_kind == kGcfBF16) return occ_adjoint_v<kGcfBF16>(variant, n);
    return hipErrorInvalidValue;
}

template <int F, bool LDS_TAB, bool DIRECT>
hipError_t launch_owner_t(const OwnerParams& p, int blocks, int waves, size_t lds, hipStream_t s) {
    if (p.n_slabs > 1)
        hipLaunchKernelGGL((grid_owner_kernel<F, LDS_TAB, true, DIRECT>), dim3(blocks), dim3(waves * kWave), lds, s, p);
    else
        hipLaunchKernelGGL((grid_owner_kernel<F, LDS_TAB, false, DIRECT>), dim3(blocks), dim3(waves * kWave), lds, s, p);
    return hipGetLastError();
}

template <int F>
hipError_t launch_owner_f(const OwnerParams& p, int blocks, int waves, size_t max_lds, hipStream_t s) {
    // the whole table in LDS where it fits beside the wavefronts' own areas
    const size_t own = (size_t)waves * kOwnerWaveBytes + (size_t)p.prob.os_w * sizeof(float4);
    const size_t with_table = own + p.prob.guv_bytes + kOwnerTablePad * GcfTraits<F>::kBytes;
    const bool lds_tab = with_table + kOwnerStaticLds <= max_lds;
    if (!p.records)
        return lds_tab ? launch_owner_t<F, true, true>(p, blocks, waves, with_table, s)
                       : launch_owner_t<F, false, true>(p, blocks, waves, own, s);
    return lds_tab ? launch_owner_t<F, true, false>(p, blocks, waves, with_table, s)
                   : launch_owner_t<F, false, false>(p, blocks, waves, own, s);
}

hipError_t launch_grid_owner(const OwnerParams& p, int gcf_kind, int n_cu, size_t max_lds, hipStream_t stream) {
    // one workgroup per CU, of as many wavefronts as there are tasks for them
    const int64_t n_runs = p.n_tasks - p.n_split + p.n_slices;
    const int waves = (int)std::min<int64_t>(kOwnerMaxWaves, std::max<int64_t>(1, (n_runs + n_cu - 1) / n_cu));
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(n_cu, (n_runs + waves - 1) / waves));
    hipError_t e = hipErrorInvalidValue;
    if (gcf_kind == kGcfF32) e = launch_owner_f<kGcfF32>(p, blocks, waves, max_lds, stream);
    if (gcf_kind == kGcfF16) e = launch_owner_f<kGcfF16>(p, blocks, waves, max_lds, stream);
    if (gcf_kind == kGcfBF16) e = launch_owner_f<kGcfBF16>(p, blocks, waves, max_lds, stream);
    if (e != hipSuccess || p.n_split == 0) return e;
    const int n_chunks = (kOwnerBand * p.segment * 2 + kWave - 1) / kWave;
    const int join = p.n_shared * n_chunks + (p.n_split - p.n_shared) * ((n_chunks + kJoinWaves - 1) / kJoinWaves);
    hipLaunchKernelGGL(grid_join_kernel, dim3((unsigned)join), dim3(kJoinWaves * kWave), 0, stream, p, n_chunks);
    return hipGetLastError();
}

hipError_t launch_grid_record(const Problem& pr, int64_t n_vis, const uint32_t* plan_start, const OwnerPlaces* place,
                              OwnerRecord* records, Ctl* ctl, Ctl* own_ctl, int max_blocks, hipStream_t stream) {
    const int64_t per_block = (int64_t)kBlockThreads * kRecordPerLane;
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n_vis + per_block - 1) / per_block, max_blocks));
    hipLaunchKernelGGL(grid_record_kernel, dim3((unsigned)blocks), dim3(kBlockThreads), 0, stream, pr, n_vis,
                       plan_start, reinterpret_cast<const uint2*>(place), reinterpret_cast<uint4*>(records), ctl,
                       own_ctl);
    return hipGetLastError();
}

template <int F>
hipError_t launch_fixup_f(const Problem& pr, const int64_t* vis_offsets, int64_t n_sub, int64_t n_vis,
                          const uint32_t* plan_start, const Ctl* own_ctl, Ctl* ctl, int blocks, hipStream_t s) {
    if (own_ctl)
        hipLaunchKernelGGL((grid_fixup_kernel<F, false>), dim3(blocks), dim3(kBlockThreads), 0, s, pr, vis_offsets, n_sub,
                           n_vis, plan_start, own_ctl, ctl);
    else
        hipLaunchKernelGGL((grid_fixup_kernel<F, true>), dim3(blocks), dim3(kBlockThreads), 0, s, pr, vis_offsets, n_sub,
                           n_vis, plan_start, own_ctl, ctl);
    return hipGetLastError();
}

hipError_t launch_grid_fixup(const Problem& pr, const int64_t* vis_offsets, int64_t n_sub, int64_t n_vis,
                             const uint32_t* plan_start, const Ctl* own_ctl, Ctl* ctl, int gcf_kind, int max_blocks,
                             hipStream_t stream) {
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n_vis + kBlockThreads - 1) / kBlockThreads, max_blocks));
    auto launch = [&](auto f) {
        return launch_fixup_f<decltype(f)::value>(pr, vis_offsets, n_sub, n_vis, plan_start, own_ctl, ctl, blocks, stream);
    };
    if (gcf_kind == kGcfF32) return launch(std::integral_constant<int, kGcfF32>{});
    if (gcf_kind == kGcfF16) return launch(std::integral_constant<int, kGcfF16>{});
    if (gcf_kind == kGcfBF16) return launch(std::integral_constant<int, kGcfBF16>{});
    return hipErrorInvalidValue;
}

}  // namespace dg
