// Plan-time work order: a stable sort of each subgrid's visibilities by the
// position of their first tap along a Hilbert curve.
//
// Tiles are cut from consecutive positions of the work order, so after this
// sort a tile holds visibilities that are close in the subgrid, and the
// tiles an XCD drains one after another cover neighbouring regions: the
// subgrid data a tile needs is then mostly in that XCD's L2 already. The sum
// each visibility receives does not depend on the order, so results are
// unchanged; only locality is.
//
// The owner-computes adjoint has an order of its own, by band of output rows
// and first column, and a list of tasks (runs of that order).
#include "dg_device.h"

#include <hipcub/hipcub.hpp>

namespace dg {
namespace {

// Position of cell (x, y) along the Hilbert curve of the 2^bits x 2^bits
// grid: level by level from the top, the rank of the cell's quadrant along
// the curve, then the coordinates turned into the orientation of that
// quadrant's sub-curve. Consecutive positions are neighbouring cells, so a
// run of positions covers a compact region (a Z-order curve jumps between
// quadrants; on the paper-scale workload this order reads 2.6 % fewer HBM
// bytes and runs about 2 % faster, cold).
__device__ __forceinline__ uint32_t hilbert(uint32_t x, uint32_t y, int bits) {
    uint32_t d = 0;
    const uint32_t ones = (1u << bits) - 1u;
    for (uint32_t s = 1u << (bits - 1); s > 0; s >>= 1) {
        const uint32_t rx = (x & s) ? 1u : 0u, ry = (y & s) ? 1u : 0u;
        d += s * s * ((3u * rx) ^ ry);
        if (ry == 0) {
            if (rx == 1) {
                x = ones - x;
                y = ones - y;
            }
            const uint32_t t = x;
            x = y;
            y = t;
        }
    }
    return d;
}

// key = subgrid << (2 bits + 1) | Hilbert position of the first tap, or
// 1 << 2 bits (the end of its subgrid) for a visibility out of range.
template <class Key>
__global__ void sort_keys_kernel(Problem pr, const int64_t* offsets, int64_t n_sub, int64_t n_vis, int bits,
                                 Key* keys, uint32_t* idx, uint32_t* plan_start) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_vis) return;
    int64_t lo = 0, hi = n_sub;   // offsets[lo] <= i < offsets[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (offsets[mid] <= i) lo = mid; else hi = mid;
    }
    int32_t cell = 0, tab = 0, ow = 0, x0 = 0, y0 = 0;
    uint64_t code = uint64_t(1) << (2 * bits);
    uint32_t st = kNoStart;
    if (vis_coords(pr, i, cell, tab, ow, x0, y0)) {
        st = ((uint32_t)y0 << 16) | (uint32_t)x0;
        code = hilbert((uint32_t)x0, (uint32_t)y0, bits);
    }
    keys[i] = (Key)(((uint64_t)lo << (2 * bits + 1)) | code);
    idx[i] = (uint32_t)i;
    plan_start[i] = st;
}

__global__ void ordered_starts_kernel(const uint32_t* perm, const uint32_t* plan_start, int64_t n_vis,
                                      uint32_t* start) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n_vis) start[p] = plan_start[perm[p]];
}

// Owner order: key = (subgrid * nby + band) * n_u + first column for each band
// a visibility reaches (slot 2 i its own, slot 2 i + 1 the next one), or
// n_keys: no such place.
template <class Key>
__global__ void owner_keys_kernel(OwnerShape h, const int64_t* offsets, const uint32_t* plan_start, Key n_keys,
                                  Key* keys, uint32_t* slots) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= h.n_vis) return;
    const uint32_t st = plan_start[i];
    Key k0 = n_keys, k1 = n_keys;
    if (st != kNoStart) {
        int64_t lo = 0, hi = h.n_sub;   // offsets[lo] <= i < offsets[hi]
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (offsets[mid] <= i) lo = mid; else hi = mid;
        }
        const int y0 = (int)(st >> 16), x0 = (int)(st & 0xFFFFu);
        k0 = (Key)((lo * h.nby + y0 / kOwnerBand) * h.n_u + x0);
        if (y0 % kOwnerBand + kSupportUV > kOwnerBand) k1 = k0 + (Key)h.n_u;
    }
    keys[2 * i] = k0;
    keys[2 * i + 1] = k1;
    slots[2 * i] = (uint32_t)(2 * i);
    slots[2 * i + 1] = (uint32_t)(2 * i + 1);
}

template <class Key>
__global__ void owner_places_kernel(const Key* keys, const uint32_t* slots, int64_t n_slots, Key n_keys,
                                    uint32_t* places) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n_slots) places[slots[p]] = keys[p] < n_keys ? (uint32_t)p : kNoPlace;
}

// (Positions past the last place hold visibilities too; no task names them.)
__global__ void owner_items_kernel(const uint32_t* slots, int64_t n_slots, uint32_t* items) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n_slots) items[p] = slots[p] >> 1;
}

// First position whose key is at least 'key'.
template <class Key>
__device__ __forceinline__ int64_t lower_bound(const Key* keys, int64_t n, Key key) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Task j before the sort by weight: segment and slab of a band. Sort key: the
// complement of its weight (records, and its columns' stores), so that the
// heaviest comes first.
template <class Key>
__global__ void owner_tasks_kernel(OwnerShape h, const Key* keys, int64_t n_slots, Key n_keys, int64_t n_tasks,
                                   OwnerTask* tasks, uint32_t* weights, uint32_t* idx) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_tasks) return;
    const int64_t per_band = (int64_t)h.n_seg * h.n_slabs;
    const int64_t band = j / per_band;
    const int place = (int)(j - band * per_band);
    const int x_lo = place / h.n_slabs * h.segment;
    const int x_hi = min(x_lo + h.segment, h.n_u);
    const Key base = (Key)(band * h.n_u);
    const int64_t b = lower_bound(keys, n_slots, (Key)(base + (Key)max(0, x_lo - (kSupportUV - 1))));
    const int64_t e = lower_bound(keys, n_slots, (Key)(base + (Key)x_hi));
    tasks[j] = OwnerTask{(uint32_t)b, (uint32_t)e, (int32_t)band, place};
    weights[j] = ~(uint32_t)min((int64_t)0x7FFFFFFF, e - b + (x_hi - x_lo));
    idx[j] = (uint32_t)j;
}

// Sum of x over the threads before this one, and over all of them in *total. part
// holds one entry per thread.
__device__ __forceinline__ uint32_t sum_before(uint32_t x, uint32_t* part, uint32_t* total) {
    const int t = (int)threadIdx.x, n = (int)blockDim.x;
    __syncthreads();
    part[t] = x;
    __syncthreads();
    for (int d = 1; d < n; d *= 2) {
        const uint32_t y = t >= d ? part[t - d] : 0u;
        __syncthreads();
        part[t] += y;
        __syncthreads();
    }
    *total = part[n - 1];
    return part[t] - x;
}

constexpr int kTaskThreads = 256;

// Slices of the tasks (j in order, heaviest first) that are longer than a slice
// may be, where the tasks are uneven; one workgroup.
template <class Key>
__device__ void cut_tasks(const OwnerShape& h, const Key* keys, int64_t n_slots, Key n_keys, const OwnerTask* tasks,
                          const uint32_t* weights, const uint32_t* order, int64_t n_tasks, int64_t room,
                          OwnerSlice* slices, uint32_t* first_slice, OwnerCounts* counts) {
    __shared__ uint32_t part[kTaskThreads];
    const int64_t n_items = lower_bound(keys, n_slots, n_keys);
    const int64_t work = n_items * h.n_slabs;
    const int64_t share = max((work + kOwnerSlices - 1) / kOwnerSlices, (int64_t)kOwnerMinSlice);
    const uint32_t longest = (uint32_t)((share + kWave - 1) / kWave * kWave);
    // weights are complements and include the columns (at most h.segment)
    const bool uneven = ~weights[0] > work / kOwnerEven + kOwnerJoin + h.segment;
    int64_t n_split = uneven ? lower_bound(weights, n_tasks, ~(longest + (uint32_t)h.segment)) : 0;
    const uint32_t many = (uint32_t)min((int64_t)0x7FFFFFFF, (int64_t)longest * kOwnerShared + h.segment);
    const int64_t n_shared = min(n_split, lower_bound(weights, n_tasks, ~many));
    auto length = [&](const OwnerTask& t) {   // of its slices: equal, whole batches of a wavefront
        const uint32_t n = t.end - t.begin, k = (n + longest - 1) / longest;
        return ((n + k - 1) / k + kWave - 1) / kWave * kWave;
    };
    uint32_t n_slices = 0;
    for (int64_t r = 0; r < n_split; r += kTaskThreads) {
        const int64_t j = r + threadIdx.x;
        uint32_t k = 0, all = 0;
        if (j < n_split) {
            const OwnerTask t = tasks[order[j]];
            const uint32_t len = length(t);
            k = (t.end - t.begin + len - 1) / len;
        }
        const uint32_t before = n_slices + sum_before(k, part, &all);
        if (j < n_split && j < room) first_slice[j] = before;
        n_slices += all;
    }
    if (n_split > room || n_slices > room) n_split = n_slices = 0;   // (see kOwnerMaxSlices: there is room)
    if (threadIdx.x == 0) first_slice[n_split] = n_slices;
    __syncthreads();
    uint32_t columns = 0;
    for (uint32_t r = 0; r < n_slices; r += kTaskThreads) {
        const uint32_t i = r + threadIdx.x;
        OwnerSlice x{};
        uint32_t all = 0;
        if (i < n_slices) {
            int64_t lo = 0, hi = n_split;   // first_slice[lo] <= i < first_slice[hi]
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (first_slice[mid] <= i) lo = mid; else hi = mid;
            }
            const OwnerTask t = tasks[order[lo]];
            const uint32_t len = length(t);
            x.begin = t.begin + (i - first_slice[lo]) * len;
            x.end = min(t.end, x.begin + len);
            x.band = t.band;
            const int seg = t.place / h.n_slabs;
            x.slab = t.place - seg * h.n_slabs;
            const int x_lo = seg * h.segment, x_hi = min(x_lo + h.segment, h.n_u);
            const Key base = (Key)((int64_t)t.band * h.n_u);
            const int c0 = (int)(keys[x.begin] - base), c1 = (int)(keys[x.end - 1] - base);
            x.x_lo = max(x_lo, c0 & ~7);
            x.width = min(x_hi, c1 + kSupportUV) - x.x_lo;
            x.task = (int32_t)lo;
        }
        x.column = columns + sum_before((uint32_t)x.width, part, &all);
        if (i < n_slices) slices[i] = x;
        columns += all;
    }
    if (threadIdx.x == 0)
        *counts = OwnerCounts{n_items, (int64_t)columns, (int32_t)n_split, (int32_t)n_slices,
                              (int32_t)min(n_split, n_shared)};
}

// Workgroup 0 cuts the heavy tasks, the others bring all tasks into order.
template <class Key>
__global__ __launch_bounds__(kTaskThreads) void order_tasks_kernel(OwnerShape h, const Key* keys, int64_t n_slots,
                                                                   Key n_keys, const OwnerTask* tasks,
                                                                   const uint32_t* weights, const uint32_t* order,
                                                                   int64_t n_tasks, int64_t room, OwnerTask* out,
                                                                   OwnerSlice* slices, uint32_t* first_slice,
                                                                   OwnerCounts* counts) {
    if (blockIdx.x == 0) {
        cut_tasks(h, keys, n_slots, n_keys, tasks, weights, order, n_tasks, room, slices, first_slice, counts);
        return;
    }
    const int64_t r = (int64_t)(blockIdx.x - 1) * kTaskThreads + threadIdx.x;
    if (r < n_tasks) out[r] = tasks[order[r]];
}

// ---------------------------------------------------------------------------
// Tiles that fit a staging box
// ---------------------------------------------------------------------------

// Minimum over lanes 0 .. l, on lane l.
__device__ __forceinline__ int prefix_min(int x) {
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) {
        const int y = __shfl_up(x, d);
        x = lane_id() >= d ? min(x, y) : x;
    }
    return x;
}

// Calls take(begin, count) for the tiles of one chunk, in order. The box of
// the first k visibilities grows with k, so the longest prefix that fits is
// found from the running box of 64 of them at once: lane k holds the box of
// the first k + 1.
template <class Take>
__device__ __forceinline__ void cut_chunk(const FitChunk& c, const uint32_t* start, const FitRule& r, Take take) {
    const int lane = lane_id();
    int at = 0;
    while (at < c.count) {
        const int n = min((int)r.nb, c.count - at);
        const uint32_t st = lane < n ? start[c.begin + at + lane] : kNoStart;
        const bool in = st != kNoStart;
        constexpr int kFar = 1 << 20;
        const int x = (int)(st & 0xFFFFu), y = (int)(st >> 16);
        const int xl = prefix_min(in ? x : kFar), xh = -prefix_min(in ? -x : kFar);
        const int yl = prefix_min(in ? y : kFar), yh = -prefix_min(in ? -y : kFar);
        bool fits = true;   // (no visibility in range so far: an empty box)
        if (xh >= xl) fits = (int64_t)(xh - xl + r.support) * (yh - yl + r.support) <= r.cap_cells;
        const uint64_t over = __ballot(!fits && lane < n);
        int k = over ? (int)__builtin_ctzll(over) : n;
        if (at + k < c.count) k = min(n, max(k, r.min_fit));   // sparse: gathered without staging
        k = max(k, 1);
        take(at, k);
        at += k;
    }
}

__global__ __launch_bounds__(256) void count_tiles_kernel(const FitChunk* chunks, int64_t n_chunks,
                                                          const uint32_t* start, FitRule rule, uint32_t* counts) {
    const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (k >= n_chunks) return;
    uint32_t n = 0;
    cut_chunk(chunks[k], start, rule, [&](int, int) { ++n; });
    if (lane_id() == 0) counts[k] = n;
}

// counts[0 .. n) to their exclusive sums, the total in counts[n] (one workgroup).
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void scan_counts_kernel(uint32_t* counts, int64_t n) {
    __shared__ uint32_t part[kScanThreads];
    const int64_t per = (n + kScanThreads - 1) / kScanThreads;
    const int64_t b = min((int64_t)threadIdx.x * per, n), e = min(b + per, n);
    uint32_t sum = 0;
    for (int64_t i = b; i < e; ++i) sum += counts[i];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < kScanThreads; d *= 2) {
        const uint32_t x = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0u;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - sum;
    for (int64_t i = b; i < e; ++i) {
        const uint32_t c = counts[i];
        counts[i] = run;
        run += c;
    }
    if (threadIdx.x == kScanThreads - 1) counts[n] = part[kScanThreads - 1];
}

__global__ __launch_bounds__(256) void write_tiles_kernel(const FitChunk* chunks, int64_t n_chunks,
                                                          const uint32_t* start, const uint32_t* perm, FitRule rule,
                                                          const uint32_t* first_tile, Tile* tiles,
                                                          uint32_t* tile_vis) {
    const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (k >= n_chunks) return;
    const FitChunk c = chunks[k];
    int64_t t = first_tile[k];
    cut_chunk(c, start, rule, [&](int at, int count) {
        const int lane = lane_id();
        if (lane == 0) tiles[t] = Tile{c.begin + at, c.sub, (uint16_t)count, 0};
        tile_vis[t * kMaxNb + lane] = perm[c.begin + at + (lane < count ? lane : 0)];
        ++t;
    });
}

// The queues of split_queues for such a list. Queue c ends after the first tile
// with which the visibilities so far, times the number of queues, reach (c + 1)
// n_vis, but holds at least one tile if there is one left. The tiles cover the
// work order without gaps, so those before tile t number tiles[t].begin.
__global__ void tile_queues_kernel(const Tile* tiles, int64_t n_tiles, int64_t n_vis, QueueSpec* q) {
    __shared__ int32_t full[kMaxQueues];
    const int nq = n_tiles < kMaxQueues ? (int)n_tiles : kMaxQueues;
    const int c = (int)threadIdx.x;
    if (c < nq) {
        int64_t lo = 0, hi = n_tiles;   // first tile count at which queue c is full
        if (c < nq - 1) {
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                const int64_t sum = tiles[mid].begin + tiles[mid].count;
                if (sum * nq >= n_vis * (c + 1)) hi = mid; else lo = mid + 1;
            }
            ++lo;
        } else {
            lo = n_tiles;
        }
        full[c] = (int32_t)lo;
    }
    __syncthreads();
    if (c != 0) return;
    q->n_queues = nq;
    int32_t at = 0;
    for (int k = 0; k < kMaxQueues; ++k) {
        q->begin[k] = k < nq ? at : 0;
        if (k < nq) at = (int32_t)min(n_tiles, (int64_t)max(full[k], at + 1));
        q->end[k] = k < nq ? at : 0;
    }
}

size_t up256(size_t b) { return (b + 255) / 256 * 256; }
unsigned grid_of(int64_t n) { return (unsigned)((n + 255) / 256); }

template <class Key>
hipError_t radix_bytes(int64_t n, int end_bit, hipStream_t stream, size_t* bytes) {
    return hipcub::DeviceRadixSort::SortPairs(nullptr, *bytes, (Key*)nullptr, (Key*)nullptr, (uint32_t*)nullptr,
                                              (uint32_t*)nullptr, n, 0, end_bit, stream);
}

template <class Key>
hipError_t sort_t(const Problem& pr, const int64_t* offsets, int64_t n_sub, int64_t n, int bits, int end_bit,
                  uint32_t* perm, uint32_t* plan_start, uint32_t* start, DeviceTemp& temp, hipStream_t stream) {
    // keys in and out, indices, the sort's own storage
    size_t sort_bytes = 0;
    hipError_t e = radix_bytes<Key>(n, end_bit, stream, &sort_bytes);
    if (e != hipSuccess) return e;
    const size_t kb = up256(sizeof(Key) * (size_t)n), ib = up256(sizeof(uint32_t) * (size_t)n);
    e = temp.ensure(2 * kb + ib + sort_bytes);
    if (e != hipSuccess) return e;
    char* base = static_cast<char*>(temp.p);
    Key* k_in = reinterpret_cast<Key*>(base);
    Key* k_out = reinterpret_cast<Key*>(base + kb);
    uint32_t* v_in = reinterpret_cast<uint32_t*>(base + 2 * kb);
    hipLaunchKernelGGL((sort_keys_kernel<Key>), dim3(grid_of(n)), dim3(256), 0, stream, pr, offsets, n_sub, n, bits,
                       k_in, v_in, plan_start);
    e = hipGetLastError();
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairs(base + 2 * kb + ib, sort_bytes, k_in, k_out, v_in, perm, n, 0, end_bit,
                                               stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(ordered_starts_kernel, dim3(grid_of(n)), dim3(256), 0, stream, perm, plan_start, n, start);
        e = hipGetLastError();
    }
    return e;
}

template <class Key>
hipError_t owner_t(const OwnerShape& h, const int64_t* offsets, const uint32_t* plan_start, OwnerPlaces* places,
                   OwnerTask* tasks, OwnerSlice* slices, uint32_t* first_slice, OwnerCounts* counts, Key n_keys,
                   int end_bit, DeviceTemp& temp, hipStream_t stream) {
    const int64_t n_slots = 2 * h.n_vis, n_tasks = h.tasks();
    size_t slot_sort = 0, task_sort = 0;
    hipError_t e = radix_bytes<Key>(n_slots, end_bit, stream, &slot_sort);
    if (e == hipSuccess) e = radix_bytes<uint32_t>(n_tasks, 32, stream, &task_sort);
    if (e != hipSuccess) return e;
    // keys and slots in and out, tasks with their weights and ranks in and
    // out, the sorts' own storage, the counts
    const size_t kb = up256(sizeof(Key) * (size_t)n_slots), sb = up256(4 * (size_t)n_slots);
    const size_t tb = up256(sizeof(OwnerTask) * (size_t)n_tasks), wb = up256(4 * (size_t)n_tasks);
    const size_t own = up256(std::max(slot_sort, task_sort));
    e = temp.ensure(2 * kb + 2 * sb + tb + 4 * wb + own + 256);
    if (e != hipSuccess) return e;
    char* at = static_cast<char*>(temp.p);
    auto take = [&](size_t bytes) {
        char* x = at;
        at += bytes;
        return x;
    };
    Key* k_in = reinterpret_cast<Key*>(take(kb));
    Key* k_out = reinterpret_cast<Key*>(take(kb));
    uint32_t* s_in = reinterpret_cast<uint32_t*>(take(sb));
    uint32_t* s_out = reinterpret_cast<uint32_t*>(take(sb));
    OwnerTask* t_in = reinterpret_cast<OwnerTask*>(take(tb));
    uint32_t* w[4];
    for (uint32_t*& x : w) x = reinterpret_cast<uint32_t*>(take(wb));
    char* sort_own = take(own);
    OwnerCounts* d_counts = reinterpret_cast<OwnerCounts*>(take(256));
    hipLaunchKernelGGL((owner_keys_kernel<Key>), dim3(grid_of(h.n_vis)), dim3(256), 0, stream, h, offsets, plan_start,
                       n_keys, k_in, s_in);
    e = hipGetLastError();
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairs(sort_own, slot_sort, k_in, k_out, s_in, s_out, n_slots, 0, end_bit,
                                               stream);
    if (e == hipSuccess) {
        if (h.direct)
            hipLaunchKernelGGL(owner_items_kernel, dim3(grid_of(n_slots)), dim3(256), 0, stream, s_out, n_slots,
                               reinterpret_cast<uint32_t*>(places));
        else
            hipLaunchKernelGGL((owner_places_kernel<Key>), dim3(grid_of(n_slots)), dim3(256), 0, stream, k_out, s_out,
                               n_slots, n_keys, reinterpret_cast<uint32_t*>(places));
        hipLaunchKernelGGL((owner_tasks_kernel<Key>), dim3(grid_of(n_tasks)), dim3(256), 0, stream, h, k_out, n_slots,
                           n_keys, n_tasks, t_in, w[0], w[2]);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = hipcub::DeviceRadixSort::SortPairs(sort_own, task_sort, w[0], w[1], w[2], w[3], n_tasks, 0, 32, stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL((order_tasks_kernel<Key>), dim3(grid_of(n_tasks) + 1), dim3(kTaskThreads), 0, stream, h, k_out,
                           n_slots, n_keys, t_in, w[1], w[3], n_tasks, h.slices(), tasks, slices, first_slice, d_counts);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(counts, d_counts, sizeof(OwnerCounts), hipMemcpyDeviceToHost, stream);
    const hipError_t es = hipStreamSynchronize(stream);
    return e == hipSuccess ? es : e;
}

}  // namespace

hipError_t sort_visibilities(const Problem& pr, const int64_t* offsets_host, const int64_t* offsets, int64_t n_sub,
                             uint32_t* perm, uint32_t* plan_start, uint32_t* start, DeviceTemp& temp,
                             hipStream_t stream) {
    const int64_t n = offsets_host[n_sub];
    if (n == 0) return hipSuccess;
    int bits = 1;   // of a first tap, per axis
    while ((1 << bits) <= std::max(pr.n_u, pr.n_v) - kSupportUV) ++bits;
    int end_bit = 2 * bits + 1;
    while ((int64_t(1) << (end_bit - 2 * bits - 1)) < n_sub) ++end_bit;
    return end_bit <= 32
               ? sort_t<uint32_t>(pr, offsets, n_sub, n, bits, end_bit, perm, plan_start, start, temp, stream)
               : sort_t<uint64_t>(pr, offsets, n_sub, n, bits, end_bit, perm, plan_start, start, temp, stream);
}

hipError_t build_owner_order(const OwnerShape& h, const int64_t* offsets, const uint32_t* plan_start,
                             OwnerPlaces* places, OwnerTask* tasks, OwnerSlice* slices, uint32_t* first_slice,
                             OwnerCounts* counts, DeviceTemp& temp, hipStream_t stream) {
    const int64_t n_keys = h.n_sub * h.nby * h.n_u;
    int end_bit = 1;
    while ((int64_t(1) << end_bit) <= n_keys) ++end_bit;
    return end_bit <= 32 ? owner_t<uint32_t>(h, offsets, plan_start, places, tasks, slices, first_slice, counts,
                                             (uint32_t)n_keys, end_bit, temp, stream)
                         : owner_t<uint64_t>(h, offsets, plan_start, places, tasks, slices, first_slice, counts,
                                             (uint64_t)n_keys, end_bit, temp, stream);
}

hipError_t launch_count_tiles(const FitChunk* chunks, int64_t n_chunks, const uint32_t* start, const FitRule& rule,
                              uint32_t* first_tile, hipStream_t stream) {
    hipLaunchKernelGGL(count_tiles_kernel, dim3(grid_of(n_chunks * kWave)), dim3(256), 0, stream, chunks, n_chunks,
                       start, rule, first_tile);
    hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(kScanThreads), 0, stream, first_tile, n_chunks);
    return hipGetLastError();
}

hipError_t launch_write_tiles(const FitChunk* chunks, int64_t n_chunks, const uint32_t* start, const uint32_t* perm,
                              const FitRule& rule, const uint32_t* first_tile, int64_t n_tiles, int64_t n_vis,
                              Tile* tiles, uint32_t* tile_vis, QueueSpec* q, hipStream_t stream) {
    hipLaunchKernelGGL(write_tiles_kernel, dim3(grid_of(n_chunks * kWave)), dim3(256), 0, stream, chunks, n_chunks,
                       start, perm, rule, first_tile, tiles, tile_vis);
    hipLaunchKernelGGL(tile_queues_kernel, dim3(1), dim3(kWave), 0, stream, tiles, n_tiles, n_vis, q);
    return hipGetLastError();
}

}  // namespace dg
