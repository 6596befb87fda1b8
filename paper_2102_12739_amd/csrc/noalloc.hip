// Degridding for callers that cannot allocate device memory (code under HIP
// graph capture, tight serving loops, harnesses that forbid hipMalloc): the
// kernels of degrid_execute_noalloc and the device scratch they use.
//
// The scratch is one file-scope device array per GPU, `scratch`, of
// kNoAllocBytes bytes, holding
//   - control blocks (the out-of-range count; the last workgroup of a launch
//     leaves its own cleared for the next). Calls that ask for the count take
//     them in turn: two that overlap in one would miscount their workgroups'
//     ends, and, with grids of two sizes, leave it so for every later call;
//   - for calls of more than kArgSubgrids subgrids, the caller's visibility
//     offsets, staged from the host ([S+1] int64), and the first tile of every
//     subgrid ([S+1] uint32, a prefix sum of ceil(N_s / n_b)).
// Host code never passes the array's name to a kernel: at a device's first
// call, hipGetSymbolAddress gives that device's copy's address, which is
// kept per device and used for every copy and launch. Every call on one GPU
// shares the array, so calls that overlap on one GPU race.
//
// Work: one tile is n_b consecutive visibilities of one subgrid, in input
// order (Section 2 gives each thread block N_b visibilities of a subgrid).
// Each XCD's workgroups take a contiguous share of the tiles, round-robin, and
// a wavefront finds a tile's subgrid by comparing it with the first tiles of 64
// subgrids at a time. The gather is the degrid kernel's cache gather
// (gather_tile), with the next tile's coordinates requested before it.
//
// Up to kArgSubgrids subgrids, the offsets travel as kernel arguments and the
// call is one launch; staging them, a prefix-sum kernel and tiles claimed one
// by one took three times as long for small calls (7500 visibilities on 9
// subgrids: 28.3 -> 12.3 us; 1.0 M uniform ones on
// 16 subgrids 358 -> 235 us).
#include "dg_device.h"

#include <algorithm>
#include <mutex>

namespace dg {
namespace {

constexpr uint32_t kNoAllocCtls = 16;
constexpr size_t kNoAllocOffsets = (kNoAllocCtls * sizeof(Ctl) + 255) / 256 * 256;   // int64 visibility offsets [S+1]
constexpr size_t kNoAllocTileOffsets = kNoAllocOffsets + sizeof(int64_t) * (kNoAllocMaxSubgrids + 1);
constexpr size_t kNoAllocUsed = kNoAllocTileOffsets + sizeof(uint32_t) * (kNoAllocMaxSubgrids + 1);
static_assert(kNoAllocUsed <= kNoAllocBytes, "scratch layout exceeds the array");

// First visibility and first tile of every subgrid, and of the end.
constexpr int kArgSubgrids = 191;
struct ArgOffsets {
    uint32_t vis[kArgSubgrids + 1];
    uint32_t tile[kArgSubgrids + 1];
};

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kSetupThreads = 1024;

// First tile of every subgrid (exclusive prefix sum of ceil(N_s / n_b)). One
// workgroup; thread k scans a contiguous run of subgrids.
__global__ __launch_bounds__(kSetupThreads) void noalloc_setup_kernel(unsigned char* scr, int64_t n_sub, int nb) {
    const int64_t* off = reinterpret_cast<const int64_t*>(scr + kNoAllocOffsets);
    uint32_t* toff = reinterpret_cast<uint32_t*>(scr + kNoAllocTileOffsets);
    __shared__ uint32_t part[kSetupThreads];
    const int64_t per = (n_sub + kSetupThreads - 1) / kSetupThreads;
    const int64_t s0 = min((int64_t)threadIdx.x * per, n_sub);
    const int64_t s1 = min(s0 + per, n_sub);
    uint32_t sum = 0;
    for (int64_t s = s0; s < s1; ++s) sum += (uint32_t)((off[s + 1] - off[s] + nb - 1) / nb);
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < kSetupThreads; d *= 2) {
        const uint32_t x = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0u;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - sum;
    for (int64_t s = s0; s < s1; ++s) {
        toff[s] = run;
        run += (uint32_t)((off[s + 1] - off[s] + nb - 1) / nb);
    }
    if (threadIdx.x == kSetupThreads - 1) toff[n_sub] = part[kSetupThreads - 1];
}

// ARGS: the offsets come as arguments, else from the scratch.
template <int G, int F, bool ARGS>
__global__ __launch_bounds__(kBlockThreads, 2) void degrid_noalloc_kernel(Problem pr, unsigned char* scr, int n_sub,
                                                                          int n_tiles, int nb, Ctl* ctl,
                                                                          unsigned long long* oob_out,
                                                                          ArgOffsets args) {
    using GT = GridTraits<G>;
    __shared__ float2 s_out[kWavesPerBlock][kMaxNb];
    __shared__ __attribute__((aligned(16))) char s_weights[kWavesPerBlock][kWeightsBytes<F>];
    const int lane = lane_id();
    const int wv = (int)(threadIdx.x / kWave);
    const int64_t* off = reinterpret_cast<const int64_t*>(scr + kNoAllocOffsets);
    const uint32_t* toff = reinterpret_cast<const uint32_t*>(scr + kNoAllocTileOffsets);
    auto first_vis = [&](int s) { return ARGS ? (int64_t)args.vis[s] : off[s]; };
    auto first_tile = [&](int s) { return ARGS ? args.tile[s] : toff[s]; };
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(pr.g_uv, pr.guv_bytes);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(pr.g_w, (uint32_t)pr.os_w * kSupportW * GcfTraits<F>::kBytes);
    const uint32_t cell_bytes = (uint32_t)pr.n_w * GT::kElemBytes;
    uint32_t wave_oob = 0;

    // this XCD's share of the tiles, and this wavefront's place among its own
    const int nq = min((int)gridDim.x, kMaxQueues);
    const int q = (int)blockIdx.x % nq;
    const int end = (int)((int64_t)n_tiles * (q + 1) / nq);
    const int stride = (((int)gridDim.x - q + nq - 1) / nq) * kWavesPerBlock;
    const int begin = (int)((int64_t)n_tiles * q / nq);
    const int rank = ((int)blockIdx.x / nq) * kWavesPerBlock + wv;
    int t = uniform(begin + min(rank, end - begin));

    // Subgrid, first visibility and count of tile t: the subgrid is the last
    // one whose first tile is at most t (empty subgrids share theirs with the
    // next one). Tiles come in increasing order, so the search starts with the
    // 64 subgrids of the previous one; where they are not enough, each step
    // divides the rest by 64 (at the limit of 16384 subgrids three loads one
    // after another; 64 subgrids after 64, up to 260: 1.0 M visibilities on
    // 16384 subgrids 300 us, now 251).
    int group = 0;
    auto locate = [&](int tile, int& sub, int64_t& beg, int& count) {
        while (true) {
            const int s = group + lane;
            const bool past = s > n_sub || first_tile(min(s, n_sub)) > (uint32_t)tile;
            const uint64_t m = __ballot(past);
            if (m == 0u) {
                group += kWave - 1;   // (the last one may still be it)
                if constexpr (!ARGS) {
                    int hi = n_sub;   // first_tile(group) <= tile < first_tile(hi)
                    while (hi - group > kWave) {
                        const int step = (hi - group + kWave - 1) / kWave;
                        const uint64_t beyond = __ballot(first_tile(min(group + (lane + 1) * step, hi)) > (uint32_t)tile);
                        const int k = (int)__builtin_ctzll(beyond);   // (lane 63 is at hi)
                        hi = uniform(min(group + (k + 1) * step, hi));
                        group = uniform(group + k * step);
                    }
                }
                continue;
            }
            sub = uniform(group + (int)__builtin_ctzll(m) - 1);
            break;
        }
        const int64_t v0 = first_vis(sub), v1 = first_vis(sub + 1);
        beg = v0 + (int64_t)((uint32_t)tile - first_tile(sub)) * nb;
        count = uniform((int)min((int64_t)nb, v1 - beg));
    };
    int sub = 0, count = 0;
    int64_t beg = 0;
    double u = 0.0, v = 0.0, w = 0.0;
    auto request = [&]() {   // coordinates of the tile at beg
        if (lane < count) {
            const double* c = pr.uvw + 3 * (beg + lane);
            u = c[0];
            v = c[1];
            w = c[2];
        }
    };
    if (t < end) {
        locate(t, sub, beg, count);
        request();
    }
    while (t < end) {
        const int64_t vis = beg + lane;
        const int n = count, s = sub;
        int32_t x0 = 0, y0 = 0, cell = 0, tab = 0, ow = 0;
        bool in_range = false;
        if (lane < n) in_range = coords_from(pr, u, v, w, cell, tab, ow, x0, y0);
        if (!in_range) ow = 0;
        wave_oob += (uint32_t)__popcll(__ballot(lane < n && !in_range));

        const char* sub_base = static_cast<const char*>(pr.subgrids) + s * (int64_t)pr.sub_bytes;
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(sub_base, pr.sub_bytes);
        t = next_dealt(t, stride, end);
        if (t < end) {
            locate(t, sub, beg, count);
            request();
        }
        const int a_off = in_range ? cell * (int)GT::kElemBytes : (int)kOutOfRange;
        // (a visibility out of range reads block 0 and is written as 0 below)
        gather_tile<G, F, false, 16>(s_out[wv], n, in_range ? table_word(tab, ow) : 0u, (uint32_t)a_off, rg, rw, ra,
                                     nullptr, s_weights[wv], ((uint64_t)pr.g_uv & 3u) == 0u, cell_bytes,
                                     (uint32_t)pr.n_u * cell_bytes);
        wave_lds_sync();
        if (lane < n) static_cast<float2*>(pr.vis)[vis] = in_range ? s_out[wv][lane] : make_float2(0.f, 0.f);
        wave_lds_sync();
    }
    if (oob_out) {   // the last workgroup hands the count over
        if (finish_launch(ctl, wave_oob))
            *oob_out = *reinterpret_cast<volatile unsigned long long*>(&ctl->oob.v[2]);
    }
}

// What every instance of the kernel is launched with.
struct NoAllocCall {
    Problem pr;
    unsigned char* scr;
    Ctl* ctl;
    int n_sub, n_tiles, nb, blocks;
    unsigned long long* oob_out;
    const ArgOffsets* args;   // nullptr: the offsets are in the scratch
    hipStream_t stream;
};

template <int G, int F>
hipError_t launch_main(const NoAllocCall& c) {
    if (c.args)
        hipLaunchKernelGGL((degrid_noalloc_kernel<G, F, true>), dim3(c.blocks), dim3(kBlockThreads), 0, c.stream,
                           c.pr, c.scr, c.n_sub, c.n_tiles, c.nb, c.ctl, c.oob_out, *c.args);
    else
        hipLaunchKernelGGL((degrid_noalloc_kernel<G, F, false>), dim3(c.blocks), dim3(kBlockThreads), 0, c.stream,
                           c.pr, c.scr, c.n_sub, c.n_tiles, c.nb, c.ctl, c.oob_out, ArgOffsets{});
    return hipGetLastError();
}

template <int G, int F>
hipError_t occupancy(int* n) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(n, degrid_noalloc_kernel<G, F, true>, kBlockThreads, 0);
}

hipError_t launch_main_any(const NoAllocCall& c, int grid_kind, int gcf_kind) {
#define DG_CALL(G, F) launch_main<G, F>(c)
    switch (grid_kind * 3 + gcf_kind) {
        case kGridC64 * 3 + kGcfF32: return DG_CALL(kGridC64, kGcfF32);
        case kGridC64 * 3 + kGcfF16: return DG_CALL(kGridC64, kGcfF16);
        case kGridC64 * 3 + kGcfBF16: return DG_CALL(kGridC64, kGcfBF16);
        case kGridCBF16 * 3 + kGcfF32: return DG_CALL(kGridCBF16, kGcfF32);
        case kGridCBF16 * 3 + kGcfF16: return DG_CALL(kGridCBF16, kGcfF16);
        case kGridCBF16 * 3 + kGcfBF16: return DG_CALL(kGridCBF16, kGcfBF16);
        case kGridCF16 * 3 + kGcfF32: return DG_CALL(kGridCF16, kGcfF32);
        case kGridCF16 * 3 + kGcfF16: return DG_CALL(kGridCF16, kGcfF16);
        case kGridCF16 * 3 + kGcfBF16: return DG_CALL(kGridCF16, kGcfBF16);
        default: return hipErrorInvalidValue;
    }
#undef DG_CALL
}

hipError_t occupancy_any(int grid_kind, int gcf_kind, int* n) {
#define DG_CALL(G, F) occupancy<G, F>(n)
    switch (grid_kind * 3 + gcf_kind) {
        case kGridC64 * 3 + kGcfF32: return DG_CALL(kGridC64, kGcfF32);
        case kGridC64 * 3 + kGcfF16: return DG_CALL(kGridC64, kGcfF16);
        case kGridC64 * 3 + kGcfBF16: return DG_CALL(kGridC64, kGcfBF16);
        case kGridCBF16 * 3 + kGcfF32: return DG_CALL(kGridCBF16, kGcfF32);
        case kGridCBF16 * 3 + kGcfF16: return DG_CALL(kGridCBF16, kGcfF16);
        case kGridCBF16 * 3 + kGcfBF16: return DG_CALL(kGridCBF16, kGcfBF16);
        case kGridCF16 * 3 + kGcfF32: return DG_CALL(kGridCF16, kGcfF32);
        case kGridCF16 * 3 + kGcfF16: return DG_CALL(kGridCF16, kGcfF16);
        case kGridCF16 * 3 + kGcfBF16: return DG_CALL(kGridCF16, kGcfBF16);
        default: return hipErrorInvalidValue;
    }
#undef DG_CALL
}

// Per device: the address of this device's copy of `scratch` and the
// resident workgroups of each kernel instance, looked up once.
constexpr int kMaxDevices = 64;
struct DeviceState {
    unsigned char* scratch = nullptr;
    int n_cu = 0;
    int occ[9] = {};
    uint32_t next_ctl = 0;
};
std::mutex g_mutex;
DeviceState g_dev[kMaxDevices];

// ctl, if given, receives the next control block.
hipError_t device_state(int grid_kind, int gcf_kind, unsigned char** scr, int* resident, Ctl** ctl = nullptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceState& d = g_dev[dev];
    if (!d.scratch) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        e = hipDeviceGetAttribute(&d.n_cu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        d.scratch = static_cast<unsigned char*>(p);
    }
    int& occ = d.occ[grid_kind * 3 + gcf_kind];
    if (occ == 0) {
        e = occupancy_any(grid_kind, gcf_kind, &occ);
        if (e != hipSuccess) return e;
        if (occ < 1) occ = 1;
    }
    *scr = d.scratch;
    *resident = d.n_cu * occ;
    if (ctl) *ctl = reinterpret_cast<Ctl*>(d.scratch) + d.next_ctl++ % kNoAllocCtls;
    return hipSuccess;
}

}  // namespace

hipError_t noalloc_resident(int grid_kind, int gcf_kind, int* resident) {
    unsigned char* scr = nullptr;
    return device_state(grid_kind, gcf_kind, &scr, resident);
}

hipError_t launch_degrid_noalloc(const Problem& pr, int grid_kind, int gcf_kind,
                                 const int64_t* offsets_host, int64_t n_sub, int nb, int64_t n_tiles,
                                 unsigned long long* oob_out, hipStream_t stream) {
    if (n_sub < 0 || n_sub > kNoAllocMaxSubgrids || nb < 1 || nb > kMaxNb) return hipErrorInvalidValue;
    NoAllocCall c{};
    int resident = 0;
    hipError_t e = device_state(grid_kind, gcf_kind, &c.scr, &resident, oob_out ? &c.ctl : nullptr);
    if (e != hipSuccess) return e;
    c.pr = pr;
    c.n_sub = (int)n_sub;
    c.n_tiles = (int)n_tiles;
    c.nb = nb;
    c.oob_out = oob_out;
    c.stream = stream;
    // (a call without tiles still clears the caller's count)
    c.blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n_tiles + kWavesPerBlock - 1) / kWavesPerBlock, resident));
    ArgOffsets args{};
    if (n_sub <= kArgSubgrids) {
        uint32_t tiles = 0;
        for (int64_t s = 0; s <= n_sub; ++s) {
            args.vis[s] = (uint32_t)offsets_host[s];
            args.tile[s] = tiles;
            if (s < n_sub) tiles += (uint32_t)((offsets_host[s + 1] - offsets_host[s] + nb - 1) / nb);
        }
        c.args = &args;
    } else {
        e = hipMemcpyAsync(c.scr + kNoAllocOffsets, offsets_host, sizeof(int64_t) * (size_t)(n_sub + 1),
                           hipMemcpyHostToDevice, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(noalloc_setup_kernel, dim3(1), dim3(kSetupThreads), 0, stream, c.scr, n_sub, nb);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_tiles == 0 && !oob_out) return hipSuccess;
    return launch_main_any(c, grid_kind, gcf_kind);
}

}  // namespace dg
