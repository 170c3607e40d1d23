// C ABI entry points of the single operations (dc_run_stack: dc_stack.hip): argument validation and launches.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "dc_internal.h"

namespace dc {

// Bytes of plan data for one conv layer, worst case.
size_t plan_bytes(int n_streams, int Hout, int Wout, const ConvTiling& t, int max_rects) {
    size_t tiles = (size_t)n_streams * ((Hout + t.th - 1) / t.th) * ((Wout + t.tw - 1) / t.tw);
    return align_up(tiles * sizeof(TileDev), 256) + align_up((size_t)n_streams * max_rects * sizeof(RectDev), 256) +
           align_up((size_t)n_streams * sizeof(RangeDev), 256);
}

PlanAddr pack_plan(const LayerPlan& plan, unsigned char* host, unsigned char* dev) {
    size_t off = 0;
    PlanAddr a;
    a.tiles = reinterpret_cast<const TileDev*>(dev + off);
    if (!plan.tiles.empty()) std::memcpy(host + off, plan.tiles.data(), plan.tiles.size() * sizeof(TileDev));
    off += align_up(plan.n_tiles * sizeof(TileDev), 256);       // the caller may fill the tile list itself
    a.rects = reinterpret_cast<const RectDev*>(dev + off);
    if (!plan.rects.empty()) std::memcpy(host + off, plan.rects.data(), plan.rects.size() * sizeof(RectDev));
    off += align_up(plan.rects.size() * sizeof(RectDev), 256);
    a.ranges = reinterpret_cast<const RangeDev*>(dev + off);
    if (!plan.ranges.empty()) std::memcpy(host + off, plan.ranges.data(), plan.ranges.size() * sizeof(RangeDev));
    off += align_up(plan.ranges.size() * sizeof(RangeDev), 256);
    a.bytes = off;
    return a;
}

// Small plans (one or a few streams) go from the pinned staging buffer to the device with a kernel that reads
// the host memory through its device address: a launch costs the host a few microseconds where an asynchronous
// copy on an idle stream measured 25.  Large plans (64 streams: megabytes) are faster through the copy engine,
// and pageable staging memory has no device address.
static __global__ void __launch_bounds__(256) upload_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n_vec) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_vec; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// Device address of a host buffer: nullptr if it is not pinned.  Asked on every call: a caller may free a
// pinned buffer and pass pageable memory at the same address later.
const unsigned char* device_alias(void* host) {
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, host, 0) != hipSuccess) { d = nullptr; (void)hipGetLastError(); }
    return static_cast<const unsigned char*>(d);
}

hipError_t upload_plans(void* dst_dev, const unsigned char* src_host, size_t bytes, void* ws_host, hipStream_t st) {
    if (bytes > 256 * 1024) return hipMemcpyAsync(dst_dev, src_host, bytes, hipMemcpyHostToDevice, st);
    const unsigned char* alias = device_alias(ws_host);
    if (!alias || bytes % 16 || reinterpret_cast<uintptr_t>(dst_dev) % 16 || reinterpret_cast<uintptr_t>(src_host) % 16)
        return hipMemcpyAsync(dst_dev, src_host, bytes, hipMemcpyHostToDevice, st);
    const unsigned char* src = alias + (src_host - static_cast<const unsigned char*>(ws_host));
    const size_t n_vec = bytes / 16;
    const unsigned grid = (unsigned)std::min<size_t>((n_vec + 255) / 256, 1024);
    hipLaunchKernelGGL(upload_kernel, dim3(grid), dim3(256), 0, st, reinterpret_cast<const uint4*>(src),
                       static_cast<uint4*>(dst_dev), n_vec);
    return hipGetLastError();
}

// The plan of one layer and the copies of its rectangles in one launch: the copies take their few rectangles as kernel
// arguments instead of waiting for the upload.  Row y < n of the grid copies rectangle y, the last one uploads.  A single 3x3
// 256->256 layer on 8 streams of 56x56 (plan 16 KB, 16 rectangles): copy engine, copies, convolution 57 us a call; upload
// kernel with two workspaces in turn 38; this 36, what the host needs.
// 32 rectangles are 1 KiB of arguments: two for each of 16 streams.  More take the upload and the copies in two launches, which
// costs 2 to 3 us (28x28 64->64, 33 and 64 rectangles 34.7 and 37.8 us a call; with room for 96 here 32.4 and 34.7, and 32
// rectangles 33.4 against 33.1); 4 KiB is what a launch takes in arguments.
constexpr int kCopyArgRects = 32;
struct CopyArgs {
    const uint4 *src, *prev;
    uint4 *dst, *out;
    int n_vec, n, Hout, Wout, pv;
    RectDev r[kCopyArgRects];
};
static __global__ void __launch_bounds__(256) upload_and_copy_kernel(CopyArgs A) {
    const int first = (int)blockIdx.x * 256 + (int)threadIdx.x, stride = (int)gridDim.x * 256;
    if ((int)blockIdx.y == A.n) {
        for (int i = first; i < A.n_vec; i += stride) A.dst[i] = A.src[i];
        return;
    }
    const RectDev r = A.r[blockIdx.y];
    const int row_v = r.w * A.pv, total = r.h * row_v;
    const size_t map = (size_t)r.stream * A.Hout * A.Wout;
    for (int i = first; i < total; i += stride) {
        const int row = i / row_v, col = i - row * row_v;
        A.out[(map + (size_t)(r.y + row) * A.Wout + r.x) * A.pv + col] = A.prev[(map + (size_t)(r.y + r.dy + row) * A.Wout + (r.x + r.dx)) * A.pv + col];
    }
}

// Brings the packed plan (in ws_host) to the device and makes its copies if both fit one launch (*copied).
static hipError_t upload_and_copy(const LayerPlan& plan, void* ws_dev, void* ws_host, size_t bytes, const void* prev, void* out,
                                  int Hout, int Wout, size_t px_bytes, bool* copied, hipStream_t st) {
    *copied = false;
    long vec = 0;                                          // of the largest rectangle
    for (const RectDev& r : plan.rects) vec = std::max(vec, (long)r.w * r.h * (long)(px_bytes / 16));
    const bool fits = !plan.rects.empty() && plan.rects.size() <= (size_t)kCopyArgRects && px_bytes % 16 == 0 && bytes % 16 == 0 && bytes <= 256 * 1024 &&
                      vec < (1l << 30) && reinterpret_cast<uintptr_t>(prev) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0 &&
                      reinterpret_cast<uintptr_t>(ws_dev) % 16 == 0 && reinterpret_cast<uintptr_t>(ws_host) % 16 == 0;
    const unsigned char* const alias = fits ? device_alias(ws_host) : nullptr;
    if (!alias) return upload_plans(ws_dev, static_cast<unsigned char*>(ws_host), bytes, ws_host, st);
    CopyArgs A;
    A.src = reinterpret_cast<const uint4*>(alias); A.dst = static_cast<uint4*>(ws_dev);
    A.prev = static_cast<const uint4*>(prev); A.out = static_cast<uint4*>(out);
    A.n_vec = (int)(bytes / 16); A.n = (int)plan.rects.size();
    A.Hout = Hout; A.Wout = Wout; A.pv = (int)(px_bytes / 16);
    std::copy(plan.rects.begin(), plan.rects.end(), A.r);
    const long blocks = std::max(std::max((vec + 1023) / 1024, ((long)A.n_vec + 1023) / 1024), 1l);      // four vectors a thread
    hipLaunchKernelGGL(upload_and_copy_kernel, dim3((unsigned)std::min(blocks, 1024l), (unsigned)A.n + 1), dim3(256), 0, st, A);
    *copied = true;
    return hipGetLastError();
}

int run_conv_planned(const dc_layer& l, const void* in, const void* w, const float* bias,
                     const void* cache_prev, void* out, int n_streams, int Hin, int Win, int dtype,
                     const ConvTiling& tiling, const LayerPlan* plan, const PlanAddr* addr, hipStream_t st,
                     Profile* prof, int gemm_slot, int copy_slot, int* kernel_id, bool copy_done, void* scratch, size_t scratch_bytes,
                     const void* w_packed, const TileDev* dev_tiles, int dev_capacity, const int* dev_count, long dev_hint,
                     const int32_t* in_origin, const int32_t* out_origin, int origin_stride, int c_frame, ConvAdd* add,
                     const uint16_t* dev_umask, ConvBatch* batch) {
    const WindowGeom wg = window_geom(l);
    const int Hout = (Hin + 2 * wg.ph - wg.eh) / l.s + 1, Wout = (Win + 2 * wg.pw - wg.ew) / l.s + 1;
    ConvLaunch c;
    c.kernel_id = kernel_id;
    if (kernel_id) *kernel_id = -1;
    c.in = in; c.w = w; c.w_packed = w_packed; c.bias = bias; c.out = out;
    c.n_streams = n_streams; c.Hin = Hin; c.Win = Win; c.Cin = l.cin;
    c.Hout = Hout; c.Wout = Wout; c.Cout = l.cout; c.k = l.k; c.s = l.s; c.p = l.p; c.relu = l.relu;
    if (!plain_square(l)) { c.kw = wg.kw; c.pw = wg.pw; c.dil = wg.dil; }
    c.dtype = dtype; c.tiling = tiling; c.c_frame = c_frame; c.add = add;
    c.scratch = scratch; c.scratch_bytes = scratch_bytes;
    c.in_origin = in_origin; c.out_origin = out_origin; c.origin_stride = origin_stride;
    auto launch = [&]() {
        if (!batch) return launch_conv(c, st);
        batch->c[batch->n++] = c;
        return hipSuccess;
    };
    if (dev_tiles) {      // a list the planning kernels built: its length is in device memory, the copies are done
        c.tiles = dev_tiles; c.n_tiles = dev_capacity; c.n_tiles_dev = dev_count; c.n_tiles_hint = dev_hint; c.umask = dev_umask;
        c.rects = nullptr; c.ranges = nullptr;
        Bracket b(prof, gemm_slot, st);
        DC_TRY_HIP(launch());
        return DC_OK;
    }
    if (!plan) {
        c.tiles = nullptr; c.n_tiles = 0; c.rects = nullptr; c.ranges = nullptr;
        Bracket b(prof, gemm_slot, st);
        DC_TRY_HIP(launch());
        return DC_OK;
    }
    int mw = 0, mh = 0;
    for (const RectDev& r : plan->rects) { mw = r.w > mw ? r.w : mw; mh = r.h > mh ? r.h : mh; }
    if (!plan->rects.empty() && !copy_done) {
        Bracket b(prof, copy_slot, st);
        DC_TRY_HIP(launch_shifted_copy(addr->rects, (int)plan->rects.size(), mw, mh, cache_prev, out, Hout, Wout,
                                       l.cout, dtype, st));
    }
    if (plan->n_tiles) {
        Bracket b(prof, gemm_slot, st);
        // (without a reusable pixel the list is every unit in raster order)
        c.tiles = plan->rects.empty() ? nullptr : addr->tiles; c.n_tiles = (int)plan->n_tiles; c.rects = addr->rects; c.ranges = addr->ranges;
        DC_TRY_HIP(launch());
    }
    return DC_OK;
}

}  // namespace dc

using namespace dc;

namespace {

bool rects_disjoint_inside(const dc_rect* r, int n, int W, int H, int dx, int dy) {
    for (int i = 0; i < n; ++i) {
        if (r[i].w <= 0 || r[i].h <= 0 || r[i].x < 0 || r[i].y < 0 || r[i].x + r[i].w > W ||
            r[i].y + r[i].h > H)
            return false;
        if (r[i].x + dx < 0 || r[i].y + dy < 0 || r[i].x + dx + r[i].w > W || r[i].y + dy + r[i].h > H)
            return false;
        for (int j = 0; j < i; ++j) {
            bool apart = r[i].x + r[i].w <= r[j].x || r[j].x + r[j].w <= r[i].x ||
                         r[i].y + r[i].h <= r[j].y || r[j].y + r[j].h <= r[i].y;
            if (!apart) return false;
        }
    }
    return true;
}

int check_conv_layer(const dc_layer* l) {
    if (l->type != DC_CONV) return DC_ERR_INVALID_ARG;
    const WindowGeom g = window_geom(*l);
    if (g.kh < 1 || g.kw < 1 || l->s < 1 || g.ph < 0 || g.pw < 0 || g.ph >= g.eh || g.pw >= g.ew || l->cin < 1 || l->cout < 1)
        return DC_ERR_INVALID_ARG;
    if (l->relu < 0 || l->relu > 2 || l->k2 < 0 || l->dil < 0 || l->dil > 64 || g.kh > 64 || g.kw > 64) return DC_ERR_INVALID_ARG;
    return DC_OK;
}

// ---- scratch of the entry point that allocates nothing ----
// Device memory that belongs to the library for the life of the process (one copy per GPU the library is loaded
// on): the plan of one conv layer (rectangles, unit masks, counts, unit list) and the partial sums of a split K.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
constexpr size_t kStaticPlanBytes = (size_t)6 << 20;      // the plan's share; the rest takes partial sums
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices] = {};           // device address of `scratch` on each GPU, asked once

// Address of this GPU's copy of the array (the array's name is not an address host code may use).
int static_scratch(unsigned char** ptr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return DC_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return DC_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> guard(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DC_ERR_HIP;
        g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return DC_OK;
}

}  // namespace

extern "C" {

const char* dc_status_string(int32_t s) {
    switch (s) {
        case DC_OK: return "ok";
        case DC_ERR_INVALID_ARG: return "invalid argument";
        case DC_ERR_NULL_PTR: return "null pointer";
        case DC_ERR_BAD_SHAPE: return "inconsistent shapes";
        case DC_ERR_UNSUPPORTED: return "unsupported configuration";
        case DC_ERR_WORKSPACE: return "workspace too small";
        case DC_ERR_CAPACITY: return "list capacity exceeded";
        case DC_ERR_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

int32_t dc_profile_create(int32_t n_slots, void** profile) {
    if (!profile) return DC_ERR_NULL_PTR;
    if (n_slots < 1 || n_slots > (1 << 20)) return DC_ERR_INVALID_ARG;
    Profile* p = new (std::nothrow) Profile();
    if (!p) return DC_ERR_WORKSPACE;
    p->ev.resize(2 * (size_t)n_slots, nullptr);
    p->used.assign(n_slots, 0);
    for (size_t i = 0; i < p->ev.size(); ++i)
        if (hipEventCreate(&p->ev[i]) != hipSuccess) {
            for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(p->ev[j]);
            delete p;
            return DC_ERR_HIP;
        }
    *profile = p;
    return DC_OK;
}

int32_t dc_profile_destroy(void* profile) {
    if (!profile) return DC_ERR_NULL_PTR;
    Profile* p = static_cast<Profile*>(profile);
    for (hipEvent_t e : p->ev) (void)hipEventDestroy(e);
    delete p;
    return DC_OK;
}

int32_t dc_profile_reset(void* profile) {
    if (!profile) return DC_ERR_NULL_PTR;
    Profile* p = static_cast<Profile*>(profile);
    std::fill(p->used.begin(), p->used.end(), 0);
    return DC_OK;
}

int32_t dc_profile_elapsed_ms(void* profile, int32_t slot, float* ms) {
    if (!profile || !ms) return DC_ERR_NULL_PTR;
    Profile* p = static_cast<Profile*>(profile);
    if (slot < 0 || (size_t)slot >= p->used.size() || !p->used[slot]) return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(hipEventElapsedTime(ms, p->ev[2 * slot], p->ev[2 * slot + 1]));
    return DC_OK;
}

int32_t dc_probe_mfma_rate(int32_t lds_reads, void* scratch_dev, size_t scratch_bytes, double* tflops, void* stream) {
    if (!scratch_dev || !tflops) return DC_ERR_NULL_PTR;
    if (scratch_bytes < ((size_t)4 << 20)) return DC_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(scratch_dev) % 16) return DC_ERR_INVALID_ARG;
    const int wgs = 256, steps = 1024, launches = 30;       // about 0.3 ms per launch
    float ms = 0.f;
    DC_TRY_HIP(probe_mfma_rate(lds_reads != 0, scratch_dev, wgs, steps, launches, &ms, as_stream(stream)));
    if (!(ms > 0.f)) return DC_ERR_HIP;
    *tflops = (double)wgs * 8 * steps * 16 * 16384.0 / (ms * 1e-3) / 1e12;
    return DC_OK;
}

int32_t dc_conv_tuning(int32_t arrangement, int32_t units_per_workgroup, int32_t k_split, int32_t chunk_index) {
    if (arrangement > 6 || units_per_workgroup > 18 || chunk_index > 1) return DC_ERR_INVALID_ARG;
    conv_set_tuning(arrangement, units_per_workgroup, k_split, chunk_index);
    return DC_OK;
}

int32_t dc_conv_kernel_name(int32_t kernel_id, char* buf, size_t n) {
    if (!buf) return DC_ERR_NULL_PTR;
    if (n < 2 || kernel_id < 0 || kernel_id == 131 || (kernel_id > 131 && !conv_kernel_built(kernel_id))) return DC_ERR_INVALID_ARG;
    conv_kernel_name(kernel_id, buf, n);
    return DC_OK;
}

int32_t dc_conv_tile_shape(const dc_layer* layer, int32_t n_streams, int32_t Hin, int32_t Win, int32_t dtype,
                           int32_t* th, int32_t* tw, int32_t* nt, int32_t* cfg) {
    if (!layer || !th || !tw || !nt || !cfg) return DC_ERR_NULL_PTR;
    int rc = check_conv_layer(layer);
    if (rc) return rc;
    if (n_streams < 1 || Hin < 1 || Win < 1) return DC_ERR_INVALID_ARG;
    const WindowGeom lg = window_geom(*layer);
    if (Hin + 2 * lg.ph < lg.eh || Win + 2 * lg.pw < lg.ew) return DC_ERR_BAD_SHAPE;
    const int Hout = (Hin + 2 * lg.ph - lg.eh) / layer->s + 1, Wout = (Win + 2 * lg.pw - lg.ew) / layer->s + 1;
    ConvTiling t = pick_tiling(*layer, Hout, Wout, n_streams, dtype);
    *th = t.th; *tw = t.tw; *nt = t.nt; *cfg = t.cfg;
    return DC_OK;
}

static int match_exhaustive(const uint8_t* cur, const uint8_t* prev, int32_t n_streams, int32_t H, int32_t W, int32_t C,
                     int32_t block, int32_t radius, int32_t k_skip, uint32_t max_block_ssd, int16_t* mv,
                     uint32_t* best_ssd, int32_t* global_mv, int32_t* n_pass, uint8_t* block_mask, void* stream) {
    if (!cur || !prev || !mv || !best_ssd || !global_mv || !n_pass || !block_mask) return DC_ERR_NULL_PTR;
    if (n_streams < 1 || n_streams > 65535 || H < 1 || W < 1 || C < 1 || block < 1 || radius < 0 || k_skip < 1)
        return DC_ERR_INVALID_ARG;
    if (block > H || block > W) return DC_ERR_BAD_SHAPE;
    if (radius > 127 || block * C > 256) return DC_ERR_UNSUPPORTED;
    const long rows = block + 2 * radius;
    if (rows * (rows * C + 16) > 60 * 1024) return DC_ERR_UNSUPPORTED;
    // 32-bit sums: B*B*C*255^2 must fit
    if ((double)block * block * C * 65025.0 * 2.0 > 4.0e9) return DC_ERR_UNSUPPORTED;
    DC_TRY_HIP(launch_match(cur, prev, n_streams, H, W, C, block, radius, k_skip, max_block_ssd, mv, best_ssd, global_mv,
                            n_pass, block_mask, as_stream(stream)));
    return DC_OK;
}

int32_t dc_match_blocks(const uint8_t* cur, const uint8_t* prev, int32_t n_streams, int32_t H, int32_t W,
                        int32_t C, int32_t block, int32_t radius, uint32_t max_block_ssd, int16_t* mv,
                        uint32_t* best_ssd, int32_t* global_mv, int32_t* n_pass, uint8_t* block_mask,
                        void* stream) {
    return match_exhaustive(cur, prev, n_streams, H, W, C, block, radius, 1, max_block_ssd, mv, best_ssd, global_mv,
                            n_pass, block_mask, stream);
}

int32_t dc_match_blocks_opt(const uint8_t* cur, const uint8_t* prev, int32_t n_streams, int32_t H, int32_t W,
                            int32_t C, int32_t block, int32_t radius, const dc_match_options* options,
                            uint32_t max_block_ssd, int16_t* mv, uint32_t* best_ssd, int32_t* global_mv,
                            int32_t* n_pass, uint8_t* block_mask, void* stream) {
    const int method = options ? options->method : DC_MATCH_EXHAUSTIVE, k = options ? options->k_skip : 1;
    if (method == DC_MATCH_DIAMOND)
        return dc_match_blocks_ds(cur, prev, n_streams, H, W, C, block, radius, k, max_block_ssd, mv, best_ssd, global_mv,
                                  n_pass, block_mask, stream);
    if (method != DC_MATCH_EXHAUSTIVE) return DC_ERR_INVALID_ARG;
    return match_exhaustive(cur, prev, n_streams, H, W, C, block, radius, k, max_block_ssd, mv, best_ssd, global_mv,
                            n_pass, block_mask, stream);
}

int32_t dc_match_blocks_ds(const uint8_t* cur, const uint8_t* prev, int32_t n_streams, int32_t H, int32_t W,
                           int32_t C, int32_t block, int32_t radius, int32_t k_skip, uint32_t max_block_ssd,
                           int16_t* mv, uint32_t* best_ssd, int32_t* global_mv, int32_t* n_pass, uint8_t* block_mask,
                           void* stream) {
    if (!cur || !prev || !mv || !best_ssd || !global_mv || !n_pass || !block_mask) return DC_ERR_NULL_PTR;
    if (n_streams < 1 || n_streams > 65535 || H < 1 || W < 1 || C < 1 || block < 1 || radius < 0 || k_skip < 1)
        return DC_ERR_INVALID_ARG;
    if (block > H || block > W) return DC_ERR_BAD_SHAPE;
    if (radius > 16383) return DC_ERR_UNSUPPORTED;                                   // vectors are int16
    if ((double)block * block * C * 65025.0 * 2.0 > 4.0e9) return DC_ERR_UNSUPPORTED;   // 32-bit sums
    if ((double)block * W * C >= 2147483648.0) return DC_ERR_UNSUPPORTED;             // 32-bit offsets inside a block
    if ((double)block * block * block * C * C >= 4294967296.0) return DC_ERR_UNSUPPORTED;   // row index by multiplication
    DC_TRY_HIP(launch_match_diamond(cur, prev, n_streams, H, W, C, block, radius, k_skip, max_block_ssd, mv, best_ssd,
                                    global_mv, n_pass, block_mask, as_stream(stream)));
    return DC_OK;
}

int32_t dc_propagate_regions(const dc_layer* layers, int32_t n_layers, int32_t H, int32_t W, int32_t block,
                             const uint8_t* block_mask, int32_t gh, int32_t gw, int32_t mx, int32_t my,
                             dc_regions* regions) {
    return dc_propagate_regions_opt(layers, n_layers, H, W, block, block_mask, gh, gw, mx, my, 0, regions);
}

int32_t dc_propagate_regions_opt(const dc_layer* layers, int32_t n_layers, int32_t H, int32_t W, int32_t block,
                                 const uint8_t* block_mask, int32_t gh, int32_t gw, int32_t mx, int32_t my,
                                 int32_t extend_borders, dc_regions* regions) {
    if (!layers || !block_mask || !regions) return DC_ERR_NULL_PTR;
    if (n_layers < 0 || H < 1 || W < 1 || block < 1 || gh < 0 || gw < 0) return DC_ERR_INVALID_ARG;
    if (gh != H / block || gw != W / block) return DC_ERR_BAD_SHAPE;
    int rc = validate_layers(layers, n_layers, H, W, n_layers ? layers[0].cin : 1, nullptr, nullptr, nullptr);
    if (rc != DC_OK) return rc;
    for (int t = 0; t <= n_layers; ++t)
        if (regions[t].capacity < 0 || (regions[t].capacity > 0 && !regions[t].rects)) return DC_ERR_NULL_PTR;
    std::vector<dc_rect> rects0;
    std::vector<TensorRegions> out;
    try {
        merge_blocks(block_mask, gh, gw, block, rects0);
        rc = propagate(layers, n_layers, H, W, rects0, mx, my, out, extend_borders != 0);
    } catch (const std::bad_alloc&) {
        return DC_ERR_WORKSPACE;
    }
    if (rc != DC_OK) return rc;
    int status = DC_OK;
    for (int t = 0; t <= n_layers; ++t) {
        dc_regions& r = regions[t];
        r.n = (int)out[t].rects.size();
        r.dx = out[t].dx; r.dy = out[t].dy; r.cum_stride = out[t].cum_stride; r.h = out[t].h; r.w = out[t].w;
        int keep = r.n < r.capacity ? r.n : r.capacity;
        if (keep) std::memcpy(r.rects, out[t].rects.data(), keep * sizeof(dc_rect));
        if (r.n > r.capacity) status = DC_ERR_CAPACITY;
    }
    return status;
}

int32_t dc_conv_workspace_bytes(const dc_layer* layer, int32_t n_streams, int32_t Hin, int32_t Win,
                                int32_t max_rects, size_t* dev_bytes, size_t* host_bytes) {
    if (!layer || !dev_bytes || !host_bytes) return DC_ERR_NULL_PTR;
    int rc = check_conv_layer(layer);
    if (rc) return rc;
    if (n_streams < 1 || Hin < 1 || Win < 1 || max_rects < 0) return DC_ERR_INVALID_ARG;
    const WindowGeom lg = window_geom(*layer);
    if (Hin + 2 * lg.ph < lg.eh || Win + 2 * lg.pw < lg.ew) return DC_ERR_BAD_SHAPE;
    const int Hout = (Hin + 2 * lg.ph - lg.eh) / layer->s + 1, Wout = (Win + 2 * lg.pw - lg.ew) / layer->s + 1;
    size_t worst = 0;
    for (int dtype = 0; dtype < 2; ++dtype) {
        size_t b = plan_bytes(n_streams, Hout, Wout, pick_tiling(*layer, Hout, Wout, n_streams, dtype), max_rects);
        worst = b > worst ? b : worst;
    }
    *dev_bytes = align_up(worst, 256) + kConvScratchBytes;   // plan + room for partial sums of a split K
    *host_bytes = worst;
    return DC_OK;
}

int32_t dc_packed_weights_bytes(const dc_layer* layer, int32_t dtype, size_t* bytes) {
    if (!layer || !bytes) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    int rc = check_conv_layer(layer);
    if (rc) return rc;
    *bytes = plain_square(*layer) ? packed_weights_bytes(layer->k, layer->s, layer->cin, layer->cout, dtype) : 0;
    return DC_OK;
}

int32_t dc_pack_conv_weights(const dc_layer* layer, const void* weights, int32_t dtype, void* packed, void* stream) {
    if (!layer || !weights || !packed) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    int rc = check_conv_layer(layer);
    if (rc) return rc;
    if (!plain_square(*layer) || !packed_weights_bytes(layer->k, layer->s, layer->cin, layer->cout, dtype)) return DC_ERR_BAD_SHAPE;
    if (reinterpret_cast<uintptr_t>(weights) % 16 || reinterpret_cast<uintptr_t>(packed) % 16 || weights == packed)
        return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(launch_pack_weights(weights, packed, layer->cin, layer->cout, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_cached_conv_layer(const dc_layer* layer, const void* in, const void* weights, const void* packed_weights,
                             const float* bias, const void* cache_prev, void* out, int32_t n_streams, int32_t Hin, int32_t Win,
                             const dc_regions* regions, int32_t dtype, void* ws_dev, size_t ws_dev_bytes,
                             void* ws_host, size_t ws_host_bytes, void* stream) {
    if (!layer || !in || !weights || !out) return DC_ERR_NULL_PTR;
    int rc = check_conv_layer(layer);
    if (rc) return rc;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || Hin < 1 || Win < 1) return DC_ERR_INVALID_ARG;
    const WindowGeom lg = window_geom(*layer);
    if (Hin + 2 * lg.ph < lg.eh || Win + 2 * lg.pw < lg.ew) return DC_ERR_BAD_SHAPE;
    const int Hout = (Hin + 2 * lg.ph - lg.eh) / layer->s + 1, Wout = (Win + 2 * lg.pw - lg.ew) / layer->s + 1;
    const ConvTiling tiling = pick_tiling(*layer, Hout, Wout, n_streams, dtype);
    hipStream_t st = as_stream(stream);
    if (!regions || !cache_prev)
        return run_conv_planned(*layer, in, weights, bias, nullptr, out, n_streams, Hin, Win, dtype, tiling, nullptr,
                                nullptr, st, nullptr, -1, -1, nullptr, false, ws_dev, ws_dev ? ws_dev_bytes : 0, packed_weights);
    if (out == cache_prev) return DC_ERR_INVALID_ARG;
    int max_rects = 0;
    for (int s = 0; s < n_streams; ++s) {
        if (regions[s].n < 0 || (regions[s].n > 0 && !regions[s].rects)) return DC_ERR_NULL_PTR;
        if (!rects_disjoint_inside(regions[s].rects, regions[s].n, Wout, Hout, regions[s].dx, regions[s].dy))
            return DC_ERR_BAD_SHAPE;
        max_rects = regions[s].n > max_rects ? regions[s].n : max_rects;
    }
    size_t need = plan_bytes(n_streams, Hout, Wout, tiling, max_rects);
    if (!ws_dev || !ws_host) return DC_ERR_NULL_PTR;
    if (ws_dev_bytes < need || ws_host_bytes < need) return DC_ERR_WORKSPACE;
    LayerPlan plan;
    try {
        for (int s = 0; s < n_streams; ++s)
            plan_stream(regions[s].rects, regions[s].n, regions[s].dx, regions[s].dy, s, Hout, Wout, tiling.th,
                        tiling.tw, plan);
    } catch (const std::bad_alloc&) {
        return DC_ERR_WORKSPACE;
    }
    plan.n_tiles = plan.tiles.size();
    PlanAddr addr = pack_plan(plan, static_cast<unsigned char*>(ws_host), static_cast<unsigned char*>(ws_dev));
    const size_t whole = align_up(addr.bytes, 16);         // (the workspaces are whole vectors unless a caller's is not)
    bool copied = false;
    DC_TRY_HIP(upload_and_copy(plan, ws_dev, ws_host, whole <= ws_dev_bytes && whole <= ws_host_bytes ? whole : addr.bytes, cache_prev, out,
                               Hout, Wout, (size_t)layer->cout * dtype_size(dtype), &copied, st));
    // whatever the workspace holds beyond the plan serves as scratch for partial sums
    const size_t plan_end = align_up(addr.bytes, 256);
    unsigned char* scratch = plan_end < ws_dev_bytes ? static_cast<unsigned char*>(ws_dev) + plan_end : nullptr;
    return run_conv_planned(*layer, in, weights, bias, cache_prev, out, n_streams, Hin, Win, dtype, tiling, &plan,
                            &addr, st, nullptr, -1, -1, nullptr, copied, scratch, scratch ? ws_dev_bytes - plan_end : 0,
                            packed_weights);
}

int32_t dc_cached_conv_layer_noalloc(const dc_layer* layer, const void* in, const void* weights, const void* packed_weights,
                                     const float* bias, const void* cache_prev, void* out, int32_t n_streams, int32_t Hin,
                                     int32_t Win, const dc_regions* regions, int32_t dtype, void* stream) {
    if (!layer || !in || !weights || !out) return DC_ERR_NULL_PTR;
    int rc = check_conv_layer(layer);
    if (rc) return rc;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || Hin < 1 || Win < 1) return DC_ERR_INVALID_ARG;
    const WindowGeom lg = window_geom(*layer);
    if (Hin + 2 * lg.ph < lg.eh || Win + 2 * lg.pw < lg.ew) return DC_ERR_BAD_SHAPE;
    const int Hout = (Hin + 2 * lg.ph - lg.eh) / layer->s + 1, Wout = (Win + 2 * lg.pw - lg.ew) / layer->s + 1;
    const ConvTiling tiling = pick_tiling(*layer, Hout, Wout, n_streams, dtype);
    hipStream_t st = as_stream(stream);
    const bool cached = regions && cache_prev;
    if (cached && out == cache_prev) return DC_ERR_INVALID_ARG;
    // sizes first: the plan of the layer must fit the library's scratch, the rectangles the kernel arguments
    PlanConvDev cv{};
    cv.tensor = 0; cv.Hout = Hout; cv.Wout = Wout; cv.units_x = (Wout + 3) / 4; cv.units_y = (Hout + 3) / 4;
    const size_t units = (size_t)cv.units_x * cv.units_y;
    cv.n_chunks = (int)((units + kPlanChunk - 1) / kPlanChunk);
    PlanArgRects args{};
    int cap = 1;
    size_t off = 0;
    size_t off_rects = 0, off_nrect = 0, off_dxy = 0, off_info = 0, off_nunits = 0, off_stats = 0, off_convs = 0;
    if (cached) {
        if (n_streams > kArgMaxStreams) return DC_ERR_CAPACITY;
        int total = 0;
        for (int s = 0; s < n_streams; ++s) {
            if (regions[s].n < 0 || (regions[s].n > 0 && !regions[s].rects)) return DC_ERR_NULL_PTR;
            if (!rects_disjoint_inside(regions[s].rects, regions[s].n, Wout, Hout, regions[s].dx, regions[s].dy))
                return DC_ERR_BAD_SHAPE;
            if (total + regions[s].n > kArgMaxRects) return DC_ERR_CAPACITY;
            args.first[s] = total;
            for (int j = 0; j < regions[s].n; ++j) args.r[total + j] = regions[s].rects[j];
            total += regions[s].n;
            args.dxy[s][0] = regions[s].dx; args.dxy[s][1] = regions[s].dy;
            cap = regions[s].n > cap ? regions[s].n : cap;
        }
        for (int s = n_streams; s <= kArgMaxStreams; ++s) args.first[s] = total;
        off_rects = off; off += align_up((size_t)n_streams * cap * sizeof(dc_rect), 256);
        off_nrect = off; off += align_up((size_t)n_streams * sizeof(int32_t), 256);
        off_dxy = off; off += align_up((size_t)n_streams * 2 * sizeof(int32_t), 256);
        off_info = off; off += align_up((size_t)n_streams * 2 * sizeof(int32_t), 256);
        off_nunits = off; off += 256;
        off_stats = off; off += 256;
        off_convs = off; off += 256;
        cv.umask_off = (int64_t)off; off += align_up((size_t)n_streams * units * sizeof(uint16_t), 256);
        cv.count_off = (int64_t)off; off += align_up((size_t)n_streams * cv.n_chunks * 2 * sizeof(int32_t), 256);
        cv.list_off = (int64_t)off; off += align_up((size_t)n_streams * units * sizeof(TileDev), 256);
        if (off > kStaticPlanBytes || (size_t)n_streams * units > 0x7fffffffull) return DC_ERR_WORKSPACE;
    }
    unsigned char* base = nullptr;
    rc = static_scratch(&base);
    if (rc) return rc;
    unsigned char* const partial = base + kStaticPlanBytes;
    const size_t partial_bytes = kStaticScratchBytes - kStaticPlanBytes;
    if (!cached)
        return run_conv_planned(*layer, in, weights, bias, nullptr, out, n_streams, Hin, Win, dtype, tiling, nullptr, nullptr,
                                st, nullptr, -1, -1, nullptr, false, partial, partial_bytes, packed_weights);
    PlanDev pd{};
    pd.layers = nullptr; pd.tensors = nullptr;
    pd.convs = reinterpret_cast<const PlanConvDev*>(base + off_convs);
    pd.n_layers = 0; pd.n_convs = 1; pd.n_streams = n_streams; pd.cap = cap;
    pd.rects = reinterpret_cast<dc_rect*>(base + off_rects);
    pd.nrect = reinterpret_cast<int32_t*>(base + off_nrect);
    pd.dxy = reinterpret_cast<int32_t*>(base + off_dxy);
    pd.stream_info = reinterpret_cast<int32_t*>(base + off_info);
    pd.n_units = reinterpret_cast<int32_t*>(base + off_nunits);
    pd.stats = base + off_stats;
    pd.area = base;
    DC_TRY_HIP(launch_plan_from_args(pd, cv, args, st));
    const size_t px_bytes = (size_t)layer->cout * dtype_size(dtype);
    const bool vec16 = px_bytes % 16 == 0 && reinterpret_cast<uintptr_t>(cache_prev) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0;
    const int vb = vec16 ? 16 : (int)dtype_size(dtype);
    const CopyUnitsLayer cl{cache_prev, out, reinterpret_cast<const uint16_t*>(base + cv.umask_off), 0, Hout, Wout,
                            cv.units_x, cv.units_y, (int32_t)(px_bytes / vb), 0, 0};
    DC_TRY_HIP(launch_shifted_copy_units(&cl, 1, pd.dxy, 1, n_streams, vb, st));
    return run_conv_planned(*layer, in, weights, bias, cache_prev, out, n_streams, Hin, Win, dtype, tiling, nullptr, nullptr, st,
                            nullptr, -1, -1, nullptr, true, partial, partial_bytes, packed_weights,
                            reinterpret_cast<const TileDev*>(base + cv.list_off), (int)((size_t)n_streams * units), pd.n_units, -1);
}

int32_t dc_frame_to_tensor(const uint8_t* frames, void* out, size_t n_pixels, int32_t c_frame, int32_t c_tensor,
                           int32_t dtype, void* stream) {
    if (!frames || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (c_frame < 1 || c_tensor < c_frame) return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(launch_frame_to_tensor(frames, out, n_pixels, c_frame, c_tensor, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_maxpool_layer(const void* in, void* out, int32_t n_streams, int32_t Hin, int32_t Win, int32_t C,
                         int32_t k, int32_t s, int32_t p, int32_t dtype, void* stream) {
    if (!in || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || Hin < 1 || Win < 1 || C < 1 || k < 1 || s < 1 || p < 0 || p >= k) return DC_ERR_INVALID_ARG;
    if (Hin + 2 * p < k || Win + 2 * p < k) return DC_ERR_BAD_SHAPE;
    DC_TRY_HIP(launch_maxpool(in, out, n_streams, Hin, Win, C, k, s, p, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_torus_read(const void* in, void* out, const int32_t* origins_dev, int32_t origin_stride, int32_t n_streams,
                      int32_t H, int32_t W, int32_t C, int32_t dtype, void* stream) {
    if (!in || !out) return DC_ERR_NULL_PTR;
    if (in == out) return DC_ERR_INVALID_ARG;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || H < 1 || W < 1 || C < 1 || (origins_dev && origin_stride < 2)) return DC_ERR_INVALID_ARG;
    if ((size_t)n_streams * H > 65535) return DC_ERR_UNSUPPORTED;
    DC_TRY_HIP(launch_torus_read(in, out, n_streams, H, W, (size_t)C * dtype_size(dtype), origins_dev, origin_stride, as_stream(stream)));
    return DC_OK;
}

int32_t dc_add_layer(const void* a, const void* b, void* out, size_t n, int32_t relu, int32_t dtype, void* stream) {
    if (!a || !b || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(launch_add(a, b, out, n, relu, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_avgpool_layer(const void* in, void* out, int32_t n_streams, int32_t Hin, int32_t Win, int32_t C,
                         int32_t k, int32_t s, int32_t p, int32_t dtype, void* stream) {
    if (!in || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || Hin < 1 || Win < 1 || C < 1 || k < 1 || s < 1 || p < 0 || p >= k) return DC_ERR_INVALID_ARG;
    if (Hin + 2 * p < k || Win + 2 * p < k) return DC_ERR_BAD_SHAPE;
    DC_TRY_HIP(launch_avgpool(in, out, n_streams, Hin, Win, C, k, s, p, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_lrn_layer(const void* in, void* out, int32_t n_streams, int32_t H, int32_t W, int32_t C, int32_t size,
                     int32_t within, float alpha, float beta, float kappa, int32_t dtype, void* stream) {
    if (!in || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || H < 1 || W < 1 || C < 1 || size < 1 || size % 2 == 0) return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(launch_lrn(in, out, n_streams, H, W, C, size, within != 0, alpha, beta, kappa, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_concat_layer(const void* const* ins, const int32_t* channels, int32_t n_in, void* out, size_t n_pixels,
                        int32_t dtype, void* stream) {
    if (!ins || !channels || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_in < 2 || n_in > 4) return DC_ERR_INVALID_ARG;
    int chans[4];
    for (int j = 0; j < n_in; ++j) {
        if (!ins[j]) return DC_ERR_NULL_PTR;
        if (channels[j] < 1) return DC_ERR_INVALID_ARG;
        if (ins[j] == out) return DC_ERR_INVALID_ARG;
        chans[j] = channels[j];
    }
    DC_TRY_HIP(launch_concat(ins, chans, n_in, out, n_pixels, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_fc_layer(const void* in, const void* weights, const float* bias, void* out, int32_t n_streams, size_t K,
                    int32_t cout, int32_t relu, int32_t dtype, void* stream) {
    if (!in || !weights || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_streams < 1 || K < 1 || cout < 1) return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(launch_fc(in, weights, bias, out, n_streams, K, cout, relu, dtype, as_stream(stream)));
    return DC_OK;
}

int32_t dc_softmax_layer(const void* in, void* out, size_t n_pixels, int32_t C, int32_t dtype, void* stream) {
    if (!in || !out) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (C < 1) return DC_ERR_INVALID_ARG;
    DC_TRY_HIP(launch_softmax(in, out, n_pixels, C, dtype, as_stream(stream)));
    return DC_OK;
}

}  // extern "C"
