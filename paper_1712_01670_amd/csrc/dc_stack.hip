// dc_run_stack: one frame of every stream through the whole path (Section 3 workflow), and what belongs to it: the
// overlap handle and its pipeline, the layout of the workspaces, the planning of a frame on the host, the order of the
// launches.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>

#include "dc_internal.h"
#include "dc_replay.h"

using namespace dc;

namespace {

// Channel count of tensor 0: the cin of the layers that read it (they must agree); it may exceed the
// frame's channel count, the extra channels are zero.
int input_channels(const dc_layer* L, int n_layers, int c_frame) {
    int c = -1;
    for (int i = 0; i < n_layers; ++i) {
        if (L[i].type == DC_CONCAT) {             // its cin is the sum of its producers' channels
            int ids[4];
            const int m = concat_inputs(L[i], ids);
            for (int j = 0; j < m; ++j)
                if (ids[j] == 0) return -1;       // a concat reads layer outputs only
            continue;
        }
        if (L[i].in0 == 0 || (L[i].type == DC_ADD && L[i].in1 == 0)) {
            if (c >= 0 && L[i].cin != c) return -1;
            c = L[i].cin;
        }
    }
    return c < 0 ? c_frame : c;
}

// Waits for an event by polling: the host thread is needed again within tens of microseconds, which a
// blocking wait's wake-up latency would double.  After 2 ms of polling it blocks instead.
hipError_t spin_wait(hipEvent_t e) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0;; ++i) {
        const hipError_t q = hipEventQuery(e);
        if (q != hipErrorNotReady) return q;
        if ((i & 63) == 63 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(2))
            return hipEventSynchronize(e);
    }
}

// ---- planning on the GPU: layout of the tables and of one frame's plan in the device workspace ----
constexpr size_t kDevHostRegion = 64 * 1024;    // tail of the host workspace: header, two counter slots, table staging
constexpr size_t kDevHostSlot = 4096;
constexpr int kPlanMaxConvs = 128;
constexpr uint64_t kDevHostMagic = 0x6463706c616e3031ull;
struct DevHostConv { int32_t layer, cout_bytes; int64_t mac_px, px_total; };
struct DevHostHeader {                          // host-only bookkeeping of the workspace pair
    uint64_t magic, signature;
    const void* ws_dev;
    int32_t n_layers, n_convs, last_slot, n_blocks;
    int64_t macs_full;
    int32_t origin_area;                        // torus frames: the plan area that holds the previous frame's origins (-1: none)
    int32_t torus;                              // 1: the last frame planned here copied nothing
    DevHostConv conv[kPlanMaxConvs];
};
static_assert(sizeof(DevHostHeader) <= kDevHostSlot, "header fits its slot");
static_assert(sizeof(PlanStatsHead) + kPlanMaxConvs * sizeof(PlanStatsConv) <= kDevHostSlot, "counters fit their slot");

struct DevPlanLayout {
    std::vector<PlanLayerDev> layers;
    std::vector<PlanTensorDev> tensors;
    std::vector<PlanConvDev> convs;
    std::vector<PlanOpDev> ops;                 // exact reuse maps
    std::vector<int> conv_layer;                // layer index of every conv
    size_t table_bytes = 0, off_tensors = 0, off_convs = 0, off_ops = 0;
    size_t frame_bytes = 0, off_nrect = 0, off_dxy = 0, off_origin = 0, off_info = 0, off_nunits = 0, off_stats = 0, off_area = 0;
    size_t off_bitmaps = 0;
    int64_t bm_words = 0;                       // words of all bitmaps of one stream (exact reuse maps)
    int cap = 0, max_chunks = 0, n_chunks = 0;
    bool ok = false;
};

// Tables and sizes for n_streams streams of this stack; ok = false if the device kernels cannot take it (the host
// path then plans the frame).
// Layer i is a 1x1 convolution and the next one sums its output with another tensor.
bool sum_behind(const dc_layer* L, int n_layers, int i) {
    if (i + 1 >= n_layers || L[i].type != DC_CONV || L[i].k != 1 || !plain_square(L[i]) || L[i + 1].type != DC_ADD) return false;
    const dc_layer& a = L[i + 1];
    return a.in0 != a.in1 && (a.in0 == i + 1 || a.in1 == i + 1);
}

void device_plan_layout(const dc_layer* L, int n_layers, const std::vector<int>& hs, const std::vector<int>& ws,
                        int n_streams, int max_rects, DevPlanLayout& d, const uint8_t* no_reuse = nullptr) {
    d.ok = false;
    const int nt = n_layers + 1;
    if (nt > kPlanMaxTensors) return;
    d.cap = max_rects < kPlanMaxRects ? max_rects : kPlanMaxRects;
    d.layers.resize(n_layers); d.tensors.resize(nt); d.convs.clear(); d.conv_layer.clear(); d.ops.clear();
    std::vector<int> depth(nt, 0);
    d.tensors[0] = PlanTensorDev{hs[0], ws[0], 1, 0};
    int64_t bm = ((int64_t)hs[0] * ((ws[0] + 31) / 32) + 63) / 64 * 64;          // every bitmap starts on a 256-byte line
    for (int i = 0; i < n_layers; ++i) {
        const dc_layer& l = L[i];
        const WindowGeom wg = window_geom(l);
        d.layers[i] = PlanLayerDev{l.type, l.k, l.s, l.p, l.in0, l.in1, l.in2, l.in3, l.within, wg.kw, wg.pw, wg.dil};
        const bool windowed = l.type == DC_CONV || l.type == DC_MAXPOOL || l.type == DC_AVGPOOL;
        const int cum = d.tensors[l.in0].cum_stride * (windowed ? l.s : 1);
        if (bm > 0x7fffffffll) return;
        d.tensors[i + 1] = PlanTensorDev{hs[i + 1], ws[i + 1], cum, (int32_t)bm};
        if (l.type == DC_ADD && d.tensors[l.in1].cum_stride != d.tensors[l.in0].cum_stride) return;
        if (l.type == DC_CONCAT) {
            int ids[4];
            const int m = concat_inputs(l, ids);
            for (int j = 1; j < m; ++j)
                if (d.tensors[ids[j]].cum_stride != d.tensors[l.in0].cum_stride) return;
        }
        if (l.type == DC_CONV) d.conv_layer.push_back(i);
        // the step that makes the tensor's bitmap, if it differs from the producer's (same size, stride and offset)
        PlanOpDev op{};
        op.src0 = d.tensors[l.in0].bm_off; op.src[0] = op.src[1] = op.src[2] = -1;
        const bool lrn_px = l.type == DC_LRN && l.within != 0;
        depth[i + 1] = depth[l.in0];
        if (l.type == DC_FC || l.type == DC_SOFTMAX) {
            op.kind = kPlanOpZero;
        } else if (l.type == DC_ADD || l.type == DC_CONCAT) {
            int ids[4] = {l.in0, l.in1, -1, -1};
            const int m = l.type == DC_CONCAT ? concat_inputs(l, ids) : 2;
            op.kind = m == 2 ? kPlanOpAnd2 : kPlanOpAnd;
            for (int j = 1; j < m; ++j) {
                op.src[j - 1] = d.tensors[ids[j]].bm_off;
                depth[i + 1] = std::max(depth[i + 1], depth[ids[j]]);
            }
        } else if ((windowed && !(wg.kh == 1 && wg.kw == 1 && l.s == 1 && wg.ph == 0 && wg.pw == 0)) || lrn_px) {
            op.kh = lrn_px ? l.k : wg.kh; op.kw = lrn_px ? l.k : wg.kw; op.s = windowed ? l.s : 1; op.dil = windowed ? wg.dil : 1;
            op.ph = lrn_px ? (l.k - 1) / 2 : wg.ph; op.pw = lrn_px ? (l.k - 1) / 2 : wg.pw;
            const bool words = (op.kw - 1) * op.dil < 32;
            op.kind = op.kh == 3 && op.kw == 3 && op.s == 1 && op.dil == 1 ? kPlanOp3x3
                    : op.kh == 2 && op.kw == 2 && op.s == 2 && op.dil == 1 ? kPlanOp2x2
                    : words && op.s == 1 ? kPlanOpStride1 : words && op.s == 2 ? kPlanOpStride2 : words && op.s <= 8 ? kPlanOpStride8 : kPlanOpSlow;
        } else {
            d.tensors[i + 1].bm_off = d.tensors[l.in0].bm_off;
            continue;
        }
        bm += ((int64_t)hs[i + 1] * ((ws[i + 1] + 31) / 32) + 63) / 64 * 64;
        ++depth[i + 1];
        op.dst = d.tensors[i + 1].bm_off;
        op.h_in = hs[l.in0]; op.w_in = ws[l.in0]; op.wpr_in = (ws[l.in0] + 31) / 32;
        op.h = hs[i + 1]; op.w = ws[i + 1]; op.wpr = (ws[i + 1] + 31) / 32;
        op.words = op.h * op.wpr;
        op.cum_stride = cum;
        op.wpr_magic = (uint32_t)((0x100000000ull + (uint64_t)op.wpr - 1) / (uint64_t)op.wpr);
        op.depth_end = depth[i + 1];                // (sorted by it below)
        d.ops.push_back(op);
    }
    std::stable_sort(d.ops.begin(), d.ops.end(), [](const PlanOpDev& a, const PlanOpDev& b) { return a.depth_end < b.depth_end; });
    for (size_t j = 0; j < d.ops.size(); ++j) d.ops[j].depth_end = j + 1 == d.ops.size() || d.ops[j + 1].depth_end != d.ops[j].depth_end ? 1 : 0;
    for (size_t j = d.ops.size(); j-- > 0;) {           // runs of small steps
        const bool small = d.ops[j].words <= 128;
        const bool goes_on = j + 1 < d.ops.size() && d.ops[j + 1].run_end > 0;
        d.ops[j].run_end = !small ? 0 : goes_on ? d.ops[j + 1].run_end : (int32_t)j + 1;
        if (!small && goes_on) d.ops[j].depth_end = 1;             // a run may go on to greater depths
    }
    if ((int)d.conv_layer.size() > kPlanMaxConvs) return;
    d.off_tensors = align_up((size_t)n_layers * sizeof(PlanLayerDev), 256);
    d.off_convs = d.off_tensors + align_up((size_t)nt * sizeof(PlanTensorDev), 256);
    d.off_ops = d.off_convs + align_up(d.conv_layer.size() * sizeof(PlanConvDev), 256);
    d.table_bytes = d.off_ops + align_up(d.ops.size() * sizeof(PlanOpDev), 256);
    size_t off = align_up((size_t)n_streams * nt * d.cap * sizeof(dc_rect), 256);
    d.off_nrect = off; off += align_up((size_t)n_streams * nt * sizeof(int32_t), 256);
    d.off_dxy = off; off += align_up((size_t)n_streams * nt * 2 * sizeof(int32_t), 256);
    d.off_origin = off; off += align_up((size_t)n_streams * nt * 2 * sizeof(int32_t), 256);
    d.off_info = off; off += align_up((size_t)n_streams * 2 * sizeof(int32_t), 256);
    d.off_nunits = off; off += align_up(d.conv_layer.size() * sizeof(int32_t), 256);
    d.off_stats = off; off += kDevHostSlot;
    d.bm_words = bm;
    d.off_bitmaps = off; off += align_up((size_t)n_streams * (size_t)bm * sizeof(uint32_t), 256);
    d.off_area = off;
    size_t area = 0;
    d.max_chunks = d.n_chunks = 0;
    for (int layer : d.conv_layer) {
        PlanConvDev c{};
        c.tensor = layer + 1; c.Hout = hs[layer + 1]; c.Wout = ws[layer + 1];
        c.no_reuse = no_reuse && no_reuse[layer] ? 1 : 0;
        c.units_x = (c.Wout + 3) / 4; c.units_y = (c.Hout + 3) / 4;
        const size_t units = (size_t)c.units_x * c.units_y;
        c.n_chunks = (int)((units + kPlanChunk - 1) / kPlanChunk);
        d.max_chunks = c.n_chunks > d.max_chunks ? c.n_chunks : d.max_chunks;
        c.chunk_base = d.n_chunks; d.n_chunks += c.n_chunks;
        c.bm_off = d.tensors[layer + 1].bm_off;
        c.list_clean = sum_behind(L, n_layers, layer) ? 1 : 0;
        c.umask_off = (int64_t)area; area += align_up((size_t)n_streams * units * sizeof(uint16_t), 256);
        c.count_off = (int64_t)area; area += align_up((size_t)n_streams * c.n_chunks * 2 * sizeof(int32_t), 256);
        c.list_off = (int64_t)area; area += align_up((size_t)n_streams * units * sizeof(TileDev), 256);
        if (units * (size_t)n_streams > 0x7fffffffull) return;
        d.convs.push_back(c);
    }
    d.frame_bytes = align_up(off + area, 256);
    d.ok = true;
}

uint64_t fnv1a(uint64_t h, const void* p, size_t n) {
    const unsigned char* b = static_cast<const unsigned char*>(p);
    for (size_t i = 0; i < n; ++i) { h ^= b[i]; h *= 0x100000001b3ull; }
    return h;
}

// Planning of one frame for dc_run_stack: per (stream, conv layer) lists built in parallel, merged by offset.
struct FramePlan {
    std::vector<int> conv_layers;          // layer indices
    std::vector<LayerPlan> part;           // [stream][conv layer], storage kept between frames
    std::vector<size_t> tile_off;          // [stream][conv layer]: first tile of the part in the layer's list
    std::vector<unsigned char*> tile_dst;  // [conv layer]: the layer's tile list in the staging buffer
    int n_streams = 0;

    // no_reuse (optional): conv layers that are computed in full (planned as if their lists were empty)
    int classify(const dc_layer* layers, int n_layers, int streams, const std::vector<std::vector<TensorRegions>>& regs,
                 const std::vector<int>& hs, const std::vector<int>& ws, const uint8_t* no_reuse) {
        n_streams = streams;
        conv_layers.clear();
        for (int i = 0; i < n_layers; ++i)
            if (layers[i].type == DC_CONV) conv_layers.push_back(i);
        const int nc = (int)conv_layers.size();
        std::vector<int> ok(streams, 1);
        try {
            if (part.size() < (size_t)streams * nc) part.resize((size_t)streams * nc);
            tile_off.assign((size_t)streams * nc, 0);
            tile_dst.assign(nc, nullptr);
        } catch (const std::bad_alloc&) {
            return DC_ERR_WORKSPACE;
        }
        parallel_for(streams, [&](int s) {
            try {
                for (int c = 0; c < nc; ++c) {
                    const int i = conv_layers[c];
                    LayerPlan& lp = part[(size_t)s * nc + c];
                    lp.rects.clear(); lp.ranges.clear(); lp.tiles.clear(); lp.reused_px = 0;
                    const TensorRegions& g = regs[s][i + 1];
                    plan_stream(g.rects.data(), (no_reuse && no_reuse[i]) ? 0 : (int)g.rects.size(), g.dx, g.dy, s, hs[i + 1], ws[i + 1], 4, 4, lp);
                }
            } catch (const std::bad_alloc&) {
                ok[s] = 0;
            }
        });
        for (int s = 0; s < streams; ++s)
            if (!ok[s]) return DC_ERR_WORKSPACE;
        return DC_OK;
    }
    // Lays layer i out in the staging buffer ([tiles][rects][ranges], as pack_plan), fills the small tables and
    // notes where each stream's tiles go.
    PlanAddr finish_layer(int layer, LayerPlan& plan, unsigned char* host, unsigned char* dev) {
        const int nc = (int)conv_layers.size();
        int c = 0;
        while (conv_layers[c] != layer) ++c;
        size_t n_tiles = 0;
        for (int s = 0; s < n_streams; ++s) {
            LayerPlan& lp = part[(size_t)s * nc + c];
            tile_off[(size_t)s * nc + c] = n_tiles;
            n_tiles += lp.tiles.size();
            RangeDev r{(int)plan.rects.size(), (int)lp.rects.size()};
            plan.rects.insert(plan.rects.end(), lp.rects.begin(), lp.rects.end());
            plan.ranges.push_back(r);
            plan.reused_px += lp.reused_px;
        }
        plan.n_tiles = n_tiles;
        tile_dst[c] = host;
        PlanAddr a = pack_plan(plan, host, dev);        // plan.tiles is empty: copies rects and ranges, sizes from n_tiles
        return a;
    }
    void copy_tiles() {
        const int nc = (int)conv_layers.size();
        parallel_for(n_streams, [&](int s) {
            for (int c = 0; c < nc; ++c) {
                const LayerPlan& lp = part[(size_t)s * nc + c];
                if (!lp.tiles.empty())
                    std::memcpy(tile_dst[c] + tile_off[(size_t)s * nc + c] * sizeof(TileDev), lp.tiles.data(),
                                lp.tiles.size() * sizeof(TileDev));
            }
        });
    }
};
FramePlan g_frame_plan;
std::mutex g_frame_plan_mutex;

}  // namespace

// The launches of one kind of frame recorded as HIP graphs, one per stage, for stacks whose frames are bound by the host
// issuing launches (StackPlan::replay).  A kernel node costs the host 0.3 us where a launch costs 2.5-3.5, but every graph
// costs its stream about 10 us on the GPU, which a frame that is bound by the GPU pays for nothing.  What the kernels' arguments
// depend on is the key; frames of a steady video go round through a handful of keys (buffer sets x plan areas).  The
// first frames of a key are launched one kernel at a time (recording costs about 5 us per kernel), later ones replay.
// The launch shapes in a graph follow the list lengths seen when it was recorded; when those of the video have moved
// away for good the graphs are dropped and recorded again.
struct dc::FrameGraphs {
    std::vector<uint64_t> key;
    uint64_t hash = 0, last_use = 0;
    int uses = 0, off_shape = 0;            // frames of this key so far; consecutive frames whose lists had other lengths
    bool ready = false;
    hipGraphExec_t exec[kMaxStages] = {};
    std::vector<int32_t> kernel_id;         // [layer]
    std::vector<long> hint;                 // [conv]
    void drop() {
        for (hipGraphExec_t& e : exec) {
            if (e) (void)hipGraphExecDestroy(e);
            e = nullptr;
        }
        ready = false;
        uses = off_shape = 0;
    }
    ~FrameGraphs() { drop(); }
};

constexpr int kSiblingReach = 12;            // layers between two that StackCall::run_with may launch together, at most

// ---- what dc_run_stack derives from a stack's description ------------------------------------------------------
// Depends on the layer table, the sizes and the options, not on the frame, its buffers or the weights.  An overlap
// handle keeps the last few (a caller runs one stack, frame after frame); without a handle it is made on every call.
struct dc::StackPlan {
    std::vector<unsigned char> key;
    std::vector<dc_layer> layers;
    std::vector<uint8_t> no_reuse;          // per layer (empty: none flagged)
    int n_streams = 0, H = 0, W = 0, C = 0, c_tensor = 0, dtype = 0;
    bool device_plan = false, exact = false, torus = false, pool_torus = false, cache_other = false, may_in_place = false;
    std::vector<int> hs, ws, cs;            // size of every tensor
    std::vector<int> last_reader;           // [tensor]: last layer that reads it (-1: none)
    std::vector<ConvTiling> tilings;        // [layer]
    std::vector<int> conv_of;               // [layer]: index among the conv layers (-1)
    std::vector<int> sibling;               // [layer]: the next 1x1 convolution of the same tensor with the same stride (-1)
    DevPlanLayout dl;                       // planning on the GPU
    bool dl_fits_host = false;              // its tables fit their place in the host workspace
    std::vector<unsigned char> tables;
    uint64_t signature = 0;
    size_t need_dev = 0, need_host = 0;
    int64_t macs_full = 0, macs_issued_full = 0;
    std::vector<int64_t> issued_full;       // [layer]
    int rc_torus = DC_OK;                   // the stack does not qualify for a torus

    // the cut into stages (see dc_internal.h): stage s is layers first[s] .. first[s + 1] - 1
    int partition = 0, n_stages = 1;
    int first[kMaxStages + 1] = {};
    bool tight[kMaxStages] = {};            // the cut before stage s crosses a tensor with a single buffer
    std::vector<float> layer_us;            // rough time of every layer, and of the matching and planning before them
    float head_us = 0.f;
    float tail_us = 0.f;                    // what the caller queues behind a frame on its own stream, the last stage's
    std::vector<char> single;               // tensors whose buffer is the same for consecutive frames: no cut may cross them
    std::vector<int> crossing;              // tensors that a later stage than their writer's reads
    // The layers' times are rough: the first frames after a cut are timed stage by stage, the times of a stage's layers are
    // scaled to what it took, and the layers are cut again if that promises a shorter longest stage.
    static constexpr int kTimedFrames = 4;
    int recuts_left = 3, timed_frames = 0;
    float timed_us[kMaxStages][kTimedFrames] = {};
    int timed_tails = 0;                    // the caller's work is known behind frames that still ran at the next call
    float timed_tail_us[kTimedFrames] = {};
    std::vector<std::unique_ptr<dc::FrameGraphs>> graphs;
    bool no_graphs = false;                 // recording failed once
    ReplayRule replay;
    std::chrono::steady_clock::time_point left;               // end of the last call
    int stage_of(int layer) const {
        int s = 0;
        while (s + 1 < n_stages && layer >= first[s + 1]) ++s;
        return s;
    }
    int writer_stage(int t) const { return t > 0 ? stage_of(t - 1) : 0; }     // (the frame's conversion heads stage 0)
    bool on_torus(int t) const {
        return torus && t > 0 && (layers[t - 1].type == DC_CONV || (pool_torus && layers[t - 1].type == DC_MAXPOOL));
    }
    bool uses_cache(int i) const { return cache_other && (layers[i].type == DC_MAXPOOL || layers[i].type == DC_ADD); }
    void cut(int max_stages);
    float longest() const {                 // by layer_us
        float most = 0.f;
        for (int s = 0; s < n_stages; ++s) most = std::max(most, stage_us(s));
        return most;
    }
    float stage_us(int s) const {
        float us = (s == 0 && device_plan ? head_us : 0.f) + (s + 1 == n_stages ? tail_us : 0.f);
        for (int i = first[s]; i < first[s + 1]; ++i) us += layer_us[i];
        return us;
    }
    float period(float longest_us, int k) const;      // of a frame in k stages
    void calibrate(int max_stages);
};

namespace {

// The producers of layer i (1 to 4 tensors).
int layer_inputs(const dc_layer& l, int* ids) {
    if (l.type == DC_CONCAT) return concat_inputs(l, ids);
    ids[0] = l.in0;
    if (l.type != DC_ADD) return 1;
    ids[1] = l.in1;
    return 2;
}

// Workspace layout.  Device: [plan areas, one per frame in flight][partial sums of split convolutions, one per stage].
// Host: [mask and motion read back][two staging halves for plans made on the host] and a tail for the planning on the GPU.
size_t scratch_region() { return (size_t)kMaxStages * kConvScratchBytes; }
void workspace_sizes(const dc_layer* layers, int n_layers, int n_streams, int H, int W, int block, int max_rects,
                     const std::vector<int>& hs, const std::vector<int>& ws, const DevPlanLayout& dl, size_t* dev_bytes, size_t* host_bytes) {
    size_t total = 0;
    for (int i = 0; i < n_layers; ++i) {
        if (layers[i].type != DC_CONV) continue;
        size_t worst = 0;
        for (int dtype = 0; dtype < 2; ++dtype) {
            size_t b = plan_bytes(n_streams, hs[i + 1], ws[i + 1], pick_tiling(layers[i], hs[i + 1], ws[i + 1], n_streams, dtype), max_rects);
            worst = b > worst ? b : worst;
        }
        total += worst;
        total += align_up((size_t)n_streams * max_rects * sizeof(RectDev), 256);   // all-layers copy table
    }
    total += align_up((size_t)n_layers * sizeof(CopyLayerDev), 256);
    const size_t nb = (size_t)n_streams * (H / block) * (W / block);
    const size_t match_host = align_up(nb, 256) + align_up((size_t)n_streams * 3 * sizeof(int32_t), 256);
    size_t area = align_up(total, 256);
    if (dl.ok && align_up(dl.table_bytes, 256) + dl.frame_bytes > area) area = align_up(dl.table_bytes, 256) + dl.frame_bytes;
    *dev_bytes = kFramesInFlight * area + scratch_region();
    *host_bytes = align_up(2 * total + match_host, 256) + kDevHostRegion;
}

// Whether the conv outputs of this stack can live on a torus: only layers whose kernels address one may touch them.
int torus_qualifies(const StackPlan& P) {
    const size_t esz = dtype_size(P.dtype);
    auto conv_output = [&](int t) { return t > 0 && P.layers[t - 1].type == DC_CONV; };
    for (size_t i = 0; i < P.layers.size(); ++i) {
        const dc_layer& l = P.layers[i];
        const int t = (int)i + 1;
        if (l.type == DC_CONV) {
            const bool first = l.in0 == 0 && P.cs[0] * esz == 16 && l.cout % 16 == 0 &&
                               ((l.k == 3 && l.s == 1) || (l.k == 7 && l.s == 2) || (l.k == 11 && l.s == 4));
            const bool gemm3 = l.k == 3 && l.s == 1 && l.cout % 64 == 0 && (l.cin * esz) % 64 == 0;
            const bool point = l.k == 1 && l.s == 1 && l.p == 0 && l.cout % 8 == 0 && (l.cin * esz) % 16 == 0;
            if (!plain_square(l) || !(first || gemm3 || point)) return DC_ERR_UNSUPPORTED;
        } else if (l.type == DC_MAXPOOL) {
            if ((conv_output(l.in0) || P.pool_torus) &&
                !(conv_output(l.in0) && l.k == 2 && l.s == 2 && l.p == 0 && (P.cs[l.in0] * esz) % 16 == 0 &&
                  (size_t)P.n_streams * P.hs[t] <= 65535))
                return DC_ERR_UNSUPPORTED;
        } else {
            if (P.pool_torus && l.type == DC_ADD) return DC_ERR_UNSUPPORTED;       // an add layer that uses the cache copies
            int ids[4];
            const int m = layer_inputs(l, ids);
            for (int j = 0; j < m; ++j)
                if (P.on_torus(ids[j])) return DC_ERR_UNSUPPORTED;
        }
    }
    return DC_OK;
}

// Rough time of a layer on its own in microseconds (for the cut into stages only): arithmetic at what the kernels reach
// on large maps, feature maps through memory, and what a launch costs at least.
float layer_cost(const StackPlan& P, int i) {
    const dc_layer& l = P.layers[i];
    const double esz = (double)dtype_size(P.dtype), n = P.n_streams;
    const double in_px = n * P.hs[l.in0] * P.ws[l.in0], out_px = n * P.hs[i + 1] * P.ws[i + 1];
    const double bytes = (in_px * P.cs[l.in0] + out_px * P.cs[i + 1]) * esz;
    double us = 3.0 + bytes / 3.5e6;
    if (l.type == DC_CONV) {
        const WindowGeom g = window_geom(l);
        const double flops = 2.0 * g.kh * g.kw * l.cin * l.cout * out_px;
        // the general kernels reach a quarter of the rate and walk over the taps one stage after another
        const bool gemm = plain_square(l) && ((l.k == 3 && l.s == 1) || l.k == 1);
        us = 5.0 + (gemm ? 0.0 : 0.8 * g.kh * g.kw) + g.kh * g.kw * l.cin * l.cout * esz / 0.8e6 * std::min(1.0, 400.0 / out_px) + std::max(bytes / 3.5e6, flops / ((P.dtype == DC_BF16 ? 0.9e9 : 0.1e9) * (gemm ? 1.0 : 0.25)));
    } else if (l.type == DC_FC) {
        const double row = (double)P.hs[l.in0] * P.ws[l.in0] * P.cs[l.in0] * esz;
        // the weights from memory, or a wavefront's walk along its neuron's row (a whole one for one stream, a sixteenth
        // for several): few neurons on long rows are that chain of loads
        us = 8.0 + std::max(row * l.cout * (1.0 + n / 6.0) / 4e6, n < 2.0 ? row / 1024.0 * 0.35 : row / 2048.0 * (0.85 + 0.035 * n));
    } else if (l.type == DC_LRN) {
        us = 3.0 + bytes / 1e6;
    }
    return (float)us;
}

// Everything but the cut; `rc` of the layer table or of the options.
int make_plan(StackPlan& P, const dc_layer* layers, int n_layers, int n_streams, int H, int W, int C, int dtype, int block,
              int radius, int max_rects, const dc_match_options* o, bool may_in_place) {
    P.n_streams = n_streams; P.H = H; P.W = W; P.C = C; P.dtype = dtype;
    P.c_tensor = input_channels(layers, n_layers, C);
    if (P.c_tensor < C) return DC_ERR_BAD_SHAPE;
    int rc = validate_layers(layers, n_layers, H, W, P.c_tensor, &P.hs, &P.ws, &P.cs);
    if (rc) return rc;
    P.layers.assign(layers, layers + n_layers);
    if (o) {
        P.device_plan = o->device_plan && !may_in_place;
        P.exact = o->exact_masks != 0;
        P.torus = o->torus != 0;
        P.pool_torus = P.torus && o->cache_pool_add;
        P.cache_other = o->cache_pool_add && o->exact_masks;
        if (o->no_reuse) P.no_reuse.assign(o->no_reuse, o->no_reuse + n_layers);
    }
    P.may_in_place = may_in_place;
    device_plan_layout(layers, n_layers, P.hs, P.ws, n_streams, max_rects, P.dl, P.no_reuse.empty() ? nullptr : P.no_reuse.data());
    P.dl_fits_host = P.dl.ok && P.dl.table_bytes <= kDevHostRegion - 3 * kDevHostSlot;
    // Asked for and possible (the kernels hold the blocks of a frame in 64 rows of 64 bits); otherwise the host plans, and the
    // stages are laid out for that: aux is left to the matching, which the host waits for.
    P.device_plan = P.device_plan && P.dl_fits_host && H / block >= 1 && W / block >= 1 && H / block <= 64 && W / block <= 64;
    if (P.dl.ok) {
        P.tables.assign(P.dl.table_bytes, 0);
        std::memcpy(P.tables.data(), P.dl.layers.data(), P.dl.layers.size() * sizeof(PlanLayerDev));
        std::memcpy(P.tables.data() + P.dl.off_tensors, P.dl.tensors.data(), P.dl.tensors.size() * sizeof(PlanTensorDev));
        if (!P.dl.convs.empty()) std::memcpy(P.tables.data() + P.dl.off_convs, P.dl.convs.data(), P.dl.convs.size() * sizeof(PlanConvDev));
        if (!P.dl.ops.empty()) std::memcpy(P.tables.data() + P.dl.off_ops, P.dl.ops.data(), P.dl.ops.size() * sizeof(PlanOpDev));
    }
    P.signature = fnv1a(0xcbf29ce484222325ull, layers, (size_t)n_layers * sizeof(dc_layer));
    const int32_t shape[8] = {n_streams, H, W, C, block, P.dl.cap, dtype, n_layers};
    P.signature = fnv1a(P.signature, shape, sizeof(shape));
    workspace_sizes(layers, n_layers, n_streams, H, W, block, max_rects, P.hs, P.ws, P.dl, &P.need_dev, &P.need_host);
    P.last_reader.assign(n_layers + 1, -1);
    P.conv_of.assign(n_layers, -1);
    P.sibling.assign(n_layers, -1);
    auto pointwise = [&](int i) { return layers[i].type == DC_CONV && layers[i].k == 1 && plain_square(layers[i]); };
    for (int i = 0; i < n_layers; ++i)
        for (int j = i + 1; pointwise(i) && j < n_layers && j <= i + kSiblingReach; ++j)      // (one with a sum behind it writes that too)
            if (pointwise(j) && layers[j].in0 == layers[i].in0 && layers[j].s == layers[i].s && !sum_behind(layers, n_layers, j)) { P.sibling[i] = j; break; }
    P.tilings.resize(n_layers);
    P.issued_full.assign(n_layers, 0);
    int conv = 0;
    for (int i = 0; i < n_layers; ++i) {
        int ids[4];
        const int m = layer_inputs(layers[i], ids);
        for (int j = 0; j < m; ++j) P.last_reader[ids[j]] = i;
        if (layers[i].type != DC_CONV) continue;
        P.conv_of[i] = conv++;
        const ConvTiling t = P.tilings[i] = pick_tiling(layers[i], P.hs[i + 1], P.ws[i + 1], n_streams, dtype);
        const WindowGeom g = window_geom(layers[i]);
        const int64_t mac_px = (int64_t)g.kh * g.kw * layers[i].cin * layers[i].cout;
        P.macs_full += (int64_t)P.hs[i + 1] * P.ws[i + 1] * n_streams * mac_px;
        P.issued_full[i] = (int64_t)n_streams * ((P.hs[i + 1] + t.th - 1) / t.th) * ((P.ws[i + 1] + t.tw - 1) / t.tw) * t.th * t.tw * mac_px;
        P.macs_issued_full += P.issued_full[i];
    }
    if (P.torus) P.rc_torus = torus_qualifies(P);
    // rough times, and the tensors that are one buffer for all frames
    const double px = (double)n_streams * H * W, cand = (2.0 * radius + 1) * (2.0 * radius + 1);
    const bool diamond = o && o->method == DC_MATCH_DIAMOND;
    P.head_us = (float)((diamond ? 50.0 + px / 25e3 : 15.0 + px * C * cand / 60e6) + (P.device_plan ? 25.0 + 0.4 * P.dl.ops.size() : 0.0));
    P.single.assign(n_layers + 1, 0);
    for (int i = 0; i < n_layers; ++i) {
        P.layer_us.push_back(layer_cost(P, i));
        if (P.on_torus(i + 1) || (may_in_place && layers[i].type == DC_CONV)) P.single[i + 1] = 1;
    }
    return DC_OK;
}

}  // namespace

// Cuts the layers into at most max_stages stages of about equal time such that no tensor with a single buffer is
// written in one stage and read in a later one (the writer's next frame would have to wait for the reader).  Where poolings
// lie on the torus too, no other cut is left, and where the caller's stream is busy with the caller's own work for long, the last
// stage should be short: there a stage may start with the only reader of the tensor that the stage before
// it writes last, and the next frame's writer waits for that one layer (an event and a wait per frame, no graphs; VGG-16
// 224x224 on one fp32 stream 384 us per frame in one stage, 259 so; 64 bf16 streams 1787 and 1620).
// A frame takes as long as its longest stage or as the host needs for it: graphs, events and cross-stream waits of a stage cost
// the host about 30 us (Dave on one fp32 stream, us per frame with 1 to 4 stages: 95, 80, 117, 133; VGG-16 224x224 bf16: 200, 140,
// 135, 147; ResNet-50: 515, 320, 257, 212), so a stage has to shorten what is the longer of the two by a tenth.  Planned on the
// host, a frame waits for its matching anyway and stages under 80 us are not worth having (VGG-16 224x224: 167, 169, 200;
// ResNet-50: 284 with two, 361 with three).
constexpr float kStageHostUs = 30.f;
constexpr float kTightTailUs = 100.f;      // the caller's work from which such a cut pays for the graphs that the stack gives up with it (VGG-16
                                           // 224x224 on one bf16 stream, us per frame without -> with it: 20 us of work 141 -> 181, 70 us 196 -> 190, 140 us 286 -> 226)
float StackPlan::period(float longest_us, int k) const { return device_plan ? std::max(longest_us, kStageHostUs * k) : longest_us; }
void StackPlan::cut(int max_stages) {
    const int n = (int)layers.size();
    std::vector<char> allowed(n, 1);       // allowed[i]: a stage may start with layer i
    for (int t = 0; t <= n; ++t)
        if (single[t])
            for (int i = t; i <= last_reader[t]; ++i)                       // the writer is layer t - 1
                allowed[i] = (pool_torus || tail_us > kTightTailUs) && i == t && last_reader[t] == t && allowed[i] == 1 ? 2 : 0;
    const float head = device_plan ? head_us : 0.f;
    float total = head;
    for (float v : layer_us) total += v;
    int k = device_plan ? max_stages : (int)(total / 80.f);
    k = std::min({std::max(k, 1), max_stages, n});
    // best[s][i]: smallest possible longest stage when layers 0 .. i - 1 form s stages
    std::vector<float> sum(n + 1, head);
    for (int i = 0; i < n; ++i) sum[i + 1] = sum[i] + layer_us[i];
    std::vector<std::vector<float>> best(k + 1, std::vector<float>(n + 1, 1e30f));
    std::vector<std::vector<int>> from(k + 1, std::vector<int>(n + 1, 0));
    for (int i = head > 0.f ? 0 : 1; i <= n; ++i) best[1][i] = sum[i];       // matching and planning alone may be a stage
    for (int s = 2; s <= k; ++s)
        for (int i = s - 1; i <= n; ++i)
            for (int j = s - 2; j < i; ++j) {
                if (!allowed[j]) continue;
                const float v = std::max(best[s - 1][j], sum[i] - sum[j]);
                if (v < best[s][i]) { best[s][i] = v; from[s][i] = j; }
            }
    // the last stage shares the caller's stream with what the caller does there
    std::vector<float> whole(k + 1, 1e30f);
    whole[1] = sum[n] + tail_us;
    for (int s = 2; s <= k; ++s)
        for (int j = s - 2; j < n; ++j) {
            const float v = allowed[j] ? std::max(best[s - 1][j], sum[n] - sum[j] + tail_us) : 1e30f;
            if (v < whole[s]) { whole[s] = v; from[s][n] = j; }
        }
    while (k > 1 && period(whole[k], k) > 0.9f * period(whole[k - 1], k - 1)) --k;          // a stage that shortens nothing
    n_stages = k;
    first[k] = n;
    for (int s = k, i = n; s > 1; --s) { i = from[s][i]; first[s - 1] = i; }
    first[0] = 0;
    for (int s = 0; s < kMaxStages; ++s) tight[s] = s > 0 && s < k && allowed[first[s]] == 2;
    crossing.clear();
    for (int t = 0; t <= n; ++t)
        if (last_reader[t] >= 0 && stage_of(last_reader[t]) > writer_stage(t) && !(single[t] && tight[stage_of(last_reader[t])])) crossing.push_back(t);
    ++partition;
}

// After kTimedFrames timed frames: scales the layers' times by what their stages took and cuts again if that pays.  A stage's
// time is the second shortest of the four: the first use of a kernel or a pause of the host between its launches is in one of
// them now and then (9 ms against 100 us: by the mean, Darknet-19 on one stream ended in stages of 66, 14 and 190 us).  The
// caller's work is taken by the same rule, the shorter of two where no more are known: a single long wait in it is not the rule.
void StackPlan::calibrate(int max_stages) {
    if (timed_frames < kTimedFrames) return;
    std::sort(timed_tail_us, timed_tail_us + timed_tails);
    const float new_tail = timed_tails ? timed_tail_us[timed_tails > 2 ? 1 : 0] : 0.f;
    float now = 0.f;
    for (int s = 0; s < n_stages; ++s) {
        const bool last = s + 1 == n_stages;
        std::nth_element(timed_us[s], timed_us[s] + 1, timed_us[s] + kTimedFrames);
        const float took = timed_us[s][1], ratio = took / std::max(stage_us(s) - (last ? tail_us : 0.f), 1.f);
        for (int i = first[s]; i < first[s + 1]; ++i) layer_us[i] *= ratio;
        if (s == 0 && device_plan) head_us *= ratio;
        now = std::max(now, took + (last && new_tail > 20.f ? new_tail : 0.f));
    }
    tail_us = new_tail > 20.f ? new_tail : 0.f;      // (the two events alone are some microseconds apart)
    timed_tails = 0;
    timed_frames = 0;
    const int old_stages = n_stages, old_partition = partition;
    int old_first[kMaxStages + 1];
    std::copy(first, first + kMaxStages + 1, old_first);
    bool old_tight[kMaxStages];
    std::copy(tight, tight + kMaxStages, old_tight);
    std::vector<int> old_crossing = crossing;
    cut(max_stages);
    if (period(longest(), n_stages) < 0.93f * period(now, old_stages)) {
        --recuts_left;
    } else {                                // as good as it gets
        recuts_left = 0;
        n_stages = old_stages; partition = old_partition;
        std::copy(old_first, old_first + kMaxStages + 1, first);
        std::copy(old_tight, old_tight + kMaxStages, tight);
        crossing.swap(old_crossing);
    }
}

namespace {

// The streams of the stages, one set per GPU for all overlap handles: the process has four hardware queues, and with
// the caller's stream these three fill them.  With streams of their own, several handles' streams shared queues in the
// order of their creation, so that stages of one handle landed in one queue and ran one after another (three runners
// taking turns, a ResNet-50 stream each: 438 us per frame against 360 for one runner alone).  All waits are for work
// that was queued earlier, so sharing cannot lock up.  The set lives as long as a handle uses it.
struct StageStreams {
    int users = 0;
    hipStream_t st[kMaxStages - 1] = {};
};
constexpr int kMaxGpus = 64;
StageStreams g_stage_streams[kMaxGpus];
std::mutex g_stage_streams_mutex;

bool acquire_stage_streams(Overlap* o) {
    if (hipGetDevice(&o->device) != hipSuccess || o->device < 0 || o->device >= kMaxGpus) { o->device = -1; return false; }
    std::lock_guard<std::mutex> guard(g_stage_streams_mutex);
    StageStreams& S = g_stage_streams[o->device];
    if (S.users == 0)
        for (hipStream_t& st : S.st)
            if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
                for (hipStream_t& made : S.st) {
                    if (made) (void)hipStreamDestroy(made);
                    made = nullptr;
                }
                o->device = -1;
                return false;
            }
    ++S.users;
    o->aux = S.st[0]; o->work[0] = S.st[1]; o->work[1] = S.st[2];
    return true;
}
void release_stage_streams(Overlap* o) {
    if (o->device < 0) return;
    std::lock_guard<std::mutex> guard(g_stage_streams_mutex);
    StageStreams& S = g_stage_streams[o->device];
    if (--S.users == 0)
        for (hipStream_t& st : S.st) {
            (void)hipStreamDestroy(st);
            st = nullptr;
        }
    o->device = -1;
}

// Waits for everything that was queued through the handle.
hipError_t drain(Overlap* o) {
    hipError_t e = hipSuccess;
    for (hipStream_t st : {o->aux, o->work[0], o->work[1]})
        if (st && e == hipSuccess) e = hipStreamSynchronize(st);
    for (FrameRecord& r : o->ring)
        if (r.valid && e == hipSuccess) e = hipEventSynchronize(r.done[r.n_stages - 1]);
    return e;
}

void release_plan(StackPlan* p) { delete p; }

// One dc_run_stack call: the arguments, then the steps in the order in which they run.
struct StackCall {
    // arguments
    const void* const* weights; const void* const* packed; const float* const* bias;
    const uint8_t *frames_cur, *frames_prev;
    void* const* tensors_cur; void* const* tensors_prev;
    int block, radius; uint32_t max_block_ssd;
    const dc_match_options* opt;
    bool cached; int32_t* in_place;
    int16_t* mv; uint32_t* best_ssd; int32_t* gmv; int32_t* n_pass; uint8_t* block_mask;
    int max_rects; dc_regions* regions_out;
    unsigned char* ws_dev; size_t ws_dev_bytes; unsigned char* ws_host; size_t ws_host_bytes;
    Profile* prof; Overlap* ov; hipStream_t caller;

    StackPlan& P;
    const int n_layers, n_streams, H, W, C, dtype;
    dc_stack_stats local;
    Overlap::Prefetch pf;

    bool pipe = false, devplan = false, inplace = false;
    bool gpu_idle = false;                   // the frames before this one were not all still running
    float blocked_us = 0.f;                  // this call's waits so far
    struct Blocked {                         // adds its own life to them
        StackCall& c;
        const std::chrono::steady_clock::time_point from = std::chrono::steady_clock::now();
        explicit Blocked(StackCall& call) : c(call) {}
        ~Blocked() { c.blocked_us += std::chrono::duration<float, std::micro>(std::chrono::steady_clock::now() - from).count(); }
    };
    int area = 0;                            // plan area of this frame
    hipStream_t stage_st[kMaxStages] = {};
    unsigned char *plan_dev = nullptr, *scratch = nullptr;
    size_t area_bytes = 0;
    std::vector<void*> eff;                  // where each tensor of this frame lives

    // planned on the GPU
    PlanDev pd{};
    DevHostHeader* hdr = nullptr;
    unsigned char *tables_host = nullptr, *tables_dev = nullptr, *slot_host = nullptr;
    const unsigned char* host_alias = nullptr;
    size_t off_stats = 0;
    std::vector<long> unit_hint;             // [conv]: list length of the last frame whose counters have arrived
    // planned on the host
    std::vector<LayerPlan> plans;
    std::vector<PlanAddr> addrs;
    struct CopyGroup { int first_layer; size_t rect_begin, rect_end, max_vec; };
    std::vector<CopyGroup> groups;
    std::vector<char> copy_fused;
    size_t all_rects_off = 0, copy_layers_off = 0;

    explicit StackCall(StackPlan& plan)
        : P(plan), n_layers((int)plan.layers.size()), n_streams(plan.n_streams), H(plan.H), W(plan.W), C(plan.C), dtype(plan.dtype) {
        std::memset(&local, 0, sizeof(local));
    }
    int gh() const { return H / block; }
    int gw() const { return W / block; }
    size_t n_blocks() const { return (size_t)n_streams * gh() * gw(); }

    int check();
    int begin();
    int prepare_device_plan();
    int launch_match(hipStream_t st);
    int emit_device_plan(hipStream_t st);
    int read_back_plan(hipStream_t st);
    int plan_on_host();
    int pack_host_plans(unsigned char* staging);
    int emit_copies(int s, hipStream_t st);
    int emit_layer(int i, hipStream_t st, ConvAdd* add = nullptr, ConvBatch* batch = nullptr);
    int run_with(int i, int end, uint32_t done, int* with) const;
    bool apart(int t, int v) const;
    bool apart(int t, int v, const void* at_v) const;
    bool sum_with(int i, ConvAdd* add) const;
    int emit_stage(int s, hipStream_t st);
    dc::FrameGraphs* find_graphs();
    int record_graphs(dc::FrameGraphs& g);
    int run();
    hipError_t wait(hipStream_t st, hipEvent_t e) const { return hipStreamWaitEvent(st, e, 0); }     // free when e is complete
    bool prefetched() const {
        return ov && pf.valid && pf.cur == frames_cur && pf.prev == frames_prev && pf.mv == mv && pf.best_ssd == best_ssd && pf.gmv == gmv &&
               pf.n_pass == n_pass && pf.mask == block_mask && pf.ws_host == ws_host && pf.n_streams == n_streams && pf.H == H &&
               pf.W == W && pf.C == C && pf.block == block && pf.radius == radius && pf.max_block_ssd == max_block_ssd &&
               pf.method == (opt ? opt->method : DC_MATCH_EXHAUSTIVE) && pf.k_skip == (opt ? opt->k_skip : 1);
    }
};

// Arguments that depend on the call and not on the stack alone.
int StackCall::check() {
    for (int t = 0; t <= n_layers; ++t)
        if (!tensors_cur[t]) return DC_ERR_NULL_PTR;
    for (int i = 0; i < n_layers; ++i)
        if ((P.layers[i].type == DC_CONV || P.layers[i].type == DC_FC) && !weights[i]) return DC_ERR_NULL_PTR;
    if (cached) {
        if (!frames_prev || !tensors_prev || !mv || !best_ssd || !gmv || !n_pass || !block_mask || !ws_dev || !ws_host)
            return DC_ERR_NULL_PTR;
        if (block > H || block > W) return DC_ERR_BAD_SHAPE;
        for (int i = 0; i < n_layers; ++i)
            if (P.layers[i].type == DC_CONV && (!tensors_prev[i + 1] || (tensors_prev[i + 1] == tensors_cur[i + 1]) != P.torus))
                return DC_ERR_NULL_PTR;     // two buffers per conv output, or the one buffer of a torus
        if (ws_dev_bytes < P.need_dev || ws_host_bytes < P.need_host) return DC_ERR_WORKSPACE;
    }
    if (regions_out)      // checked before anything is launched: every list fits
        for (size_t i = 0; i < (size_t)n_streams * (n_layers + 1); ++i)
            if (regions_out[i].capacity < max_rects || !regions_out[i].rects) return DC_ERR_CAPACITY;
    if (P.torus) {
        if (P.rc_torus) return P.rc_torus;
        for (int t = 1; t <= n_layers; ++t)
            if (P.on_torus(t) && (!tensors_prev || tensors_prev[t] != tensors_cur[t])) return DC_ERR_INVALID_ARG;     // one buffer
    }
    if (cached && P.cache_other)      // max-pooling and add layers that use the cache
        for (int i = 0; i < n_layers; ++i)
            if (P.uses_cache(i)) {
                if (!tensors_prev[i + 1] || (tensors_prev[i + 1] == tensors_cur[i + 1]) != P.pool_torus) return DC_ERR_NULL_PTR;
                if ((P.cs[i + 1] * dtype_size(dtype)) % 16 || (size_t)n_streams * P.hs[i + 1] > 65535 ||
                    reinterpret_cast<uintptr_t>(tensors_prev[i + 1]) % 16 || reinterpret_cast<uintptr_t>(tensors_cur[i + 1]) % 16)
                    return DC_ERR_UNSUPPORTED;
            }
    return DC_OK;
}

// Streams of the stages, place in the workspace, and the waits that order this frame behind the earlier ones where
// the streams do not.
int StackCall::begin() {
    pipe = ov && ov->pipeline;
    if (pipe) {     // the end of what the caller has queued behind the last frame: known to the GPU while that frame still runs
        FrameRecord& last = ov->ring[(ov->frame_no + kFramesInFlight - 1) % kFramesInFlight];
        if (last.valid && last.timed && !last.tail && last.plan == &P && last.caller == caller && hipEventQuery(last.done[last.n_stages - 1]) == hipErrorNotReady) {
            if (!last.after) DC_TRY_HIP(hipEventCreate(&last.after));
            DC_TRY_HIP(hipEventRecord(last.after, caller));
            last.tail = true;
        }
    }
    // With a pipeline and planning on the GPU, matching and planning head stage 0; planned on the host they run on aux,
    // because the host waits for them.
    const int most = P.device_plan ? kMaxStages : kMaxStages - 1;
    if (pipe && P.partition == 0) P.cut(most);
    if (pipe && P.recuts_left > 0) {
        FrameRecord& old = ov->ring[ov->frame_no % kFramesInFlight];
        if (old.valid && old.timed && old.plan == &P && old.partition == P.partition) {
            const Blocked b(*this);
            DC_TRY_HIP(hipEventSynchronize(old.done[old.n_stages - 1]));      // (the first few frames only)
            float ms = 0.f;
            for (int s = 0; s < old.n_stages; ++s) {
                DC_TRY_HIP(hipEventElapsedTime(&ms, old.start[s], old.done[s]));
                P.timed_us[s][P.timed_frames] = ms * 1e3f;
            }
            if (old.tail) {
                DC_TRY_HIP(hipEventSynchronize(old.after));
                DC_TRY_HIP(hipEventElapsedTime(&ms, old.done[old.n_stages - 1], old.after));
                P.timed_tail_us[P.timed_tails++] = ms * 1e3f;
            }
            ++P.timed_frames;
            const int before = P.partition;
            P.calibrate(most);
            ov->counters.recuts += P.partition != before ? 1 : 0;
        }
    }
    const int k = pipe ? P.n_stages : 1;
    if (pipe) {
        hipStream_t inner[kMaxStages - 1] = {ov->aux, ov->work[0], ov->work[1]};
        const int skip = P.device_plan ? 0 : 1;
        for (int s = 0; s + 1 < k; ++s) stage_st[s] = inner[s + skip];
    }
    stage_st[k - 1] = caller;
    area = ov ? (int)(ov->frame_no % kFramesInFlight) : 0;
    if (ws_dev && ws_dev_bytes >= scratch_region()) {
        const size_t plans_all = ws_dev_bytes - scratch_region();
        area_bytes = plans_all / kFramesInFlight / 256 * 256;
        plan_dev = ws_dev + (size_t)area * area_bytes;
        scratch = ws_dev + plans_all / 256 * 256;
    }
    devplan = cached && P.device_plan &&
              align_up(P.dl.table_bytes, 256) + P.dl.frame_bytes <= area_bytes && ws_host_bytes >= kDevHostRegion + 256;
    if (P.torus && cached && !devplan) return DC_ERR_UNSUPPORTED;      // a torus frame is planned on the GPU or not at all
    if (!ov) return DC_OK;
    FrameRecord& rec = ov->ring[area];
    for (int s = 0; s < k; ++s) {
        if (!rec.done[s]) DC_TRY_HIP(hipEventCreate(&rec.done[s]));
        if (!rec.start[s]) DC_TRY_HIP(hipEventCreate(&rec.start[s]));
        if (P.tight[s] && !rec.read[s]) DC_TRY_HIP(hipEventCreateWithFlags(&rec.read[s], hipEventDisableTiming));
    }
    // the plan area's (and the record's) last frame has to be over
    hipStream_t head = devplan && !pipe ? ov->aux : stage_st[0];
    if (rec.valid) DC_TRY_HIP(wait(head, rec.done[rec.n_stages - 1]));
    const FrameRecord& next = ov->ring[(area + 1) % kFramesInFlight];
    if (pipe && rec.valid && next.valid && rec.plan == &P && next.plan == &P) {
        gpu_idle = hipEventQuery(next.done[next.n_stages - 1]) == hipSuccess;
        float ms = 0.f;
        if (gpu_idle && hipEventElapsedTime(&ms, rec.done[rec.n_stages - 1], next.done[next.n_stages - 1]) == hipSuccess) P.replay.period(ms * 1e3f);
    }
    const FrameRecord& prev = ov->ring[(area + kFramesInFlight - 1) % kFramesInFlight];
    if (prev.valid && (prev.plan != &P || prev.partition != P.partition || prev.n_stages != k || prev.caller != caller)) {
        // other stages or streams than the previous frame's: its end comes first, on every stream
        const hipEvent_t end = prev.done[prev.n_stages - 1];
        for (int s = 0; s < k; ++s) DC_TRY_HIP(wait(stage_st[s], end));
        DC_TRY_HIP(wait(ov->aux, end));
    }
    return DC_OK;
}

// Host side of planning on the GPU: where the plan goes, and the counters of an earlier frame as launch hints.
int StackCall::prepare_device_plan() {
    const DevPlanLayout& dl = P.dl;
    unsigned char* const region = ws_host + ((ws_host_bytes - kDevHostRegion) & ~(size_t)255);
    hdr = reinterpret_cast<DevHostHeader*>(region);
    unsigned char* const slots = region + kDevHostSlot;
    tables_host = region + 3 * kDevHostSlot;
    // The layer tables travel with every frame (a few KB): what the device workspace holds from earlier calls is never
    // trusted.  The staging copy is rewritten only when it differs, and then nothing may still be reading it.
    if (std::memcmp(tables_host, P.tables.data(), dl.table_bytes) != 0) {
        const Blocked b(*this);
        if (ov) {
            DC_TRY_HIP(hipStreamSynchronize(ov->aux));
            for (hipStream_t w : ov->work) DC_TRY_HIP(hipStreamSynchronize(w));
        }
        DC_TRY_HIP(hipStreamSynchronize(caller));
        std::memcpy(tables_host, P.tables.data(), dl.table_bytes);
    }
    if (hdr->magic != kDevHostMagic || hdr->signature != P.signature || hdr->ws_dev != ws_dev || (hdr->last_slot != 0 && hdr->last_slot != 1)) {
        std::memset(region, 0, 3 * kDevHostSlot);          // other stack or workspace: the counters start afresh
        hdr->last_slot = 1;
        hdr->origin_area = -1;
        hdr->magic = kDevHostMagic; hdr->signature = P.signature; hdr->ws_dev = ws_dev;
        hdr->n_layers = n_layers; hdr->n_convs = (int32_t)dl.convs.size();
        hdr->macs_full = P.macs_full;
        hdr->n_blocks = (int32_t)n_blocks();
        for (size_t c = 0; c < dl.convs.size(); ++c) {
            const dc_layer& l = P.layers[dl.conv_layer[c]];
            hdr->conv[c] = DevHostConv{dl.conv_layer[c], (int32_t)(l.cout * dtype_size(dtype)), (int64_t)window_geom(l).kh * window_geom(l).kw * l.cin * l.cout,
                                       (int64_t)n_streams * dl.convs[c].Hout * dl.convs[c].Wout};
        }
    }
    unit_hint.assign(dl.convs.size(), -1);
    const PlanStatsConv* seen = reinterpret_cast<const PlanStatsConv*>(slots + (size_t)hdr->last_slot * kDevHostSlot + sizeof(PlanStatsHead));
    for (size_t c = 0; c < dl.convs.size(); ++c) {
        const int32_t v = *reinterpret_cast<const volatile int32_t*>(&seen[c].n_units);
        unit_hint[c] = v > 0 ? v : -1;
    }
    const int slot = ov ? area & 1 : hdr->last_slot ^ 1;
    tables_dev = plan_dev;
    unsigned char* const frame = plan_dev + align_up(dl.table_bytes, 256);
    pd.layers = reinterpret_cast<const PlanLayerDev*>(tables_dev);
    pd.tensors = reinterpret_cast<const PlanTensorDev*>(tables_dev + dl.off_tensors);
    pd.convs = reinterpret_cast<const PlanConvDev*>(tables_dev + dl.off_convs);
    pd.ops = reinterpret_cast<const PlanOpDev*>(tables_dev + dl.off_ops);
    pd.n_layers = n_layers; pd.n_convs = (int32_t)dl.convs.size(); pd.n_streams = n_streams; pd.cap = dl.cap;
    pd.n_ops = (int32_t)dl.ops.size(); pd.n_chunks = dl.n_chunks;
    pd.rects = reinterpret_cast<dc_rect*>(frame);
    pd.nrect = reinterpret_cast<int32_t*>(frame + dl.off_nrect);
    pd.dxy = reinterpret_cast<int32_t*>(frame + dl.off_dxy);
    pd.stream_info = reinterpret_cast<int32_t*>(frame + dl.off_info);
    pd.n_units = reinterpret_cast<int32_t*>(frame + dl.off_nunits);
    pd.area = frame + dl.off_area;
    pd.bitmaps = reinterpret_cast<uint32_t*>(frame + dl.off_bitmaps);
    pd.bm_words = dl.bm_words;
    pd.origin = nullptr; pd.origin_prev = nullptr; pd.pool_torus = P.pool_torus ? 1 : 0;
    if (P.torus) {          // this frame's origins follow from the previous frame's, which its plan area still holds
        pd.origin = reinterpret_cast<int32_t*>(frame + dl.off_origin);
        if (hdr->origin_area >= 0 && hdr->origin_area < kFramesInFlight)
            pd.origin_prev = reinterpret_cast<const int32_t*>(ws_dev + (size_t)hdr->origin_area * area_bytes + align_up(dl.table_bytes, 256) + dl.off_origin);
        hdr->origin_area = area;
    } else {
        hdr->origin_area = -1;
    }
    hdr->torus = P.torus ? 1 : 0;
    slot_host = slots + (size_t)slot * kDevHostSlot;
    hdr->last_slot = slot;
    off_stats = align_up(dl.table_bytes, 256) + dl.off_stats;
    host_alias = device_alias(ws_host);
    pd.stats = host_alias ? const_cast<unsigned char*>(host_alias) + (slot_host - ws_host) : plan_dev + off_stats;
    return DC_OK;
}

int StackCall::launch_match(hipStream_t st) {
    return dc_match_blocks_opt(frames_cur, frames_prev, n_streams, H, W, C, block, radius, opt, max_block_ssd, mv, best_ssd, gmv, n_pass,
                               block_mask, st);
}

// Step 5 and the propagation on the GPU, into this frame's plan area.
int StackCall::emit_device_plan(hipStream_t st) {
    const DevPlanLayout& dl = P.dl;
    DC_TRY_HIP(upload_plans(tables_dev, tables_host, dl.table_bytes, ws_host, st));
    const int ext = opt->extend_borders;
    if (P.exact) DC_TRY_HIP(launch_plan_exact(pd, block_mask, gmv, gh(), gw(), block, ext, dl.max_chunks, true, st));
    else DC_TRY_HIP(launch_plan(pd, block_mask, gmv, gh(), gw(), block, ext, dl.max_chunks, st));
    if (!host_alias)
        DC_TRY_HIP(hipMemcpyAsync(slot_host, plan_dev + off_stats, sizeof(PlanStatsHead) + dl.convs.size() * sizeof(PlanStatsConv),
                                  hipMemcpyDeviceToHost, st));
    return DC_OK;
}

// For inspection only: waits for the plan and reads origins and rectangle lists back.
int StackCall::read_back_plan(hipStream_t st) {
    const DevPlanLayout& dl = P.dl;
    if (P.torus && opt->origins_out) {
        DC_TRY_HIP(hipStreamSynchronize(st));
        DC_TRY_HIP(hipMemcpy(opt->origins_out, pd.origin, (size_t)n_streams * (n_layers + 1) * 2 * sizeof(int32_t), hipMemcpyDeviceToHost));
    }
    if (regions_out) {
        const int nt = n_layers + 1;
        std::vector<int32_t> h_n((size_t)n_streams * nt), h_d((size_t)n_streams * nt * 2);
        std::vector<dc_rect> h_r((size_t)n_streams * nt * dl.cap);
        DC_TRY_HIP(hipStreamSynchronize(st));
        DC_TRY_HIP(hipMemcpy(h_n.data(), pd.nrect, h_n.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
        DC_TRY_HIP(hipMemcpy(h_d.data(), pd.dxy, h_d.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
        DC_TRY_HIP(hipMemcpy(h_r.data(), pd.rects, h_r.size() * sizeof(dc_rect), hipMemcpyDeviceToHost));
        for (int s = 0; s < n_streams; ++s)
            for (int t = 0; t < nt; ++t) {
                dc_regions& r = regions_out[(size_t)s * nt + t];
                const size_t at = (size_t)s * nt + t;
                r.n = h_n[at]; r.dx = h_d[2 * at]; r.dy = h_d[2 * at + 1];
                r.cum_stride = dl.tensors[t].cum_stride; r.h = P.hs[t]; r.w = P.ws[t];
                if (r.n) std::memcpy(r.rects, h_r.data() + at * dl.cap, (size_t)r.n * sizeof(dc_rect));   // n <= cap <= capacity
            }
    }
    return DC_OK;
}

// Steps 1 to 5 and the propagation with the host in the loop: waits for the matching, merges, propagates, lists the
// dirty units of every conv layer and packs the plans into pinned staging memory.
int StackCall::plan_on_host() {
    // With an overlap handle the matching runs on its own stream, next to whatever is still queued of earlier frames;
    // only that stream is waited for.
    hipStream_t mst = ov ? ov->aux : caller;
    const size_t nb = n_blocks();
    unsigned char* hbase = ws_host;
    uint8_t* h_mask = hbase;
    int32_t* h_gmv = reinterpret_cast<int32_t*>(hbase + align_up(nb, 256));
    const bool ahead = prefetched();    // a match started ahead of time with exactly these arguments is on its way or done
    if (ov && pf.valid && !ahead) DC_TRY_HIP(hipStreamSynchronize(mst));   // let the stale match finish first
    if (!ahead) {
        const int rc = launch_match(mst);
        if (rc) return rc;
        DC_TRY_HIP(hipMemcpyAsync(h_mask, block_mask, nb, hipMemcpyDeviceToHost, mst));
        DC_TRY_HIP(hipMemcpyAsync(h_gmv, gmv, (size_t)n_streams * 2 * sizeof(int32_t), hipMemcpyDeviceToHost, mst));
    }
    if (ov) {
        if (!ahead) DC_TRY_HIP(hipEventRecord(ov->match_done, mst));
        DC_TRY_HIP(spin_wait(ov->match_done));
    } else {
        DC_TRY_HIP(hipStreamSynchronize(mst));
    }
    if (in_place) {     // no stream moved: the previous frame's conv outputs can be updated where they are
        inplace = true;
        for (int s = 0; s < n_streams; ++s) inplace = inplace && h_gmv[2 * s] == 0 && h_gmv[2 * s + 1] == 0;
        *in_place = inplace ? 1 : 0;
    }
    std::vector<std::vector<TensorRegions>> regs(n_streams);  // [stream][tensor]
    {   // per stream: count, merge (Step 5), propagate (Section 5); streams are independent
        std::vector<int> stream_rc(n_streams, DC_OK), stream_reusable(n_streams, 0), stream_over(n_streams, 0);
        parallel_for(n_streams, [&](int s) {
            try {
                std::vector<dc_rect> rects0;
                const uint8_t* m = h_mask + (size_t)s * gh() * gw();
                int cnt = 0;
                for (int i = 0; i < gh() * gw(); ++i) cnt += m[i] ? 1 : 0;
                stream_reusable[s] = cnt;
                merge_blocks(m, gh(), gw(), block, rects0);
                int r = propagate(P.layers.data(), n_layers, H, W, rects0, h_gmv[2 * s], h_gmv[2 * s + 1], regs[s],
                                  opt && opt->extend_borders != 0);
                // a list longer than the caller allows: the stream reuses nothing in this frame (always valid)
                bool over = false;
                for (int t = 0; r == DC_OK && t <= n_layers; ++t) over = over || (int)regs[s][t].rects.size() > max_rects;
                if (over) {
                    for (int t = 0; t <= n_layers; ++t) regs[s][t].rects.clear();
                    stream_over[s] = 1;
                }
                stream_rc[s] = r;
            } catch (const std::bad_alloc&) {
                stream_rc[s] = DC_ERR_WORKSPACE;
            }
        });
        for (int s = 0; s < n_streams; ++s) {
            if (stream_rc[s]) return stream_rc[s];
            local.n_reusable_blocks += stream_reusable[s];
            local.n_overflow_streams += stream_over[s];
        }
    }
    hbase += align_up(nb, 256) + align_up((size_t)n_streams * 3 * sizeof(int32_t), 256);
    if (ov) {
        // two staging halves: the upload of the frame before last must have left the half reused now
        const size_t half = (ws_host_bytes - kDevHostRegion - (size_t)(hbase - ws_host)) / 2 / 256 * 256;
        hbase += (size_t)ov->parity * half;
        if (ov->pending[ov->parity]) {
            DC_TRY_HIP(spin_wait(ov->upload_done[ov->parity]));
            ov->pending[ov->parity] = false;
        }
    }
    if (regions_out)
        for (int s = 0; s < n_streams; ++s)
            for (int t = 0; t <= n_layers; ++t) {
                dc_regions& r = regions_out[(size_t)s * (n_layers + 1) + t];
                const TensorRegions& g = regs[s][t];
                r.n = (int)g.rects.size(); r.dx = g.dx; r.dy = g.dy; r.cum_stride = g.cum_stride; r.h = g.h; r.w = g.w;
                if (r.n) std::memcpy(r.rects, g.rects.data(), r.n * sizeof(dc_rect));     // n <= max_rects <= capacity
            }
    // The tiles of every (stream, conv layer) are classified in parallel over the streams into per-stream lists,
    // the per-layer offsets follow from their sizes, and the lists are then copied straight into the pinned
    // staging buffer, again in parallel (64 streams: 550 k tiles per frame).
    plans.resize(n_layers);
    addrs.resize(n_layers);
    size_t off = 0;
    {
        std::lock_guard<std::mutex> guard(g_frame_plan_mutex);
        FramePlan& fp = g_frame_plan;
        const int rc = fp.classify(P.layers.data(), n_layers, n_streams, regs, P.hs, P.ws, P.no_reuse.empty() ? nullptr : P.no_reuse.data());
        if (rc) return rc;
        for (int i = 0; i < n_layers; ++i) {
            const dc_layer& l = P.layers[i];
            if (l.type != DC_CONV) continue;
            const int64_t px = (int64_t)P.hs[i + 1] * P.ws[i + 1] * n_streams;
            const int64_t mac_px = (int64_t)window_geom(l).kh * window_geom(l).kw * l.cin * l.cout;
            LayerPlan& plan = plans[i];
            addrs[i] = fp.finish_layer(i, plan, hbase + off, plan_dev + off);
            off += addrs[i].bytes;
            const int64_t issued = (int64_t)plan.n_tiles * P.tilings[i].th * P.tilings[i].tw * mac_px;
            local.macs_needed += (px - plan.reused_px) * mac_px;
            local.macs_issued += issued;
            if (!inplace) local.copy_bytes += 2 * plan.reused_px * l.cout * (int64_t)dtype_size(dtype);
            if (local.layer_reused_px) local.layer_reused_px[i] = plan.reused_px;
            if (local.layer_issued_macs) local.layer_issued_macs[i] = issued;
        }
        fp.copy_tiles();
    }
    // The shifted copies of a stage's layers go out in one launch (16-byte vector path only): a layer's cache is
    // complete when its stage starts.
    copy_fused.assign(n_layers, inplace ? 1 : 0);        // in place every reusable pixel already holds its value
    if (!inplace) {
        std::vector<RectDev> all_rects;
        std::vector<CopyLayerDev> copy_layers;
        for (int i = 0; i < n_layers; ++i) {
            if (P.layers[i].type != DC_CONV || plans[i].rects.empty()) continue;
            const size_t px_bytes = (size_t)P.layers[i].cout * dtype_size(dtype);
            if (px_bytes % 16 || reinterpret_cast<uintptr_t>(tensors_prev[i + 1]) % 16 || reinterpret_cast<uintptr_t>(tensors_cur[i + 1]) % 16)
                continue;
            copy_fused[i] = 1;
            const int pv = (int)(px_bytes / 16);
            if (groups.empty() || (pipe && P.stage_of(groups.back().first_layer) != P.stage_of(i)))
                groups.push_back(CopyGroup{i, all_rects.size(), all_rects.size(), 0});
            CopyGroup& g = groups.back();
            for (RectDev r : plans[i].rects) {
                r.pad = (int)copy_layers.size();
                all_rects.push_back(r);
                g.max_vec = std::max(g.max_vec, (size_t)r.w * r.h * pv);
            }
            g.rect_end = all_rects.size();
            copy_layers.push_back(CopyLayerDev{tensors_prev[i + 1], tensors_cur[i + 1], P.hs[i + 1], P.ws[i + 1], pv, 0});
        }
        if (!all_rects.empty()) {
            all_rects_off = off;
            std::memcpy(hbase + off, all_rects.data(), all_rects.size() * sizeof(RectDev));
            off += align_up(all_rects.size() * sizeof(RectDev), 256);
            copy_layers_off = off;
            std::memcpy(hbase + off, copy_layers.data(), copy_layers.size() * sizeof(CopyLayerDev));
            off += align_up(copy_layers.size() * sizeof(CopyLayerDev), 256);
        }
    }
    if (off) {
        DC_TRY_HIP(upload_plans(plan_dev, hbase, off, ws_host, stage_st[0]));
        if (ov) {
            DC_TRY_HIP(hipEventRecord(ov->upload_done[ov->parity], stage_st[0]));
            ov->pending[ov->parity] = true;
            ov->parity ^= 1;
        }
    }
    return DC_OK;
}

// Section 5 "Reuse", step 1, for the conv layers of stage s.
int StackCall::emit_copies(int s, hipStream_t st) {
    if (!cached || P.torus || inplace) return DC_OK;
    if (!devplan) {
        for (const CopyGroup& g : groups) {
            if (P.stage_of(g.first_layer) != s && pipe) continue;
            Bracket b(prof, n_layers + g.first_layer, st);
            DC_TRY_HIP(launch_shifted_copy_all(reinterpret_cast<const RectDev*>(plan_dev + all_rects_off) + g.rect_begin,
                                               (int)(g.rect_end - g.rect_begin),
                                               reinterpret_cast<const CopyLayerDev*>(plan_dev + copy_layers_off), g.max_vec, st));
        }
        return DC_OK;
    }
    const int end = pipe ? P.first[s + 1] : n_layers;
    std::vector<CopyUnitsLayer> L;
    int vec_bytes = 0, group_first = -1;
    auto flush = [&]() -> int {
        if (L.empty()) return DC_OK;
        Bracket b(prof, n_layers + group_first, st);
        DC_TRY_HIP(launch_shifted_copy_units(L.data(), (int)L.size(), pd.dxy, n_layers + 1, n_streams, vec_bytes, st));
        L.clear();
        return DC_OK;
    };
    for (int i = pipe ? P.first[s] : 0; i < end; ++i) {
        const int c = P.conv_of[i];
        if (c < 0 || (!P.no_reuse.empty() && P.no_reuse[i])) continue;        // nothing of a flagged layer comes from the cache
        const size_t px_bytes = (size_t)P.layers[i].cout * dtype_size(dtype);
        const bool vec16 = px_bytes % 16 == 0 && reinterpret_cast<uintptr_t>(tensors_prev[i + 1]) % 16 == 0 &&
                           reinterpret_cast<uintptr_t>(tensors_cur[i + 1]) % 16 == 0;
        const int vb = vec16 ? 16 : (int)dtype_size(dtype);
        if (vb != vec_bytes) {
            const int rc = flush();
            if (rc) return rc;
        }
        if (L.empty()) group_first = i;
        vec_bytes = vb;
        const PlanConvDev& cv = P.dl.convs[c];
        L.push_back(CopyUnitsLayer{tensors_prev[i + 1], tensors_cur[i + 1], reinterpret_cast<const uint16_t*>(pd.area + cv.umask_off), cv.tensor,
                                   cv.Hout, cv.Wout, cv.units_x, cv.units_y, (int32_t)(px_bytes / vb), 0, 0});
    }
    return flush();
}

// No byte of tensor t lies in tensor v.
bool StackCall::apart(int t, int v) const { return apart(t, v, eff[v]); }
bool StackCall::apart(int t, int v, const void* at_v) const {
    auto bytes = [&](int x) { return (size_t)n_streams * P.hs[x] * P.ws[x] * P.cs[x] * dtype_size(dtype); };
    const uintptr_t a = reinterpret_cast<uintptr_t>(eff[t]), b = reinterpret_cast<uintptr_t>(at_v);
    return a + bytes(t) <= b || b + bytes(v) <= a;
}

// The later 1x1 convolutions (before layer `end`) that may be launched with layer i because they read its input: the layers
// between must neither read nor write their outputs, which buffers that a caller lets tensors share could make them do.
// Bit d of `done`: layer i + d has been launched (with a layer before i, where one between them could not be).
int StackCall::run_with(int i, int end, uint32_t done, int* with) const {
    if (prof || inplace || P.torus) return 0;
    int n = 0;
    for (int j = P.sibling[i]; j >= 0 && j < end && n < kConvBatch - 1; j = P.sibling[j]) {
        bool free = !((done >> (j - i)) & 1);
        for (int k = i; k < j && free; ++k) {
            int ids[4];
            const int m = layer_inputs(P.layers[k], ids);
            for (int x = 0; x < m; ++x) free = free && apart(j + 1, ids[x]);
            free = free && apart(j + 1, k + 1);
            if (cached && (P.layers[k].type == DC_CONV || P.uses_cache(k))) free = free && apart(j + 1, k + 1, tensors_prev[k + 1]);
        }
        if (free) with[n++] = j;
    }
    return n;
}

// The sum behind conv layer i, where a kernel may write both: in the order of the layers the sum's output is written when the
// convolution has read its input, so buffers that a caller lets tensors share must not be those.
bool StackCall::sum_with(int i, ConvAdd* add) const {
    if (!sum_behind(P.layers.data(), n_layers, i) || (cached && !devplan) || inplace || P.torus || prof || (devplan && P.uses_cache(i + 1))) return false;
    const dc_layer& sum = P.layers[i + 1];
    const int other = sum.in0 == i + 1 ? sum.in1 : sum.in0;
    if (!apart(i + 2, P.layers[i].in0) || !apart(i + 2, i + 1) || !(eff[i + 2] == eff[other] || apart(i + 2, other)) || !apart(i + 1, other)) return false;
    *add = ConvAdd{eff[other], eff[i + 2], sum.relu, false};
    return true;
}

int StackCall::emit_layer(int i, hipStream_t st, ConvAdd* add, ConvBatch* batch) {
    const dc_layer& l = P.layers[i];
    const int a = l.in0, t = i + 1;
    const std::vector<int>&hs = P.hs, &ws = P.ws, &cs = P.cs;
    // torus frames: where the origins of tensor t start (a stream's are 2 (n_layers + 1) ints apart); nullptr: the
    // tensor starts at its buffer's start (every tensor of a full frame, everything but conv outputs otherwise)
    auto origin_of = [&](int tensor) -> const int32_t* { return (devplan && P.on_torus(tensor)) ? pd.origin + 2 * tensor : nullptr; };
    const bool from_cache = devplan && P.uses_cache(i);
    const CachedMap cm{pd.bitmaps, pd.bm_words, devplan ? P.dl.tensors[t].bm_off : 0, pd.dxy, n_layers + 1, t};
    const size_t out_px = (size_t)n_streams * hs[t] * ws[t];
    switch (l.type) {
        case DC_CONV: {
            const int c = P.conv_of[i];
            unsigned char* const my_scratch = scratch ? scratch + (size_t)(pipe ? P.stage_of(i) : 0) * kConvScratchBytes : nullptr;
            return run_conv_planned(l, eff[a], weights[i], bias ? bias[i] : nullptr, cached ? tensors_prev[t] : nullptr, eff[t], n_streams,
                                    hs[a], ws[a], dtype, P.tilings[i], cached && !devplan ? &plans[i] : nullptr,
                                    cached && !devplan ? &addrs[i] : nullptr, st, prof, i, n_layers + i,
                                    local.layer_kernel_id ? &local.layer_kernel_id[i] : nullptr, devplan || (cached && copy_fused[i]),
                                    my_scratch, my_scratch ? kConvScratchBytes : 0, packed ? packed[i] : nullptr,
                                    devplan ? reinterpret_cast<const TileDev*>(pd.area + P.dl.convs[c].list_off) : nullptr,
                                    devplan ? n_streams * P.dl.convs[c].units_x * P.dl.convs[c].units_y : 0,
                                    devplan ? pd.n_units + c : nullptr, devplan ? unit_hint[c] : -1, origin_of(a), origin_of(t),
                                    2 * (n_layers + 1), a == 0 ? C : 0, add,
                                    devplan ? reinterpret_cast<const uint16_t*>(pd.area + P.dl.convs[c].umask_off) : nullptr, batch);
        }
        case DC_MAXPOOL:
            if (origin_of(a))            // its input lies on a torus, and with the cache its output too
                DC_TRY_HIP(launch_maxpool2x2_torus(eff[a], eff[t], n_streams, hs[a], ws[a], cs[a], dtype, origin_of(a), origin_of(t),
                                                   2 * (n_layers + 1), origin_of(t) && from_cache ? &cm : nullptr, st));
            else if (from_cache)
                DC_TRY_HIP(launch_maxpool_cached(eff[a], tensors_prev[t], eff[t], n_streams, hs[a], ws[a], cs[a], l.k, l.s, l.p, dtype, cm, st));
            else
                DC_TRY_HIP(launch_maxpool(eff[a], eff[t], n_streams, hs[a], ws[a], cs[a], l.k, l.s, l.p, dtype, st));
            return DC_OK;
        case DC_ADD:
            if (from_cache)
                DC_TRY_HIP(launch_add_cached(eff[a], eff[l.in1], tensors_prev[t], eff[t], n_streams, hs[t], ws[t], cs[t], l.relu, dtype, cm, st));
            else
                DC_TRY_HIP(launch_add(eff[a], eff[l.in1], eff[t], out_px * cs[t], l.relu, dtype, st));
            return DC_OK;
        case DC_AVGPOOL:
            DC_TRY_HIP(launch_avgpool(eff[a], eff[t], n_streams, hs[a], ws[a], cs[a], l.k, l.s, l.p, dtype, st));
            return DC_OK;
        case DC_LRN:
            DC_TRY_HIP(launch_lrn(eff[a], eff[t], n_streams, hs[a], ws[a], cs[a], l.k, l.within, l.alpha, l.beta, l.kappa, dtype, st));
            return DC_OK;
        case DC_CONCAT: {
            int ids[4], chans[4];
            const void* ins[4];
            const int m = concat_inputs(l, ids);
            for (int j = 0; j < m; ++j) { ins[j] = eff[ids[j]]; chans[j] = cs[ids[j]]; }
            DC_TRY_HIP(launch_concat(ins, chans, m, eff[t], out_px, dtype, st));
            return DC_OK;
        }
        case DC_FC:
            DC_TRY_HIP(launch_fc(eff[a], weights[i], bias ? bias[i] : nullptr, eff[t], n_streams, (size_t)hs[a] * ws[a] * cs[a], l.cout, l.relu, dtype, st));
            return DC_OK;
        case DC_SOFTMAX:
            DC_TRY_HIP(launch_softmax(eff[a], eff[t], out_px, cs[t], dtype, st));
            return DC_OK;
        default:
            DC_TRY_HIP(launch_add(eff[a], nullptr, eff[t], out_px * cs[t], 1, dtype, st));
            return DC_OK;
    }
}

int StackCall::emit_stage(int s, hipStream_t st) {
    int rc = emit_copies(s, st);
    const int end = pipe ? P.first[s + 1] : n_layers;
    static_assert((kConvBatch - 1) * kSiblingReach < 32, "a bit for every layer that may run early");
    uint32_t done = 0;                              // bit d: layer i + d has been launched
    for (int i = pipe ? P.first[s] : 0; i < end && !rc; ++i, done >>= 1) {
        if (done & 1) continue;
        if (pipe && i + 1 == end && s + 1 < P.n_stages && P.tight[s + 1]) {
            // the last frame's next stage has to have read the tensor that this layer writes (with another cut its end
            // has been waited for)
            const FrameRecord& last = ov->ring[(area + kFramesInFlight - 1) % kFramesInFlight];
            if (last.valid && last.plan == &P && last.partition == P.partition) DC_TRY_HIP(wait(st, last.read[s + 1]));
        }
        ConvAdd add{};
        // (no such wait for a sum: its tensor has a buffer per frame, and only one of a single buffer is waited for)
        const bool both = i + 1 < end && sum_with(i, &add);
        int with[kConvBatch - 1];
        const int n_with = both ? 0 : run_with(i, pipe && s + 1 < P.n_stages && P.tight[s + 1] ? end - 1 : end, done, with);
        if (n_with) {
            ConvBatch batch;
            rc = emit_layer(i, st, nullptr, &batch);
            for (int m = 0; m < n_with && !rc; ++m) {
                rc = emit_layer(with[m], st, nullptr, &batch);
                done |= 1u << (with[m] - i);
            }
            if (!rc) DC_TRY_HIP(launch_conv_batch(batch, st));
        } else {
            rc = emit_layer(i, st, both ? &add : nullptr);
        }
        if (pipe && i == P.first[s] && P.tight[s] && !rc) DC_TRY_HIP(hipEventRecord(ov->ring[area].read[s], st));
        if (add.done) { ++i; done >>= 1; }          // the sum is written
    }
    return rc;
}

constexpr size_t kMaxFrameGraphs = 16;       // keys kept per stack
constexpr int kGraphUses = 2;               // frames of a key that are launched kernel by kernel before it is recorded
constexpr int kGraphOffShape = 8;           // consecutive frames with other list lengths before a graph is recorded anew:
constexpr int kGraphOffUnits = 16;          // a layer's differs by more than a quarter and this many units (the launch of a few is as good as any)

// The entry for this frame's key, or nullptr if the frame cannot be replayed from a graph: everything its kernels take
// as arguments has to be part of the key, and nothing may wait for the host or go through a copy in between.
dc::FrameGraphs* StackCall::find_graphs() {
    const bool wanted = ov && (ov->replay_mode < 0 ? P.replay.on && !P.replay.refresh() : ov->replay_mode == 1 && opt && P.device_plan);
    if (!pipe || !wanted || (cached && !devplan) || prof || regions_out || P.no_graphs) return nullptr;
    for (bool tight : P.tight)      // (a wait in the middle of a stage)
        if (tight) return nullptr;
    if (cached && (!host_alias || (P.torus && opt->origins_out))) return nullptr;
    const size_t n = n_layers;
    std::vector<uint64_t> key;
    key.reserve(5 * n + 16);
    auto put = [&](const void* const* v, size_t m) {
        for (size_t i = 0; i < m; ++i) key.push_back(v ? reinterpret_cast<uint64_t>(v[i]) : 0);
    };
    put(weights, n); put(packed, n); put(reinterpret_cast<const void* const*>(bias), n);
    put(tensors_cur, n + 1);
    put(cached ? tensors_prev : nullptr, n + 1);
    key.push_back(reinterpret_cast<uint64_t>(scratch));
    if (cached)
        for (const void* v : {static_cast<const void*>(plan_dev), static_cast<const void*>(host_alias), static_cast<const void*>(tables_host),
                              static_cast<const void*>(pd.stats), static_cast<const void*>(pd.origin_prev),
                              static_cast<const void*>(block_mask), static_cast<const void*>(gmv)})
            key.push_back(reinterpret_cast<uint64_t>(v));
    key.push_back((uint64_t)P.partition << 32 | (cached ? 1 : 0) | (opt->extend_borders ? 2 : 0));
    for (int v : conv_tuning().v) key.push_back((uint64_t)(int64_t)v);
    uint64_t h = 0x9e3779b97f4a7c15ull;
    for (uint64_t v : key) { h = (h ^ v) * 0xff51afd7ed558ccdull; h ^= h >> 32; }
    for (auto& g : P.graphs)
        if (g->hash == h && g->key == key) {
            g->last_use = ov->frame_no;
            return g.get();
        }
    if (P.graphs.size() >= kMaxFrameGraphs) {        // the least recently used entry goes
        size_t old = 0;
        for (size_t i = 1; i < P.graphs.size(); ++i)
            if (P.graphs[i]->last_use < P.graphs[old]->last_use) old = i;
        if (P.graphs[old]->ready) {
            const Blocked b(*this);
            if (drain(ov) != hipSuccess) return nullptr;      // (its graphs may still be running)
            ++ov->counters.evicted;
        }
        P.graphs.erase(P.graphs.begin() + old);
    }
    P.graphs.emplace_back(new dc::FrameGraphs());
    dc::FrameGraphs* g = P.graphs.back().get();
    g->key.swap(key);
    g->hash = h;
    g->last_use = ov->frame_no;
    return g;
}

// Records the launches of every stage (nothing is executed).
int StackCall::record_graphs(dc::FrameGraphs& g) {
    g.kernel_id.assign(n_layers, -1);
    int32_t* const caller_ids = local.layer_kernel_id;
    local.layer_kernel_id = g.kernel_id.data();
    // The handle's own stream, on which nothing is executed: what another thread's handle launches on a stage stream while
    // that stream is captured would end up in this graph.
    if (!ov->record && hipStreamCreateWithFlags(&ov->record, hipStreamNonBlocking) != hipSuccess) ov->record = nullptr;
    const hipStream_t st = ov->record;
    int rc = st ? DC_OK : DC_ERR_HIP;
    for (int s = 0; s < P.n_stages && !rc; ++s) {
        hipGraph_t graph = nullptr;
        if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) != hipSuccess) { rc = DC_ERR_HIP; break; }
        if (s == 0 && cached) rc = emit_device_plan(st);
        if (!rc) rc = emit_stage(s, st);
        if (hipStreamEndCapture(st, &graph) != hipSuccess || !graph) rc = DC_ERR_HIP;
        size_t nodes = 0;
        if (!rc && hipGraphGetNodes(graph, nullptr, &nodes) != hipSuccess) rc = DC_ERR_HIP;
        if (!rc && nodes && hipGraphInstantiate(&g.exec[s], graph, nullptr, nullptr, 0) != hipSuccess) rc = DC_ERR_HIP;
        if (graph) (void)hipGraphDestroy(graph);
    }
    local.layer_kernel_id = caller_ids;
    g.hint = unit_hint;
    if (rc) { g.drop(); (void)hipGetLastError(); }
    g.ready = rc == DC_OK;
    ++(rc ? ov->counters.failed : ov->counters.recorded);
    return rc;
}

int StackCall::run() {
    const auto t_start = std::chrono::steady_clock::now();
    int rc = check();
    if (rc) return rc;
    // a look-ahead match is for the very next call only (the caller may reuse its frame buffers after that)
    if (ov) { pf = ov->prefetch; ov->prefetch.valid = false; }
    rc = begin();
    if (rc) return rc;
    local.full = cached ? 0 : 1;
    local.n_blocks = (int32_t)n_blocks();
    local.macs_full = P.macs_full;
    if (in_place) *in_place = 0;
    if (P.torus && opt->origins_dev_out) *opt->origins_dev_out = nullptr;
    if (P.torus && !cached && ws_host && ws_host_bytes >= kDevHostRegion + 256) {
        // a full frame writes every tensor at its buffer's start: the next cached frame starts from origins (0, 0)
        DevHostHeader* h = reinterpret_cast<DevHostHeader*>(ws_host + ((ws_host_bytes - kDevHostRegion) & ~(size_t)255));
        if (h->magic == kDevHostMagic) h->origin_area = -1;
    }
    const int k = pipe ? P.n_stages : 1;
    FrameRecord* const rec = ov ? &ov->ring[area] : nullptr;
    if (rec) rec->valid = false;
    const bool timed = devplan && pipe && P.recuts_left > 0;      // (planned on the host, a stage takes what the host takes to issue it)
    if (timed) DC_TRY_HIP(hipEventRecord(rec->start[0], stage_st[0]));

    // ---- matching and planning ----
    hipStream_t head = devplan && ov && !pipe ? ov->aux : stage_st[0];
    // A look-ahead match, taken or not, writes the match buffers and reads the caller's frames on aux: a frame that does not
    // start there comes after it, a full one too (the next cached frame matches on the stream that it starts on).  The
    // other stages, the caller's stream and the later frames follow from this one; planned on the host, the host waits.
    if (pf.valid && (devplan || !cached) && head != ov->aux) DC_TRY_HIP(wait(head, ov->match_done));
    if (devplan) {
        rc = prepare_device_plan();
        if (rc) return rc;
        // (the match buffers are shared by consecutive frames: their matching and planning follow one another on one stream)
        if (!prefetched()) {
            rc = launch_match(head);
            if (rc) return rc;
        }
        if (P.torus && opt->origins_dev_out) *opt->origins_dev_out = pd.origin;
        if (ov) { ov->head = head; ov->planned = false; }
    } else if (cached) {
        rc = plan_on_host();
        if (rc) return rc;
    } else {
        local.macs_needed = P.macs_full;
        local.macs_issued = P.macs_issued_full;
        for (int i = 0; i < n_layers; ++i) {
            if (P.layers[i].type != DC_CONV) continue;
            if (local.layer_reused_px) local.layer_reused_px[i] = 0;
            if (local.layer_issued_macs) local.layer_issued_macs[i] = P.issued_full[i];
        }
        if (regions_out)
            for (size_t i = 0; i < (size_t)n_streams * (n_layers + 1); ++i) {
                dc_regions& r = regions_out[i];
                const int t = (int)(i % (n_layers + 1));
                r.n = 0; r.dx = r.dy = 0; r.cum_stride = 0; r.h = P.hs[t]; r.w = P.ws[t];
            }
    }

    // ---- layers ----
    // an in-place frame keeps the conv outputs in the previous frame's buffers
    eff.resize(n_layers + 1);
    for (int t = 0; t <= n_layers; ++t)
        eff[t] = (inplace && t > 0 && P.layers[t - 1].type == DC_CONV) ? tensors_prev[t] : tensors_cur[t];
    // a tensor that a later stage reads: the readers of the frame that last used its buffer have to be done.  (Tensors
    // that stay inside a stage are ordered by its stream.)
    bool recut = false;
    if (pipe)
        for (int t : P.crossing)
            for (int g = 1; g < kFramesInFlight; ++g) {
                const FrameRecord& r = ov->ring[(area + kFramesInFlight - g) % kFramesInFlight];
                if (!r.valid || r.plan != &P || r.partition != P.partition) break;
                if (r.bufs[t] != eff[t]) continue;
                DC_TRY_HIP(wait(stage_st[P.writer_stage(t)], r.done[P.stage_of(P.last_reader[t])]));
                if (g == 1 && !P.single[t]) { P.single[t] = 1; recut = true; }
                break;
            }
    dc::FrameGraphs* g = find_graphs();
    if (g && g->ready && cached) {      // a graph is kept while every layer's list is about as long as when it was recorded
        bool off = false;
        for (size_t c = 0; c < unit_hint.size(); ++c) {
            const long a = std::max(unit_hint[c], 0l), b = std::max(g->hint[c], 0l);
            off = off || std::abs(a - b) * 4 > std::max(a, b) + 4 * kGraphOffUnits;
        }
        g->off_shape = off ? g->off_shape + 1 : 0;
        if (g->off_shape >= kGraphOffShape) {
            const Blocked b(*this);
            DC_TRY_HIP(drain(ov));
            g->drop();
            ++ov->counters.dropped;
        }
    }
    const bool recorded = g && !g->ready && g->uses++ >= kGraphUses;
    if (recorded && record_graphs(*g) != DC_OK) P.no_graphs = true;
    const bool replay = g && g->ready;

    DC_TRY_HIP(launch_frame_to_tensor(frames_cur, eff[0], (size_t)n_streams * H * W, C, P.c_tensor, dtype, stage_st[0]));
    if (devplan && !replay) {
        rc = emit_device_plan(head);
        if (!rc) rc = read_back_plan(head);
        if (rc) return rc;
        if (head != stage_st[0]) {
            DC_TRY_HIP(hipEventRecord(ov->plan_done, head));
            DC_TRY_HIP(wait(stage_st[0], ov->plan_done));
        } else if (ov && ov->looks_ahead && head != ov->aux) {
            DC_TRY_HIP(hipEventRecord(ov->plan_done, head));
            ov->planned = true;
        }
    }
    for (int s = 0; s < k; ++s) {
        if (s > 0) {
            DC_TRY_HIP(wait(stage_st[s], rec->done[s - 1]));
            if (timed) DC_TRY_HIP(hipEventRecord(rec->start[s], stage_st[s]));
        }
        if (!replay) rc = emit_stage(s, stage_st[s]);
        else if (g->exec[s]) DC_TRY_HIP(hipGraphLaunch(g->exec[s], stage_st[s]));
        if (rc) return rc;
        if (rec) DC_TRY_HIP(hipEventRecord(rec->done[s], stage_st[s]));
    }
    if (pipe && (devplan || (!cached && P.device_plan))) {
        const auto t_end = std::chrono::steady_clock::now();
        auto us = [](auto a, auto b) { return std::chrono::duration<float, std::micro>(b - a).count(); };
        if (replay) P.replay.replayed();
        else if (!recorded && !timed) P.replay.issued(us(t_start, t_end) - blocked_us, gpu_idle || P.replay.refresh());
        P.replay.between(us(P.left, t_start));
        P.left = t_end;
    }
    if (replay && local.layer_kernel_id) std::copy(g->kernel_id.begin(), g->kernel_id.end(), local.layer_kernel_id);
    if (rec) {
        rec->plan = &P; rec->partition = P.partition; rec->n_stages = k; rec->caller = caller;
        rec->bufs.assign(eff.begin(), eff.end());
        rec->timed = timed;
        rec->tail = false;
        rec->valid = true;
        ++ov->frame_no;
        ++ov->counters.frames;
        ov->counters.replayed += replay ? 1 : 0;
        ov->counters.stages = k;
        ov->counters.last_layers = pipe ? P.first[k] - P.first[k - 1] : n_layers;
    }
    if (recut) {
        ++ov->counters.recuts;
        P.cut(P.device_plan ? kMaxStages : kMaxStages - 1);
        P.timed_frames = P.timed_tails = 0;
    }
    return DC_OK;
}

}  // namespace

extern "C" {

int32_t dc_overlap_create(void** overlap) {
    if (!overlap) return DC_ERR_NULL_PTR;
    Overlap* o = new (std::nothrow) Overlap();
    if (!o) return DC_ERR_WORKSPACE;
    bool ok = acquire_stage_streams(o);
    for (int i = 0; i < 2 && ok; ++i) ok = hipEventCreateWithFlags(&o->upload_done[i], hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&o->match_done, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&o->plan_done, hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        (void)dc_overlap_destroy(o);
        return DC_ERR_HIP;
    }
    *overlap = o;
    return DC_OK;
}

int32_t dc_overlap_destroy(void* overlap) {
    if (!overlap) return DC_ERR_NULL_PTR;
    Overlap* o = static_cast<Overlap*>(overlap);
    (void)drain(o);
    for (StackPlan* p : o->plans) release_plan(p);
    for (hipEvent_t e : o->upload_done)
        if (e) (void)hipEventDestroy(e);
    for (FrameRecord& r : o->ring)
        for (int s = 0; s < kMaxStages; ++s) {
            if (r.done[s]) (void)hipEventDestroy(r.done[s]);
            if (r.start[s]) (void)hipEventDestroy(r.start[s]);
            if (r.read[s]) (void)hipEventDestroy(r.read[s]);
        }
    for (FrameRecord& r : o->ring)
        if (r.after) (void)hipEventDestroy(r.after);
    if (o->match_done) (void)hipEventDestroy(o->match_done);
    if (o->plan_done) (void)hipEventDestroy(o->plan_done);
    if (o->record) (void)hipStreamDestroy(o->record);
    release_stage_streams(o);
    delete o;
    return DC_OK;
}

int32_t dc_overlap_pipeline(void* overlap, int32_t frames_in_flight) {
    if (!overlap) return DC_ERR_NULL_PTR;
    if (frames_in_flight < 1 || frames_in_flight > 2) return DC_ERR_INVALID_ARG;
    Overlap* o = static_cast<Overlap*>(overlap);
    DC_TRY_HIP(drain(o));
    for (FrameRecord& r : o->ring) r.valid = false;
    o->pipeline = frames_in_flight == 2;
    return DC_OK;
}

int32_t dc_overlap_replay(void* overlap, int32_t mode) {
    if (!overlap) return DC_ERR_NULL_PTR;
    if (mode < -1 || mode > 1) return DC_ERR_INVALID_ARG;
    static_cast<Overlap*>(overlap)->replay_mode = mode;
    return DC_OK;
}

int32_t dc_overlap_stats(const void* overlap, dc_overlap_counters* counters) {
    if (!overlap || !counters) return DC_ERR_NULL_PTR;
    *counters = static_cast<const Overlap*>(overlap)->counters;
    return DC_OK;
}

int32_t dc_prefetch_match(void* overlap, const uint8_t* frames_next, const uint8_t* frames_cur,
                          int32_t n_streams, int32_t H, int32_t W, int32_t C, int32_t block, int32_t radius,
                          uint32_t max_block_ssd, const dc_match_options* match_options,
                          int16_t* mv, uint32_t* best_ssd, int32_t* global_mv, int32_t* n_pass,
                          uint8_t* block_mask, void* ws_host, size_t ws_host_bytes) {
    if (!overlap || !frames_next || !frames_cur || !global_mv || !block_mask || !ws_host) return DC_ERR_NULL_PTR;
    if (n_streams < 1 || H < 1 || W < 1 || C < 1 || block < 1) return DC_ERR_INVALID_ARG;
    if (block > H || block > W) return DC_ERR_BAD_SHAPE;
    Overlap* ov = static_cast<Overlap*>(overlap);
    const size_t nb = (size_t)n_streams * (H / block) * (W / block);
    if (ws_host_bytes < align_up(nb, 256) + align_up((size_t)n_streams * 3 * sizeof(int32_t), 256)) return DC_ERR_WORKSPACE;
    if (ov->prefetch.valid) {     // an unused look-ahead is dropped once its kernels are out of the way
        DC_TRY_HIP(hipStreamSynchronize(ov->aux));
        ov->prefetch.valid = false;
    }
    if (ov->head && ov->head != ov->aux) {     // the current frame's planning on the GPU still reads the match buffers
        const FrameRecord& last = ov->ring[(ov->frame_no + kFramesInFlight - 1) % kFramesInFlight];
        if (ov->planned) DC_TRY_HIP(hipStreamWaitEvent(ov->aux, ov->plan_done, 0));
        else if (last.valid) DC_TRY_HIP(hipStreamWaitEvent(ov->aux, last.done[0], 0));      // (planned in a graph)
    }
    ov->looks_ahead = true;
    int rc = dc_match_blocks_opt(frames_next, frames_cur, n_streams, H, W, C, block, radius, match_options, max_block_ssd,
                                 mv, best_ssd, global_mv, n_pass, block_mask, ov->aux);
    if (rc) return rc;
    unsigned char* hbase = static_cast<unsigned char*>(ws_host);
    DC_TRY_HIP(hipMemcpyAsync(hbase, block_mask, nb, hipMemcpyDeviceToHost, ov->aux));
    DC_TRY_HIP(hipMemcpyAsync(hbase + align_up(nb, 256), global_mv, (size_t)n_streams * 2 * sizeof(int32_t),
                              hipMemcpyDeviceToHost, ov->aux));
    DC_TRY_HIP(hipEventRecord(ov->match_done, ov->aux));
    Overlap::Prefetch& pf = ov->prefetch;
    pf.cur = frames_next; pf.prev = frames_cur; pf.mv = mv; pf.best_ssd = best_ssd; pf.gmv = global_mv; pf.n_pass = n_pass;
    pf.mask = block_mask; pf.ws_host = ws_host; pf.n_streams = n_streams; pf.H = H; pf.W = W; pf.C = C; pf.block = block;
    pf.radius = radius; pf.max_block_ssd = max_block_ssd;
    pf.method = match_options ? match_options->method : DC_MATCH_EXHAUSTIVE;
    pf.k_skip = match_options ? match_options->k_skip : 1;
    pf.valid = true;
    return DC_OK;
}

int32_t dc_stack_workspace_bytes(const dc_layer* layers, int32_t n_layers, int32_t n_streams, int32_t H, int32_t W,
                                 int32_t C, int32_t block, int32_t max_rects, size_t* dev_bytes, size_t* host_bytes) {
    if (!layers || !dev_bytes || !host_bytes) return DC_ERR_NULL_PTR;
    if (n_layers < 1 || n_streams < 1 || block < 1 || max_rects < 1) return DC_ERR_INVALID_ARG;
    try {
        std::vector<int> hs, ws, cs;
        const int c_tensor = input_channels(layers, n_layers, C);
        if (c_tensor < C) return DC_ERR_BAD_SHAPE;
        int rc = validate_layers(layers, n_layers, H, W, c_tensor, &hs, &ws, &cs);
        if (rc) return rc;
        DevPlanLayout dl;                              // planning on the GPU lays the same area out differently
        device_plan_layout(layers, n_layers, hs, ws, n_streams, max_rects, dl);
        workspace_sizes(layers, n_layers, n_streams, H, W, block, max_rects, hs, ws, dl, dev_bytes, host_bytes);
    } catch (const std::bad_alloc&) {
        return DC_ERR_WORKSPACE;
    }
    return DC_OK;
}

int32_t dc_run_stack(const dc_layer* layers, int32_t n_layers, const void* const* weights,
                     const void* const* packed_weights, const float* const* bias,
                     const uint8_t* frames_cur, const uint8_t* frames_prev, void* const* tensors_cur,
                     void* const* tensors_prev, int32_t n_streams, int32_t H, int32_t W, int32_t C,
                     int32_t dtype, int32_t block, int32_t radius, uint32_t max_block_ssd,
                     const dc_match_options* match_options, int32_t force_full, int32_t* in_place,
                     int16_t* mv, uint32_t* best_ssd, int32_t* global_mv, int32_t* n_pass, uint8_t* block_mask,
                     int32_t max_rects, dc_regions* regions_out, void* ws_dev, size_t ws_dev_bytes, void* ws_host,
                     size_t ws_host_bytes, dc_stack_stats* stats, void* overlap, void* stream) {
    if (!layers || !weights || !frames_cur || !tensors_cur) return DC_ERR_NULL_PTR;
    if (dtype != DC_F32 && dtype != DC_BF16) return DC_ERR_INVALID_ARG;
    if (n_layers < 1 || n_streams < 1 || n_streams > 65535 || block < 1 || radius < 0 || max_rects < 1) return DC_ERR_INVALID_ARG;
    const dc_match_options* o = match_options;
    if (o) {
        if (o->method != DC_MATCH_EXHAUSTIVE && o->method != DC_MATCH_DIAMOND) return DC_ERR_INVALID_ARG;
        if (o->k_skip < 1) return DC_ERR_INVALID_ARG;
        if (o->exact_masks && (!o->device_plan || in_place)) return DC_ERR_UNSUPPORTED;   // planned on the GPU only
        if (o->cache_pool_add && !o->exact_masks) return DC_ERR_UNSUPPORTED;
        if (o->torus && (!o->device_plan || in_place)) return DC_ERR_UNSUPPORTED;
    }
    Overlap* const ov = static_cast<Overlap*>(overlap);
    try {
        // the stack's plan: the handle's, if its last calls were for this stack
        const int32_t head[16] = {n_layers, n_streams, H, W, C, dtype, block, radius, max_rects, in_place ? 1 : 0, o ? o->method : -1,
                                  o ? o->exact_masks : 0, o ? o->cache_pool_add : 0, o ? o->torus : 0, o ? o->device_plan : 0,
                                  o && o->no_reuse ? 1 : 0};
        const size_t layer_bytes = (size_t)n_layers * sizeof(dc_layer), flag_bytes = o && o->no_reuse ? (size_t)n_layers : 0;
        auto same = [&](const StackPlan& p) {
            const unsigned char* k = p.key.data();
            return p.key.size() == sizeof(head) + layer_bytes + flag_bytes && std::memcmp(k, head, sizeof(head)) == 0 &&
                   std::memcmp(k + sizeof(head), layers, layer_bytes) == 0 &&
                   (!flag_bytes || std::memcmp(k + sizeof(head) + layer_bytes, o->no_reuse, flag_bytes) == 0);
        };
        std::unique_ptr<StackPlan> fresh;
        StackPlan* plan = nullptr;
        if (ov)
            for (size_t i = 0; i < ov->plans.size() && !plan; ++i)
                if (same(*ov->plans[i])) {
                    plan = ov->plans[i];
                    std::rotate(ov->plans.begin(), ov->plans.begin() + i, ov->plans.begin() + i + 1);
                }
        if (!plan) {
            fresh.reset(new StackPlan());
            const int rc = make_plan(*fresh, layers, n_layers, n_streams, H, W, C, dtype, block, radius, max_rects, o, in_place != nullptr);
            if (rc) return rc;
            fresh->key.resize(sizeof(head) + layer_bytes + flag_bytes);
            std::memcpy(fresh->key.data(), head, sizeof(head));
            std::memcpy(fresh->key.data() + sizeof(head), layers, layer_bytes);
            if (flag_bytes) std::memcpy(fresh->key.data() + sizeof(head) + layer_bytes, o->no_reuse, flag_bytes);
            plan = fresh.get();
            if (ov) {
                constexpr size_t kKept = 4;
                ov->plans.reserve(kKept + 1);
                if (ov->plans.size() >= kKept) {        // the least recently used one goes; nothing of it may be in flight
                    DC_TRY_HIP(drain(ov));
                    for (FrameRecord& r : ov->ring)
                        if (r.plan == ov->plans.back()) r.valid = false;
                    release_plan(ov->plans.back());
                    ov->plans.pop_back();
                }
                ov->plans.insert(ov->plans.begin(), fresh.release());
            }
        }
        StackCall c(*plan);
        c.weights = weights; c.packed = packed_weights; c.bias = bias;
        c.frames_cur = frames_cur; c.frames_prev = frames_prev;
        c.tensors_cur = tensors_cur; c.tensors_prev = tensors_prev;
        c.block = block; c.radius = radius; c.max_block_ssd = max_block_ssd;
        c.opt = o; c.cached = !force_full; c.in_place = in_place;
        c.mv = mv; c.best_ssd = best_ssd; c.gmv = global_mv; c.n_pass = n_pass; c.block_mask = block_mask;
        c.max_rects = max_rects; c.regions_out = regions_out;
        c.ws_dev = static_cast<unsigned char*>(ws_dev); c.ws_dev_bytes = ws_dev_bytes;
        c.ws_host = static_cast<unsigned char*>(ws_host); c.ws_host_bytes = ws_host_bytes;
        c.prof = stats ? static_cast<Profile*>(stats->profile) : nullptr;
        c.ov = ov; c.caller = as_stream(stream);
        if (stats) {
            c.local.layer_reused_px = stats->layer_reused_px;
            c.local.layer_issued_macs = stats->layer_issued_macs;
            c.local.profile = stats->profile;
            c.local.layer_kernel_id = stats->layer_kernel_id;
        }
        const int rc = c.run();
        if (rc) return rc;
        if (stats) *stats = c.local;
    } catch (const std::bad_alloc&) {
        return DC_ERR_WORKSPACE;
    }
    return DC_OK;
}

int32_t dc_propagate_masks_size(const dc_layer* layers, int32_t n_layers, int32_t H, int32_t W, int32_t C,
                                size_t* words_per_stream, int64_t* tensor_offset, size_t* ws_dev_bytes) {
    if (!layers || !words_per_stream || !ws_dev_bytes) return DC_ERR_NULL_PTR;
    if (n_layers < 1 || H < 1 || W < 1 || C < 1) return DC_ERR_INVALID_ARG;
    std::vector<int> hs, ws, cs;
    const int c_tensor = input_channels(layers, n_layers, C);
    if (c_tensor < C) return DC_ERR_BAD_SHAPE;
    int rc = validate_layers(layers, n_layers, H, W, c_tensor, &hs, &ws, &cs);
    if (rc) return rc;
    try {
        DevPlanLayout dl;
        device_plan_layout(layers, n_layers, hs, ws, 1, 1, dl);
        if (!dl.ok) return DC_ERR_UNSUPPORTED;
        *words_per_stream = (size_t)dl.bm_words;
        *ws_dev_bytes = dl.table_bytes + 256;
        if (tensor_offset)
            for (int t = 0; t <= n_layers; ++t) tensor_offset[t] = dl.tensors[t].bm_off;
    } catch (const std::bad_alloc&) {
        return DC_ERR_WORKSPACE;
    }
    return DC_OK;
}

int32_t dc_propagate_masks(const dc_layer* layers, int32_t n_layers, int32_t n_streams, int32_t H, int32_t W, int32_t C,
                           int32_t block, const uint8_t* block_mask, const int32_t* global_mv, int32_t extend_borders,
                           uint32_t* bitmaps, int32_t* dxy, void* ws_dev, size_t ws_dev_bytes, void* stream) {
    if (!layers || !block_mask || !global_mv || !bitmaps || !dxy || !ws_dev) return DC_ERR_NULL_PTR;
    if (n_layers < 1 || n_streams < 1 || H < 1 || W < 1 || C < 1 || block < 1) return DC_ERR_INVALID_ARG;
    if (block > H || block > W) return DC_ERR_BAD_SHAPE;
    std::vector<int> hs, ws, cs;
    const int c_tensor = input_channels(layers, n_layers, C);
    if (c_tensor < C) return DC_ERR_BAD_SHAPE;
    int rc = validate_layers(layers, n_layers, H, W, c_tensor, &hs, &ws, &cs);
    if (rc) return rc;
    hipStream_t st = as_stream(stream);
    try {
        DevPlanLayout dl;
        device_plan_layout(layers, n_layers, hs, ws, n_streams, 1, dl);
        if (!dl.ok) return DC_ERR_UNSUPPORTED;
        if (ws_dev_bytes < dl.table_bytes + 256) return DC_ERR_WORKSPACE;
        std::vector<unsigned char> tables(dl.table_bytes, 0);
        std::memcpy(tables.data(), dl.layers.data(), dl.layers.size() * sizeof(PlanLayerDev));
        std::memcpy(tables.data() + dl.off_tensors, dl.tensors.data(), dl.tensors.size() * sizeof(PlanTensorDev));
        if (!dl.ops.empty()) std::memcpy(tables.data() + dl.off_ops, dl.ops.data(), dl.ops.size() * sizeof(PlanOpDev));
        unsigned char* const table_dev = static_cast<unsigned char*>(ws_dev);
        DC_TRY_HIP(hipMemcpyAsync(table_dev, tables.data(), dl.table_bytes, hipMemcpyHostToDevice, st));
        DC_TRY_HIP(hipStreamSynchronize(st));          // `tables` goes away with this scope
        PlanDev pd{};
        pd.layers = reinterpret_cast<const PlanLayerDev*>(table_dev);
        pd.tensors = reinterpret_cast<const PlanTensorDev*>(table_dev + dl.off_tensors);
        pd.ops = reinterpret_cast<const PlanOpDev*>(table_dev + dl.off_ops);
        pd.n_layers = n_layers; pd.n_convs = 0; pd.n_streams = n_streams; pd.cap = 1;
        pd.n_ops = (int32_t)dl.ops.size();
        pd.dxy = dxy;
        // the kernel also leaves a block count and empty rectangle lists: into the tail of the workspace
        int32_t* tail = reinterpret_cast<int32_t*>(table_dev + dl.table_bytes);
        if (ws_dev_bytes < dl.table_bytes + 256 + (size_t)n_streams * (n_layers + 3) * sizeof(int32_t)) return DC_ERR_WORKSPACE;
        pd.stream_info = tail + 64;
        pd.nrect = tail + 64 + 2 * n_streams;
        pd.bitmaps = bitmaps; pd.bm_words = dl.bm_words;
        DC_TRY_HIP(launch_plan_exact(pd, block_mask, global_mv, H / block, W / block, block, extend_borders, 0, false, st));
    } catch (const std::bad_alloc&) {
        return DC_ERR_WORKSPACE;
    }
    return DC_OK;
}

int32_t dc_stack_stats_fetch(const void* ws_host, size_t ws_host_bytes, dc_stack_stats* stats) {
    if (!ws_host || !stats) return DC_ERR_NULL_PTR;
    if (ws_host_bytes < kDevHostRegion + 256) return DC_ERR_WORKSPACE;
    const unsigned char* region = static_cast<const unsigned char*>(ws_host) + ((ws_host_bytes - kDevHostRegion) & ~(size_t)255);
    const DevHostHeader* hdr = reinterpret_cast<const DevHostHeader*>(region);
    if (hdr->magic != kDevHostMagic || hdr->n_convs < 0 || hdr->n_convs > kPlanMaxConvs) return DC_ERR_INVALID_ARG;
    const unsigned char* slot = region + kDevHostSlot + (size_t)hdr->last_slot * kDevHostSlot;
    const PlanStatsHead* sh = reinterpret_cast<const PlanStatsHead*>(slot);
    const PlanStatsConv* sc = reinterpret_cast<const PlanStatsConv*>(slot + sizeof(PlanStatsHead));
    stats->full = 0;
    stats->n_blocks = hdr->n_blocks;
    stats->n_reusable_blocks = sh->n_reusable_blocks;
    stats->n_overflow_streams = sh->n_overflow_streams;
    stats->macs_full = hdr->macs_full;
    stats->macs_needed = 0; stats->macs_issued = 0; stats->copy_bytes = 0;
    for (int c = 0; c < hdr->n_convs; ++c) {
        const DevHostConv& hc = hdr->conv[c];
        const int64_t issued = (int64_t)sc[c].n_units * 16 * hc.mac_px;
        stats->macs_needed += (hc.px_total - sc[c].reused_px) * hc.mac_px;
        stats->macs_issued += issued;
        if (!hdr->torus) stats->copy_bytes += 2 * sc[c].reused_px * hc.cout_bytes;
        if (stats->layer_reused_px) stats->layer_reused_px[hc.layer] = sc[c].reused_px;
        if (stats->layer_issued_macs) stats->layer_issued_macs[hc.layer] = issued;
    }
    return DC_OK;
}

}  // extern "C"
