// Host side of the FlashOptim C ABI (include/flashoptim.h): argument validation, the
// cached device tables that let one call cover a whole parameter list, per-call scalar
// set-up, and the checkpoint container.
//
// Nothing here computes on the CPU what the GPU should: if HIP is unavailable every
// compute entry point returns FLASHOPTIM_ERR_HIP.

#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstdint>
#include <cstring>
#include <list>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

#include "flashoptim.h"
#include "flashoptim_device.h"

namespace {

using fo::CopySegment;
using fo::StepArgs;
using fo::StepConsts;
using fo::TensorDev;

constexpr int64_t kMaxNumel = (int64_t)1 << 40;
constexpr int kVersion = (0 << 16) | 1;

thread_local int g_last_hip_error = 0;

#define FO_HIP(expr)                                         \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) {                              \
            g_last_hip_error = (int)e_;                      \
            (void)hipGetLastError();                         \
            return FLASHOPTIM_ERR_HIP;                       \
        }                                                    \
    } while (0)

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int64_t n_groups(int64_t n) { return (n + fo::kGroup - 1) / fo::kGroup; }
inline int64_t align64(int64_t x) { return (x + 63) & ~(int64_t)63; }

// Whether what is enqueued on `stream` is being captured into a graph.  (An error means that another stream's capture
// forbids the question for the default stream: that stream itself is not capturing.)
bool is_capturing(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return status != hipStreamCaptureStatusNone;
}

// The calls that wait for values from the device refuse a capturing stream before anything is enqueued: their kernels
// would run with the graph only, on memory that this call gives back.
int refuse_capture(hipStream_t stream) {
    if (!is_capturing(stream)) return FLASHOPTIM_OK;
    g_last_hip_error = (int)hipErrorStreamCaptureUnsupported;
    return FLASHOPTIM_ERR_HIP;
}

// ----------------------------------------------------- cached device tables --
//
// A "plan" is what a multi-tensor launch needs on the device: the table of tensors (for copies, of
// segments) and a coarse index table into it by workgroup.  It belongs to the list's identity (device, operation, every state pointer and
// numel; NOT the gradient pointers or lr/wd, which legitimately change from step to step).
// What a later call on the same list may change (gradient pointer, rates, weight decay) is written into the
// tensor table in stream order, from kernel arguments, only when it differs from what the device already holds; a
// new learning rate that all tensors share goes with the step's own launch.
//
// A call finds its plan through a 64-bit hash of the identity and then compares the descriptors themselves, so a
// collision costs time and nothing else.  (With the identity as a string key, built and hashed byte by byte on
// every call, a step over 161 tensors spent 5 us on the host beyond the launch, a checkpoint pack 20.)

struct PlanTag {
    int32_t device, op, kind, flags;    // op: a LiveOp, or kOpPack / kOpUnpack
    const void* blob;                   // copies: the blob
};
inline bool operator==(const PlanTag& a, const PlanTag& b) {
    return a.device == b.device && a.op == b.op && a.kind == b.kind && a.flags == b.flags && a.blob == b.blob;
}

bool same_identity(const TensorDev& a, const TensorDev& b) {
    return a.param == b.param && a.rho == b.rho && a.m_q == b.m_q && a.m_scale == b.m_scale && a.v_q == b.v_q &&
           a.v_scale == b.v_scale && a.theta32 == b.theta32 && a.m32 == b.m32 && a.v32 == b.v32 && a.numel == b.numel;
}

uint64_t identity_hash(const PlanTag& tag, const std::vector<TensorDev>& t) {
    const uint64_t k = 0x9e3779b97f4a7c15ull;
    uint64_t h = ((uint64_t)(uint32_t)tag.device + ((uint64_t)(uint32_t)tag.op << 16) + ((uint64_t)(uint32_t)tag.kind << 32) +
                  ((uint64_t)(uint32_t)tag.flags << 48)) * k + (uint64_t)reinterpret_cast<uintptr_t>(tag.blob);
    auto w = [](const void* p) { return (uint64_t)reinterpret_cast<uintptr_t>(p); };
    for (const TensorDev& d : t) {
        const uint64_t x = w(d.param) + 3 * w(d.rho) + 5 * w(d.m_q) + 7 * w(d.m_scale) + 11 * w(d.v_q) + 13 * w(d.v_scale);
        const uint64_t y = 17 * w(d.theta32) + 19 * w(d.m32) + 23 * w(d.v32) + 29 * (uint64_t)d.numel;
        h = (h ^ (h >> 29) ^ (x + y)) * k;
    }
    return h ^ (h >> 32);
}

struct Plan {
    PlanTag tag = {};
    uint64_t hash = 0;
    std::vector<TensorDev> tensors;    // the list; for steps and conversions also what the device table holds
    bool table_known = true;           // false: a call failed part of the way, so the table is written as a whole next
    bool in_graphs = false;            // an update was captured: replays write the table, so every call writes it as a whole
    void* d_mem = nullptr;         // one allocation: the table, the index, the header
    void* d_table = nullptr;       // TensorDev[] or CopySegment[]
    void* d_index = nullptr;       // uint32 coarse table: workgroup -> tensor (steps, conversions) or segment (copies)
    int64_t n_chunks = 0;          // workgroups of a launch over this plan
    uint32_t coarse_shift = 0;     // copies only
    void* d_header = nullptr;      // copies only: the blob's header and table, all but the step
    void* h_mem = nullptr;         // pinned source of d_mem's upload, kept until the plan is freed
    size_t bytes = 0;              // of each
    bool uploaded = false;         // an upload has been enqueued (one that was captured runs with the graph, if at all)
};

std::mutex g_mu;
std::list<Plan> g_plans;            // most recently used first
std::unordered_multimap<uint64_t, std::list<Plan>::iterator> g_index;
constexpr size_t kMaxPlans = 256;   // least recently used beyond this are freed (after a device synchronisation)

// Frees a plan's device and pinned buffers.  Work that was enqueued with this plan may still read them, so
// the plan's own device is synchronised first (plans are freed rarely: on eviction and on release_cache).
void destroy_plan(Plan& p) {
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(p.tag.device);
    if (p.d_mem) (void)hipDeviceSynchronize();
    if (p.d_mem) (void)hipFree(p.d_mem);
    if (p.h_mem) (void)hipHostFree(p.h_mem);
    p.d_mem = nullptr; p.h_mem = nullptr;
    (void)hipSetDevice(cur);
}

// Finds the plan of a list and makes it the most recently used one; nullptr if there is none.
Plan* find_plan(const PlanTag& tag, uint64_t hash, const std::vector<TensorDev>& tensors) {
    const auto range = g_index.equal_range(hash);
    for (auto it = range.first; it != range.second; ++it) {
        const Plan& p = *it->second;
        if (!(p.tag == tag) || p.tensors.size() != tensors.size()) continue;
        bool same = true;
        for (size_t i = 0; i < tensors.size() && same; ++i) same = same_identity(p.tensors[i], tensors[i]);
        if (!same) continue;
        g_plans.splice(g_plans.begin(), g_plans, it->second);
        return &g_plans.front();
    }
    return nullptr;
}

// What a plan puts on the device.
struct PlanSource {
    const void* table;
    size_t table_bytes;
    const std::vector<uint32_t>& index;
    const std::vector<uint8_t>& header;
};

// Uploads a plan's tables in stream order on `stream`, ahead of the launch that the calling call enqueues there, unless
// an earlier call has (calls with the same list touch the same tensors, so the caller orders them like any other work on
// those tensors).
int upload_tables(Plan& p, hipStream_t stream) {
    if (p.uploaded) return FLASHOPTIM_OK;
    FO_HIP(fo::launch_move(p.h_mem, p.d_mem, p.bytes, stream));
    if (is_capturing(stream)) p.in_graphs = true;       // (a replay brings back the entries that the list began with)
    else p.uploaded = true;
    return FLASHOPTIM_OK;
}

// Makes the plan of a list that has none, its tables in pinned memory of the plan.  Nothing here waits for the stream.
int make_plan(const PlanTag& tag, uint64_t hash, const std::vector<TensorDev>& tensors, const PlanSource& src,
              int64_t n_chunks, Plan** out) {
    Plan p;
    p.tag = tag;
    p.hash = hash;
    p.tensors = tensors;
    p.n_chunks = n_chunks;
    const size_t index_bytes = src.index.size() * sizeof(uint32_t);
    const size_t index_at = (size_t)align64((int64_t)src.table_bytes);
    const size_t header_at = index_at + (size_t)align64((int64_t)index_bytes);
    const size_t all = header_at + (size_t)align64((int64_t)src.header.size());
    p.bytes = all > 0 ? all : 64;
    hipError_t e = hipMalloc(&p.d_mem, p.bytes);
    if (e == hipSuccess) e = hipHostMalloc(&p.h_mem, p.bytes, hipHostMallocCoherent);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        (void)hipGetLastError();
        destroy_plan(p);
        return FLASHOPTIM_ERR_HIP;
    }
    p.d_table = p.d_mem;
    p.d_index = static_cast<uint8_t*>(p.d_mem) + index_at;
    p.d_header = static_cast<uint8_t*>(p.d_mem) + header_at;
    uint8_t* h = static_cast<uint8_t*>(p.h_mem);
    std::memset(h, 0, p.bytes);
    if (src.table_bytes) std::memcpy(h, src.table, src.table_bytes);
    if (index_bytes) std::memcpy(h + index_at, src.index.data(), index_bytes);
    if (!src.header.empty()) std::memcpy(h + header_at, src.header.data(), src.header.size());
    g_plans.push_front(std::move(p));
    g_index.emplace(hash, g_plans.begin());
    while (g_plans.size() > kMaxPlans) {
        Plan& old = g_plans.back();
        destroy_plan(old);
        const auto range = g_index.equal_range(old.hash);
        for (auto it = range.first; it != range.second; ++it)
            if (&*it->second == &old) { g_index.erase(it); break; }
        g_plans.pop_back();
    }
    *out = &g_plans.front();
    return FLASHOPTIM_OK;
}

// Brings a step's table up to date in stream order if any descriptor has changed since its last update.  A rate that all
// tensors share, if it is all that has changed of the rates, is left to the launch (*lr_by_launch): its kernels take the
// rate from their arguments and write it into the table.  Not in a captured call, whose kernels read the table at every
// replay, as the latest call on the list has left it.  The new values travel as kernel arguments: no staging memory is
// involved, so nothing is waited for however far the stream is behind, and a captured update writes the same values at
// every replay (from the first one on, what the table holds when a later call runs is not known here).
int refresh_table(Plan& p, const std::vector<TensorDev>& tensors, bool shared_lr, hipStream_t stream, bool* lr_by_launch) {
    auto bits = [](float x) { uint32_t u; std::memcpy(&u, &x, sizeof(u)); return u; };
    uint64_t grad = 0;          // bits that differ (the same list: what a call can change are these three)
    uint32_t lr = 0, wd = 0;
    const size_t n = tensors.size();
    for (size_t i = 0; i < n; ++i) {
        const TensorDev &x = p.tensors[i], &y = tensors[i];
        grad |= (uint64_t)reinterpret_cast<uintptr_t>(x.grad) ^ (uint64_t)reinterpret_cast<uintptr_t>(y.grad);
        lr |= bits(x.lr) ^ bits(y.lr);
        wd |= bits(x.wd) ^ bits(y.wd);
    }
    *lr_by_launch = false;
    if (p.in_graphs) p.table_known = false;
    if (p.table_known && !grad && !lr && !wd) return FLASHOPTIM_OK;
    const bool capturing = is_capturing(stream);
    fo::TableUpdate u;
    u.fields = fo::kUpdateGrad | fo::kUpdateLr | fo::kUpdateWd;
    if (p.table_known) {
        *lr_by_launch = lr && shared_lr && !capturing;
        u.fields = (grad ? fo::kUpdateGrad : 0) | (lr && !*lr_by_launch ? fo::kUpdateLr : 0) | (wd ? fo::kUpdateWd : 0);
    }
    if (*lr_by_launch)
        for (size_t i = 0; i < n; ++i) p.tensors[i].lr = tensors[i].lr;
    if (!u.fields) return FLASHOPTIM_OK;
    if (capturing) p.in_graphs = true;
    const uint32_t most = fo::update_batch(u.fields);
    p.table_known = false;      // until every launch has been accepted
    for (size_t first = 0; first < n; first += u.count) {
        u.first = (uint32_t)first;
        u.count = n - first < most ? (uint32_t)(n - first) : most;
        uint32_t* w = u.words;
        for (size_t i = first; i < first + u.count; ++i) {
            TensorDev& x = p.tensors[i];
            const TensorDev& y = tensors[i];
            if (u.fields & fo::kUpdateGrad) {
                x.grad = y.grad;
                const uint64_t g = (uint64_t)reinterpret_cast<uintptr_t>(y.grad);
                *w++ = (uint32_t)g;
                *w++ = (uint32_t)(g >> 32);
            }
            if (u.fields & fo::kUpdateLr) *w++ = bits(x.lr = y.lr);
            if (u.fields & fo::kUpdateWd) *w++ = bits(x.wd = y.wd);
        }
        FO_HIP(fo::launch_table_update(u, static_cast<TensorDev*>(p.d_table), stream));
    }
    p.table_known = true;
    return FLASHOPTIM_OK;
}

// ------------------------------------------------------------------- steps --

int validate_tensors(const flashoptim_tensor* t, int64_t n, bool has_v) {
    if (n < 0 || (n > 0 && t == nullptr)) return FLASHOPTIM_ERR_INVALID_ARG;
    for (int64_t i = 0; i < n; ++i) {
        const flashoptim_tensor& x = t[i];
        if (x.numel < 0 || x.numel >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
        if (x.numel == 0) continue;
        if (!x.param || !x.rho || !x.m_q || !x.m_scale) return FLASHOPTIM_ERR_INVALID_ARG;
        if (has_v && (!x.v_q || !x.v_scale)) return FLASHOPTIM_ERR_INVALID_ARG;
        if (!aligned16(x.param) || !aligned16(x.rho) || !aligned16(x.m_q) || !aligned16(x.m_scale))
            return FLASHOPTIM_ERR_MISALIGNED;
        if (has_v && (!aligned16(x.v_q) || !aligned16(x.v_scale))) return FLASHOPTIM_ERR_MISALIGNED;
    }
    return FLASHOPTIM_OK;
}

TensorDev to_dev(const flashoptim_tensor& x, bool has_v) {
    TensorDev d;
    std::memset(&d, 0, sizeof(d));
    d.param = x.param; d.rho = x.rho; d.grad = x.grad; d.m_q = x.m_q; d.m_scale = x.m_scale;
    d.v_q = has_v ? x.v_q : nullptr; d.v_scale = has_v ? x.v_scale : nullptr;
    d.numel = x.numel; d.lr = x.lr; d.wd = x.weight_decay;
    return d;
}

// Validation and conversion of the extended descriptors of the ablation entry points: only the
// buffers that the chosen variant uses are required (and passed on).
int to_dev_ex(const flashoptim_tensor_ex* t, int64_t n, bool has_v, bool split, bool quant,
              std::vector<TensorDev>& live) {
    if (n < 0 || (n > 0 && t == nullptr)) return FLASHOPTIM_ERR_INVALID_ARG;
    for (int64_t i = 0; i < n; ++i) {
        const flashoptim_tensor_ex& x = t[i];
        if (x.t.numel < 0 || x.t.numel >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
        if (x.t.numel == 0) continue;
        const void* need[8];
        int k = 0;
        need[k++] = x.t.grad;
        if (split) { need[k++] = x.t.param; need[k++] = x.t.rho; } else need[k++] = x.theta;
        if (quant) {
            need[k++] = x.t.m_q; need[k++] = x.t.m_scale;
            if (has_v) { need[k++] = x.t.v_q; need[k++] = x.t.v_scale; }
        } else {
            need[k++] = x.m;
            if (has_v) need[k++] = x.v;
        }
        for (int j = 0; j < k; ++j) if (!need[j]) return FLASHOPTIM_ERR_INVALID_ARG;
        for (int j = 0; j < k; ++j) if (!aligned16(need[j])) return FLASHOPTIM_ERR_MISALIGNED;
    }
    for (int64_t i = 0; i < n; ++i) {
        const flashoptim_tensor_ex& x = t[i];
        if (x.t.numel == 0) continue;
        TensorDev d;
        std::memset(&d, 0, sizeof(d));
        d.grad = x.t.grad; d.numel = x.t.numel; d.lr = x.t.lr; d.wd = x.t.weight_decay;
        if (split) { d.param = x.t.param; d.rho = x.t.rho; } else d.theta32 = x.theta;
        if (quant) {
            d.m_q = x.t.m_q; d.m_scale = x.t.m_scale;
            if (has_v) { d.v_q = x.t.v_q; d.v_scale = x.t.v_scale; }
        } else {
            d.m32 = x.m;
            if (has_v) d.v32 = x.v;
        }
        live.push_back(d);
    }
    return FLASHOPTIM_OK;
}

// What a multi-tensor launch runs: an optimizer step (kOpStepExact: with the exactly rounded division of
// the AdamW update), a layout conversion, or the stream probe.
enum LiveOp { kOpStep = 0, kOpCompress = 1, kOpDecompress = 2, kOpProbe = 3, kOpStepExact = 4 };
constexpr int32_t kOpPack = 5, kOpUnpack = 6;

hipError_t launch_segment(LiveOp op, int kind, bool direct, bool split, bool quant, fo::StepShape shape, const StepArgs& a,
                          int64_t blocks, hipStream_t stream) {
    if (op == kOpStep || op == kOpStepExact)
        return fo::launch_step(kind, direct, split, quant, shape, op == kOpStepExact, a, blocks, stream);
    if (op == kOpProbe) return fo::launch_probe(kind, direct, shape, a, blocks, stream);
    return fo::launch_convert(kind == FLASHOPTIM_ADAMW, op == kOpCompress, direct, a, blocks, stream);
}

// The workgroups 0 .. blocks-1 of one logical launch (each handles `tile_elems` elements), issued as
// back-to-back launches on the same stream, each covering at most kSegmentElems elements.
hipError_t launch_op(LiveOp op, int kind, bool direct, bool split, bool quant, fo::StepShape shape, StepArgs a, int64_t blocks,
                     int64_t tile_elems, hipStream_t stream) {
    const auto launch_part = [&](int64_t first, int64_t n, bool through) {
        a.block_offset = (uint32_t)first;
        a.through = through;
        return launch_segment(op, kind, direct, split, quant, shape, a, n, stream);
    };
    if (op != kOpCompress && op != kOpDecompress) return fo::for_each_step_segment(kind, split, quant, blocks, tile_elems, launch_part);
    return fo::for_each_segment(blocks, tile_elems, [&](int64_t first, int64_t n) { return launch_part(first, n, a.through); });
}

// Launches one operation over the live tensors (already validated and converted).
int launch_live(int kind, bool split, bool quant, std::vector<TensorDev>& live, const StepConsts& c,
                hipStream_t stream, LiveOp op = kOpStep, const float* sqrt_min_word = nullptr) {
    if (live.empty()) return FLASHOPTIM_OK;
    StepArgs a;
    std::memset(&a, 0, sizeof(a));
    a.c = c;
    a.sqrt_min_word = sqrt_min_word;
    int64_t elems = 0;
    for (const TensorDev& d : live) elems += d.numel;
    const fo::StepShape shape = fo::step_shape(kind, split, quant, elems);
    const bool convert = op == kOpCompress || op == kOpDecompress;
    if (convert) a.through = fo::convert_through(elems);
    const int64_t ce = convert ? fo::convert_chunk(op == kOpCompress, a.through) : fo::chunk_elems(split, quant, shape);
    // one workgroup per chunk: the launch grid is a 31-bit count
    uint32_t log2_ce = 0;
    while (((int64_t)1 << log2_ce) < ce) ++log2_ce;        // every tile size is a power of two
    int64_t total_chunks = 0;
    for (TensorDev& d : live) {
        const int64_t tiles = (d.numel + ce - 1) >> log2_ce;
        d.first_tile = (uint32_t)total_chunks;             // (in range once the total has been checked)
        d.n_tiles = (uint32_t)tiles;
        total_chunks += tiles;
    }
    if (total_chunks > (int64_t)0x7fffffff) return FLASHOPTIM_ERR_NUMEL_RANGE;

    if (live.size() == 1) {
        // gradient-release call: no table, no allocation, no lock
        a.single = live[0];
        FO_HIP(launch_op(op, kind, true, split, quant, shape, a, total_chunks, ce, stream));
        return FLASHOPTIM_OK;
    }

    const bool step = op == kOpStep || op == kOpStepExact;
    bool shared_lr = true;
    for (TensorDev& d : live) {
        if (!step) d.lr = d.wd = 0.0f;         // not used
        shared_lr = shared_lr && std::memcmp(&d.lr, &live[0].lr, sizeof(float)) == 0;
    }

    PlanTag tag = {0, (int32_t)op, kind, (int32_t)(split ? 1 : 0) | (int32_t)(quant ? 2 : 0), nullptr};
    FO_HIP(hipGetDevice(&tag.device));
    const uint64_t hash = identity_hash(tag, live);
    const uint32_t shift = fo::coarse_shift(total_chunks);
    std::lock_guard<std::mutex> lock(g_mu);
    Plan* plan = find_plan(tag, hash, live);
    int rc = FLASHOPTIM_OK;
    if (!plan) {
        // the coarse workgroup -> tensor table
        std::vector<uint32_t> coarse((size_t)fo::coarse_entries(total_chunks, shift));
        size_t ti = 0;
        for (size_t j = 0; j < coarse.size(); ++j) {
            const int64_t b = (int64_t)j << shift;
            while ((int64_t)live[ti].first_tile + live[ti].n_tiles <= b) ++ti;
            coarse[j] = (uint32_t)ti;
        }
        coarse.push_back((uint32_t)live.size() - 1);
        const std::vector<uint8_t> no_header;
        rc = make_plan(tag, hash, live, {live.data(), live.size() * sizeof(TensorDev), coarse, no_header},
                       total_chunks, &plan);
    }
    if (rc == FLASHOPTIM_OK) rc = upload_tables(*plan, stream);
    bool lr_by_launch = false;
    if (rc == FLASHOPTIM_OK) rc = refresh_table(*plan, live, shared_lr, stream, &lr_by_launch);
    if (rc != FLASHOPTIM_OK) return rc;
    a.table_lr_mask = lr_by_launch ? 0u : ~0u;
    if (lr_by_launch) std::memcpy(&a.shared_lr_bits, &live[0].lr, sizeof(float));
    a.tensors = static_cast<TensorDev*>(plan->d_table);
    a.coarse = static_cast<const uint32_t*>(plan->d_index);
    a.coarse_shift = shift;
    const hipError_t e = launch_op(op, kind, false, split, quant, shape, a, plan->n_chunks, ce, stream);
    if (e != hipSuccess) plan->table_known = false;        // the launches that were accepted may have written a rate
    FO_HIP(e);
    return FLASHOPTIM_OK;
}

// The short square root of the AdamW kernels (reciprocal-square-root estimate plus one correction) is
// exactly rounded on a device only if the hardware estimate makes it so.  The kernels therefore read the
// smallest v_t they may give to it from a word of device memory that starts at +inf (never: sqrtf
// throughout).  The first AdamW step on a device puts the check of every value of the sequence's range on
// its stream, ahead of its own kernels (about 4 ms on MI355X), followed by a one-lane kernel that lowers
// the word to 2^-96 if every value passed.  Nothing is allocated and the host does not wait: work that
// runs before the verdict has landed (another stream's, say) uses sqrtf and gets the same results.
// FLASHOPTIM_FORCE_GENERAL_SQRT in the environment leaves the word at +inf (for testing that path).
constexpr int kMaxDevices = 64;
static __device__ float sqrt_min_word = __builtin_inff();
static __device__ unsigned long long sqrt_check_counters[fo::kSelftestCounters];

__global__ void sqrt_verdict_kernel(unsigned long long* counters, float* word, unsigned long long expected) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const bool ok = counters[4] == expected && counters[5] == 0;
        *word = ok ? 1.2621774483536189e-29f /* 2^-96 */ : __builtin_inff();
        counters[4] = 0;
        counters[5] = 0;
    }
}

struct SqrtCheck {
    std::atomic<int> state;       // 0 not started, 1 verified, 2 not to be used, 3 on its way (see `done`)
    float* word;                  // device address of sqrt_min_word on this device
    hipEvent_t done;              // recorded behind the verdict kernel
};
SqrtCheck g_sqrt[kMaxDevices];
std::mutex g_sqrt_mu;

// Device address of the word the AdamW kernels read on the current device.  With `start`, the check is put
// on `stream` first if this device has not had it yet (not while the stream is being captured: the check
// belongs in front of a graph, not inside it).
int sqrt_min_word_of_device(hipStream_t stream, bool start, const float** out) {
    int dev = 0;
    FO_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return FLASHOPTIM_ERR_INVALID_ARG;
    SqrtCheck& s = g_sqrt[dev];
    if (s.state.load(std::memory_order_acquire) == 0 || !s.word) {
        std::lock_guard<std::mutex> lock(g_sqrt_mu);
        if (!s.word) {
            void* sym = nullptr;
            FO_HIP(hipGetSymbolAddress(&sym, HIP_SYMBOL(sqrt_min_word)));
            if (!sym) return FLASHOPTIM_ERR_HIP;
            s.word = static_cast<float*>(sym);
        }
        if (start && s.state.load(std::memory_order_acquire) == 0) {
            hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
            FO_HIP(hipStreamIsCapturing(stream, &cap));
            const char* force = std::getenv("FLASHOPTIM_FORCE_GENERAL_SQRT");
            if (force && force[0] != '\0' && force[0] != '0') {
                s.state.store(2, std::memory_order_release);
            } else if (cap == hipStreamCaptureStatusNone) {
                void* sym = nullptr;
                FO_HIP(hipGetSymbolAddress(&sym, HIP_SYMBOL(sqrt_check_counters)));
                if (!sym) return FLASHOPTIM_ERR_HIP;
                unsigned long long* counters = static_cast<unsigned long long*>(sym);
                if (!s.done) FO_HIP(hipEventCreateWithFlags(&s.done, hipEventDisableTiming));
                StepConsts c0;
                std::memset(&c0, 0, sizeof(c0));
                FO_HIP(fo::launch_selftest(counters, 2, c0, 1.0f, stream));
                hipLaunchKernelGGL(sqrt_verdict_kernel, dim3(1), dim3(64), 0, stream, counters, s.word,
                                   (unsigned long long)fo::kSelftestSqrtValues);
                FO_HIP(hipGetLastError());
                FO_HIP(hipEventRecord(s.done, stream));
                s.state.store(3, std::memory_order_release);
            }
        }
    }
    *out = s.word;
    return FLASHOPTIM_OK;
}

// Operand limits of the short square root and division of the AdamW kernels for this call (StepConsts).
void set_ranges(StepConsts& c) {
    c.sqrt_min = INFINITY;      // the kernels replace it by the device's word
    const bool eps_ok = c.eps >= fo::kDivFastLo && c.eps <= 1.0f;
    const double slack = 1.0 - 1.0 / 1048576.0;       // the limits are rounded to FP32: stay below the exact quotient
    c.v_max = eps_ok ? (float)((double)fo::kDivFastHi / (double)c.rbc2 * slack) : -1.0f;
    c.m_max = eps_ok ? (float)((double)fo::kDivFastHi / (double)c.rbc1 * slack) : -1.0f;
}

int run_step(int kind, const flashoptim_tensor* tensors, int64_t n_tensors, const StepConsts& c, void* stream_,
             LiveOp op = kOpStep) {
    const bool has_v = (kind == FLASHOPTIM_ADAMW);
    int rc = validate_tensors(tensors, n_tensors, has_v);
    if (rc != FLASHOPTIM_OK) return rc;
    for (int64_t i = 0; i < n_tensors; ++i) {
        if (tensors[i].numel == 0) continue;
        if (!tensors[i].grad) return FLASHOPTIM_ERR_INVALID_ARG;
        if (!aligned16(tensors[i].grad)) return FLASHOPTIM_ERR_MISALIGNED;
    }
    std::vector<TensorDev> live;
    live.reserve((size_t)n_tensors);
    for (int64_t i = 0; i < n_tensors; ++i)
        if (tensors[i].numel > 0) live.push_back(to_dev(tensors[i], has_v));
    StepConsts cc = c;
    const float* word = nullptr;
    if (has_v && op != kOpProbe && !live.empty()) {
        rc = sqrt_min_word_of_device(static_cast<hipStream_t>(stream_), true, &word);
        if (rc != FLASHOPTIM_OK) return rc;
        set_ranges(cc);
    }
    return launch_live(kind, true, true, live, cc, static_cast<hipStream_t>(stream_), op, word);
}

// Conversion between the FP32 state and the compressed layout: every buffer of both layouts is needed.
int run_convert(int kind, const flashoptim_tensor_ex* t, int64_t n, bool compress, void* stream_) {
    if (kind < 0 || kind > 2) return FLASHOPTIM_ERR_INVALID_ARG;
    const bool has_v = (kind == FLASHOPTIM_ADAMW);
    if (n < 0 || (n > 0 && t == nullptr)) return FLASHOPTIM_ERR_INVALID_ARG;
    std::vector<TensorDev> live;
    for (int64_t i = 0; i < n; ++i) {
        const flashoptim_tensor_ex& x = t[i];
        if (x.t.numel < 0 || x.t.numel >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
        if (x.t.numel == 0) continue;
        const void* need[10] = {x.t.param, x.t.rho, x.t.m_q, x.t.m_scale, x.theta, x.m,
                                has_v ? (const void*)x.t.v_q : x.theta, has_v ? (const void*)x.t.v_scale : x.theta,
                                has_v ? (const void*)x.v : x.theta, x.theta};
        for (const void* p : need) if (!p) return FLASHOPTIM_ERR_INVALID_ARG;
        for (const void* p : need) if (!aligned16(p)) return FLASHOPTIM_ERR_MISALIGNED;
    }
    for (int64_t i = 0; i < n; ++i) {
        const flashoptim_tensor_ex& x = t[i];
        if (x.t.numel == 0) continue;
        TensorDev d = to_dev(x.t, has_v);
        d.grad = nullptr;
        d.theta32 = x.theta; d.m32 = x.m; d.v32 = has_v ? x.v : nullptr;
        live.push_back(d);
    }
    StepConsts c;
    std::memset(&c, 0, sizeof(c));
    return launch_live(kind, true, true, live, c, static_cast<hipStream_t>(stream_), compress ? kOpCompress : kOpDecompress);
}

int run_step_ex(int kind, const flashoptim_tensor_ex* tensors, int64_t n_tensors, const StepConsts& c,
                unsigned flags, void* stream_) {
    if (flags & ~(unsigned)(FLASHOPTIM_SPLIT_WEIGHTS | FLASHOPTIM_QUANTIZE_STATES)) return FLASHOPTIM_ERR_INVALID_ARG;
    const bool split = (flags & FLASHOPTIM_SPLIT_WEIGHTS) != 0, quant = (flags & FLASHOPTIM_QUANTIZE_STATES) != 0;
    std::vector<TensorDev> live;
    int rc = to_dev_ex(tensors, n_tensors, kind == FLASHOPTIM_ADAMW, split, quant, live);
    if (rc != FLASHOPTIM_OK) return rc;
    StepConsts cc = c;
    const float* word = nullptr;
    if (kind == FLASHOPTIM_ADAMW && !live.empty()) {
        rc = sqrt_min_word_of_device(static_cast<hipStream_t>(stream_), true, &word);
        if (rc != FLASHOPTIM_OK) return rc;
        set_ranges(cc);
    }
    // the ablation and reference variants always use the exactly rounded arithmetic
    return launch_live(kind, split, quant, live, cc, static_cast<hipStream_t>(stream_), kOpStepExact, word);
}

// 1 / (float)(1 - beta^t): the bias correction is formed in double and rounded to FP32
// once; its reciprocal is one FP32 division.
float recip_bias_correction(float beta, int64_t t) {
    const float bc = (float)(1.0 - std::pow((double)beta, (double)t));
    return 1.0f / bc;
}

// ---------------------------------------------------------------- checkpoint --

const char kMagic[8] = {'F', 'O', 'P', 'T', 'C', 'K', 'P', 'T'};

int64_t tensor_payload(int64_t n, int kind) {
    int64_t b = align64(2 * n) + align64(n) + align64(n) + align64(2 * n_groups(n));
    if (kind == FLASHOPTIM_ADAMW) b += align64(n) + align64(2 * n_groups(n));
    return b;
}

void put_i64(uint8_t* p, int64_t v) { for (int i = 0; i < 8; ++i) p[i] = (uint8_t)((uint64_t)v >> (8 * i)); }
void put_u32(uint8_t* p, uint32_t v) { for (int i = 0; i < 4; ++i) p[i] = (uint8_t)(v >> (8 * i)); }

int64_t header_size(int64_t n) { return 64 + align64(16 * n); }

std::vector<uint8_t> build_header(int kind, const flashoptim_tensor* t, int64_t n, int64_t step, int64_t total) {
    std::vector<uint8_t> h((size_t)header_size(n), 0);
    std::memcpy(h.data(), kMagic, 8);
    put_u32(h.data() + 8, 1u);
    put_u32(h.data() + 12, (uint32_t)kind);
    put_i64(h.data() + fo::kHeaderStepAt, step);
    put_i64(h.data() + 24, n);
    put_i64(h.data() + 32, total);
    int64_t off = (int64_t)h.size();
    for (int64_t i = 0; i < n; ++i) {
        put_i64(h.data() + 64 + 16 * i, t[i].numel);
        put_i64(h.data() + 64 + 16 * i + 8, off);
        off += tensor_payload(t[i].numel, kind);
    }
    return h;
}

// Segments (one per section per tensor) between the tensors' buffers and the blob.
void build_segments(int kind, const flashoptim_tensor* t, int64_t n, uint8_t* blob, bool pack,
                    std::vector<CopySegment>& segs) {
    int64_t off = header_size(n);
    auto add = [&](const void* tensor_buf, int64_t bytes) {
        if (bytes > 0) {
            CopySegment s;
            if (pack) { s.src = static_cast<const uint8_t*>(tensor_buf); s.dst = blob + off; s.pad_bytes = align64(bytes); }
            else { s.src = blob + off; s.dst = static_cast<uint8_t*>(const_cast<void*>(tensor_buf)); s.pad_bytes = bytes; }
            s.bytes = bytes;
            s.first_piece = s.n_pieces = 0;
            segs.push_back(s);
        }
        off += align64(bytes);
    };
    for (int64_t i = 0; i < n; ++i) {
        const int64_t ne = t[i].numel, ng = n_groups(ne);
        add(t[i].param, 2 * ne); add(t[i].rho, ne); add(t[i].m_q, ne); add(t[i].m_scale, 2 * ng);
        if (kind == FLASHOPTIM_ADAMW) { add(t[i].v_q, ne); add(t[i].v_scale, 2 * ng); }
    }
}

int check_elementwise(const void* a, const void* b, const void* c, int64_t n) {
    if (n < 0 || n >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
    if (n == 0) return FLASHOPTIM_OK;
    if (!a || !b || !c) return FLASHOPTIM_ERR_INVALID_ARG;
    if (!aligned16(a) || !aligned16(b) || !aligned16(c)) return FLASHOPTIM_ERR_MISALIGNED;
    return FLASHOPTIM_OK;
}

// ------------------------------------------------------------ workspaces of waiting calls --
//
// The calls that return values to the host (quantisation error, unpack's header check) let a kernel write them to
// pinned memory, which they watch; unpack also needs a word of device memory by which its check admits its copy.  They are kept from
// call to call (allocating and freeing them cost ~20 us a call, and freeing waits for every stream of the device); a call takes a
// workspace out of the pool for as long as it runs, so calls of several threads and streams never share one, and a
// workspace goes back only once its kernels have written all that they write there or their stream has been waited for.  One kernel
// may still be to run then: the copy of an unpack that was admitted, which reads the word and stands any later use of it
// (verdict_word in flashoptim_launch.h).
struct CallSpace {
    int device = 0;
    uint64_t* verdict = nullptr;    // device memory: the word
    uint8_t* host = nullptr;        // pinned and coherent: kSpaceHost bytes, the flag and the quantisation error's words behind them
    uint64_t seq = 0;               // the workspace's uses so far: the ticket of the current one

    uint32_t ticket() const { return (uint32_t)seq; }      // (never 0)
    uint32_t* flag() const;
    uint64_t* words() const;
};
constexpr size_t kSpaceHost = 64;               // two values of eight bytes
constexpr size_t kFlagStride = 64;              // bytes: the flag has a cache line of its own
constexpr size_t kSpaceWords = (size_t)fo::kNmseMaxBlocks * fo::kNmseWords * sizeof(uint64_t);
uint32_t* CallSpace::flag() const { return reinterpret_cast<uint32_t*>(host + kSpaceHost); }
uint64_t* CallSpace::words() const { return reinterpret_cast<uint64_t*>(host + kSpaceHost + kFlagStride); }
std::mutex g_space_mu;
constexpr int kMaxIdleSpaces = 16;              // 32 KB of pinned memory and 64 bytes of device memory each; what more calls
CallSpace g_space_idle[kMaxIdleSpaces];         // than that give back at once is freed
int g_space_n_idle = 0;

// Frees a workspace, after everything on its device: a copy that was admitted may still read its word.
void destroy_space(CallSpace& w) {
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(w.device);
    if (w.verdict) (void)hipDeviceSynchronize();
    if (w.verdict) (void)hipFree(w.verdict);
    if (w.host) (void)hipHostFree(w.host);
    (void)hipSetDevice(cur);
    w = CallSpace();
}

int take_space(CallSpace& w) {
    FO_HIP(hipGetDevice(&w.device));
    {
        std::lock_guard<std::mutex> lock(g_space_mu);
        for (int i = 0; i < g_space_n_idle; ++i) {
            if (g_space_idle[i].device != w.device) continue;
            w = g_space_idle[i];
            g_space_idle[i] = g_space_idle[--g_space_n_idle];
            ++w.seq;
            if (w.ticket() == 0) {      // tickets start over: no word may hold one that comes again
                std::memset(w.host, 0, kSpaceHost + kFlagStride + kSpaceWords);
                ++w.seq;
            }
            return FLASHOPTIM_OK;
        }
    }
    hipError_t e = hipMalloc((void**)&w.verdict, 64);
    if (e == hipSuccess) e = hipHostMalloc((void**)&w.host, kSpaceHost + kFlagStride + kSpaceWords, hipHostMallocCoherent);
    if (e != hipSuccess) {
        destroy_space(w);
        g_last_hip_error = (int)e;
        (void)hipGetLastError();
        return FLASHOPTIM_ERR_HIP;
    }
    std::memset(w.host, 0, kSpaceHost + kFlagStride + kSpaceWords);
    w.seq = 1;
    return FLASHOPTIM_OK;
}

// Takes a workspace back whose work is known to have finished.
void give_space(CallSpace& w) {
    std::lock_guard<std::mutex> lock(g_space_mu);
    if (g_space_n_idle < kMaxIdleSpaces) g_space_idle[g_space_n_idle++] = w;
    else destroy_space(w);
}

// Waits until is_set() finds in the pinned memory of `w` what the work that uses it (launched with result `e`) writes there.  For up
// to 2 ms the host watches it without a pause: it sees it some microseconds before the runtime reports the stream idle (2^24 momentum
// values, when that was written: 31.5 -> 27.9 us a call).  Longer work is waited for through the stream if nothing is behind it (`last`).  Otherwise the
// host goes on watching, with pauses, and now and then asks whether the stream has failed or run dry without it: waiting for the
// stream would be waiting for what is enqueued behind as well (unpack's copy, 14 ms for 41 GB).  If anything failed the workspace is
// freed, which waits for whatever may still use it.
template <typename F>
int wait_space(CallSpace& w, hipError_t e, hipStream_t stream, bool last, F is_set) {
    auto done = [&] {
        if (!is_set()) return false;
        std::atomic_thread_fence(std::memory_order_acquire);
        return true;
    };
    if (e == hipSuccess) {
        const auto t0 = std::chrono::steady_clock::now();
        for (uint32_t k = 1;; ++k) {
            if (done()) return FLASHOPTIM_OK;
            if (k % 64 == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(2)) break;
        }
        for (uint32_t k = 1;; ++k) {
            if (last) {
                e = hipStreamSynchronize(stream);
            } else {
                std::this_thread::sleep_for(std::chrono::microseconds(20));
                e = k % 256 == 0 ? hipStreamQuery(stream) : hipErrorNotReady;
                if (k % 256 == 0) (void)hipGetLastError();      // ("not ready" is no error of a later launch's)
            }
            if ((e == hipSuccess || e == hipErrorNotReady) && done()) return FLASHOPTIM_OK;
            if (e == hipSuccess) e = hipErrorUnknown;           // (never: the kernel that sets it has run)
            if (e != hipErrorNotReady) break;
        }
    }
    g_last_hip_error = (int)e;
    (void)hipGetLastError();
    destroy_space(w);
    return FLASHOPTIM_ERR_HIP;
}

// ------------------------------------------------------------------- copies --

// Copies between the list's buffers and the blob.  The blob's header and table follow from the list but for the step, so the
// plan holds them on the device.  When packing they go with the copy, and the step is an argument of the kernel: nothing is
// staged per call, calls behind any amount of earlier work never wait, and a captured one can be replayed.  When unpacking
// (check: the workspace that the host will wait for) a kernel compares them with the blob's ahead of the copy, which does
// nothing unless they agree, or the workgroups of the copy do so themselves (checked_copy).
int run_copy(int kind, const flashoptim_tensor* t, int64_t n, uint8_t* blob, bool pack, int64_t total_bytes, int64_t step,
             hipStream_t stream, CallSpace* check = nullptr) {
    // the identity: every tensor, those without elements included (they lengthen the header and move the sections)
    std::vector<TensorDev> list;
    list.reserve((size_t)n);
    for (int64_t i = 0; i < n; ++i) {
        TensorDev d = to_dev(t[i], kind == FLASHOPTIM_ADAMW);
        d.grad = nullptr;
        d.lr = d.wd = 0.0f;
        list.push_back(d);
    }
    PlanTag tag = {0, pack ? kOpPack : kOpUnpack, kind, 0, blob};
    FO_HIP(hipGetDevice(&tag.device));
    const uint64_t hash = identity_hash(tag, list);
    int64_t total = 0;
    for (const TensorDev& d : list) total += tensor_payload(d.numel, kind);
    // (one workgroup per piece, sections included that end in a short piece, and one for the header: a 32-bit index)
    if (total / fo::kCopyPiece + 6 * n + 1 > (int64_t)0x7fffffff) return FLASHOPTIM_ERR_NUMEL_RANGE;
    std::lock_guard<std::mutex> lock(g_mu);
    Plan* plan = find_plan(tag, hash, list);
    if (!plan) {
        std::vector<CopySegment> segs;
        build_segments(kind, t, n, blob, pack, segs);
        int64_t n_pieces = 0;
        for (CopySegment& sg : segs) {
            sg.first_piece = (uint32_t)n_pieces;
            sg.n_pieces = (uint32_t)((sg.pad_bytes + fo::kCopyPiece - 1) / fo::kCopyPiece);
            n_pieces += sg.n_pieces;
        }
        const uint32_t shift = fo::coarse_shift(n_pieces);
        std::vector<uint32_t> coarse((size_t)fo::coarse_entries(n_pieces, shift));
        size_t si = 0;
        for (size_t j = 0; j < coarse.size(); ++j) {
            const int64_t b = (int64_t)j << shift;
            while ((int64_t)segs[si].first_piece + segs[si].n_pieces <= b) ++si;
            coarse[j] = (uint32_t)si;
        }
        coarse.push_back(segs.empty() ? 0 : (uint32_t)segs.size() - 1);
        const std::vector<uint8_t> header = build_header(kind, t, n, 0, total_bytes);
        const int rc = make_plan(tag, hash, list, {segs.data(), segs.size() * sizeof(CopySegment), coarse, header},
                                 n_pieces, &plan);
        if (rc != FLASHOPTIM_OK) return rc;
        plan->coarse_shift = shift;
    }
    const int rc = upload_tables(*plan, stream);
    if (rc != FLASHOPTIM_OK) return rc;
    fo::CopyArgs a;
    std::memset(&a, 0, sizeof(a));
    a.segs = static_cast<const CopySegment*>(plan->d_table);
    a.coarse = static_cast<const uint32_t*>(plan->d_index);
    a.coarse_shift = plan->coarse_shift;
    a.n_pieces = (uint32_t)plan->n_chunks;
    int64_t* found = pack ? nullptr : reinterpret_cast<int64_t*>(check->host);
    if (pack) {
        a.header = static_cast<const uint4*>(plan->d_header);
        a.header_n16 = (uint32_t)(header_size(n) / 16);
        a.header_dst = reinterpret_cast<uint4*>(blob);
        a.step = step;
    } else if (a.n_pieces > 0 && fo::checked_copy(total_bytes, header_size(n))) {
        fo::CheckedCopyArgs c(a);
        c.header = static_cast<const uint4*>(plan->d_header);
        c.header_n16 = (uint32_t)(header_size(n) / 16);
        c.ticket = check->seq;
        c.found = reinterpret_cast<const uint4*>(blob);
        c.out = found;
        c.flag = check->flag();
        FO_HIP(fo::launch_checked_copy(c, stream));
        return FLASHOPTIM_OK;
    } else {
        FO_HIP(fo::launch_check_header(plan->d_header, blob, (size_t)header_size(n), check->verdict, found,
                                       check->flag(), check->seq, stream));
        a.verdict = check->verdict;
        a.ticket = check->seq;
    }
    FO_HIP(fo::launch_copy(a, stream));
    return FLASHOPTIM_OK;
}

// ------------------------------------------ the step entry point that allocates nothing --
//
// For callers that cannot allocate device memory (stream capture, tight serving loops): the two device
// tables of a multi-tensor launch live in a fixed array that every GPU holds from library load to process
// end, instead of in a cached allocation.  `scratch` is the array's host-side stand-in: host code never
// passes it anywhere; it asks the runtime once per device for the array's device address and uses that.
constexpr int64_t kShardUnit = 256;     // elements: a shard that starts on a multiple has every stream 16-byte aligned
constexpr int kNoAllocMaxTensors = 1024;
constexpr size_t kScratchTableBytes = kNoAllocMaxTensors * sizeof(TensorDev);                 // 106,496
constexpr size_t kScratchBytes = kScratchTableBytes + (fo::kCoarseMaxEntries + 1) * sizeof(uint32_t);   // + 65,540
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

std::atomic<unsigned char*> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mu;

// Device address of the array on `dev`, which must be the current device.
int scratch_of_device(int dev, unsigned char** out) {
    if (dev < 0 || dev >= kMaxDevices) return FLASHOPTIM_ERR_INVALID_ARG;
    unsigned char* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        p = g_scratch_ptr[dev].load(std::memory_order_acquire);
        if (!p) {
            void* sym = nullptr;
            FO_HIP(hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)));
            if (!sym) return FLASHOPTIM_ERR_HIP;
            p = static_cast<unsigned char*>(sym);
            g_scratch_ptr[dev].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return FLASHOPTIM_OK;
}

// Tensor descriptors reach the table as kernel arguments (no host-to-device copy, hence no staging memory).
constexpr int kTableBatch = 32;
struct TableBatch {
    uint32_t first, count;
    TensorDev t[kTableBatch];
};
static_assert(sizeof(TableBatch) <= 4096, "kernel arguments");
__global__ __launch_bounds__(64) void noalloc_fill_table(TableBatch b, TensorDev* table) {
    if (threadIdx.x < b.count) table[b.first + threadIdx.x] = b.t[threadIdx.x];
}
// coarse[j] = the tensor that holds tile j << shift: the last one whose first tile is not beyond it (every tensor of the
// table has at least one tile, so first_tile increases strictly).  The last of the n_coarse entries is the last tensor.
__global__ __launch_bounds__(256) void noalloc_fill_coarse(const TensorDev* table, uint32_t n_tensors,
                                                           uint32_t* coarse, uint32_t n_coarse, uint32_t shift) {
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_coarse) return;
    coarse[j] = j + 1 == n_coarse ? n_tensors - 1
                                  : fo::entry_of(j << shift, 0, n_tensors - 1, [&](uint32_t i) { return table[i].first_tile; });
}

}  // namespace

extern "C" {

// 255 * sqrt(1 / rbc2), evaluated in double and handed to the kernels as two floats.
static void set_k255(StepConsts& c) {
    const double k = 255.0 * std::sqrt(1.0 / (double)c.rbc2);
    c.k255_hi = (float)k;
    c.k255_lo = (float)(k - (double)c.k255_hi);
}

static bool adamw_consts(const flashoptim_adamw_hp* hp, StepConsts& c) {
    if (!hp || hp->step < 1) return false;
    std::memset(&c, 0, sizeof(c));
    c.beta1 = hp->beta1; c.beta2 = hp->beta2;
    c.omb1 = 1.0f - hp->beta1; c.omb2 = 1.0f - hp->beta2;
    c.rbc1 = recip_bias_correction(hp->beta1, hp->step);
    c.rbc2 = recip_bias_correction(hp->beta2, hp->step);
    c.eps = hp->eps;
    set_k255(c);
    return true;
}
static bool sgd_consts(const flashoptim_sgd_hp* hp, StepConsts& c) {
    if (!hp) return false;
    std::memset(&c, 0, sizeof(c));
    c.beta1 = hp->momentum;
    return true;
}
static bool lion_consts(const flashoptim_lion_hp* hp, StepConsts& c) {
    if (!hp) return false;
    std::memset(&c, 0, sizeof(c));
    c.beta1 = hp->beta1; c.beta2 = hp->beta2;
    c.omb1 = 1.0f - hp->beta1; c.omb2 = 1.0f - hp->beta2;
    return true;
}

int flashoptim_adamw_step(const flashoptim_tensor* tensors, int64_t n_tensors, const flashoptim_adamw_hp* hp,
                          void* stream) {
    StepConsts c;
    if (!adamw_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step(FLASHOPTIM_ADAMW, tensors, n_tensors, c, stream);
}

int flashoptim_adamw_step_exact(const flashoptim_tensor* tensors, int64_t n_tensors, const flashoptim_adamw_hp* hp,
                                void* stream) {
    StepConsts c;
    if (!adamw_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step(FLASHOPTIM_ADAMW, tensors, n_tensors, c, stream, kOpStepExact);
}

int flashoptim_sgd_step(const flashoptim_tensor* tensors, int64_t n_tensors, const flashoptim_sgd_hp* hp,
                        void* stream) {
    StepConsts c;
    if (!sgd_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step(FLASHOPTIM_SGD, tensors, n_tensors, c, stream);
}

int flashoptim_lion_step(const flashoptim_tensor* tensors, int64_t n_tensors, const flashoptim_lion_hp* hp,
                         void* stream) {
    StepConsts c;
    if (!lion_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step(FLASHOPTIM_LION, tensors, n_tensors, c, stream);
}

int flashoptim_adamw_step_ex(const flashoptim_tensor_ex* tensors, int64_t n_tensors, const flashoptim_adamw_hp* hp,
                             unsigned flags, void* stream) {
    StepConsts c;
    if (!adamw_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step_ex(FLASHOPTIM_ADAMW, tensors, n_tensors, c, flags, stream);
}

int flashoptim_sgd_step_ex(const flashoptim_tensor_ex* tensors, int64_t n_tensors, const flashoptim_sgd_hp* hp,
                           unsigned flags, void* stream) {
    StepConsts c;
    if (!sgd_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step_ex(FLASHOPTIM_SGD, tensors, n_tensors, c, flags, stream);
}

int flashoptim_lion_step_ex(const flashoptim_tensor_ex* tensors, int64_t n_tensors, const flashoptim_lion_hp* hp,
                            unsigned flags, void* stream) {
    StepConsts c;
    if (!lion_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    return run_step_ex(FLASHOPTIM_LION, tensors, n_tensors, c, flags, stream);
}

int flashoptim_stream_probe(int kind, const flashoptim_tensor* tensors, int64_t n_tensors, void* stream) {
    if (kind < 0 || kind > 2) return FLASHOPTIM_ERR_INVALID_ARG;
    StepConsts c;
    std::memset(&c, 0, sizeof(c));
    return run_step(kind, tensors, n_tensors, c, stream, kOpProbe);
}

int flashoptim_compress_state(int kind, const flashoptim_tensor_ex* tensors, int64_t n_tensors, void* stream) {
    return run_convert(kind, tensors, n_tensors, true, stream);
}

int flashoptim_decompress_state(int kind, const flashoptim_tensor_ex* tensors, int64_t n_tensors, void* stream) {
    return run_convert(kind, tensors, n_tensors, false, stream);
}

int flashoptim_split_weights(const float* theta, void* param_bf16, int8_t* rho, int64_t n, void* stream) {
    int rc = check_elementwise(theta, param_bf16, rho, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_split(8, theta, param_bf16, rho, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_reconstruct_weights(const void* param_bf16, const int8_t* rho, float* theta, int64_t n, void* stream) {
    int rc = check_elementwise(param_bf16, rho, theta, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_reconstruct(8, param_bf16, rho, theta, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_split_weights_i16(const float* theta, void* param_bf16, int16_t* rho, int64_t n, void* stream) {
    int rc = check_elementwise(theta, param_bf16, rho, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_split(16, theta, param_bf16, rho, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_reconstruct_weights_i16(const void* param_bf16, const int16_t* rho, float* theta, int64_t n,
                                       void* stream) {
    int rc = check_elementwise(param_bf16, rho, theta, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_reconstruct(16, param_bf16, rho, theta, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

// Runs the sweep and copies the first n_stats statistics to the host.
static int run_sweep(int correction_bits, int ulp_reading, uint64_t first, uint64_t stride, double* stats,
                     int n_stats, void* stream_) {
    if ((correction_bits != 8 && correction_bits != 16) || (ulp_reading != 0 && ulp_reading != 1) || stride == 0 ||
        !stats)
        return FLASHOPTIM_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const uint64_t limit = 1ull << 32;
    const uint64_t count = first < limit ? (limit - first + stride - 1) / stride : 0;
    for (int i = 0; i < n_stats; ++i) stats[i] = 0.0;
    if (count == 0) return FLASHOPTIM_OK;
    const int rc = refuse_capture(stream);
    if (rc != FLASHOPTIM_OK) return rc;
    double* d = nullptr;
    FO_HIP(hipMalloc((void**)&d, fo::kSweepStats * sizeof(double)));
    hipError_t e = hipMemsetAsync(d, 0, fo::kSweepStats * sizeof(double), stream);
    if (e == hipSuccess) e = fo::launch_sweep(correction_bits, ulp_reading == 1, first, stride, count, d, stream);
    if (e == hipSuccess) e = hipMemcpyAsync(stats, d, (size_t)n_stats * sizeof(double), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    (void)hipFree(d);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        (void)hipGetLastError();
        return FLASHOPTIM_ERR_HIP;
    }
    return FLASHOPTIM_OK;
}

int flashoptim_reconstruction_sweep(int correction_bits, uint64_t first, uint64_t stride, double* stats,
                                    void* stream) {
    return run_sweep(correction_bits, 0, first, stride, stats, 8 + 2 * 256, stream);
}

int flashoptim_reconstruction_sweep_ex(int correction_bits, int ulp_reading, uint64_t first, uint64_t stride,
                                       double* stats, void* stream) {
    return run_sweep(correction_bits, ulp_reading, first, stride, stats, fo::kSweepStats, stream);
}

int flashoptim_quantize_momentum(const float* m, int8_t* q, uint16_t* scale, int64_t n, void* stream) {
    int rc = check_elementwise(m, q, scale, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_quantize(false, false, m, q, scale, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_dequantize_momentum(const int8_t* q, const uint16_t* scale, float* m, int64_t n, void* stream) {
    int rc = check_elementwise(q, scale, m, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_dequantize(false, false, q, scale, m, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_quantize_variance(const float* v, uint8_t* q, uint16_t* scale, int64_t n, void* stream) {
    int rc = check_elementwise(v, q, scale, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_quantize(true, false, v, q, scale, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_dequantize_variance(const uint8_t* q, const uint16_t* scale, float* v, int64_t n, void* stream) {
    int rc = check_elementwise(q, scale, v, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_dequantize(true, false, q, scale, v, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_quantize_state(int state, int linear, const float* x, void* q, uint16_t* scale, int64_t n,
                              void* stream) {
    if (state < 0 || state > 1 || linear < 0 || linear > 1) return FLASHOPTIM_ERR_INVALID_ARG;
    int rc = check_elementwise(x, q, scale, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_quantize(state == 1, linear == 1, x, q, scale, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_dequantize_state(int state, int linear, const void* q, const uint16_t* scale, float* x, int64_t n,
                                void* stream) {
    if (state < 0 || state > 1 || linear < 0 || linear > 1) return FLASHOPTIM_ERR_INVALID_ARG;
    int rc = check_elementwise(q, scale, x, n);
    if (rc != FLASHOPTIM_OK || n == 0) return rc;
    FO_HIP(fo::launch_dequantize(state == 1, linear == 1, q, scale, x, n, static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_quantization_nmse(int state, int linear, const float* x, int64_t n, double* sums, void* stream_) {
    if (state < 0 || state > 1 || linear < 0 || linear > 1 || !sums) return FLASHOPTIM_ERR_INVALID_ARG;
    if (n < 0 || n >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
    sums[0] = sums[1] = 0.0;
    if (n == 0) return FLASHOPTIM_OK;
    if (!x) return FLASHOPTIM_ERR_INVALID_ARG;
    if (!aligned16(x)) return FLASHOPTIM_ERR_MISALIGNED;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    int rc = refuse_capture(stream);
    if (rc != FLASHOPTIM_OK) return rc;
    CallSpace w;
    rc = take_space(w);
    if (rc != FLASHOPTIM_OK) return rc;
    // the workgroups' pairs are added up in their order, each as soon as it is there
    const int blocks = fo::nmse_blocks(n);
    const volatile uint64_t* words = w.words();
    const uint32_t ticket = w.ticket();
    double err = 0.0, ref = 0.0;
    int next = 0;
    rc = wait_space(w, fo::launch_nmse(state == 1, linear == 1, x, n, w.words(), ticket, stream), stream, true, [&] {
        for (; next < blocks; ++next) {
            uint64_t pair[fo::kNmseWords];
            for (int k = 0; k < fo::kNmseWords; ++k) pair[k] = words[next * fo::kNmseWords + k];
            if (!fo::nmse_ready(pair, ticket)) return false;
            // (what the device has written is in no cache of the host's: 16 lines ahead)
            if (next + 32 < blocks) __builtin_prefetch(const_cast<const uint64_t*>(words) + (next + 32) * fo::kNmseWords);
            const uint64_t bits[2] = {fo::nmse_sum(pair, 0), fo::nmse_sum(pair, 1)};
            double d[2];
            std::memcpy(d, bits, sizeof(d));
            err += d[0];
            ref += d[1];
        }
        return true;
    });
    if (rc != FLASHOPTIM_OK) return rc;
    sums[0] = err;
    sums[1] = ref;
    give_space(w);
    return FLASHOPTIM_OK;
}

int64_t flashoptim_checkpoint_size(int kind, const int64_t* numels, int64_t n_tensors) {
    if (kind < 0 || kind > 2 || n_tensors < 0 || (n_tensors > 0 && !numels)) return FLASHOPTIM_ERR_INVALID_ARG;
    int64_t total = header_size(n_tensors);
    for (int64_t i = 0; i < n_tensors; ++i) {
        if (numels[i] < 0 || numels[i] >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
        total += tensor_payload(numels[i], kind);
    }
    return total;
}

static int64_t list_size(int kind, const flashoptim_tensor* t, int64_t n) {
    std::vector<int64_t> numels((size_t)n);
    for (int64_t i = 0; i < n; ++i) numels[(size_t)i] = t[i].numel;
    return flashoptim_checkpoint_size(kind, numels.data(), n);
}

int flashoptim_checkpoint_pack(int kind, const flashoptim_tensor* tensors, int64_t n_tensors, int64_t step,
                               void* blob, int64_t blob_bytes, void* stream_) {
    if (kind < 0 || kind > 2 || !blob) return FLASHOPTIM_ERR_INVALID_ARG;
    int rc = validate_tensors(tensors, n_tensors, kind == FLASHOPTIM_ADAMW);
    if (rc != FLASHOPTIM_OK) return rc;
    if (!aligned16(blob)) return FLASHOPTIM_ERR_MISALIGNED;
    const int64_t total = list_size(kind, tensors, n_tensors);
    if (total < 0) return (int)total;
    if (blob_bytes < total) return FLASHOPTIM_ERR_BAD_BLOB;
    // (header and table reach the blob in stream order, like the sections: earlier work may still be using it)
    return run_copy(kind, tensors, n_tensors, static_cast<uint8_t*>(blob), true, total, step,
                    static_cast<hipStream_t>(stream_));
}

int flashoptim_checkpoint_unpack(int kind, const void* blob, int64_t blob_bytes, const flashoptim_tensor* tensors,
                                 int64_t n_tensors, int64_t* step_out, void* stream_) {
    if (kind < 0 || kind > 2 || !blob || !step_out) return FLASHOPTIM_ERR_INVALID_ARG;
    int rc = validate_tensors(tensors, n_tensors, kind == FLASHOPTIM_ADAMW);
    if (rc != FLASHOPTIM_OK) return rc;
    if (!aligned16(blob)) return FLASHOPTIM_ERR_MISALIGNED;
    const int64_t total = list_size(kind, tensors, n_tensors);
    if (total < 0) return (int)total;
    if (blob_bytes < total) return FLASHOPTIM_ERR_BAD_BLOB;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    rc = refuse_capture(stream);
    if (rc != FLASHOPTIM_OK) return rc;
    CallSpace w;
    rc = take_space(w);
    if (rc != FLASHOPTIM_OK) return rc;
    rc = run_copy(kind, tensors, n_tensors, static_cast<uint8_t*>(const_cast<void*>(blob)), false, total, 0, stream, &w);
    if (rc != FLASHOPTIM_OK) {
        destroy_space(w);       // (the check may be on its way: freeing waits for it)
        return rc;
    }
    const volatile uint32_t* flag = w.flag();
    rc = wait_space(w, hipSuccess, stream, false, [&] { return *flag == w.ticket(); });
    if (rc != FLASHOPTIM_OK) return rc;
    int64_t found[2];
    std::memcpy(found, w.host, sizeof(found));
    if (!found[0]) {
        // The copy that was not admitted has to have run before the workspace's next use can write its word.  (One that checks the blob
        // itself has no word; it is waited for all the same, so that a refused call leaves nothing to run.)
        const hipError_t e = hipStreamSynchronize(stream);
        if (e != hipSuccess) destroy_space(w);
        FO_HIP(e);
        give_space(w);
        return FLASHOPTIM_ERR_BAD_BLOB;
    }
    give_space(w);
    *step_out = found[1];
    return FLASHOPTIM_OK;
}

// Runs the self-test sections and copies the raw device counters to h.
static int run_selftest(unsigned long long (&h)[fo::kSelftestCounters], bool only_faithful, void* stream_) {
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    const int rc = refuse_capture(stream);
    if (rc != FLASHOPTIM_OK) return rc;
    unsigned long long* d = nullptr;
    FO_HIP(hipMalloc((void**)&d, fo::kSelftestCounters * sizeof(unsigned long long)));
    hipError_t e = hipMemsetAsync(d, 0, fo::kSelftestCounters * sizeof(unsigned long long), stream);
    StepConsts c;
    std::memset(&c, 0, sizeof(c));
    if (e == hipSuccess) e = fo::launch_selftest(d, 6, c, 1.0f, stream);
    if (!only_faithful) {
        for (int section = 0; section < 4 && e == hipSuccess; ++section) e = fo::launch_selftest(d, section, c, 1.0f, stream);
        if (e == hipSuccess) e = fo::launch_selftest(d, 5, c, 1.0f, stream);
        // variance codes: the estimate depends on the call's bias correction (rbc2 and the constant derived from it), so
        // the section runs with the pairs of steps 1..20 and of a log-spaced set up to 10^6, for four
        // values of beta2, each with three group scales
        const float beta2s[4] = {0.95f, 0.99f, 0.999f, 0.9999f};
        const float scales[3] = {0.000244140625f /* 2^-12 */, 0.00131988525390625f, 0.03125f};
        for (int b = 0; b < 4 && e == hipSuccess; ++b) {
            for (int i = 0; i < fo::kSelftestVarSteps && e == hipSuccess; ++i) {
                c.rbc2 = recip_bias_correction(beta2s[b], fo::selftest_var_step(i));
                set_k255(c);
                for (int k = 0; k < 3 && e == hipSuccess; ++k) e = fo::launch_selftest(d, 4, c, 1.0f / scales[k], stream);
            }
        }
    }
    if (e == hipSuccess) e = hipMemcpyAsync(h, d, sizeof(h), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    (void)hipFree(d);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        (void)hipGetLastError();
        return FLASHOPTIM_ERR_HIP;
    }
    return FLASHOPTIM_OK;
}

int flashoptim_selftest(int64_t* n_checked, int64_t* n_failed, void* stream) {
    if (!n_checked || !n_failed) return FLASHOPTIM_ERR_INVALID_ARG;
    unsigned long long h[fo::kSelftestCounters] = {0};
    const int rc = run_selftest(h, false, stream);
    if (rc != FLASHOPTIM_OK) return rc;
    int64_t failed = 0;
    for (int sct = 0; sct < fo::kSelftestSectionCount; ++sct) {
        n_checked[sct] = (int64_t)h[2 * sct];
        n_failed[sct] = (int64_t)h[2 * sct + 1];
        failed += n_failed[sct];
    }
    return failed == 0 ? FLASHOPTIM_OK : FLASHOPTIM_ERR_SELFTEST;
}

int flashoptim_faithful_rounding_stats(int64_t* counts, void* stream) {
    if (!counts) return FLASHOPTIM_ERR_INVALID_ARG;
    unsigned long long h[fo::kSelftestCounters] = {0};
    const int rc = run_selftest(h, true, stream);
    if (rc != FLASHOPTIM_OK) return rc;
    counts[0] = (int64_t)h[12]; counts[1] = (int64_t)h[14];     // operand pairs, quotients that are not the exactly rounded one
    return h[13] == 0 ? FLASHOPTIM_OK : FLASHOPTIM_ERR_SELFTEST;
}

int flashoptim_clock_monitor(uint64_t* samples, int64_t n_samples, double seconds_per_sample, double* tick_hz,
                             void* stream) {
    // the kernel's lifetime is bounded by n_samples x seconds_per_sample: at most ten seconds in all
    if (!samples || n_samples < 1 || n_samples > 100000 || !(seconds_per_sample > 0.0) || seconds_per_sample > 1.0 ||
        (double)n_samples * seconds_per_sample > 10.0 || !tick_hz)
        return FLASHOPTIM_ERR_INVALID_ARG;
    int dev = 0, khz = 0;
    FO_HIP(hipGetDevice(&dev));
    FO_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (khz <= 0) return FLASHOPTIM_ERR_HIP;
    *tick_hz = 1e3 * (double)khz;
    const unsigned long long ticks = (unsigned long long)(seconds_per_sample * *tick_hz);
    FO_HIP(fo::launch_clock_monitor(reinterpret_cast<unsigned long long*>(samples), (int)n_samples, ticks ? ticks : 1,
                                    static_cast<hipStream_t>(stream)));
    return FLASHOPTIM_OK;
}

int flashoptim_short_sqrt_state(void) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return FLASHOPTIM_ERR_HIP; }
    if (dev < 0 || dev >= kMaxDevices) return 2;
    const float* word_dev = nullptr;
    const int rc = sqrt_min_word_of_device(nullptr, false, &word_dev);
    if (rc != FLASHOPTIM_OK) return rc;
    SqrtCheck& s = g_sqrt[dev];
    std::lock_guard<std::mutex> lock(g_sqrt_mu);
    int st = s.state.load(std::memory_order_acquire);
    if (st == 1) return st;
    // read the word the kernels read: after the verdict if the check is on its way; in the other states it
    // must still hold +inf
    float word = 0.0f;
    if (st == 3) FO_HIP(hipEventSynchronize(s.done));
    FO_HIP(hipMemcpy(&word, word_dev, sizeof(word), hipMemcpyDeviceToHost));
    if (st == 3) {
        st = word < INFINITY ? 1 : 2;
        s.state.store(st, std::memory_order_release);
    } else if (!(word == INFINITY)) {
        return FLASHOPTIM_ERR_SELFTEST;
    }
    return st;
}

int flashoptim_shard_range(int64_t numel, int64_t world, int64_t rank, int64_t* begin, int64_t* len) {
    if (numel < 0 || numel >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
    if (world < 1 || rank < 0 || rank >= world || !begin || !len) return FLASHOPTIM_ERR_INVALID_ARG;
    const int64_t units = (numel + kShardUnit - 1) / kShardUnit;      // the last unit may be short
    const int64_t base = units / world, extra = units % world;
    const int64_t first = rank * base + (rank < extra ? rank : extra);
    const int64_t count = base + (rank < extra ? 1 : 0);
    const int64_t b = first * kShardUnit, e = (first + count) * kShardUnit;
    *begin = b < numel ? b : numel;
    *len = (e < numel ? e : numel) - *begin;
    return FLASHOPTIM_OK;
}

int flashoptim_adamw_step_noalloc(const flashoptim_tensor* tensors, int64_t n_tensors, const flashoptim_adamw_hp* hp,
                                  void* stream_) {
    StepConsts c;
    if (!adamw_consts(hp, c)) return FLASHOPTIM_ERR_INVALID_ARG;
    int rc = validate_tensors(tensors, n_tensors, true);
    if (rc != FLASHOPTIM_OK) return rc;
    int64_t elems = 0;
    for (int64_t i = 0; i < n_tensors; ++i) elems += tensors[i].numel;
    const fo::StepShape shape = fo::step_shape(FLASHOPTIM_ADAMW, true, true, elems);
    const int64_t ce = fo::chunk_elems(true, true, shape);
    int64_t n_live = 0, total_tiles = 0, only = -1;
    for (int64_t i = 0; i < n_tensors; ++i) {
        if (tensors[i].numel == 0) continue;
        if (!tensors[i].grad) return FLASHOPTIM_ERR_INVALID_ARG;
        if (!aligned16(tensors[i].grad)) return FLASHOPTIM_ERR_MISALIGNED;
        ++n_live;
        only = i;
        total_tiles += (tensors[i].numel + ce - 1) / ce;
    }
    if (n_live == 0) return FLASHOPTIM_OK;
    if (n_live > kNoAllocMaxTensors) return FLASHOPTIM_ERR_LIST_TOO_LONG;
    if (total_tiles > (int64_t)0x7fffffff) return FLASHOPTIM_ERR_NUMEL_RANGE;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    int dev = 0;
    FO_HIP(hipGetDevice(&dev));
    // the short square root only where an earlier call has put its check on a stream of this device (that
    // creates an event, so it is not started from here); sqrtf otherwise: same results
    const float* word = nullptr;
    rc = sqrt_min_word_of_device(stream, false, &word);
    if (rc != FLASHOPTIM_OK) return rc;
    set_ranges(c);
    StepArgs a;
    std::memset(&a, 0, sizeof(a));
    a.c = c;
    a.sqrt_min_word = word;
    if (n_live == 1) {          // one tensor: no table at all
        a.single = to_dev(tensors[only], true);
        FO_HIP(launch_op(kOpStepExact, FLASHOPTIM_ADAMW, true, true, true, shape, a, total_tiles, ce, stream));
        return FLASHOPTIM_OK;
    }
    unsigned char* base = nullptr;
    rc = scratch_of_device(dev, &base);
    if (rc != FLASHOPTIM_OK) return rc;
    TensorDev* table = reinterpret_cast<TensorDev*>(base);
    uint32_t* coarse = reinterpret_cast<uint32_t*>(base + kScratchTableBytes);
    // the tensor table travels as kernel arguments, 32 descriptors per small launch
    TableBatch batch;
    batch.first = 0; batch.count = 0;
    int64_t first_tile = 0;
    for (int64_t i = 0; i < n_tensors; ++i) {
        if (tensors[i].numel == 0) continue;
        TensorDev d = to_dev(tensors[i], true);
        d.first_tile = (uint32_t)first_tile;
        d.n_tiles = (uint32_t)((d.numel + ce - 1) / ce);
        first_tile += d.n_tiles;
        batch.t[batch.count++] = d;
        if (batch.count == kTableBatch) {
            hipLaunchKernelGGL(noalloc_fill_table, dim3(1), dim3(64), 0, stream, batch, table);
            FO_HIP(hipGetLastError());
            batch.first += batch.count; batch.count = 0;
        }
    }
    if (batch.count) {
        hipLaunchKernelGGL(noalloc_fill_table, dim3(1), dim3(64), 0, stream, batch, table);
        FO_HIP(hipGetLastError());
    }
    const uint32_t shift = fo::coarse_shift(total_tiles);
    const uint32_t n_coarse = (uint32_t)fo::coarse_entries(total_tiles, shift) + 1;
    hipLaunchKernelGGL(noalloc_fill_coarse, dim3((n_coarse + 255) / 256), dim3(256), 0, stream, table,
                       (uint32_t)n_live, coarse, n_coarse, shift);
    FO_HIP(hipGetLastError());
    a.tensors = table;
    a.coarse = coarse;
    a.coarse_shift = shift;
    a.table_lr_mask = ~0u;
    FO_HIP(launch_op(kOpStepExact, FLASHOPTIM_ADAMW, false, true, true, shape, a, total_tiles, ce, stream));
    return FLASHOPTIM_OK;
}

const char* flashoptim_strerror(int status) {
    switch (status) {
        case FLASHOPTIM_OK: return "ok";
        case FLASHOPTIM_ERR_INVALID_ARG: return "invalid argument";
        case FLASHOPTIM_ERR_MISALIGNED: return "device pointer is not 16-byte aligned";
        case FLASHOPTIM_ERR_NUMEL_RANGE: return "numel out of range";
        case FLASHOPTIM_ERR_HIP: return "HIP runtime error";
        case FLASHOPTIM_ERR_BAD_BLOB: return "checkpoint blob too small or does not match the tensor list";
        case FLASHOPTIM_ERR_SELFTEST: return "device self-test found a hardware operation outside its documented error bound";
        case FLASHOPTIM_ERR_LIST_TOO_LONG: return "list has more tensors than the entry point without allocation holds (1024)";
        default: return "unknown status";
    }
}

int flashoptim_last_hip_error(void) { return g_last_hip_error; }

int64_t flashoptim_step_launch_count(int kind, const int64_t* numels, int64_t n_tensors) {
    if (kind < 0 || kind > 2 || n_tensors < 0 || (n_tensors > 0 && !numels)) return FLASHOPTIM_ERR_INVALID_ARG;
    int64_t tiles = 0, elems = 0;
    for (int64_t i = 0; i < n_tensors; ++i) {
        if (numels[i] < 0 || numels[i] >= kMaxNumel) return FLASHOPTIM_ERR_NUMEL_RANGE;
        elems += numels[i];
    }
    const int64_t ce = fo::chunk_elems(true, true, fo::step_shape(kind, true, true, elems));
    for (int64_t i = 0; i < n_tensors; ++i) {
        tiles += (numels[i] + ce - 1) / ce;
    }
    const int64_t seg = fo::kSegmentElems / ce > 0 ? fo::kSegmentElems / ce : 1;
    return (tiles + seg - 1) / seg;
}

int flashoptim_release_cache(void) {
    std::lock_guard<std::mutex> lock(g_mu);
    for (Plan& p : g_plans) destroy_plan(p);
    g_plans.clear();
    g_index.clear();
    std::lock_guard<std::mutex> space_lock(g_space_mu);
    while (g_space_n_idle > 0) destroy_space(g_space_idle[--g_space_n_idle]);
    return FLASHOPTIM_OK;
}

int flashoptim_version(void) { return kVersion; }

}  // extern "C"
