// C ABI of the library: argument checks, launch geometry, kernel dispatch.
//
// Every check runs before the first HIP call, so invalid calls fail the same
// way with or without a GPU.  Launch geometry follows the paper's knobs:
// the split factor decides how many vectors each work-group owns, the
// work-group size and vector width pick the kernel instance.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <new>
#include <numeric>
#include <utility>
#include <vector>

#include "lift.h"
#include "lift_apps.hpp"
#include "lift_internal.hpp"

using namespace lift;

namespace {

thread_local int g_last_hip_error = 0;
thread_local hipEvent_t g_time_start = nullptr;  // armed by lift_time_next_launch
thread_local hipEvent_t g_time_stop = nullptr;
thread_local uint64_t *g_stamps = nullptr;       // armed by lift_stamp_next_launch
thread_local int64_t g_stamp_capacity = 0;
thread_local int32_t g_rounds = COMBINE_ROUNDS;  // set by lift_combine_rounds_next_launch

int32_t take_rounds() { return std::exchange(g_rounds, COMBINE_ROUNDS); }

constexpr int MAX_DEVICES = 64;
std::atomic<int> g_cu_count[MAX_DEVICES];

lift_status hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return LIFT_EHIP;
}

// Compute units of the current device (cached per device).
lift_status cu_count(int *out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e);
    if (dev < 0 || dev >= MAX_DEVICES)
        return LIFT_EUNSUPPORTED;
    int c = g_cu_count[dev].load(std::memory_order_relaxed);
    if (c <= 0) {
        e = hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess)
            return hip_fail(e);
        if (c <= 0)
            c = 256;
        g_cu_count[dev].store(c, std::memory_order_relaxed);
    }
    *out = c;
    return LIFT_OK;
}

// The largest work-group a kernel was compiled for (its launch bound),
// cached per kernel.
lift_status max_block(const void *kernel, int *out)
{
    static std::mutex mu;
    static std::vector<std::pair<const void *, int>> cache;
    std::lock_guard<std::mutex> lock(mu);
    for (const auto &kv : cache)
        if (kv.first == kernel) {
            *out = kv.second;
            return LIFT_OK;
        }
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, kernel);
    if (e != hipSuccess)
        return hip_fail(e);
    cache.emplace_back(kernel, attr.maxThreadsPerBlock);
    *out = attr.maxThreadsPerBlock;
    return LIFT_OK;
}

// How many work-groups of `block` threads of a kernel fit on one compute
// unit at once (registers, LDS, wave slots), cached per kernel and size.
lift_status resident_per_cu(const void *kernel, int block, int *out)
{
    static std::mutex mu;
    static std::vector<std::pair<std::pair<const void *, int>, int>> cache;
    std::lock_guard<std::mutex> lock(mu);
    for (const auto &kv : cache)
        if (kv.first.first == kernel && kv.first.second == block) {
            *out = kv.second;
            return LIFT_OK;
        }
    int n = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, block, 0);
    if (e != hipSuccess)
        return hip_fail(e);
    n = std::max(n, 1);
    cache.emplace_back(std::make_pair(kernel, block), n);
    *out = n;
    return LIFT_OK;
}

// Work-items of one dispatch are counted in 32 bits (the dispatch packet's
// grid size).
constexpr int64_t MAX_DISPATCH_ITEMS = 0xFFFFFFFFLL;

lift_status launch(const void *kernel, int64_t grid, int block, void *args, hipStream_t s)
{
    if (grid <= 0 || block <= 0 || grid * block > MAX_DISPATCH_ITEMS)
        return LIFT_EUNSUPPORTED;
    void *argv[] = {args};
    hipError_t e;
    if (g_time_start || g_time_stop) {
        e = hipExtLaunchKernel(kernel, dim3((unsigned)grid), dim3((unsigned)block), argv, 0, s, g_time_start,
                               g_time_stop, 0);
        g_time_start = g_time_stop = nullptr;
    } else {
        e = hipLaunchKernel(kernel, dim3((unsigned)grid), dim3((unsigned)block), argv, 0, s);
    }
    if (e != hipSuccess)
        return hip_fail(e);
    return LIFT_OK;
}

int elem_bytes(int dt)
{
    switch (dt) {
    case LIFT_F32: return 4;
    case LIFT_BF16:
    case LIFT_F16: return 2;
    case LIFT_F64: return 8;
    default: return 0;
    }
}

bool aligned(const void *p, int64_t a) { return ((uintptr_t)p % (uintptr_t)a) == 0; }

// [p, p + bytes) and [q, q + qbytes) share a byte.
bool overlaps(const void *p, int64_t bytes, const void *q, int64_t qbytes)
{
    if (!p || !q || bytes <= 0 || qbytes <= 0)
        return false;
    uintptr_t a = (uintptr_t)p, b = (uintptr_t)q;
    return a < b + (uintptr_t)qbytes && b < a + (uintptr_t)bytes;
}

bool pow2_in(int64_t v, int64_t lo, int64_t hi)
{
    return v >= lo && v <= hi && (v & (v - 1)) == 0;
}

// Resolved launch knobs.
struct Knobs {
    int block, vec_bytes, unroll, rows;
    int64_t split;
    int wg_per_cu;
    int row_split;  // 1: wavefront per row group, 2: work-group per row
    int lanes;      // MD: lanes per particle
    int interleave; // reductions: 1 = grid-stride steps, 0 = contiguous chunks
    int lane_form;  // reductions: a lift_lane_form value
};

// Checks the caller's knobs (0 = default) and merges them with defaults.
// `lanes`: the op takes lane forms (asum / dot), whose sequential forms
// allow work-groups of 1 to 32 lanes.
lift_status resolve(const lift_knobs *k, Knobs def, int ebytes, Knobs *out, bool lanes = false)
{
    *out = def;
    if (!k)
        return LIFT_OK;
    if (k->lane_form < LIFT_LANES_TREE || k->lane_form > LIFT_LANES_RUNS_SEQ)
        return LIFT_EINVAL;
    if (lanes)
        out->lane_form = k->lane_form;
    if (k->block) {
        if (!pow2_in(k->block, lanes && (k->lane_form & LIFT_LANES_SEQ) ? 1 : 64, 1024))
            return LIFT_EINVAL;
        out->block = k->block;
    }
    if (k->vec_bytes) {
        if (!pow2_in(k->vec_bytes, 2, 16) || k->vec_bytes < ebytes)
            return LIFT_EINVAL;
        out->vec_bytes = k->vec_bytes;
    }
    if (k->unroll) {
        if (!pow2_in(k->unroll, 1, 8))
            return LIFT_EINVAL;
        out->unroll = k->unroll;
    }
    if (k->rows_per_wave) {
        if (!pow2_in(k->rows_per_wave, 1, 4))
            return LIFT_EINVAL;
        out->rows = k->rows_per_wave;
    }
    if (k->split < 0)
        return LIFT_EINVAL;
    if (k->split)
        out->split = k->split;
    if (k->wg_per_cu < 0 || k->wg_per_cu > 64 || k->row_split < 0 || k->row_split > 2)
        return LIFT_EINVAL;
    if (k->wg_per_cu)
        out->wg_per_cu = k->wg_per_cu;
    if (k->row_split)
        out->row_split = k->row_split;
    if (k->lanes_per_item) {
        if (!pow2_in(k->lanes_per_item, 1, 16))
            return LIFT_EINVAL;
        out->lanes = k->lanes_per_item;
    }
    if (k->interleave < LIFT_INTERLEAVE_DEFAULT || k->interleave > LIFT_INTERLEAVE_CHUNK)
        return LIFT_EINVAL;
    if (k->interleave)
        out->interleave = k->interleave == LIFT_INTERLEAVE_STRIDE;
    return LIFT_OK;
}

// Defaults, from the knob search on MI355X (256 CUs): reductions run about
// one long-lived work-group per CU (fewer partials, shorter combine tail),
// scal many one-step work-groups, gemv a work-group per row with x held in
// registers where one step covers a row (row_split 0 = chosen per shape).
constexpr Knobs DEF_SCAL = {256, 4, 8, 1, 0, 32, 1, 1, 0};
constexpr Knobs DEF_REDUCE = {256, 16, 8, 1, 0, 1, 1, 1, 0};
constexpr Knobs DEF_GEMV = {256, 16, 8, 1, 0, 0, 0, 1, 0};
constexpr Knobs DEF_BATCH = {256, 16, 4, 1, 65536, 2, 1, 1, 0};
constexpr Knobs DEF_BS = {256, 4, 4, 1, 0, 16, 1, 1, 0};
constexpr Knobs DEF_MD = {256, 16, 2, 1, 0, 0, 1, 16, 0};
constexpr Knobs DEF_STREAM = {256, 16, 8, 1, 0, 1, 1, 1, 0};

// ---- knobs for calls that pass none --------------------------------------
//
// A call with knobs == NULL runs with, in this order: the LIFT_FORCE_CONFIG
// override (read once from the environment), the autotuned entry for its
// op / storage / accumulation / log2 size bucket on a device of the same
// architecture and compute-unit count (generated at build time from the
// tuner's cache), or the defaults above.

enum TunedOp { TOP_SCAL = 0, TOP_ASUM, TOP_DOT, TOP_GEMV, TOP_BATCH, TOP_BS, TOP_MD, TOP_COUNT };

struct TunedEntry {
    const char *arch;  // e.g. "gfx950"; nullptr ends the table
    int cus, op, storage, acc, bucket;
    int row_bucket;    // gemv: floor(log2(n)); -1: any
    lift_knobs knobs;
};

const TunedEntry TUNED_TABLE[] = {
#include "lift_tuned_table.inc"
    {nullptr, 0, 0, 0, 0, 0, -1, {0, 0, 0, 0, 0, 0, 0, 0, 0}},
};

const char *const TUNED_OP_NAMES[TOP_COUNT] = {"scal", "asum", "dot", "gemv", "batch", "blackscholes", "md"};

int log2_bucket(int64_t elements)
{
    int b = 0;
    while (elements > 1) {
        elements >>= 1;
        ++b;
    }
    return b;
}

const TunedEntry *tuned_entry(const char *arch, int cus, int op, int storage, int acc, int64_t elements,
                              int64_t row_length)
{
    const int bucket = op == TOP_BATCH ? 0 : log2_bucket(elements);
    const int row_bucket = log2_bucket(row_length);
    for (const TunedEntry *e = TUNED_TABLE; e->arch; ++e)
        if (e->cus == cus && e->op == op && e->storage == storage && e->acc == acc && e->bucket == bucket &&
            (e->row_bucket < 0 || e->row_bucket == row_bucket) && std::strcmp(e->arch, arch) == 0)
            return e;
    return nullptr;
}

// LIFT_FORCE_CONFIG="key=value,...": keys block (or wg), vec, unroll, rpw,
// split, wgcu, rowsplit, lanes, interleave (stride | chunk), laneform; values are
// non-negative integers.  Parsed once; a malformed string makes every call
// without knobs fail with LIFT_EINVAL.
struct Forced {
    bool present = false, valid = true;
    lift_knobs knobs{};
};

bool parse_forced(const char *text, lift_knobs *k)
{
    std::memset(k, 0, sizeof *k);
    const char *p = text;
    while (*p) {
        const char *eq = std::strchr(p, '=');
        if (!eq)
            return false;
        std::string key(p, eq);
        const char *v = eq + 1;
        const char *end = std::strchr(v, ',');
        std::string val = end ? std::string(v, end) : std::string(v);
        p = end ? end + 1 : v + val.size();
        if (key == "interleave" && (val == "stride" || val == "chunk")) {
            k->interleave = val == "stride" ? LIFT_INTERLEAVE_STRIDE : LIFT_INTERLEAVE_CHUNK;
            continue;
        }
        if (val.empty() || val.size() > 12 || val.find_first_not_of("0123456789") != std::string::npos)
            return false;
        const long long x = std::stoll(val);
        if (key == "block" || key == "wg")
            k->block = (int32_t)x;
        else if (key == "vec")
            k->vec_bytes = (int32_t)x;
        else if (key == "unroll")
            k->unroll = (int32_t)x;
        else if (key == "rpw")
            k->rows_per_wave = (int32_t)x;
        else if (key == "split")
            k->split = (int64_t)x;
        else if (key == "wgcu")
            k->wg_per_cu = (int32_t)x;
        else if (key == "rowsplit")
            k->row_split = (int32_t)x;
        else if (key == "lanes")
            k->lanes_per_item = (int32_t)x;
        else if (key == "interleave")
            k->interleave = (int32_t)x;
        else if (key == "laneform")
            k->lane_form = (int32_t)x;
        else
            return false;
        if (x > INT32_MAX && key != "split")
            return false;
    }
    return true;
}

const Forced &forced_config()
{
    static Forced f;
    static std::once_flag once;
    std::call_once(once, [] {
        const char *env = std::getenv("LIFT_FORCE_CONFIG");
        if (env && *env) {
            f.present = true;
            f.valid = parse_forced(env, &f.knobs);
        }
    });
    return f;
}

// LIFT_IGNORE_TUNED set: calls without knobs go without tuned entries too.
bool ignore_tuned()
{
    static const bool set = std::getenv("LIFT_IGNORE_TUNED") != nullptr;
    return set;
}

// Architecture name (up to the first ':') and CU count of the current
// device, cached per device; false if the device cannot be queried.
bool device_identity(const char **arch, int *cus)
{
    static std::mutex mu;
    static char names[MAX_DEVICES][64];
    static int counts[MAX_DEVICES];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES)
        return false;
    std::lock_guard<std::mutex> lock(mu);
    if (counts[dev] == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess)
            return false;
        size_t i = 0;
        for (; i + 1 < sizeof names[dev] && prop.gcnArchName[i] && prop.gcnArchName[i] != ':'; ++i)
            names[dev][i] = prop.gcnArchName[i];
        names[dev][i] = 0;
        counts[dev] = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : -1;
    }
    *arch = names[dev];
    *cus = counts[dev];
    return true;
}

// The knobs a call runs with: the caller's, else forced, else tuned for this
// device, else nullptr (defaults).  *st is LIFT_EINVAL for a malformed
// LIFT_FORCE_CONFIG.
const lift_knobs *effective_knobs(const lift_knobs *given, int op, int storage, int acc, int64_t elements,
                                  lift_status *st, int64_t row_length = 0)
{
    *st = LIFT_OK;
    if (given)
        return given;
    const Forced &f = forced_config();
    if (f.present) {
        if (!f.valid)
            *st = LIFT_EINVAL;
        return &f.knobs;
    }
    const char *arch = nullptr;
    int cus = 0;
    if (ignore_tuned() || !device_identity(&arch, &cus))  // no device: defaults (the launch reports the HIP error)
        return nullptr;
    const TunedEntry *e = tuned_entry(arch, cus, op, storage, acc, elements, row_length);
    return e ? &e->knobs : nullptr;
}

// Split a range of n elements of `ebytes` bytes at base address p into a
// scalar head (up to the first vb-aligned address), whole vb-byte vectors,
// and a scalar tail.  Both p and q (if given) must share the head length.
struct Split3 {
    int64_t head, nvec;
};

bool split3(const void *p, const void *q, int64_t n, int ebytes, int vb, Split3 *out)
{
    const int64_t e = vb / ebytes;
    int64_t mis = (int64_t)((uintptr_t)p % (uintptr_t)vb);
    int64_t head = mis ? (vb - mis) / ebytes : 0;
    if (q) {
        int64_t mq = (int64_t)((uintptr_t)q % (uintptr_t)vb);
        if (mq != mis)
            return false;
    }
    head = std::min(head, n);
    out->head = head;
    out->nvec = (n - head) / e;
    return true;
}

// Vectors per work-group: the requested split (elements) or the default
// grid, rounded up to whole block * unroll steps, with the grid capped.
int64_t chunk_for(int64_t nvec, int64_t elems_per_vec, const Knobs &k, int cus, int64_t max_wg)
{
    const int64_t wg_per_cu = k.wg_per_cu;
    const int64_t step = (int64_t)k.block * k.unroll;
    int64_t chunk;
    if (k.split > 0) {
        chunk = (k.split + elems_per_vec - 1) / elems_per_vec;
    } else {
        int64_t target = (int64_t)cus * wg_per_cu;
        chunk = (nvec + target - 1) / std::max<int64_t>(target, 1);
    }
    chunk = std::max<int64_t>(step, (chunk + step - 1) / step * step);
    if ((nvec + chunk - 1) / chunk > max_wg) {
        chunk = (nvec + max_wg - 1) / max_wg;
        chunk = (chunk + step - 1) / step * step;
    }
    return chunk;
}

// Loads in flight per thread of a reduction whose launch is the library's
// choice: as few as let every work-group take one step on a compute unit of
// its own.  A vector that one work-group covers stays with it (there is no
// combine then: 16384 bf16 2.3 us against 2.7 to 2.8 over several).
//
// Replayed from a graph, us, at the fixed 8 (asum) or 4 (dot) loads and now:
// 2^16 fp32 asum 2.90 | 2.66, 2^18 fp32 3.32 | 2.97, 2^18 bf16 3.41 | 2.82, 2^20
// bf16 3.63 | 3.19; dot 2^18 bf16 3.54 | 2.89, 2^19 fp32 3.78 | 3.38.  One step
// more than that on a compute unit costs a round trip: 2^20 fp32 asum with 2
// loads 3.86, with 4 3.61.
int spread_unroll(int64_t nvec, int block, int unroll, int cus)
{
    const auto groups = [&](int u) { return (nvec + (int64_t)block * u - 1) / ((int64_t)block * u); };
    while (unroll > 1 && groups(unroll) > 1 && groups(unroll / 2) <= cus)
        unroll /= 2;
    return unroll;
}

const void *reduce_table(int dt, int op, int acc, int vb, int unroll)
{
    switch (dt) {
    case LIFT_F32: return reduce_kernel_f32(op, acc, vb, unroll);
    case LIFT_BF16: return reduce_kernel_bf16(op, acc, vb, unroll);
    case LIFT_F16: return reduce_kernel_f16(op, acc, vb, unroll);
    default: return nullptr;
    }
}

const void *dot_shifted_table(int dt, int acc)
{
    switch (dt) {
    case LIFT_F32: return dot_shifted_kernel_f32(acc);
    case LIFT_BF16: return dot_shifted_kernel_bf16(acc);
    case LIFT_F16: return dot_shifted_kernel_f16(acc);
    default: return nullptr;
    }
}

const void *gemv_table(int dt, int acc, int vb, int rows, int unroll)
{
    switch (dt) {
    case LIFT_F32: return gemv_kernel_f32(acc, vb, rows, unroll);
    case LIFT_BF16: return gemv_kernel_bf16(acc, vb, rows, unroll);
    case LIFT_F16: return gemv_kernel_f16(acc, vb, rows, unroll);
    default: return nullptr;
    }
}

const void *gemv_split_table(int dt, int acc, int vb, int rows, int unroll, bool xs)
{
    switch (dt) {
    case LIFT_F32: return gemv_split_kernel_f32(acc, vb, rows, unroll, xs);
    case LIFT_BF16: return gemv_split_kernel_bf16(acc, vb, rows, unroll, xs);
    case LIFT_F16: return gemv_split_kernel_f16(acc, vb, rows, unroll, xs);
    default: return nullptr;
    }
}

const void *gemv_rows_table(int dt, int acc, int vb, int lanes, int v, int r)
{
    switch (dt) {
    case LIFT_F32: return gemv_rows_kernel_f32(acc, vb, lanes, v, r);
    case LIFT_BF16: return gemv_rows_kernel_bf16(acc, vb, lanes, v, r);
    case LIFT_F16: return gemv_rows_kernel_f16(acc, vb, lanes, v, r);
    default: return nullptr;
    }
}

const void *gemv_rows_wg_table(int dt, int acc, int v)
{
    switch (dt) {
    case LIFT_F32: return gemv_rows_wg_kernel_f32(acc, v);
    case LIFT_BF16: return gemv_rows_wg_kernel_bf16(acc, v);
    case LIFT_F16: return gemv_rows_wg_kernel_f16(acc, v);
    default: return nullptr;
    }
}

const void *gemv_panel_table(int dt, int acc, int r)
{
    switch (dt) {
    case LIFT_F32: return gemv_panel_kernel_f32(acc, r);
    case LIFT_BF16: return gemv_panel_kernel_bf16(acc, r);
    case LIFT_F16: return gemv_panel_kernel_f16(acc, r);
    default: return nullptr;
    }
}

// Checks of a reduction's operands (everything but the workspace).
lift_status reduce_check(int op, int64_t n, int xt, const void *x, const void *y, int acc, int rt,
                         const void *result)
{
    if (n < 0)
        return LIFT_EINVAL;
    if (xt != LIFT_F32 && xt != LIFT_BF16 && xt != LIFT_F16)
        return LIFT_EINVAL;
    if (rt != LIFT_F32 && rt != LIFT_F64)
        return LIFT_EINVAL;
    if (acc != LIFT_ACC_F32 && acc != LIFT_ACC_F32_COMP && acc != LIFT_ACC_F32_F64COMBINE)
        return LIFT_EINVAL;
    const int eb = elem_bytes(xt), rb = elem_bytes(rt);
    if (!result || !aligned(result, rb))
        return LIFT_EINVAL;
    if (n > 0 && (!x || !aligned(x, eb)))
        return LIFT_EINVAL;
    if (op == OP_DOT && n > 0 && (!y || !aligned(y, eb)))
        return LIFT_EINVAL;
    const int64_t xbytes = n * eb;
    if (overlaps(result, rb, x, xbytes) || overlaps(result, rb, y, op == OP_DOT ? xbytes : 0))
        return LIFT_EINVAL;
    return LIFT_OK;
}

lift_status reduce_common(int op, int64_t n, int xt, const void *x, const void *y, int acc, int rt,
                          void *result, void *ws, size_t ws_bytes, const lift_knobs *knobs,
                          hipStream_t stream)
{
    lift_status st0 = reduce_check(op, n, xt, x, y, acc, rt, result);
    if (st0 != LIFT_OK)
        return st0;
    const int eb = elem_bytes(xt), rb = elem_bytes(rt);
    if (!ws || ws_bytes < lift_workspace_bytes())
        return LIFT_EWORKSPACE;
    if (!aligned(ws, 16))
        return LIFT_EINVAL;
    if (overlaps(result, rb, ws, (int64_t)ws_bytes))
        return LIFT_EINVAL;
    lift_status st = LIFT_OK;
    const bool choose = !knobs && !forced_config().present;   // the launch is the library's choice
    knobs = effective_knobs(knobs, op == OP_DOT ? TOP_DOT : TOP_ASUM, xt, acc, n, &st);
    if (st != LIFT_OK)
        return st;
    Knobs k;
    Knobs def = DEF_REDUCE;
    if (op == OP_DOT) {
        def.unroll = 4;  // two streams: grid-stride steps of 4 loads of each in flight
        def.interleave = 1;
    }
    st = resolve(knobs, def, eb, &k, true);
    if (st != LIFT_OK)
        return st;
    if (k.lane_form) {
        // the other lane forms: binary32 accumulation, the chunk partition
        if (acc != LIFT_ACC_F32 || (xt != LIFT_F32 && xt != LIFT_BF16))
            return LIFT_EUNSUPPORTED;
        if (knobs->interleave == LIFT_INTERLEAVE_STRIDE)
            return LIFT_EINVAL;
        k.interleave = 0;
    }

    // Vector width: the requested one if x (and y) share its alignment
    // phase, else the element size (scalar loads).
    Split3 sp{0, 0};
    int vb = k.vec_bytes;
    bool shifted = false;
    if (n > 0 && !split3(x, op == OP_DOT ? y : nullptr, n, eb, vb, &sp)) {
        // Operands of a dot in different phases: where the launch is the
        // library's choice, 16-byte loads of both, y's from wherever they
        // start (x[1:] . x[:-1] of 2^24 fp32: element loads 39.2, now 15.5 us;
        // bf16: 34.1, now 11.7 us), 512 threads x 2 loads of each; else
        // element loads, as the knobs' contract says.
        shifted = choose && !g_stamps;
        if (shifted)
            k = {512, 16, 2, 1, 0, 1, 1, 1, 1, 0};
        vb = shifted ? 16 : eb;
        split3(x, nullptr, n, eb, vb, &sp);
        while (shifted && k.block > 64 && sp.nvec <= k.block)   // half as many threads still take it in one step
            k.block /= 2;
    }
    int cus = 0;
    // Only where the order of the binary32 sums does not matter beyond the last
    // digit: asum (no cancellation) to a binary32 result, and compensated sums.
    // A dot's binary32 sums keep theirs, and so does a binary64 result.
    if (choose && !knobs && vb == 16 && !shifted &&
        (acc == LIFT_ACC_F32_COMP || (op == OP_ASUM && rt == LIFT_F32))) {
        st = cu_count(&cus);
        if (st != LIFT_OK)
            return st;
        k.unroll = spread_unroll(sp.nvec, k.block, k.unroll, cus);
    }
    const void *kern = shifted ? dot_shifted_table(xt, acc)
                       : !k.lane_form ? reduce_table(xt, op, acc, vb, k.unroll)
                       : xt == LIFT_F32 ? reduce_lanes_kernel_f32(op, vb, k.unroll, k.lane_form)
                                        : reduce_lanes_kernel_bf16(op, vb, k.unroll, k.lane_form);
    if (!kern)
        return LIFT_EUNSUPPORTED;
    st = cu_count(&cus);
    if (st != LIFT_OK)
        return st;
    const int64_t e = vb / eb;
    const int64_t chunk = chunk_for(sp.nvec, e, k, cus, MAX_WORKGROUPS);
    const int64_t grid = std::max<int64_t>(1, (sp.nvec + chunk - 1) / chunk);

    ReduceArgs a;
    a.x = x;
    a.y = y;
    a.n = n;
    a.head = sp.head;
    a.nvec = sp.nvec;
    a.chunk = chunk;
    a.ws = ws;
    a.result = result;
    a.result_f64 = rt == LIFT_F64;
    a.interleave = k.interleave;
    a.rounds = take_rounds();
    a.stamps = nullptr;
    if (g_stamps) {  // the stamped instance of the same kernel (one-shot)
        uint64_t *buf = g_stamps;
        const int64_t cap = g_stamp_capacity;
        g_stamps = nullptr;
        if (xt != LIFT_F32 || acc != LIFT_ACC_F32 || vb != 16 || k.lane_form)
            return LIFT_EUNSUPPORTED;
        if (grid > cap)
            return LIFT_EINVAL;
        kern = reduce_kernel_stamped_f32(op, k.unroll);
        if (!kern)
            return LIFT_EUNSUPPORTED;
        a.stamps = buf;
    }
    return launch(kern, grid, k.block, &a, stream);
}

// gemv whose launch is left to the library (no knobs and no tuned entry for
// its shape and alignment, or all-zero knobs): the kernels of
// lift_gemv_rows.hpp by row length.  n >= 1, m >= 1.  ws: a reduction
// workspace, or null.
//
// Measured on MI355X (us, back to back, cold inputs; before = the launch the
// library took until these kernels):
//   rows (m x n)        storage  before    now
//   1000000 x 33        f32      339       21
//   65536 x 64          f32      27        4.7
//   65536 x 257         bf16     28        10.5
//   16384 x 1000        bf16     13.8      7.6
//   20000 x 4099        bf16     42        26.9
//   20000 x 4099        f32      61        49.9
//   16384 x 8191        bf16     63        41.4
//   32 x 1048576        f32      435       27 (workspace)
lift_status gemv_by_rows(int64_t m, int64_t n, float alpha, int at, const void *A, int64_t lda, const float *x,
                         float beta, float *y, int acc, char *ws, hipStream_t stream)
{
    const int eb = elem_bytes(at);
    const int64_t e = 16 / eb;
    int cus = 0;
    lift_status st = cu_count(&cus);
    if (st != LIFT_OK)
        return st;
    GemvRowsArgs a;
    a.A = A;
    a.x = x;
    a.y = y;
    a.m = m;
    a.n = n;
    a.lda = lda;
    a.alpha = alpha;
    a.beta = beta;
    // 16-bit rows that start between two dwords have a head column; with an
    // odd pitch every other row does
    const bool odd_pitch = eb == 2 && lda % 2 != 0 && m > 1;
    a.classes = odd_pitch ? 2 : 1;
    a.heads = eb == 2 && (odd_pitch || !aligned(A, 4));
    const int64_t P = a.classes;

    const int64_t vecs = (n + e - 1) / e;      // 16-byte vectors of a row
    if (vecs <= 64 * 8) {
        // One wavefront step covers a row: as few lanes as do, several rows
        // per wavefront.  8 / v rows in flight keep 8 loads per lane in
        // flight; with fewer than 4 wavefronts per CU that way, one row each
        // spreads the rows wider (1024 x 1024 fp32: 3.95 against 4.53 us).
        // Fewer elements than one vector: element loads.
        const int vb = n < e ? eb : 16;
        int lanes = 8, v = 1, r = 8;
        if (vb == 16) {
            while (lanes < 64 && lanes < vecs)
                lanes *= 2;
            v = (int)((vecs + lanes - 1) / lanes);
            r = 8 / v;
        }
        const int64_t side = lanes < 64 ? 64 / lanes : 1;
        int64_t units = (m + side * r - 1) / (side * r);
        if (vb == 16 && units < (int64_t)cus * 4) {
            r = 1;
            units = (m + side - 1) / side;
        }
        const void *kern = gemv_rows_table(at, acc, vb, lanes, v, r);
        if (!kern)
            return LIFT_EUNSUPPORTED;
        // 8 work-groups per CU; 2 where a lane has more than one vector per
        // row (5 to 8 loads in flight with several rows, 2 to 8 with one):
        // 4096 x 4096 bf16 8.1 against 9.4, 16384 x 1000 bf16 7.5 against 7.7,
        // but 1000000 x 33 fp32 22.2 against 21.6 us
        const int64_t grid = std::min<int64_t>((units + 3) / 4, (int64_t)cus * (v > 1 ? 2 : 8));
        return launch(kern, grid, 256, &a, stream);
    }
    if (vecs <= 64 * 8 * 8) {
        // One work-group step covers a row: 3 .. 8 wavefronts x v vectors per
        // lane with the least left over (ties: the fewest wavefronts).  The
        // grid keeps about 40 KiB of loads in flight per CU (16 KiB rows:
        // 2 work-groups per CU 49.9, 4: 53.7, 8: 54.0 us for 20000 x 4099
        // fp32; rows of 12 to 13 KiB, 3 wavefronts x 5 vectors: 3 per CU, 39000 x
        // 6400 bf16 81.8 with 2, 74.4); rows of 32 KiB and more do better as more, shorter-lived
        // work-groups (16384 x 8191 fp32: 16 per CU 80.3, 2 per CU 82.8 us)
        // of at least 4 rows, each reading its part of x once (3000 x 25137
        // bf16: one row each 35.6, 2 work-groups per CU 27.9 us) -- but not
        // between 32 and 56 KiB, where a work-group has 5 to 7 wavefronts, no
        // multiple of a CU's 4 SIMDs: 2 per CU, 3 from 48 KiB on (us, as the
        // others | this: 14000 x 9800 fp32 89.3 | 86.2, 13000 x 8400 fp32 70.0 |
        // 67.4, 13000 x 20000 bf16 84.7 | 82.2, 7900 x 12000 fp32 57.4 | 56.4,
        // 12000 x 24000 bf16 88.6 | 85.6; 8500 x 16000 fp32, 64 KiB, 16 per CU
        // 77.6, 2 per CU 80.1).
        int waves = 8, v = 8;
        const int64_t need = (vecs + 63) / 64;
        for (int w = 8; w >= 3; --w)
            for (int q = 3; q <= 8; ++q)
                if ((int64_t)w * q >= need && (int64_t)w * (q - 1) * 64 < vecs && w * q <= waves * v) {
                    waves = w;
                    v = q;
                }
        const void *kern = gemv_rows_wg_table(at, acc, v);
        if (!kern)
            return LIFT_EUNSUPPORTED;
        const int64_t bytes = (int64_t)waves * v * 1024;
        int64_t per_cu = bytes > 32768 && bytes < 57344 ? (bytes < 49152 ? 2 : 3)
                         : bytes >= 32768 ? std::max<int64_t>(2, std::min<int64_t>(16, m / (4 * (int64_t)cus)))
                                          : std::max<int64_t>(2, 40960 / (need * 1024));
        // The compensated sums need wavefronts for their arithmetic: 9 of them
        // per CU at least, and from 56 KiB of 16-bit storage on the two
        // work-groups that are resident anyway (us, as the others | this:
        // 35511 x 7040 bf16 98.1 | 80.2, 32894 x 7600 bf16 92.4 | 80.5, 35511 x
        // 3520 fp32 81.4 | 74.8, 8928 x 28000 bf16 90.4 | 80.9; slower by 5 %
        // than before these kernels stay 14880 x 16800 bf16, 97, and 8928 x
        // 14000 fp32, 83).
        if (acc == LIFT_ACC_F32_COMP)
            per_cu = waves == 3 ? std::max<int64_t>(3, per_cu) : eb == 2 && bytes >= 57344 ? 2 : per_cu;
        int64_t grid = std::min<int64_t>(m, (int64_t)cus * per_cu);
        if (P == 2)
            grid -= grid % 2;
        return launch(kern, grid, waves * 64, &a, stream);
    }
    // Rows longer than that: panels of r rows, whole rows while there are
    // enough of them (3000 x 25137 fp32: r = 4 49.1, 2: 50.9, 1: 56.8 us; 4 from
    // 6 rows per CU on, where as many turns of work-groups take them: us, r = 2 |
    // 4: 1540 x 60000 bf16 42.7 | 38.6, 2047 x 60000 bf16 47.1 | 42.7, 1700 x 60000
    // fp32 71.4 | 66.7, but 1500 x 60000 bf16 36.0 | 38.4),
    // else cut in chunks (at least 16 KiB each) so that one or two
    // work-groups per CU come out as nearly even as can be.  Up to 32 KiB per
    // CU the work-groups count, not the x they share: single rows (us, r = 2
    // with chunks of 32 KiB | r = 1 with 16: 8 x 33000 bf16 6.5 | 4.4, 22 x
    // 60184 bf16 6.6 | 4.6, 64 x 45000 bf16 8.0 | 5.4, 8 x 262144 fp32 6.0 | 5.2;
    // but r = 2 | 1 with 16 KiB of 120 x 65539 bf16 7.2 | 7.4, 16 x 524288
    // fp32 8.7 | 8.9).
    const int64_t per_class = (m + P - 1) / P;
    const bool split = ws && per_class * P <= (int64_t)cus;
    const int r = per_class * P > (int64_t)cus * 6 ? 4
                  : split && m * n * eb <= (int64_t)cus * 32768 ? 1
                  : per_class > 1 && (ws || per_class * P > cus) ? 2 : 1;
    GemvPanelArgs p;
    p.rows = a;
    p.groups = P * ((per_class + r - 1) / r);
    p.chunks = 1;
    if (ws && p.groups <= cus) {
        int64_t one = cus / p.groups, two = 2 * cus / p.groups;
        int64_t c = two * p.groups * 100 > 2 * one * p.groups * 110 ? two : one;
        c = std::min<int64_t>(c, std::max<int64_t>(1, n * eb / 16384));
        c = std::min<int64_t>(c, MAX_WORKGROUPS / (p.groups * r));
        p.chunks = std::max<int64_t>(1, c);
    }
    const int64_t nv = n / e;   // the head moves a boundary by one vector at most: the last chunk ends at the row
    p.chunk = (nv + p.chunks - 1) / p.chunks;
    p.chunks = std::max<int64_t>(1, (nv + p.chunk - 1) / p.chunk);
    p.ws = ws;
    p.rounds = take_rounds();
    const void *kern = gemv_panel_table(at, acc, r);
    if (!kern)
        return LIFT_EUNSUPPORTED;
    return launch(kern, p.groups * p.chunks, 512, &p, stream);
}

bool all_zero(const lift_knobs *k)
{
    return !k->block && !k->vec_bytes && !k->unroll && !k->rows_per_wave && !k->split && !k->wg_per_cu &&
           !k->row_split && !k->lanes_per_item && !k->interleave && !k->lane_form;
}

// ws (with ws_bytes): null, or the workspace of lift_gemv_ex_ws.
lift_status gemv_common(int64_t m, int64_t n, float alpha, int at, const void *A, int64_t lda,
                        const float *x, float beta, float *y, int acc, const lift_knobs *knobs,
                        hipStream_t stream, void *ws = nullptr)
{
    if (m < 0 || n < 0 || lda < std::max<int64_t>(1, n))
        return LIFT_EINVAL;
    if (at != LIFT_F32 && at != LIFT_BF16 && at != LIFT_F16)
        return LIFT_EINVAL;
    if (acc != LIFT_ACC_F32 && acc != LIFT_ACC_F32_COMP && acc != LIFT_ACC_F32_F64COMBINE)
        return LIFT_EINVAL;
    const int eb = elem_bytes(at);
    if (m > 0 && (!y || !aligned(y, 4)))
        return LIFT_EINVAL;
    if (m > 0 && n > 0 && (!A || !x || !aligned(A, eb) || !aligned(x, 4)))
        return LIFT_EINVAL;
    const int64_t abytes = m > 0 && n > 0 ? ((m - 1) * lda + n) * eb : 0;
    if (overlaps(y, m * 4, A, abytes) || overlaps(y, m * 4, x, m > 0 ? n * 4 : 0))
        return LIFT_EINVAL;
    lift_status st = LIFT_OK;
    const lift_knobs *given = knobs;
    knobs = effective_knobs(knobs, TOP_GEMV, at, acc, m * n, &st, n);
    if (st != LIFT_OK)
        return st;
    Knobs k;
    st = resolve(knobs, DEF_GEMV, eb, &k);
    if (st != LIFT_OK)
        return st;
    if (m == 0)
        return LIFT_OK;

    // Vector path needs every row start and x aligned for the chosen width.
    int vb = k.vec_bytes;
    int64_t e = vb / eb;
    const int64_t xalign = std::min<int64_t>(e * 4, 16);
    const bool vec = n > 0 && aligned(A, vb) && (lda * eb) % vb == 0 && aligned(x, xalign);
    // The launch is the library's choice: without knobs, unless a tuned entry
    // (found on aligned rows of a power of two) or the environment override
    // decides it.  An entry stands for rows that take as many of its steps as
    // that power of two; one more step, mostly empty, or x no longer in
    // registers costs more than the row-length form (us, tuned | by rows: 9000 x
    // 30000 bf16 128 | 87, 12000 x 12000 fp32 91.3 | 85.7, 10000 x 20000 fp32 121
    // | 114, 5000 x 4104 fp32 15.7 | 14.3; but 4096 x 4096 fp32 11.5 | 12.1,
    // 8192 x 16384 fp32 76.0 | 77.6).
    const int64_t row_step = (int64_t)(k.row_split == 2 ? k.block : 64) * k.unroll * e;
    const auto steps = [&](int64_t columns) { return (columns + row_step - 1) / row_step; };
    const bool as_tuned = vec && steps(n) == steps((int64_t)1 << log2_bucket(n));
    const bool choose = given ? all_zero(given) : !forced_config().present && (!knobs || !as_tuned);
    if (choose && n > 0)
        return gemv_by_rows(m, n, alpha, at, A, lda, x, beta, y, acc, static_cast<char *>(ws), stream);
    if (!vec) {
        vb = eb;
        e = 1;
    }
    if (k.row_split == 0) {
        // library choice: a work-group per row where one step of at most 512
        // threads covers the row (x then stays in registers), sized to the row
        // unless the caller fixed the work-group size
        const int64_t nvec = n / e;
        const bool fits = (vb == 16 || vb == eb) && nvec <= (int64_t)512 * k.unroll;
        k.row_split = fits ? 2 : 1;
        if (fits && (!knobs || !knobs->block)) {
            k.block = 64;
            while ((int64_t)k.block * k.unroll < nvec && k.block < 512)
                k.block *= 2;
        }
    }
    if (!knobs || !knobs->rows_per_wave)  // wavefront form on long matrices: share x loads over 2 rows
        k.rows = k.row_split == 1 && m * n > ((int64_t)1 << 25) ? 2 : 1;
    int cus = 0;
    const void *kern;
    int64_t grid;
    int bound = 0;
    if (k.row_split == 2) {
        // the work-group streams whole rows: 16-byte loads or element loads
        if (vb != eb && vb != 16) {
            vb = eb;
            e = 1;
        }
        kern = gemv_split_table(at, acc, vb, k.rows, k.unroll, false);
        if (!kern)
            return LIFT_EUNSUPPORTED;
        st = cu_count(&cus);
        if (st == LIFT_OK)
            st = max_block(kern, &bound);  // the x-stationary instance has the same bound
        if (st != LIFT_OK)
            return st;
        k.block = std::min(k.block, bound);
        // rows that one step of the work-group covers: x stays in registers
        const bool xs = n / e <= (int64_t)k.block * k.unroll;
        if (xs)
            kern = gemv_split_table(at, acc, vb, k.rows, k.unroll, true);
        const int64_t per_cu = k.wg_per_cu ? k.wg_per_cu : (xs ? 8 : 16);
        grid = std::min<int64_t>((m + k.rows - 1) / k.rows, (int64_t)cus * per_cu);
    } else {
        kern = gemv_table(at, acc, vb, k.rows, k.unroll);
        if (!kern)
            return LIFT_EUNSUPPORTED;
        st = cu_count(&cus);
        if (st == LIFT_OK)
            st = max_block(kern, &bound);
        if (st != LIFT_OK)
            return st;
        k.block = std::min(k.block, bound);
        const int64_t waves = (m + k.rows - 1) / k.rows;
        const int64_t wpb = k.block / 64;
        grid = std::min<int64_t>((waves + wpb - 1) / wpb, (int64_t)cus * 64);
    }

    GemvArgs a;
    a.A = A;
    a.x = x;
    a.y = y;
    a.m = m;
    a.n = n;
    a.lda = lda;
    a.nvec = n / e;
    a.alpha = alpha;
    a.beta = beta;
    return launch(kern, grid, k.block, &a, stream);
}

const void *batch_table(int dt, int acc, int vb, int unroll, bool gemv)
{
    switch (dt) {
    case LIFT_F32: return batch_kernel_f32(acc, vb, unroll, gemv);
    case LIFT_BF16: return batch_kernel_bf16(acc, vb, unroll, gemv);
    case LIFT_F16: return batch_kernel_f16(acc, vb, unroll, gemv);
    default: return nullptr;
    }
}

// True if any interval of `outs` shares a byte with another interval of
// `outs` or with any interval of `ins` ([begin, end) byte ranges).
bool any_overlap(std::vector<std::pair<uintptr_t, uintptr_t>> outs,
                 std::vector<std::pair<uintptr_t, uintptr_t>> ins)
{
    std::sort(outs.begin(), outs.end());
    for (size_t i = 1; i < outs.size(); ++i)
        if (outs[i].first < outs[i - 1].second)
            return true;
    std::sort(ins.begin(), ins.end());
    // prefix maximum of input ends, to test each output against every input
    std::vector<uintptr_t> maxend(ins.size());
    uintptr_t m = 0;
    for (size_t i = 0; i < ins.size(); ++i)
        maxend[i] = m = std::max(m, ins[i].second);
    for (const auto &o : outs) {
        // inputs starting before o.second; overlap if any of them ends after o.first
        size_t k = std::lower_bound(ins.begin(), ins.end(), std::make_pair(o.second, (uintptr_t)0)) - ins.begin();
        if (k > 0 && maxend[k - 1] > o.first)
            return true;
    }
    return false;
}

// The bandwidth reference kernels: checks, then the reductions' partition
// (chunk_for) over 16-byte vectors.
lift_status stream_common(bool copy, int64_t n, const float *x, float *out, const lift_knobs *knobs,
                          hipStream_t stream)
{
    if (n < 0 || n % 4 != 0)
        return LIFT_EINVAL;
    if (n > 0 && (!x || !out || !aligned(x, 16) || !aligned(out, copy ? 16 : 4)))
        return LIFT_EINVAL;
    if (overlaps(x, n * 4, out, copy ? n * 4 : 4))
        return LIFT_EINVAL;
    Knobs k;
    lift_status st = resolve(knobs, DEF_STREAM, 4, &k);
    if (st != LIFT_OK)
        return st;
    if (k.vec_bytes != 16)
        return LIFT_EUNSUPPORTED;
    if (n == 0)
        return LIFT_OK;
    const void *kern = stream_kernel(copy, k.unroll);
    if (!kern)
        return LIFT_EUNSUPPORTED;
    int cus = 0;
    st = cu_count(&cus);
    if (st != LIFT_OK)
        return st;
    const int64_t nvec = n / 4;
    const int64_t chunk = chunk_for(nvec, 4, k, cus, MAX_DISPATCH_ITEMS / k.block);
    StreamArgs a;
    a.x = x;
    a.out = out;
    a.nvec = nvec;
    a.chunk = chunk;
    a.interleave = k.interleave;
    return launch(kern, std::max<int64_t>(1, (nvec + chunk - 1) / chunk), k.block, &a, stream);
}

// ---- allocation-free reductions --------------------------------------------
//
// lift_dot_ex_noalloc keeps its counters and partial slots in this file-scope
// device array instead of a caller workspace: one copy per device, zero-filled
// when the library's code object is loaded on it, and left as the next call
// needs it by every call (the work-group that combines clears the slots and
// counters that were used), so nothing is cleared per call.  In host code `scratch` names
// a host-side stand-in; the device address of each device's copy comes from
// hipGetSymbolAddress with that device current, once, and only that address
// is handed to kernels.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)(WS_HEADER + (int64_t)MAX_WORKGROUPS * WS_SLOT);
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

lift_status static_scratch(void **out)
{
    static std::mutex mu;
    static void *addr[MAX_DEVICES];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e);
    if (dev < 0 || dev >= MAX_DEVICES)
        return LIFT_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return hip_fail(e);
        if (!p)
            return LIFT_EHIP;
        addr[dev] = p;
    }
    *out = addr[dev];
    return LIFT_OK;
}

}  // namespace

// A planned batch: one launch over the reduction tiles ([0]) and one over
// the gemv tiles ([1]), each with its own tile table and counters.
struct lift_batch {
    int device = 0;
    int64_t nprobs = 0;
    int64_t bytes = 0;
    int block = 0;
    void *dmem = nullptr;
    int64_t ntiles[2] = {0, 0};
    int64_t grid[2] = {0, 0};
    const void *kern[2] = {nullptr, nullptr};
    BatchArgs args[2]{};
    hipEvent_t ev[2] = {nullptr, nullptr};  // inner ends of a timed two-launch run
    int storage = 0, acc = 0, vb = 0, unroll = 0;  // for the stamped gemv instance
    bool waves = false;       // one launch of wavefront tiles (grid[0], kern[0], wave_args)
    BatchWaveArgs wave_args{};
};

namespace {

const void *batch_wave_table(int dt, int acc, bool stamped)
{
    switch (dt) {
    case LIFT_F32: return batch_wave_f32(acc, stamped);
    case LIFT_BF16: return batch_wave_bf16(acc, stamped);
    case LIFT_F16: return batch_wave_f16(acc, stamped);
    default: return nullptr;
    }
}

// Work-groups of the wavefront kernel that the device holds, a multiple of
// DRAW_LISTS.
lift_status batch_wave_groups(int storage, int acc, const void **kern, int64_t *groups)
{
    *kern = batch_wave_table(storage, acc, false);
    if (!*kern)
        return LIFT_EUNSUPPORTED;
    int cus = 0, fit = 1;
    lift_status st = cu_count(&cus);
    if (st == LIFT_OK)
        st = resident_per_cu(*kern, 256, &fit);
    *groups = std::max<int64_t>(DRAW_LISTS, (int64_t)cus * std::min(fit, 4) / DRAW_LISTS * DRAW_LISTS);
    return st;
}

// How a wavefront takes the rows of a gemv tile (wave_gemv): `rows` of them in
// `steps` rounds of loads.
struct WaveRows {
    int64_t rows, steps;
};

WaveRows wave_rows_step(int64_t n, int64_t eb, int acc)
{
    const int64_t vecs = (n * eb + 15) / 16;
    if (vecs <= 64) {
        int64_t lanes = 8;
        while (lanes < 64 && lanes < vecs)
            lanes *= 2;
        return {4 * 64 / lanes, 1};
    }
    if (vecs <= 128 || (vecs <= 192 && eb == 4))
        return {2, 1};
    if (vecs <= 448 && (vecs <= 384 || eb == 4 || acc != LIFT_ACC_F32_COMP))
        return {1, 1};
    if ((vecs <= 512 && (eb == 4 || acc != LIFT_ACC_F32_COMP)) || (vecs <= 1024 && eb == 4 && acc == LIFT_ACC_F32))
        return {1, (vecs + 255) / 256};
    return {2, (vecs + 255) / 256};
}

// What a wavefront's rounds of loads cost, in bytes: one that moves less than
// 8 KiB takes no less time.
constexpr int64_t WAVE_STEP = 8192;

// A problem's share of a batch of wavefront tiles, in such bytes (a gemv row's,
// or the whole reduction's).
double wave_cost(const lift_problem &q, int64_t eb, int acc)
{
    if (q.kind != LIFT_KIND_GEMV)
        return std::max<double>(WAVE_STEP, (double)q.n * eb * (q.kind == LIFT_KIND_DOT ? 2 : 1));
    const WaveRows w = wave_rows_step(q.n, eb, acc);
    return std::max<double>((double)q.n * eb, (double)w.steps * WAVE_STEP / w.rows);
}

// Bytes of x, y and A that a batch reads, and the problems that read any.
double batch_reads(const lift_problem *probs, int32_t count, int64_t eb, int64_t *filled)
{
    double total = 0;
    *filled = 0;
    for (int32_t i = 0; i < count; ++i) {
        const lift_problem &q = probs[i];
        const double n = (double)q.n * eb * (q.kind == LIFT_KIND_GEMV ? (double)q.m : q.kind == LIFT_KIND_DOT ? 2 : 1);
        total += std::max(0.0, n);
        *filled += n > 0;
    }
    return total;
}

// Up to this many bytes per wavefront (268 MB on 256 CUs) a batch without
// knobs runs as wavefront tiles, above it as the two launches of work-group
// tiles.  Measured in us, two launches | wavefronts: 1.8 MB bf16 13.4 | 7.3,
// 94 MB f32 108 | 18, 163 MB bf16 102 | 30, 180 MB of f32 gemv 44 | 43, 194 MB
// bf16 50 | 38; but 301 MB of bf16 gemv 66 | 83, 332 MB of f32 gemv 68 | 81,
// 1.57 GB f32 250 | 303, 3.7 GB bf16 630 | 682: independent wavefronts that
// draw their tiles stream at 5.2 to 5.5 TB/s, work-groups at 5.9 to 6.5.
constexpr double BATCH_WAVE_SHARE = 65536;

// The library's choice for a batch without knobs: wavefront tiles or (false)
// work-group tiles, then with *red_split elements per reduction tile.
//
// A work-group takes 70 us for a tile of 4 MB, so with the largest tile that
// the default gives, a batch of some 100 MB ends on one.  A quarter of a
// work-group's share (2 per CU) evens that out; below 65536 elements the cost
// per tile shows (3.7 GB bf16: 624 us at 2^20, 645 at 65536, 673 at 32768).
// At the default split and with this, us: 314 MB f32 111 | 63, 514 MB bf16
// 160 | 102, 645 MB f32 181 | 117, 1.47 GB f32 243 | 235.
bool batch_choose(const lift_problem *probs, int32_t count, int storage, int acc, int64_t *red_split)
{
    const void *kern = nullptr;
    int64_t groups = 0, filled = 0;
    int cus = 0;
    const int error = g_last_hip_error;
    if (batch_wave_groups(storage, acc, &kern, &groups) != LIFT_OK || cu_count(&cus) != LIFT_OK) {
        g_last_hip_error = error;  // no device: the plan itself reports that, if its problems are in order
        return false;
    }
    const int eb = elem_bytes(storage);
    const double total = batch_reads(probs, count, eb, &filled);
    if (total <= BATCH_WAVE_SHARE * 4 * groups)
        return true;
    *red_split = std::min(*red_split, (int64_t)std::max(65536.0, std::min(1e15, total / (2 * cus) / 4 / eb)));
    return false;
}

// The plan of a batch without knobs (lift_batch_wave.hpp), its problems
// already checked.
//
// Tile size (in bytes as of wave_cost): what gives every wavefront about one
// tile (problems shorter than that leave more tiles than wavefronts, which are
// then drawn).  Never below one step of loads.
lift_status batch_plan_waves(const lift_problem *probs, int32_t count, int storage, int acc, int rt, int64_t bytes,
                             lift_batch *b)
{
    const int64_t eb = elem_bytes(storage), e = 16 / eb;
    const void *kern = nullptr;
    int64_t most = 0, filled = 0;
    lift_status st = batch_wave_groups(storage, acc, &kern, &most);
    if (st != LIFT_OK)
        return st;
    const int64_t waves = most * 4;
    double total = 0;
    batch_reads(probs, count, eb, &filled);
    for (int32_t i = 0; i < count; ++i)
        total += wave_cost(probs[i], eb, acc) * (probs[i].kind == LIFT_KIND_GEMV ? (double)probs[i].m : 1);
    const int64_t tile =
        (int64_t)std::max<double>(WAVE_STEP, std::min(1e15, total / std::max<int64_t>(waves / 2, waves - filled)));

    // Equal tiles of one problem, one after the other: a, b and out advance by
    // these many bytes, a reduction's slot and its number in its problem by 1.
    struct Run {
        WaveTile t;
        int64_t count, cost, da, db, dout;
    };
    std::vector<Run> runs;
    runs.reserve(2 * (size_t)count);
    int64_t slots = 0, kinds[2] = {0, 0};
    bool grouped = false;   // some reduction has more than TILE_GROUP tiles
    // `total` units in tiles of `unit`: a run of whole ones and the rest
    const auto cut = [&](Run r, int64_t total_units, int64_t unit, int32_t WaveTile::*length, int64_t unit_bytes) {
        const int64_t whole = total_units / unit, rest = total_units - whole * unit;
        for (int last = 0; last < 2; ++last) {
            Run part = r;
            part.count = last ? rest > 0 || total_units == 0 : whole;
            if (part.count == 0)
                continue;
            part.t.*length = (int32_t)(last ? rest : unit);
            part.cost = (last ? rest : unit) * unit_bytes + 4096;
            if (last) {
                const auto advance = [&](const void *p, int64_t d) {
                    return p ? static_cast<const char *>(p) + whole * d : nullptr;
                };
                part.t.a = advance(r.t.a, r.da);
                part.t.b = advance(r.t.b, r.db);
                part.t.out = static_cast<char *>(r.t.out) + whole * r.dout;
                if (r.t.kind != LIFT_KIND_GEMV) {
                    part.t.rows += (int32_t)whole;
                    part.t.slot += (int32_t)whole;
                }
            }
            kinds[r.t.kind == LIFT_KIND_GEMV] += part.count;
            runs.push_back(part);
        }
    };
    for (int32_t i = 0; i < count; ++i) {
        const lift_problem &q = probs[i];
        Run r;
        std::memset(&r, 0, sizeof r);
        r.t.kind = q.kind;
        r.t.problem = i;
        r.t.alpha = q.alpha;
        r.t.beta = q.beta;
        r.t.out = q.out;
        if (q.kind == LIFT_KIND_GEMV) {
            if (q.m == 0)
                continue;
            if (q.n > INT32_MAX)
                return LIFT_EUNSUPPORTED;
            // whole groups of the rows that a wavefront has in flight (pairs of
            // long rows share x: single ones only where each is several tiles)
            const WaveRows w = wave_rows_step(q.n, eb, acc);
            const double cost = wave_cost(q, eb, acc);
            const int64_t unit = w.rows == 2 && w.steps > 1 && cost > 4 * (double)tile ? 1 : w.rows;
            const int64_t want = std::max<int64_t>(unit, (int64_t)std::ceil((double)tile / cost));
            const int64_t nt = (q.m + want - 1) / want;
            int64_t rows = (q.m + nt - 1) / nt;
            rows = std::min<int64_t>((rows + unit - 1) / unit * unit, 1 << 30);
            r.t.a = q.a;
            r.t.b = q.b;
            r.t.pitch = q.lda * eb;
            r.t.n = (int32_t)q.n;
            r.t.ntiles = 1;
            r.da = rows * q.lda * eb;
            r.dout = rows * 4;
            cut(r, q.m, rows, &WaveTile::rows, (int64_t)cost);
        } else {
            const int64_t streams = q.kind == LIFT_KIND_DOT ? 2 : 1;
            const int64_t want = std::max<int64_t>(64 * e, tile / (eb * streams));
            int64_t nt = std::max<int64_t>(1, (q.n + want - 1) / want);
            int64_t len = (q.n + nt - 1) / nt;
            len = std::min<int64_t>(std::max<int64_t>(64 * e, (len + 64 * e - 1) / (64 * e) * (64 * e)), 1 << 30);
            nt = std::max<int64_t>(1, (q.n + len - 1) / len);
            grouped |= nt > TILE_GROUP;
            if (nt > TILE_GROUP)
                slots = (slots + TILE_GROUP - 1) / TILE_GROUP * TILE_GROUP;
            if (slots + nt > INT32_MAX)
                return LIFT_EUNSUPPORTED;
            r.t.a = q.n ? q.a : nullptr;
            r.t.b = q.n && streams == 2 ? q.b : nullptr;
            r.t.ntiles = (int32_t)nt;
            r.t.slot = (int32_t)slots;
            r.da = r.db = len * eb;
            cut(r, q.n, len, &WaveTile::n, eb * streams);
            slots += nt;
        }
    }
    const int64_t ntiles = kinds[0] + kinds[1];
    if (ntiles >= 1 << 30)
        return LIFT_EUNSUPPORTED;
    std::stable_sort(runs.begin(), runs.end(), [](const Run &x, const Run &y) { return x.cost > y.cost; });
    const int64_t grid = std::min<int64_t>(most, (std::max<int64_t>(ntiles, 1) + DRAW_LISTS - 1) / DRAW_LISTS * DRAW_LISTS);

    int dev = 0;
    hipError_t he = hipGetDevice(&dev);
    if (he != hipSuccess)
        return hip_fail(he);
    // one allocation: draw counters | counter and groups of work-groups that
    // left | per-problem counters | counters of groups of tiles | tiles | records
    // | slots; all but the slots in one upload
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    const int64_t off_done = up(DRAW_LISTS * WS_GROUP_STRIDE), off_groups = off_done + 256;
    const int64_t off_pc = off_groups + up((grid + ARRIVAL_GROUP - 1) / ARRIVAL_GROUP * WS_GROUP_STRIDE);
    const int64_t off_gc = off_pc + up(std::max<int64_t>(count, 1) * 4);
    const int64_t off_ti = off_gc + (grouped ? up((slots / TILE_GROUP + 1) * WS_GROUP_STRIDE) : 0);
    const int64_t off_re = off_ti + up(std::max<int64_t>(ntiles, 1) * (int64_t)sizeof(WaveTile));
    const int64_t off_sl = off_re + up(std::max<int64_t>(ntiles, 1) * 4);
    const std::unique_ptr<char[]> image(new char[(size_t)off_sl]);
    std::memset(image.get(), 0, (size_t)off_ti);
    WaveTile *table = reinterpret_cast<WaveTile *>(image.get() + off_ti);
    int32_t *records = reinterpret_cast<int32_t *>(image.get() + off_re);   // stamps: reductions first, then gemv
    int64_t at[2] = {0, kinds[0]};
    for (const Run &r : runs) {
        WaveTile w = r.t;
        for (int64_t k = 0; k < r.count; ++k) {
            *table++ = w;
            *records++ = (int32_t)at[w.kind == LIFT_KIND_GEMV]++;
            w.a = w.a ? static_cast<const char *>(w.a) + r.da : nullptr;
            w.b = w.b ? static_cast<const char *>(w.b) + r.db : nullptr;
            w.out = static_cast<char *>(w.out) + r.dout;
            if (w.kind != LIFT_KIND_GEMV) {
                ++w.rows;
                ++w.slot;
            }
        }
    }
    void *mem = nullptr;
    he = hipMalloc(&mem, (size_t)(off_sl + std::max<int64_t>(slots, 1) * WS_SLOT));
    if (he != hipSuccess)
        return hip_fail(he);
    char *base = static_cast<char *>(mem);
    if ((he = hipMemcpy(base, image.get(), (size_t)off_sl, hipMemcpyHostToDevice)) != hipSuccess) {
        hipFree(mem);
        return hip_fail(he);
    }
    b->device = dev;
    b->storage = storage;
    b->acc = acc;
    b->nprobs = count;
    b->bytes = bytes;
    b->block = 256;
    b->dmem = mem;
    b->waves = true;
    b->ntiles[0] = kinds[0];
    b->ntiles[1] = kinds[1];
    b->grid[0] = grid;
    b->kern[0] = kern;
    BatchWaveArgs &a = b->wave_args;
    a.tiles = reinterpret_cast<const WaveTile *>(base + off_ti);
    a.ntiles = (int32_t)ntiles;
    a.lists = base;
    a.done = reinterpret_cast<unsigned *>(base + off_done);
    a.groups = base + off_groups;
    a.pcount = reinterpret_cast<unsigned *>(base + off_pc);
    a.gcount = base + off_gc;
    a.slots = base + off_sl;
    a.result_f64 = rt == LIFT_F64;
    a.dynamic = ntiles > grid * 4;
    a.records = reinterpret_cast<const int32_t *>(base + off_re);
    return LIFT_OK;
}

// One run of such a plan; an armed stamp hook takes the stamped instance.
lift_status batch_run_waves(lift_batch *b, hipStream_t stream)
{
    BatchWaveArgs a = b->wave_args;
    const void *kern = b->kern[0];
    if (g_stamps) {
        a.stamps = g_stamps;
        const int64_t cap = g_stamp_capacity;
        g_stamps = nullptr;
        if (b->acc != LIFT_ACC_F32 || (b->storage != LIFT_F32 && b->storage != LIFT_BF16))
            return LIFT_EUNSUPPORTED;
        if (a.ntiles > cap)
            return LIFT_EINVAL;
        kern = batch_wave_table(b->storage, b->acc, true);
        if (!kern)
            return LIFT_EUNSUPPORTED;
    }
    return launch(kern, b->grid[0], b->block, &a, stream);
}

lift_status batch_plan(const lift_problem *probs, int32_t count, int storage, int acc, int rt,
                       const lift_knobs *knobs, lift_batch *b)
{
    if (count < 0 || (count > 0 && !probs))
        return LIFT_EINVAL;
    if (storage != LIFT_F32 && storage != LIFT_BF16 && storage != LIFT_F16)
        return LIFT_EINVAL;
    if (acc != LIFT_ACC_F32 && acc != LIFT_ACC_F32_COMP && acc != LIFT_ACC_F32_F64COMBINE)
        return LIFT_EINVAL;
    if (rt != LIFT_F32 && rt != LIFT_F64)
        return LIFT_EINVAL;
    const int eb = elem_bytes(storage), rb = elem_bytes(rt);
    lift_status st = LIFT_OK;
    const bool unset = !knobs && !forced_config().present;   // the plan is the library's choice
    knobs = effective_knobs(knobs, TOP_BATCH, storage, acc, 0, &st);
    if (st != LIFT_OK)
        return st;
    Knobs k;
    st = resolve(knobs, DEF_BATCH, eb, &k);
    if (st != LIFT_OK)
        return st;
    if (k.vec_bytes < 4)
        return LIFT_EUNSUPPORTED;  // the batched kernels load at least a dword per lane
    if (k.block > 512)
        return LIFT_EUNSUPPORTED;  // built for at most 512 threads (no register spills at 8 loads in flight)
    if (k.row_split == 2)
        return LIFT_EUNSUPPORTED;  // batch gemv tiles use one wavefront per row pair
    const int vb = k.vec_bytes;
    const int64_t e = vb / eb;
    int64_t red_split = k.split;
    const bool choose = unset && batch_choose(probs, count, storage, acc, &red_split);   // wavefront tiles

    std::vector<std::pair<uintptr_t, uintptr_t>> outs, ins;
    std::vector<BatchProblem> hp((size_t)count);
    std::vector<BatchTile> tiles[2];   // reduction tiles, gemv tiles
    std::vector<int64_t> cost[2];
    int64_t slots = 0, bytes = 0;
    const int64_t step = (int64_t)k.block * k.unroll;
    const int64_t waves = k.block / 64;
    for (int32_t i = 0; i < count; ++i) {
        const lift_problem &q = probs[i];
        BatchProblem &p = hp[(size_t)i];
        std::memset(&p, 0, sizeof p);
        if (q.reserved != 0)
            return LIFT_EINVAL;
        p.kind = q.kind;
        p.n = q.n;
        p.a = q.a;
        p.b = q.b;
        p.out = q.out;
        p.alpha = q.alpha;
        p.beta = q.beta;
        if (q.kind == LIFT_KIND_ASUM || q.kind == LIFT_KIND_DOT) {
            const bool dot = q.kind == LIFT_KIND_DOT;
            if (q.n < 0 || !q.out || !aligned(q.out, rb))
                return LIFT_EINVAL;
            if (q.n > 0 && (!q.a || !aligned(q.a, eb) || (dot && (!q.b || !aligned(q.b, eb)))))
                return LIFT_EINVAL;
            outs.push_back({(uintptr_t)q.out, (uintptr_t)q.out + rb});
            if (q.n > 0) {
                ins.push_back({(uintptr_t)q.a, (uintptr_t)q.a + q.n * eb});
                if (dot)
                    ins.push_back({(uintptr_t)q.b, (uintptr_t)q.b + q.n * eb});
            }
            Split3 sp{0, 0};
            int64_t unit_e = e;
            p.vec = 1;
            if (q.n > 0 && !split3(q.a, dot ? q.b : nullptr, q.n, eb, vb, &sp)) {
                p.vec = 0;
                unit_e = 1;
                sp.head = 0;
                sp.nvec = q.n;
            }
            p.head = sp.head;
            p.nvec = sp.nvec;
            // tile length in units (vectors or elements), whole steps
            int64_t len = std::max<int64_t>(1, (red_split + unit_e - 1) / unit_e);
            len = (len + step - 1) / step * step;
            const int64_t nt = std::max<int64_t>(1, (p.nvec + len - 1) / len);
            if (nt > INT32_MAX)
                return LIFT_EUNSUPPORTED;
            p.ntiles = (int32_t)nt;
            p.slot_base = slots;
            slots += nt;
            for (int64_t t = 0; t < nt && !choose; ++t) {
                BatchTile tl{i, (int32_t)t, t * len, std::min(len, p.nvec - t * len)};
                if (tl.len < 0)
                    tl.len = 0;
                tiles[0].push_back(tl);
                cost[0].push_back(tl.len * unit_e * eb * (dot ? 2 : 1));
            }
            bytes += q.n * eb * (dot ? 2 : 1) + rb;
        } else if (q.kind == LIFT_KIND_GEMV) {
            if (q.m < 0 || q.n < 0 || q.lda < std::max<int64_t>(1, q.n))
                return LIFT_EINVAL;
            p.m = q.m;
            p.lda = q.lda;
            if (q.m > 0 && (!q.out || !aligned(q.out, 4)))
                return LIFT_EINVAL;
            if (q.m > 0 && q.n > 0 && (!q.a || !q.b || !aligned(q.a, eb) || !aligned(q.b, 4)))
                return LIFT_EINVAL;
            if (q.m == 0)
                continue;
            outs.push_back({(uintptr_t)q.out, (uintptr_t)q.out + q.m * 4});
            if (q.n > 0) {
                ins.push_back({(uintptr_t)q.a, (uintptr_t)q.a + ((q.m - 1) * q.lda + q.n) * eb});
                ins.push_back({(uintptr_t)q.b, (uintptr_t)q.b + q.n * 4});
            }
            const int64_t xalign = std::min<int64_t>(e * 4, 16);
            p.vec = q.n > 0 && aligned(q.a, vb) && (q.lda * eb) % vb == 0 && aligned(q.b, xalign);
            // rows with heads against shifted copies of x in LDS, for rows with
            // at least one vector per lane (shorter ones keep element loads,
            // two rows per wavefront)
            if (!p.vec && e > 1 && vb <= 8 && q.n >= 64 * e && e * ((q.n + 3) / 4 * 4) <= BATCH_LDS_X)
                p.vec = 2;
            p.nvec = p.vec == 1 ? q.n / e : q.n;
            int64_t rows = std::max<int64_t>(1, k.split / std::max<int64_t>(1, q.n));
            // a wavefront pays a memory round trip per row pair whatever the
            // rows' length: at most 16 row pairs per wavefront in a tile, so
            // short rows spread over many work-groups
            rows = std::min<int64_t>(rows, waves * 2 * 16);
            rows = (rows + waves - 1) / waves * waves;
            const int64_t nt = (q.m + rows - 1) / rows;
            if (nt > INT32_MAX)
                return LIFT_EUNSUPPORTED;
            p.ntiles = (int32_t)nt;
            for (int64_t t = 0; t < nt && !choose; ++t) {
                BatchTile tl{i, (int32_t)t, t * rows, std::min(rows, q.m - t * rows)};
                tiles[1].push_back(tl);
                // a row shorter than one step of loads costs about a whole step
                cost[1].push_back(tl.len * std::max<int64_t>(q.n, 64 * k.unroll * e) * eb);
            }
            bytes += q.m * q.n * eb + q.n * 4 + q.m * 4 + (q.beta != 0.f ? q.m * 4 : 0);
        } else {
            return LIFT_EINVAL;
        }
    }
    if (any_overlap(outs, ins))
        return LIFT_EINVAL;
    if (choose)
        return batch_plan_waves(probs, count, storage, acc, rt, bytes, b);
    if ((int64_t)tiles[0].size() > INT32_MAX || (int64_t)tiles[1].size() > INT32_MAX || count > 0x7fffffff)
        return LIFT_EUNSUPPORTED;

    // each kind's tiles largest first, so its dynamic schedule ends on small ones
    std::vector<BatchTile> sorted[2];
    for (int kd = 0; kd < 2; ++kd) {
        std::vector<int64_t> order(tiles[kd].size());
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(),
                         [&](int64_t x, int64_t y) { return cost[kd][x] > cost[kd][y]; });
        sorted[kd].resize(tiles[kd].size());
        for (size_t i = 0; i < order.size(); ++i)
            sorted[kd][i] = tiles[kd][(size_t)order[i]];
    }

    // Each launch's grid: at most wg_per_cu work-groups per CU, and no more
    // than fit on one at once.  (A persistent grid larger than what the CUs
    // hold would park the excess work-groups until resident ones drain the
    // tile counter; each would then run its first tile, taken by index and
    // among the largest, at the end of the launch.)
    const void *kern[2] = {batch_table(storage, acc, vb, k.unroll, false),
                           batch_table(storage, acc, vb, k.unroll, true)};
    if (!kern[0] || !kern[1])
        return LIFT_EUNSUPPORTED;
    int cus = 0;
    st = cu_count(&cus);
    if (st != LIFT_OK)
        return st;
    int64_t resident[2];
    for (int kd = 0; kd < 2; ++kd) {
        int fit = 1;
        st = resident_per_cu(kern[kd], k.block, &fit);
        if (st != LIFT_OK)
            return st;
        resident[kd] = (int64_t)cus * std::min<int64_t>(k.wg_per_cu, fit);
    }
    // The gemv launch's last round of tiles (one per work-group) is cut in
    // quarters of whole row groups: the launch then ends on short tiles, so
    // its work-groups finish within a fraction of a tile of one another.
    // (A gemv row's result does not depend on its tile; the reduction tiles
    // are the problems' work-group chunks and stay as planned.)
    {
        std::vector<BatchTile> &g = sorted[1];
        const size_t cut = g.size() - (size_t)std::min<int64_t>((int64_t)g.size(), resident[1]);
        std::vector<std::pair<int64_t, BatchTile>> pieces;
        for (size_t i = cut; i < g.size(); ++i) {
            const BatchTile tl = g[i];
            const int64_t n = hp[tl.problem].n;
            const int64_t group = 2 * e;   // a row pair, or a heads tile's pairs of every phase
            const int64_t sub = std::max<int64_t>(group, ((tl.len + 3) / 4 + group - 1) / group * group);
            for (int64_t r = 0; r < tl.len; r += sub) {
                BatchTile pc{tl.problem, tl.index, tl.begin + r, std::min(sub, tl.len - r)};
                pieces.push_back({pc.len * std::max<int64_t>(n, 64 * k.unroll * e) * eb, pc});
            }
        }
        std::stable_sort(pieces.begin(), pieces.end(),
                         [](const auto &x, const auto &y) { return x.first > y.first; });
        g.resize(cut);
        for (const auto &pc : pieces)
            g.push_back(pc.second);
    }
    int dev = 0;
    hipError_t he = hipGetDevice(&dev);
    if (he != hipSuccess)
        return hip_fail(he);

    // one allocation: per launch (reductions, gemv) counters | group
    // counters, then per-problem counters | problems | reduction tiles | gemv
    // tiles | slots
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    int64_t grid[2], off_ct[2], off_gc[2], off = 0;
    for (int kd = 0; kd < 2; ++kd) {
        grid[kd] = std::max<int64_t>(1, std::min<int64_t>(resident[kd], (int64_t)sorted[kd].size()));
        off_ct[kd] = off;
        off_gc[kd] = off + 256;
        off = off_gc[kd] + up((grid[kd] + ARRIVAL_GROUP - 1) / ARRIVAL_GROUP * WS_GROUP_STRIDE);
    }
    const int64_t off_pc = off;
    const int64_t off_pr = off_pc + up(std::max<int64_t>(count, 1) * 4);
    const int64_t off_ti0 = off_pr + up(std::max<int64_t>(count, 1) * (int64_t)sizeof(BatchProblem));
    const int64_t off_ti1 = off_ti0 + up(std::max<int64_t>((int64_t)sorted[0].size(), 1) * (int64_t)sizeof(BatchTile));
    const int64_t off_sl = off_ti1 + up(std::max<int64_t>((int64_t)sorted[1].size(), 1) * (int64_t)sizeof(BatchTile));
    const int64_t total = off_sl + std::max<int64_t>(slots, 1) * WS_SLOT;
    void *mem = nullptr;
    he = hipMalloc(&mem, (size_t)total);
    if (he != hipSuccess)
        return hip_fail(he);
    char *base = (char *)mem;
    if ((he = hipMemset(base, 0, (size_t)off_pr)) != hipSuccess ||
        (count > 0 && (he = hipMemcpy(base + off_pr, hp.data(), hp.size() * sizeof(BatchProblem),
                                      hipMemcpyHostToDevice)) != hipSuccess) ||
        (!sorted[0].empty() && (he = hipMemcpy(base + off_ti0, sorted[0].data(), sorted[0].size() * sizeof(BatchTile),
                                               hipMemcpyHostToDevice)) != hipSuccess) ||
        (!sorted[1].empty() && (he = hipMemcpy(base + off_ti1, sorted[1].data(), sorted[1].size() * sizeof(BatchTile),
                                               hipMemcpyHostToDevice)) != hipSuccess)) {
        hipFree(mem);
        return hip_fail(he);
    }
    for (hipEvent_t &ev : b->ev) {
        if ((he = hipEventCreate(&ev)) != hipSuccess) {
            for (hipEvent_t &e2 : b->ev)
                if (e2) {
                    hipEventDestroy(e2);
                    e2 = nullptr;
                }
            hipFree(mem);
            return hip_fail(he);
        }
    }
    b->device = dev;
    b->storage = storage;
    b->acc = acc;
    b->vb = vb;
    b->unroll = k.unroll;
    b->nprobs = count;
    b->bytes = bytes;
    b->block = k.block;
    b->dmem = mem;
    for (int kd = 0; kd < 2; ++kd) {
        b->ntiles[kd] = (int64_t)sorted[kd].size();
        b->grid[kd] = grid[kd];
        b->kern[kd] = kern[kd];
        BatchArgs &a = b->args[kd];
        a.probs = (const BatchProblem *)(base + off_pr);
        a.tiles = (const BatchTile *)(base + (kd == 0 ? off_ti0 : off_ti1));
        a.counters = (unsigned *)(base + off_ct[kd]);
        a.groups = base + off_gc[kd];
        a.pcount = (unsigned *)(base + off_pc);
        a.slots = base + off_sl;
        a.ntiles = b->ntiles[kd];
        a.result_f64 = rt == LIFT_F64;
    }
    return LIFT_OK;
}

}  // namespace

// ---- workspaces of graphs --------------------------------------------------

namespace {

// A graph may be replayed at any time, next to whatever else runs, so the calls
// captured into it have a workspace that is the graph's own: one per capture
// and stream, given back by the runtime when the graph and all its instances
// are gone and none of their replays runs any more.
struct GraphWorkspace {
    unsigned long long capture;
    hipStream_t stream;
    int device;
    void *mem;
};

// Never destroyed: graphs may end after this library's own statics have.
struct GraphWorkspaces {
    std::mutex mu;   // not held over a HIP call: the runtime calls give_back() on its own
    std::vector<GraphWorkspace *> owned, spare;
};

// Given back and kept for later captures (164 KB each); more are freed.
constexpr size_t SPARE_WORKSPACES = 32;

GraphWorkspaces &graph_workspaces()
{
    static GraphWorkspaces *all = new GraphWorkspaces;
    return *all;
}

void give_back(void *p)
{
    GraphWorkspaces &all = graph_workspaces();
    std::lock_guard<std::mutex> lock(all.mu);
    const auto at = std::find(all.owned.begin(), all.owned.end(), static_cast<GraphWorkspace *>(p));
    if (at != all.owned.end()) {
        all.spare.push_back(*at);
        all.owned.erase(at);
    }
}

// While one lives, this thread may allocate although a stream is captured
// (what it does is on no captured stream).
struct OutsideCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Zeros in mem, memory of the current device, when this returns: on a stream
// that is kept per device (making one for each capture takes 0.4 ms).
hipError_t zero_now(void *mem, size_t bytes, int dev)
{
    static std::atomic<hipStream_t> sides[MAX_DEVICES];
    hipStream_t side = sides[dev].load(std::memory_order_acquire);
    if (!side) {
        hipStream_t made = nullptr;
        const hipError_t e = hipStreamCreateWithFlags(&made, hipStreamNonBlocking);
        if (e != hipSuccess)
            return e;
        if (sides[dev].compare_exchange_strong(side, made))
            side = made;
        else
            (void)hipStreamDestroy(made);   // another thread was first
    }
    const hipError_t e = hipMemsetAsync(mem, 0, bytes, side);
    return e == hipSuccess ? hipStreamSynchronize(side) : e;
}

lift_status capture_workspace(hipStream_t stream, void **ws)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamGetCaptureInfo_v2(stream, &status, &id, &graph, nullptr, nullptr);
    if (e != hipSuccess)
        return hip_fail(e);
    if (status != hipStreamCaptureStatusActive)
        return LIFT_OK;
    int dev = 0;
    e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e);
    if (dev < 0 || dev >= MAX_DEVICES)
        return LIFT_EUNSUPPORTED;
    GraphWorkspaces &all = graph_workspaces();
    GraphWorkspace *mine = nullptr;
    std::vector<GraphWorkspace *> over;
    {
        std::lock_guard<std::mutex> lock(all.mu);
        for (const GraphWorkspace *w : all.owned)
            if (w->capture == id && w->stream == stream && w->device == dev) {
                *ws = w->mem;
                return LIFT_OK;
            }
        for (size_t i = all.spare.size(); i-- > 0 && !mine;)
            if (all.spare[i]->device == dev) {
                mine = all.spare[i];
                all.spare.erase(all.spare.begin() + (std::ptrdiff_t)i);
            }
        while (all.spare.size() > SPARE_WORKSPACES) {
            over.push_back(all.spare.back());
            all.spare.pop_back();
        }
    }
    OutsideCapture outside;
    for (GraphWorkspace *w : over) {
        (void)hipFree(w->mem);
        delete w;
    }
    if (!mine) {
        mine = new (std::nothrow) GraphWorkspace{0, nullptr, dev, nullptr};
        if (!mine)
            return hip_fail(hipErrorOutOfMemory);
        e = hipMalloc(&mine->mem, lift_workspace_bytes());
    }
    if (e == hipSuccess)
        e = zero_now(mine->mem, lift_workspace_bytes(), dev);
    if (e != hipSuccess) {
        (void)hipFree(mine->mem);
        delete mine;
        return hip_fail(e);
    }
    mine->capture = id;
    mine->stream = stream;
    {
        std::lock_guard<std::mutex> lock(all.mu);
        all.owned.push_back(mine);
    }
    hipUserObject_t object = nullptr;
    e = hipUserObjectCreate(&object, mine, give_back, 1, hipUserObjectNoDestructorSync);
    if (e != hipSuccess)
        give_back(mine);
    else {
        e = hipGraphRetainUserObject(graph, object, 1, hipGraphUserObjectMove);
        if (e != hipSuccess)
            (void)hipUserObjectRelease(object, 1);   // gives it back
    }
    if (e != hipSuccess)
        return hip_fail(e);
    *ws = mine->mem;
    return LIFT_OK;
}

}  // namespace

extern "C" {

size_t lift_workspace_bytes(void) { return (size_t)(WS_HEADER + (int64_t)MAX_WORKGROUPS * WS_SLOT); }

int32_t lift_max_workgroups(void) { return MAX_WORKGROUPS; }

lift_status lift_scal_ex(int64_t n, float alpha, const float *x, float *out, const lift_knobs *knobs,
                         hipStream_t stream)
{
    if (n < 0)
        return LIFT_EINVAL;
    if (n > 0 && (!x || !out || !aligned(x, 4) || !aligned(out, 4)))
        return LIFT_EINVAL;
    if (x != out && overlaps(x, n * 4, out, n * 4))
        return LIFT_EINVAL;
    lift_status st = LIFT_OK;
    knobs = effective_knobs(knobs, TOP_SCAL, LIFT_F32, LIFT_ACC_F32, n, &st);
    if (st != LIFT_OK)
        return st;
    Knobs k;
    // Up to 16 MiB a vector of 16 bytes per thread where x and out share that
    // alignment: the shortest chain of a load and a store, and the most
    // work-groups (replayed from a graph, us, with 8 dwords per thread | this:
    // 2^20 3.25 | 2.84, 3000001 7.2 | 5.4, 2^21 4.06 | 3.82, 2^22 6.85 | 6.86,
    // 2^23 12.18 | 12.28).  Else, from 4 to 8 MiB, 4 dwords (8 | 4: 1100000 3.31 |
    // 3.12, 2000000 5.60 | 4.44; but 1000000 3.55 | 3.67, 2108370 5.39 | 5.99).
    Split3 sp;
    Knobs def = DEF_SCAL;
    if (!knobs && n > 0 && n <= 1 << 22 && split3(x, out, n, 4, 16, &sp))
        def = {256, 16, 1, 1, 0, 32, 1, 1, 0};
    else if (!knobs && n >= 1 << 20 && n < 1 << 21)
        def.unroll = 4;
    st = resolve(knobs, def, 4, &k);
    if (st != LIFT_OK)
        return st;
    if (k.vec_bytes < 4)
        return LIFT_EINVAL;
    if (n == 0)
        return LIFT_OK;
    int vb = k.vec_bytes;
    if (!split3(x, out, n, 4, vb, &sp)) {
        vb = 4;
        split3(x, nullptr, n, 4, vb, &sp);
    }
    const void *kern = scal_kernel(vb, k.unroll);
    if (!kern)
        return LIFT_EUNSUPPORTED;
    int cus = 0;
    st = cu_count(&cus);
    if (st != LIFT_OK)
        return st;
    const int64_t chunk = chunk_for(sp.nvec, vb / 4, k, cus, MAX_DISPATCH_ITEMS / k.block);
    const int64_t grid = std::max<int64_t>(1, (sp.nvec + chunk - 1) / chunk);
    ScalArgs a;
    a.x = x;
    a.out = out;
    a.n = n;
    a.head = sp.head;
    a.nvec = sp.nvec;
    a.chunk = chunk;
    a.alpha = alpha;
    return launch(kern, grid, k.block, &a, stream);
}

lift_status lift_scal(int64_t n, float alpha, const float *x, float *out, hipStream_t stream)
{
    return lift_scal_ex(n, alpha, x, out, nullptr, stream);
}

lift_status lift_asum(int64_t n, const float *x, float *result, void *ws, size_t ws_bytes,
                      hipStream_t stream)
{
    return reduce_common(OP_ASUM, n, LIFT_F32, x, nullptr, LIFT_ACC_F32, LIFT_F32, result, ws,
                         ws_bytes, nullptr, stream);
}

lift_status lift_dot(int64_t n, const float *x, const float *y, float *result, void *ws,
                     size_t ws_bytes, hipStream_t stream)
{
    return reduce_common(OP_DOT, n, LIFT_F32, x, y, LIFT_ACC_F32, LIFT_F32, result, ws, ws_bytes,
                         nullptr, stream);
}

lift_status lift_asum_ex(int64_t n, lift_dtype xt, const void *x, lift_acc acc, lift_dtype rt,
                         void *result, void *ws, size_t ws_bytes, const lift_knobs *knobs,
                         hipStream_t stream)
{
    return reduce_common(OP_ASUM, n, xt, x, nullptr, acc, rt, result, ws, ws_bytes, knobs, stream);
}

lift_status lift_dot_ex(int64_t n, lift_dtype xt, const void *x, const void *y, lift_acc acc,
                        lift_dtype rt, void *result, void *ws, size_t ws_bytes,
                        const lift_knobs *knobs, hipStream_t stream)
{
    return reduce_common(OP_DOT, n, xt, x, y, acc, rt, result, ws, ws_bytes, knobs, stream);
}

lift_status lift_dot_ex_noalloc(int64_t n, lift_dtype xt, const void *x, const void *y, lift_acc acc,
                                lift_dtype rt, void *result, const lift_knobs *knobs, hipStream_t stream)
{
    lift_status st = reduce_check(OP_DOT, n, xt, x, y, acc, rt, result);
    if (st != LIFT_OK)
        return st;
    Knobs checked;  // explicit knobs and the override are checked before the first HIP call
    if (knobs && (st = resolve(knobs, DEF_REDUCE, elem_bytes(xt), &checked, true)) != LIFT_OK)
        return st;
    if (!knobs && forced_config().present && !forced_config().valid)
        return LIFT_EINVAL;
    static_assert(STATIC_SCRATCH_BYTES >= (size_t)(WS_HEADER + (int64_t)MAX_WORKGROUPS * WS_SLOT),
                  "the array holds a partial for the largest grid a reduction launches");
    void *ws = nullptr;
    st = static_scratch(&ws);
    if (st != LIFT_OK)
        return st;
    return reduce_common(OP_DOT, n, xt, x, y, acc, rt, result, ws, STATIC_SCRATCH_BYTES, knobs, stream);
}

lift_status lift_blackscholes_ex(int64_t n, const float *s, float strike, float rate, float volatility,
                                 float years, float *call_put, const lift_knobs *knobs, hipStream_t stream)
{
    if (n < 0)
        return LIFT_EINVAL;
    if (n > 0 && (!s || !call_put || !aligned(s, 4) || !aligned(call_put, 8)))
        return LIFT_EINVAL;
    if (overlaps(s, n * 4, call_put, n * 8))
        return LIFT_EINVAL;
    if (!(strike > 0.f) || !std::isfinite(strike) || !(volatility > 0.f) || !std::isfinite(volatility) ||
        !(years > 0.f) || !std::isfinite(years) || !std::isfinite(rate))
        return LIFT_EINVAL;
    lift_status st = LIFT_OK;
    knobs = effective_knobs(knobs, TOP_BS, LIFT_F32, LIFT_ACC_F32, n, &st);
    if (st != LIFT_OK)
        return st;
    Knobs k;
    st = resolve(knobs, DEF_BS, 4, &k);
    if (st != LIFT_OK)
        return st;
    if (k.vec_bytes < 4)
        return LIFT_EINVAL;
    if (n == 0)
        return LIFT_OK;
    // vector path: prices vb-aligned after the head, and the head's pairs
    // aligned for the pair stores (2 vb bytes, at most 16 per store)
    int vb = k.vec_bytes;
    Split3 sp;
    split3(s, nullptr, n, 4, vb, &sp);
    const uintptr_t out_head = reinterpret_cast<uintptr_t>(call_put) + (uintptr_t)sp.head * 8;
    if (out_head % (uintptr_t)std::min(2 * vb, 16) != 0) {
        vb = 4;
        split3(s, nullptr, n, 4, vb, &sp);
    }
    const void *kern = blackscholes_kernel_table(vb, k.unroll);
    if (!kern)
        return LIFT_EUNSUPPORTED;
    int cus = 0;
    st = cu_count(&cus);
    if (st != LIFT_OK)
        return st;
    const int64_t chunk = chunk_for(sp.nvec, vb / 4, k, cus, MAX_DISPATCH_ITEMS / k.block);
    BsArgs a;
    a.s = s;
    a.call_put = call_put;
    a.n = n;
    a.head = sp.head;
    a.nvec = sp.nvec;
    a.chunk = chunk;
    const double K = strike, r = rate, v = volatility, T = years;
    const double vst = v * std::sqrt(T);
    a.ln2_over_vst = (float)(std::log(2.0) / vst);
    a.d1_offset = (float)(((r + 0.5 * v * v) * T - std::log(K)) / vst);
    a.vol_sqrt_t = (float)vst;
    a.strike_disc = (float)(K * std::exp(-r * T));
    const int64_t grid = std::max<int64_t>(1, (sp.nvec + chunk - 1) / chunk);
    return launch(kern, grid, k.block, &a, stream);
}

lift_status lift_blackscholes(int64_t n, const float *s, float strike, float rate, float volatility,
                              float years, float *call_put, hipStream_t stream)
{
    return lift_blackscholes_ex(n, s, strike, rate, volatility, years, call_put, nullptr, stream);
}

// MD in passes over slices of the positions (md_packed_kernel): the particles
// whose neighbours lie near them are done by the first launch, the others
// marked, and each pass adds their neighbours in one slice.  v: indices per
// load; kn: lanes and loads in flight of the first launch.
static lift_status md_passes(const MdArgs &args, int slices, int v, const Knobs &kn, hipStream_t stream)
{
    MdArgs a = args;
    const int64_t span = (a.n + slices - 1) / slices;
    a.near = (uint32_t)(a.n / 12);
    const void *sort = md_sort_kernel_table(kn.lanes, v, kn.unroll), *packed = md_packed_kernel_table(std::min(v, 2));
    if (!sort || !packed)
        return LIFT_EUNSUPPORTED;
    int cus = 0, fit = 1;
    lift_status st = cu_count(&cus);
    if (st == LIFT_OK)
        st = resident_per_cu(packed, 256, &fit);
    if (st != LIFT_OK)
        return st;
    // 4 work-groups per CU: the lists' and the gathers' lines compete for the
    // L1's outstanding misses, more wavefronts change nothing (3 slices of 2^20
    // particles, us: 2 per CU 1023, 3: 839, 4: 795, 6: 798, 8: 791)
    const int64_t grid = std::min<int64_t>((a.n + 15) / 16, (int64_t)cus * std::min(fit, 4));
    // an armed timing hook spans the launches
    const hipEvent_t t0 = g_time_start, t1 = g_time_stop;
    g_time_stop = nullptr;
    st = launch(sort, (a.n * kn.lanes + 255) / 256, 256, &a, stream);
    for (int p = 0; p < slices && st == LIFT_OK; ++p) {
        MdPackedArgs s;
        s.md = a;
        s.lo = (uint32_t)(p * span);
        s.hi = (uint32_t)std::min<int64_t>(a.n, (p + 1) * span);
        if (p == slices - 1 && t0)
            g_time_stop = t1;
        st = launch(packed, grid, 256, &s, stream);
    }
    g_time_start = g_time_stop = nullptr;
    return st;
}

lift_status lift_md_ex(int64_t n, const float *pos, int64_t k, const int32_t *nbr, float cutoff,
                       float epsilon, float sigma, float *force, const lift_knobs *knobs,
                       hipStream_t stream)
{
    if (n < 0 || k < 0 || n > INT32_MAX)
        return LIFT_EINVAL;
    if (n > 0 && (!pos || !force || !aligned(pos, 16) || !aligned(force, 16)))
        return LIFT_EINVAL;
    if (n > 0 && k > 0 && (!nbr || !aligned(nbr, 4)))
        return LIFT_EINVAL;
    if (n > 0 && k > INT64_MAX / 4 / n)
        return LIFT_EINVAL;
    if (overlaps(force, n * 16, pos, n * 16) || overlaps(force, n * 16, nbr, n > 0 ? n * k * 4 : 0))
        return LIFT_EINVAL;
    if (!(cutoff >= 0.f) || !std::isfinite(cutoff) || !(sigma > 0.f) || !std::isfinite(sigma) ||
        !std::isfinite(epsilon))
        return LIFT_EINVAL;
    lift_status st = LIFT_OK;
    const bool choose = !knobs && !forced_config().present;   // the launch is the library's choice
    knobs = effective_knobs(knobs, TOP_MD, LIFT_F32, LIFT_ACC_F32, n * k, &st);
    if (st != LIFT_OK)
        return st;
    Knobs kn;
    st = resolve(knobs, DEF_MD, 4, &kn);
    if (st != LIFT_OK)
        return st;
    if (kn.vec_bytes < 4 || kn.unroll > 4)
        return LIFT_EINVAL;
    // one thread per lane of each particle (16 lanes where the library chooses)
    if (n * (choose ? DEF_MD.lanes : kn.lanes) > MAX_DISPATCH_ITEMS - kn.block)
        return LIFT_EINVAL;
    if (n == 0)
        return LIFT_OK;
    // V indices per load when every row starts V-aligned
    int v = kn.vec_bytes / 4;
    while (v > 1 && (k % v != 0 || !aligned(nbr, (size_t)v * 4)))
        v /= 2;
    if (choose && !knobs) {
        // 8 lanes per particle, with as many loads in flight as cover a row
        // and no more (a load past the row still costs its pairs' arithmetic);
        // 16 with two loads in flight for longer rows while 8 would leave
        // wavefront slots empty, and where an index vector is not 4 of them
        // (graph replays, us, random and lattice order, 16 lanes | 8: 32768 x 24
        // 6.5 5.4 | 5.5 3.5, 262144 x 32 50.9 26.4 | 46.2 17.0, 262144 x 256 330
        // 120 | 327 109; but 12288 x 128 5.9 | 6.6 in random order, and rows of 65,
        // 343000 x 65 164.9 64.1 | 177.0 71.8).
        const int64_t vecs = k / v;
        const bool wide = n < 65536 ? vecs >= 16 : v < 4 && vecs > 16;
        kn.lanes = wide ? 16 : 8;
        kn.unroll = wide && v < 4 ? 2 : 1;
        while (kn.unroll < (v < 4 ? 2 : 4) && (int64_t)kn.lanes * kn.unroll < vecs)
            kn.unroll *= 2;
    }
    const void *kern = md_kernel_table(kn.lanes, v, kn.unroll);
    if (!kern)
        return LIFT_EUNSUPPORTED;
    MdArgs a;
    a.pos = pos;
    a.nbr = nbr;
    a.force = force;
    a.n = n;
    a.k = k;
    a.t2 = (float)((double)cutoff * (double)cutoff);
    a.sigma2 = (float)((double)sigma * (double)sigma);
    a.eps24 = (float)(24.0 * (double)epsilon);
    a.near = 0;
    // Slices of about 5 MB of positions (an XCD's L2 holds 4 MiB), where there
    // are 2 to 4 of them: below 7.5 MB one pass is as fast (474552 particles in
    // random order, 7.6 MB, 128 slots: 316 us, 2 slices 284 us), and beyond 4
    // the lists' extra readings cost what the misses did.
    const int slices = (int)std::min<int64_t>(5, (n * 16 + 2500000) / 5000000);
    // A pass costs its reading of the lists and of the marks, whatever they
    // hold; a gather costs by neighbours.  So short lists take one pass (2^20
    // particles in random order, full lists, us, one pass | passes: of 16 222 |
    // 530, of 40 551 | 560, of 48 656 | 587, of 64 879 | 651; lists of 64 that are
    // 5/8 full 565 | 571; 512000 particles: of 64 291 | 267 and, 5/8 full, 191 |
    // 212, of 96 433 | 348 and 285 | 272).
    const bool long_lists = k >= (slices == 2 ? 96 : 64);
    if (choose && !knobs && slices >= 2 && slices <= 4 && long_lists)
        return md_passes(a, slices, v, kn, stream);
    const int64_t threads = n * kn.lanes;
    const int64_t grid = (threads + kn.block - 1) / kn.block;
    return launch(kern, grid, kn.block, &a, stream);
}

lift_status lift_md(int64_t n, const float *pos, int64_t k, const int32_t *nbr, float cutoff, float epsilon,
                    float sigma, float *force, hipStream_t stream)
{
    return lift_md_ex(n, pos, k, nbr, cutoff, epsilon, sigma, force, nullptr, stream);
}

lift_status lift_gemv(int64_t m, int64_t n, float alpha, const float *A, int64_t lda,
                      const float *x, float beta, float *y, hipStream_t stream)
{
    return gemv_common(m, n, alpha, LIFT_F32, A, lda, x, beta, y, LIFT_ACC_F32, nullptr, stream);
}

lift_status lift_gemv_ex(int64_t m, int64_t n, float alpha, lift_dtype at, const void *A,
                         int64_t lda, const float *x, float beta, float *y, lift_acc acc,
                         const lift_knobs *knobs, hipStream_t stream)
{
    return gemv_common(m, n, alpha, at, A, lda, x, beta, y, acc, knobs, stream);
}

lift_status lift_gemv_ex_ws(int64_t m, int64_t n, float alpha, lift_dtype at, const void *A, int64_t lda,
                            const float *x, float beta, float *y, lift_acc acc, void *ws, size_t ws_bytes,
                            const lift_knobs *knobs, hipStream_t stream)
{
    if (!ws || ws_bytes < lift_workspace_bytes())
        return LIFT_EWORKSPACE;
    if (!aligned(ws, 16))
        return LIFT_EINVAL;
    if (m > 0 && overlaps(y, m * 4, ws, (int64_t)ws_bytes))
        return LIFT_EINVAL;
    return gemv_common(m, n, alpha, at, A, lda, x, beta, y, acc, knobs, stream, ws);
}

lift_status lift_batch_create(const lift_problem *probs, int32_t count, lift_dtype storage, lift_acc acc,
                              lift_dtype rt, const lift_knobs *knobs, lift_batch **out)
{
    if (!out)
        return LIFT_EINVAL;
    *out = nullptr;
    lift_batch *b = new (std::nothrow) lift_batch();
    if (!b)
        return LIFT_EUNSUPPORTED;
    lift_status st = batch_plan(probs, count, storage, acc, rt, knobs, b);
    if (st != LIFT_OK) {
        delete b;
        return st;
    }
    *out = b;
    return LIFT_OK;
}

lift_status lift_batch_run(lift_batch *b, hipStream_t stream)
{
    if (!b)
        return LIFT_EINVAL;
    if (b->ntiles[0] + b->ntiles[1] == 0)
        return LIFT_OK;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e);
    if (dev != b->device)
        return LIFT_EINVAL;
    if (b->waves)
        return batch_run_waves(b, stream);
    // An armed timing hook covers the whole run: its start event goes with
    // the first launch and its stop event with the last (the batch's own
    // pair of events fills the other ends when there are two launches).
    const hipEvent_t t0 = g_time_start, t1 = g_time_stop;
    g_time_start = g_time_stop = nullptr;
    // an armed stamp hook takes both launches' stamped instances (one-shot)
    const void *kern[2] = {b->kern[0], b->kern[1]};
    int64_t grid[2] = {b->grid[0], b->grid[1]};
    uint64_t *stamps = nullptr;
    if (g_stamps) {
        stamps = g_stamps;
        const int64_t cap = g_stamp_capacity;
        g_stamps = nullptr;
        if (b->acc != LIFT_ACC_F32 || (b->storage != LIFT_F32 && b->storage != LIFT_BF16))
            return LIFT_EUNSUPPORTED;
        if (b->ntiles[0] + b->ntiles[1] > cap)
            return LIFT_EINVAL;
        int cus = 0;
        lift_status st = cu_count(&cus);
        if (st != LIFT_OK)
            return st;
        for (int kd = 0; kd < 2; ++kd) {
            kern[kd] = b->storage == LIFT_F32 ? batch_stamped_f32(b->vb, b->unroll, kd == 1)
                                              : batch_stamped_bf16(b->vb, b->unroll, kd == 1);
            if (!kern[kd])
                return LIFT_EUNSUPPORTED;
            int fit = 1;
            if ((st = resident_per_cu(kern[kd], b->block, &fit)) != LIFT_OK)
                return st;
            grid[kd] = std::min<int64_t>(grid[kd], (int64_t)cus * fit);
        }
    }
    const int first = b->ntiles[0] > 0 ? 0 : 1, last = b->ntiles[1] > 0 ? 1 : 0;
    for (int kd = first; kd <= last; ++kd) {
        if (b->ntiles[kd] == 0)
            continue;
        if (t0) {
            g_time_start = kd == first ? t0 : b->ev[1];
            g_time_stop = kd == last ? t1 : b->ev[0];
        }
        BatchArgs a = b->args[kd];
        if (stamps)  // the reduction tiles' words first, then the gemv tiles'
            a.stamps = stamps + (kd == 1 ? b->ntiles[0] : 0) * STAMPS_PER_TILE;
        lift_status st = launch(kern[kd], grid[kd], b->block, &a, stream);
        if (st != LIFT_OK) {
            g_time_start = g_time_stop = nullptr;
            return st;
        }
    }
    return LIFT_OK;
}

lift_status lift_batch_capture(lift_batch *b, hipStream_t stream, hipGraphExec_t *exec)
{
    if (!b || !exec || !stream)
        return LIFT_EINVAL;
    *exec = nullptr;
    hipError_t e = hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess)
        return hip_fail(e);
    lift_status st = lift_batch_run(b, stream);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(stream, &graph);
    if (st != LIFT_OK) {
        if (graph)
            hipGraphDestroy(graph);
        return st;
    }
    if (e != hipSuccess)
        return hip_fail(e);
    e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    hipGraphDestroy(graph);
    if (e != hipSuccess) {
        *exec = nullptr;
        return hip_fail(e);
    }
    return LIFT_OK;
}

lift_status lift_batch_info(const lift_batch *b, int64_t *tiles, int64_t *grid, int64_t *bytes)
{
    if (!b)
        return LIFT_EINVAL;
    if (tiles)
        *tiles = b->ntiles[0] + b->ntiles[1];
    if (grid)
        *grid = b->waves ? (b->ntiles[0] + b->ntiles[1] ? b->grid[0] : 0)
                         : (b->ntiles[0] ? b->grid[0] : 0) + (b->ntiles[1] ? b->grid[1] : 0);
    if (bytes)
        *bytes = b->bytes;
    return LIFT_OK;
}

void lift_batch_destroy(lift_batch *b)
{
    if (!b)
        return;
    if (b->dmem)
        hipFree(b->dmem);
    for (hipEvent_t ev : b->ev)
        if (ev)
            hipEventDestroy(ev);
    delete b;
}

lift_status lift_stream_read(int64_t n, const float *x, float *sink, const lift_knobs *knobs,
                             hipStream_t stream)
{
    return stream_common(false, n, x, sink, knobs, stream);
}

lift_status lift_stream_copy(int64_t n, const float *x, float *out, const lift_knobs *knobs,
                             hipStream_t stream)
{
    return stream_common(true, n, x, out, knobs, stream);
}

int32_t lift_default_knobs(const char *op, lift_dtype storage, lift_acc acc, int64_t elements, int64_t row_length,
                           const char *arch, int32_t cus, lift_knobs *out)
{
    if (!op || !out || elements < 0 || row_length < 0)
        return LIFT_EINVAL;
    if (storage != LIFT_F32 && storage != LIFT_BF16 && storage != LIFT_F16)
        return LIFT_EINVAL;
    if (acc != LIFT_ACC_F32 && acc != LIFT_ACC_F32_COMP && acc != LIFT_ACC_F32_F64COMBINE)
        return LIFT_EINVAL;
    int top = -1;
    for (int i = 0; i < TOP_COUNT; ++i)
        if (std::strcmp(op, TUNED_OP_NAMES[i]) == 0)
            top = i;
    if (top < 0)
        return LIFT_EINVAL;
    std::memset(out, 0, sizeof *out);
    const Forced &f = forced_config();
    if (f.present) {
        if (!f.valid)
            return LIFT_EINVAL;
        *out = f.knobs;
        return 2;
    }
    if (!arch && !device_identity(&arch, &cus))
        return LIFT_EHIP;
    if (ignore_tuned())
        return 0;
    const TunedEntry *e = tuned_entry(arch, cus, top, storage, acc, elements, row_length);
    if (!e)
        return 0;
    *out = e->knobs;
    return 1;
}

const char *lift_status_string(lift_status s)
{
    switch (s) {
    case LIFT_OK: return "ok";
    case LIFT_EINVAL: return "invalid argument";
    case LIFT_EWORKSPACE: return "workspace missing or too small";
    case LIFT_EHIP: return "HIP runtime error";
    case LIFT_EUNSUPPORTED: return "unsupported combination";
    default: return "unknown status";
    }
}

int lift_last_hip_error(void) { return g_last_hip_error; }

lift_status lift_time_next_launch(hipEvent_t start, hipEvent_t stop)
{
    if ((start == nullptr) != (stop == nullptr))
        return LIFT_EINVAL;
    g_time_start = start;
    g_time_stop = stop;
    return LIFT_OK;
}

lift_status lift_stamp_next_launch(uint64_t *stamps, int64_t capacity, int32_t *clock_khz)
{
    if (!stamps) {
        g_stamps = nullptr;
        g_stamp_capacity = 0;
        return LIFT_OK;
    }
    if (capacity <= 0 || !aligned(stamps, 8) || !clock_khz)
        return LIFT_EINVAL;
    int dev = 0, khz = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess)
        return hip_fail(e);
    *clock_khz = khz;
    g_stamps = stamps;
    g_stamp_capacity = capacity;
    return LIFT_OK;
}

lift_status lift_capture_workspace(hipStream_t stream, void **ws)
{
    if (!ws)
        return LIFT_EINVAL;
    *ws = nullptr;
    return stream ? capture_workspace(stream, ws) : LIFT_OK;   // the null stream cannot be captured
}

lift_status lift_combine_rounds_next_launch(int32_t rounds)
{
    if (rounds < 0)
        return LIFT_EINVAL;
    g_rounds = rounds;
    return LIFT_OK;
}

const char *lift_version(void) { return "lift-mi355x 0.1 gfx950"; }

}  // extern "C"
