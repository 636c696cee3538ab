// asum and dot: one streaming pass, one launch.
//
// The kernel is the paper's fused reduction (the asum derivation of Fig. 8,
// eq. 8, and the GPU expressions of Fig. 9) laid out for CDNA4:
//
//   reduce-seq o join o map-workgroup(
//       toGlobal(...)                              partial -> workspace slot
//     o iterate(part-red) with toLocal             DPP wave butterfly + LDS
//     o map-local(reduce-seq(lambda acc, a: acc + term(a), 0))
//     o split o reorder-stride                     lane t reads vector t, t+B, ..
//   ) o asVector o split^chunk                      dwordx4 loads, chunk per WG
//
// term(a) = |a| (asum) or a_x * a_y (dot, zip fused into the load).  The
// final reduce-seq o join runs in the same launch: every work-group stores
// its partial with a tag that shows its arrival, and one wavefront of the
// grid's last work-group folds all partials (lane t: partials t, t + 64, ...;
// then the wave butterfly) as they arrive, writes the result and clears the
// tags for the next call.  No float atomics, so the result is deterministic.
// The last work-group's wait is bounded: past it the work-group whose partial
// is the last to come folds instead (meet()), so the grid drains in whatever
// order its work-groups run.
//
// Cross-XCD visibility without cache maintenance: the partials are written
// and read with agent-scope atomics, which gfx950 performs device-coherently
// (past the per-XCD L2), value and tag in one word.  An agent-scope
// release/acquire fence would instead write back and invalidate the whole L2
// of the XCD in every work-group.
#pragma once

#include "lift_device.hpp"
#include "lift_internal.hpp"

namespace lift {

// Per-lane accumulator of the streaming phase.
template <int ACC, int E>
struct LaneAcc;

// binary32: E independent sums (one per vector component), folded pairwise
// at the end.
template <int E>
struct LaneAcc<ACC_F32, E> {
    float s[E];
    __device__ __forceinline__ LaneAcc()
    {
#pragma unroll
        for (int e = 0; e < E; ++e)
            s[e] = 0.f;
    }
    // asum / dot-with-product-given
    __device__ __forceinline__ void add_terms(const float *t)
    {
#pragma unroll
        for (int e = 0; e < E; ++e)
            s[e] += t[e];
    }
    __device__ __forceinline__ void add_products(const float *a, const float *b)
    {
#pragma unroll
        for (int e = 0; e < E; ++e)
            s[e] = fmaf(a[e], b[e], s[e]);
    }
    __device__ __forceinline__ void add_scalar(float v) { s[0] += v; }
    __device__ __forceinline__ void add_scalar_product(float a, float b) { s[0] = fmaf(a, b, s[0]); }
    __device__ __forceinline__ float value() const
    {
        float t[E];
#pragma unroll
        for (int e = 0; e < E; ++e)
            t[e] = s[e];
#pragma unroll
        for (int w = 1; w < E; w <<= 1)
#pragma unroll
            for (int e = 0; e + w < E; e += 2 * w)
                t[e] = t[e] + t[e + w];
        return t[0];
    }
};

// binary32 with a binary64 cross-work-group combine: same lane arithmetic.
template <int E>
struct LaneAcc<ACC_F64, E> : LaneAcc<ACC_F32, E> {};

// Compensated: the E terms of one load are summed pairwise, then added to
// the lane's (sum, error) pair with TwoSum; binary32 products contribute
// their exact rounding error (fma(a, b, -a*b), the TwoProduct of Ogita,
// Rump and Oishi) to the error term.
template <int E>
struct LaneAcc<ACC_COMP, E> {
    Pair p{0.f, 0.f};
    __device__ __forceinline__ static float tree(float *t)
    {
#pragma unroll
        for (int w = 1; w < E; w <<= 1)
#pragma unroll
            for (int e = 0; e + w < E; e += 2 * w)
                t[e] = t[e] + t[e + w];
        return t[0];
    }
    __device__ __forceinline__ void add_terms(const float *t)
    {
        float u[E];
#pragma unroll
        for (int e = 0; e < E; ++e)
            u[e] = t[e];
        p = pair_add(p, tree(u));
    }
    template <bool EXACT_PRODUCTS>
    __device__ __forceinline__ void add_products_c(const float *a, const float *b)
    {
        float q[E], r[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            q[e] = a[e] * b[e];
            r[e] = EXACT_PRODUCTS ? 0.f : fmaf(a[e], b[e], -q[e]);
        }
        p = pair_add(p, tree(q));
        if (!EXACT_PRODUCTS)
            p.c += tree(r);
    }
    __device__ __forceinline__ void add_scalar(float v) { p = pair_add(p, v); }
    template <bool EXACT_PRODUCTS>
    __device__ __forceinline__ void add_scalar_product_c(float a, float b)
    {
        float q = a * b;
        p = pair_add(p, q);
        if (!EXACT_PRODUCTS)
            p.c += fmaf(a, b, -q);
    }
    __device__ __forceinline__ Pair value() const { return p; }
};

// Partial slot type written by each work-group.
template <int ACC> struct SlotT { using type = float; };
template <> struct SlotT<ACC_COMP> { using type = Pair; };
template <> struct SlotT<ACC_F64> { using type = double; };

template <int ACC> struct BlockT { using type = float; };
template <> struct BlockT<ACC_COMP> { using type = Pair; };

__device__ __forceinline__ double to_f64(float v) { return (double)v; }
__device__ __forceinline__ double to_f64(double v) { return v; }
__device__ __forceinline__ double to_f64(Pair p) { return (double)p.s + (double)p.c; }
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(double v) { return (float)v; }
__device__ __forceinline__ float to_f32(Pair p) { return p.s + p.c; }

template <int ACC>
__device__ __forceinline__ typename SlotT<ACC>::type to_slot(typename BlockT<ACC>::type v)
{
    return typename SlotT<ACC>::type(v);
}
template <>
__device__ __forceinline__ Pair to_slot<ACC_COMP>(Pair v)
{
    return v;
}

template <class S>
__device__ __forceinline__ S zero_of();
template <> __device__ __forceinline__ float zero_of<float>() { return 0.f; }
template <> __device__ __forceinline__ double zero_of<double>() { return 0.0; }
template <> __device__ __forceinline__ Pair zero_of<Pair>() { return Pair{0.f, 0.f}; }

// Agent-coherent (all XCDs) store / load of a partial slot.
__device__ __forceinline__ void store_coherent(char *p, float v)
{
    __hip_atomic_store(reinterpret_cast<uint32_t *>(p), __builtin_bit_cast(uint32_t, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent(char *p, double v)
{
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent(char *p, Pair v)
{
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
template <class S>
__device__ __forceinline__ S load_coherent(const char *p);
template <>
__device__ __forceinline__ float load_coherent<float>(const char *p)
{
    return __builtin_bit_cast(float, __hip_atomic_load(reinterpret_cast<const uint32_t *>(p), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT));
}
template <>
__device__ __forceinline__ double load_coherent<double>(const char *p)
{
    return __builtin_bit_cast(double, __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT));
}
template <>
__device__ __forceinline__ Pair load_coherent<Pair>(const char *p)
{
    return __builtin_bit_cast(Pair, __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT));
}

// Partials whose arrival shows in the slot itself: one 64-bit word per
// partial, written at once, so a reader sees all of it or none and needs
// no counter and no ordering between stores.  A word of zeros (the workspace
// before its first use, and again once the reader has cleared what it took)
// or of ones has not arrived:
//   binary32       : the value and a tag;
//   (sum, error)   : the pair XOR a constant whose sum half is a signalling
//                    NaN; both halves come out of additions, which never
//                    return one, so the word is not 0, and not ~0 as the
//                    complement's error half is one too;
//   binary64       : the value XOR a signalling NaN; ~0 would be a subnormal,
//                    and these partials are sums of binary32 values and
//                    products, multiples of 2^-298.
constexpr uint32_t SLOT_TAG = 0x4c494654u;
constexpr uint64_t SLOT_PAIR = 0x805ffffe7fa5c3e1ull;   // error half above, sum half below
constexpr uint64_t SLOT_F64 = 0x7ff4c3e15a96f00dull;
// Left in the slot of a partial that has not arrived by a reader that waits no
// longer (meet()): no partial's word, by the same reasons.
constexpr uint64_t SLOT_MARK = 1;

__device__ __forceinline__ uint64_t to_word(float v)
{
    return ((uint64_t)SLOT_TAG << 32) | __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint64_t to_word(double v) { return __builtin_bit_cast(uint64_t, v) ^ SLOT_F64; }
__device__ __forceinline__ uint64_t to_word(Pair v) { return __builtin_bit_cast(uint64_t, v) ^ SLOT_PAIR; }
template <class S>
__device__ __forceinline__ bool word_arrived(uint64_t w)
{
    if constexpr (sizeof(S) == 4)
        return (uint32_t)(w >> 32) == SLOT_TAG;
    else
        return w + 1 > 2;   // not 0, ~0 or SLOT_MARK
}
template <class S>
__device__ __forceinline__ S from_word(uint64_t w);
template <> __device__ __forceinline__ float from_word<float>(uint64_t w) { return bits_to_float((uint32_t)w); }
template <> __device__ __forceinline__ double from_word<double>(uint64_t w)
{
    return __builtin_bit_cast(double, w ^ SLOT_F64);
}
template <> __device__ __forceinline__ Pair from_word<Pair>(uint64_t w)
{
    return __builtin_bit_cast(Pair, w ^ SLOT_PAIR);
}
// The word of partial i is the second half of its 16-byte slot; the untagged
// partials of other kernels (the small lane forms) go into the first.
__device__ __forceinline__ uint64_t *slot_word(char *ws, int64_t i)
{
    return reinterpret_cast<uint64_t *>(ws + WS_HEADER + i * WS_SLOT + 8);
}
__device__ __forceinline__ void store_word(uint64_t *p, uint64_t w)
{
    __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_word(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Two-level arrival of this work-group (called by one thread, after its
// partial's store has completed).  Work-group b counts in on the group
// counter at group_base + (b / ARRIVAL_GROUP) * WS_GROUP_STRIDE; the last of
// a group resets that counter and counts the group in on `global`.  Returns
// true in the one work-group that arrives last overall; by then every
// partial is stored.  The caller resets `global`.
__device__ __forceinline__ bool arrive(unsigned *global, char *group_base)
{
    const unsigned g = blockIdx.x / ARRIVAL_GROUP;
    const unsigned groups = (gridDim.x + ARRIVAL_GROUP - 1) / ARRIVAL_GROUP;
    const unsigned size = min((unsigned)ARRIVAL_GROUP, gridDim.x - g * ARRIVAL_GROUP);
    unsigned *gc = reinterpret_cast<unsigned *>(group_base + g * WS_GROUP_STRIDE);
    unsigned prev = __hip_atomic_fetch_add(gc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (prev != size - 1)
        return false;
    __hip_atomic_store(gc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    prev = __hip_atomic_fetch_add(global, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return prev == groups - 1;
}

// Lane i's value, for the whole wave.
__device__ __forceinline__ float lane_value(float v, int i) { return readlane(v, i); }
__device__ __forceinline__ Pair lane_value(Pair v, int i) { return {readlane(v.s, i), readlane(v.c, i)}; }
__device__ __forceinline__ double lane_value(double v, int i)
{
    const uint64_t w = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)w, i), hi = __builtin_amdgcn_readlane((uint32_t)(w >> 32), i);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <class S>
__device__ __forceinline__ void write_result(void *result, int f64, S v)
{
    if (f64)
        *reinterpret_cast<double *>(result) = to_f64(v);
    else
        *reinterpret_cast<float *>(result) = to_f32(v);
}

// 16-bit products are exact in binary32 (8- or 11-bit significands).
template <class T> struct ExactProducts { static constexpr bool value = T::bytes == 2; };

template <class T, int OP, int ACC, int E>
__device__ __forceinline__ void accumulate(LaneAcc<ACC, E> &acc, const float *a, const float *b)
{
    if constexpr (OP == OP_ASUM) {
        float t[E];
#pragma unroll
        for (int e = 0; e < E; ++e)
            t[e] = fabsf(a[e]);
        acc.add_terms(t);
    } else if constexpr (ACC == ACC_COMP) {
        acc.template add_products_c<ExactProducts<T>::value>(a, b);
    } else {
        acc.add_products(a, b);
    }
}

template <class T, int OP, int ACC, int E>
__device__ __forceinline__ void accumulate_scalar(LaneAcc<ACC, E> &acc, float a, float b)
{
    if constexpr (OP == OP_ASUM) {
        acc.add_scalar(fabsf(a));
    } else if constexpr (ACC == ACC_COMP) {
        acc.template add_scalar_product_c<ExactProducts<T>::value>(a, b);
    } else {
        acc.add_scalar_product(a, b);
    }
}

// Clock reading for the stamped instances (s_memrealtime: 100 MHz, shared
// by all XCDs), written by thread 0 with an ordinary vector store.
template <bool STAMP>
__device__ __forceinline__ void stamp(const ReduceArgs &a, int k)
{
    if constexpr (STAMP) {
        if (threadIdx.x == 0)
            a.stamps[(int64_t)blockIdx.x * STAMPS_PER_WG + k] = (uint64_t)wall_clock64();
    }
}

// Stamped instances, thread 0 of a work-group whose partial is on its way:
// the time (store, arrival and end alike, unless it combines), its ids and
// whether it combines.
template <bool STAMP>
__device__ __forceinline__ void stamp_arrival(const ReduceArgs &a, int last)
{
    if constexpr (STAMP) {
        __builtin_amdgcn_sched_barrier(0);
        uint64_t *w = a.stamps + (int64_t)blockIdx.x * STAMPS_PER_WG;
        const uint64_t now = (uint64_t)wall_clock64();
        w[3] = now;
        w[4] = now;
        w[5] = now;
        const uint32_t xcc = __builtin_amdgcn_s_getreg((20 << 0) | (0 << 6) | (3 << 11));  // XCC_ID[3:0]
        const uint32_t hw = __builtin_amdgcn_s_getreg((4 << 0) | (8 << 6) | (7 << 11));    // HW_ID[15:8]: CU, SH, SE
        w[6] = ((uint64_t)(unsigned)last << 32) | ((uint64_t)xcc << 16) | hw;
    }
}

// Lane t of a wavefront folds partials t, t + 64, ... of [0, last) and
// `own`, partial `last`, into v in that order, each as soon as it is there.
// LOADS loads in flight, all issued again while one of them is missing, `rounds`
// times in all: it ends negative if one still is (v is then of no use).  CLEAR:
// the last LOADS x 64 slots are cleared on the way, all of their partials having
// come (after the fold this takes 0.1 us of every reduction).
template <class ST, int LOADS, bool CLEAR>
__device__ __forceinline__ void fold_slots(char *ws, int64_t slot0, int64_t last, ST own, int &rounds, ST &v)
{
    const int t = threadIdx.x & 63;
    for (int64_t base = 0; base <= last; base += 64 * LOADS) {
        uint64_t w[LOADS];
        bool waits;
        do {
            waits = false;
            if constexpr (LOADS == 1) {
                w[0] = base + t < last ? load_word(slot_word(ws, slot0 + base + t)) : 0;
                waits = base + t < last && !word_arrived<ST>(w[0]);
            } else {
#pragma unroll
                for (int k = 0; k < LOADS; ++k)
                    w[k] = load_word(slot_word(ws, slot0 + min(base + t + 64 * k, last - 1)));
#pragma unroll
                for (int k = 0; k < LOADS; ++k)
                    waits |= base + t + 64 * k < last && !word_arrived<ST>(w[k]);
            }
        } while (__any(waits) && rounds-- > 0);
        const bool clears = CLEAR && rounds >= 0 && base + 64 * LOADS > last;   // uniform
#pragma unroll
        for (int k = 0; k < LOADS; ++k) {
            const int64_t i = base + t + 64 * k;
            if (clears && i < last)
                store_word(slot_word(ws, slot0 + i), 0);
            if (i <= last)
                v = merge(v, i == last ? own : from_word<ST>(w[k]));
        }
    }
}

// Where `count` (at least 2) work-groups meet: each calls meet() with one
// wavefront, its `index`, and in lane i < R its partial of row i (the slots are
// [row][index] from slot0 on).  Exactly one of them, as a whole wavefront, then
// calls finish(v), with lane t of v[i] the fold of row i's partials t, t + 64,
// ... (LOADS of them in flight, twice as many where there are more rounds of
// that), when it has cleared the slots.
//
// The last work-group waits for the others' partials, but not for good: which
// work-groups run at the same time is the hardware's choice, and another
// kernel may hold the places that theirs need.  After `rounds` looks in vain
// it puts a mark into every slot whose partial has not come, says in `pending`
// how many marks it left, and is done.  A work-group that finds the mark where
// it puts its partial counts itself off there, and the one that brings the
// count to zero, the last, folds in the waiter's place: the same slots in the
// same order.  So every wait ends, whatever runs when, and the result's bits do
// not depend on it.  (Two runs that share their slots, which they must not,
// get wrong numbers from that, and end.)
//
// To the others this costs an exchange that returns instead of a store, which
// takes no longer (asum fp32 of 2^16, 2^18, 2^20 back to back in a HIP graph,
// us: 2.49 2.55 3.07 with the store, 2.46 2.53 3.10 with the exchange).
template <class ST, int R>
struct Meeting {
    char *ws;
    unsigned *pending;
    int64_t slot0, count, index;
    ST own;
    ST (&v)[R];

    __device__ __forceinline__ uint64_t *slot(int64_t i) const { return slot_word(ws, slot0 + i); }

    template <int LOADS>
    __device__ __forceinline__ bool fold(int rounds)
    {
        const int64_t last = count - 1;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            v[i] = zero_of<ST>();
            const ST mine = lane_value(own, i);
            if (i == R - 1)
                fold_slots<ST, LOADS, true>(ws, slot0 + i * count, last, mine, rounds, v[i]);
            else
                fold_slots<ST, LOADS, false>(ws, slot0 + i * count, last, mine, rounds, v[i]);
        }
        if (__builtin_expect(rounds < 0, 0))
            return false;
        const int64_t left = (R - 1) * count + last / (64 * LOADS) * (64 * LOADS);   // not cleared on the way
        for (int64_t i = threadIdx.x & 63; i < left; i += 64)
            store_word(slot(i), 0);
        return true;
    }

    // The waiter has waited in vain, or a work-group has found `marks` marks.
    __device__ __forceinline__ bool hand_over(unsigned marks)
    {
        const int t = threadIdx.x & 63;
        const int64_t last = count - 1;
        if (index == last) {
            if (t < R)
                store_word(slot(t * count + last), to_word(own));
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0);   // its own partials are there before the marks count
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            marks = 0;
            for (int64_t i = t; i < R * count; i += 64) {
                uint64_t w = load_word(slot(i));
                if (!word_arrived<ST>(w) && __hip_atomic_compare_exchange_strong(slot(i), &w, SLOT_MARK, __ATOMIC_RELAXED,
                                                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    --marks;
            }
#pragma unroll
            for (int m = 1; m < 64; m <<= 1)
                marks += __shfl_xor(marks, m, 64);
        }
        int finishes = 0;
        if (t == 0)
            finishes = __hip_atomic_fetch_add(pending, marks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + marks == 0;
        if (!__builtin_amdgcn_readfirstlane(finishes))
            return false;
        // every partial is in its slot now
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (t < R)
            own = from_word<ST>(load_word(slot(t * count + last)));
        fold<1>(0);
        if (t < R)
            store_word(slot(t * count + last), 0);
        return true;
    }
};

template <int LOADS, class ST, int R, class F>
__device__ __forceinline__ void meet(char *ws, unsigned *pending, int64_t slot0, int64_t count, int64_t index, ST own,
                                     int rounds, F &&finish)
{
    ST v[R];
    Meeting<ST, R> m{ws, pending, slot0, count, index, own, v};
    const int t = threadIdx.x & 63;
    unsigned marks = 0;
    if (index != count - 1) {
        bool marked = false;
        if (t < R)
            marked = __hip_atomic_exchange(m.slot(t * count + index), to_word(own), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT) == SLOT_MARK;
        marks = __popcll(__ballot(marked));
        if (__builtin_expect(marks == 0, 1))
            return;
    } else {
        // the common case's code follows at once: what lies in between costs a
        // miss of the instruction cache each (0.1 us)
        if (__builtin_expect(LOADS == 1 || count <= 64 * LOADS, 1)) {
            if (__builtin_expect(m.template fold<LOADS>(rounds), 1)) {
                finish(v);
                return;
            }
        } else if (__builtin_expect(m.template fold<2 * LOADS>(rounds), 1)) {
            finish(v);
            return;
        }
    }
    if (m.hand_over(marks))
        finish(v);
}

// The work-group's partial wg (valid in thread 0; every thread calls this
// after the work-group tree) goes to the combine: with one work-group it is
// the result; else one wavefront of each brings it to where they meet, and the
// one that has them all -- lane t folded partials t, t + 64, t + 128, ... in
// that order -- takes the wave butterfly and writes the result.  No barrier on
// this path.
//
// Against a wait for the store's completion, two levels of arrival counters
// and the last arriver reading the slots (four dependent device-scope round
// trips), this leaves the partial's way and the read's.  Back to back in a HIP
// graph, before and now (us): asum fp32 of 2^16 3.8 -> 2.9, 2^18 4.0 -> 3.2,
// 2^20 4.6 -> 3.4, 2^24 14.0 -> 13.4; compensated bf16 of 2^22 5.9 -> 4.8.
// The loads of a round are what the poll costs (each of the 64 lanes is its
// own device-scope request), hence one word per partial and 4 loads per lane
// where they do: with two words per partial the compensated form gained
// nothing, and re-reading only what is missing lost what fp32 had gained.
template <int ACC, bool STAMP, class W>
__device__ __forceinline__ void combine_partials(const ReduceArgs &a, W wg)
{
    using ST = typename SlotT<ACC>::type;
    const int t = threadIdx.x;
    if (gridDim.x == 1) {
        if (t == 0) {
            write_result(a.result, a.result_f64, wg);
            stamp_arrival<STAMP>(a, 1);  // the only work-group combines: stored, arrived and done at once
        }
        return;
    }

    // The rest is wave 0's: the other waves are done once the tree has their
    // values (block_sum ends with a barrier).
    if (t >= 64)
        return;
    char *ws = reinterpret_cast<char *>(a.ws);
    unsigned *pending = reinterpret_cast<unsigned *>(ws + WS_PENDING);
    const int64_t count = gridDim.x;
    if (t == 0)
        stamp_arrival<STAMP>(a, 0);

    // the final reduce-seq o join, by one wavefront
    meet<4, ST, 1>(ws, pending, 0, count, blockIdx.x, ST(wg), a.rounds, [&](ST(&v)[1]) {
        const ST total = wave_sum(v[0]);
        if (t == 0)
            write_result(a.result, a.result_f64, total);
        if constexpr (STAMP) {
            if (t == 0)
                a.stamps[(int64_t)blockIdx.x * STAMPS_PER_WG + 6] |= 1ull << 32;
            __builtin_amdgcn_sched_barrier(0);
            stamp<STAMP>(a, 5);
        }
    });
}

// SHIFTED (dot, 16-byte vectors): y does not share x's 16-byte phase and is
// read from wherever its vectors start; the lanes' binary32 sums meet in
// binary64 (a dot that cancels loses nothing in the trees).
template <class T, int OP, int ACC, int VB, int U, bool STAMP = false, bool SHIFTED = false>
__global__ void __launch_bounds__(1024) reduce_kernel(ReduceArgs a)
{
    constexpr int E = Elems<T, VB>::value;
    using V = typename Vec<VB>::type;
    using BT = typename BlockT<ACC>::type;
    __shared__ BT lds_block[16];

    stamp<STAMP>(a, 0);
    const int t = threadIdx.x;
    const int64_t B = blockDim.x;
    const char *xv = reinterpret_cast<const char *>(a.x) + a.head * T::bytes;
    const char *yv = OP == OP_DOT ? reinterpret_cast<const char *>(a.y) + a.head * T::bytes : nullptr;
    const auto load_y = [&](int64_t i) {
        if constexpr (SHIFTED)
            return load_stream_any<T, VB>(yv + i * VB);
        else
            return load_stream<VB>(yv, i);
    };

    // The work-group's steps of B * U vectors: one contiguous chunk
    // (split^chunk), or every G-th step starting at its own (the chunking of
    // a reorder-stride-G over steps: all work-groups then stream neighbouring
    // steps at the same time).
    const int64_t step = B * U;
    const int64_t vbeg = a.interleave ? (int64_t)blockIdx.x * step : (int64_t)blockIdx.x * a.chunk;
    const int64_t vend = a.interleave ? a.nvec : min(vbeg + a.chunk, a.nvec);
    const int64_t stride = a.interleave ? (int64_t)gridDim.x * step : step;

    LaneAcc<ACC, E> acc;
    int64_t base = vbeg;
    // full steps: U independent loads per lane (per operand) in flight
    for (; base + step <= vend; base += stride) {
        V vx[U], vy[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            vx[k] = load_stream<VB>(xv, base + t + k * B);
            if constexpr (OP == OP_DOT)
                vy[k] = load_y(base + t + k * B);
        }
        loads_in_flight();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            float fx[E], fy[E];
            decode<T, VB>(vx[k], fx);
            if constexpr (OP == OP_DOT)
                decode<T, VB>(vy[k], fy);
            accumulate<T, OP, ACC, E>(acc, fx, fy);
        }
    }
    // the last, partial step of this work-group
    if (base < vend) {
        // Final partial step: fewer than U vectors per lane.  Every lane loads
        // U vectors at clamped (in-range) indices so all loads are in flight
        // without branches; the ones past the end are replaced by zeros, which
        // leave every sum unchanged.
        V vx[U], vy[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t i = min(base + t + k * B, vend - 1);
            vx[k] = load_stream<VB>(xv, i);
            if constexpr (OP == OP_DOT)
                vy[k] = load_y(i);
        }
        loads_in_flight();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool in = base + t + k * B < vend;
            float fx[E], fy[E];
            decode<T, VB>(vx[k], fx);
            if constexpr (OP == OP_DOT)
                decode<T, VB>(vy[k], fy);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                fx[e] = in ? fx[e] : 0.f;
                if constexpr (OP == OP_DOT)
                    fy[e] = in ? fy[e] : 0.f;
            }
            accumulate<T, OP, ACC, E>(acc, fx, fy);
        }
    }
    // scalar head (work-group 0) and tail (last work-group), fewer than E each
    if (blockIdx.x == 0 && t < a.head) {
        float fy = OP == OP_DOT ? load_elem<T>(a.y, t) : 0.f;
        accumulate_scalar<T, OP, ACC, E>(acc, load_elem<T>(a.x, t), fy);
    }
    const int64_t tail0 = a.head + a.nvec * E;
    if (blockIdx.x == gridDim.x - 1 && t < a.n - tail0) {
        float fy = OP == OP_DOT ? load_elem<T>(a.y, tail0 + t) : 0.f;
        accumulate_scalar<T, OP, ACC, E>(acc, load_elem<T>(a.x, tail0 + t), fy);
    }

    if constexpr (STAMP) {  // every load of the streaming loop has been consumed
        __builtin_amdgcn_sched_barrier(0);
        stamp<STAMP>(a, 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (SHIFTED && ACC != ACC_COMP) {
        __shared__ double lds_wide[16];
        combine_partials<ACC_F64, STAMP>(a, block_sum<double>((double)acc.value(), lds_wide));
    } else {
        BT wg = block_sum<BT>(acc.value(), lds_block);
        stamp<STAMP>(a, 2);
        combine_partials<ACC, STAMP>(a, wg);
    }
}

// Table of instantiated reduce kernels for storage T.
template <class T, int OP, int ACC, int VB>
const void *pick_unroll(int unroll)
{
    switch (unroll) {
    case 1: return reinterpret_cast<const void *>(&reduce_kernel<T, OP, ACC, VB, 1>);
    case 2: return reinterpret_cast<const void *>(&reduce_kernel<T, OP, ACC, VB, 2>);
    case 4: return reinterpret_cast<const void *>(&reduce_kernel<T, OP, ACC, VB, 4>);
    case 8: return reinterpret_cast<const void *>(&reduce_kernel<T, OP, ACC, VB, 8>);
    default: return nullptr;
    }
}

template <class T, int OP, int ACC>
const void *pick_vec(int vec_bytes, int unroll)
{
    switch (vec_bytes) {
    case 2:
        if constexpr (T::bytes == 2)
            return pick_unroll<T, OP, ACC, 2>(unroll);
        return nullptr;
    case 4: return pick_unroll<T, OP, ACC, 4>(unroll);
    case 8: return pick_unroll<T, OP, ACC, 8>(unroll);
    case 16: return pick_unroll<T, OP, ACC, 16>(unroll);
    default: return nullptr;
    }
}

template <class T, int OP>
const void *pick_acc(int acc, int vec_bytes, int unroll)
{
    switch (acc) {
    case ACC_F32: return pick_vec<T, OP, ACC_F32>(vec_bytes, unroll);
    case ACC_COMP: return pick_vec<T, OP, ACC_COMP>(vec_bytes, unroll);
    case ACC_F64: return pick_vec<T, OP, ACC_F64>(vec_bytes, unroll);
    default: return nullptr;
    }
}

template <class T>
const void *pick_reduce(int op, int acc, int vec_bytes, int unroll)
{
    if (op == OP_ASUM)
        return pick_acc<T, OP_ASUM>(acc, vec_bytes, unroll);
    if (op == OP_DOT)
        return pick_acc<T, OP_DOT>(acc, vec_bytes, unroll);
    return nullptr;
}

// dot of operands in different 16-byte phases.
template <class T>
const void *pick_dot_shifted(int acc)
{
    switch (acc) {
    case ACC_F32: return reinterpret_cast<const void *>(&reduce_kernel<T, OP_DOT, ACC_F32, 16, 2, false, true>);
    case ACC_COMP: return reinterpret_cast<const void *>(&reduce_kernel<T, OP_DOT, ACC_COMP, 16, 2, false, true>);
    case ACC_F64: return reinterpret_cast<const void *>(&reduce_kernel<T, OP_DOT, ACC_F64, 16, 2, false, true>);
    default: return nullptr;
    }
}

// The stamped instances (binary32 storage and accumulation, 16-byte loads).
template <int OP>
const void *pick_stamped(int unroll)
{
    switch (unroll) {
    case 1: return reinterpret_cast<const void *>(&reduce_kernel<F32, OP, ACC_F32, 16, 1, true>);
    case 2: return reinterpret_cast<const void *>(&reduce_kernel<F32, OP, ACC_F32, 16, 2, true>);
    case 4: return reinterpret_cast<const void *>(&reduce_kernel<F32, OP, ACC_F32, 16, 4, true>);
    case 8: return reinterpret_cast<const void *>(&reduce_kernel<F32, OP, ACC_F32, 16, 8, true>);
    default: return nullptr;
    }
}

}  // namespace lift
