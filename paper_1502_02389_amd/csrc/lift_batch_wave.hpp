// Batched form without knobs, up to 64 KiB per wavefront: one launch, every
// wavefront on its own.
//
// The host cuts all problems of a batch into tiles of one wavefront each --
// reductions: runs of elements; gemv: runs of rows -- and sorts them largest
// first; a persistent grid of independent wavefronts takes them.  No barrier
// and no LDS in the loop: a wavefront that ends a short problem goes on to the
// next while its neighbours stream, and the work-group form's costs per tile
// (tree across waves, staging x in LDS, two barriers around the draw) are
// gone, as is the second launch's ramp.
//   reduction tile -> lane reduce-seq over 16-byte vectors from wherever the
//                     tile starts, wave butterfly; a problem of one tile
//                     writes its result, else the partial goes to its slot and
//                     the wavefront that counts in last folds the problem's
//                     partials in tile order (groups of 64 first);
//   gemv tile      -> the columns of a lane stay the same over all rows of the
//                     tile, so its part of x stays in registers (rows of up to
//                     64 floats of x per lane; longer ones read x from the
//                     cache, two rows sharing it).
// Every tile's arithmetic and every fold's order are fixed by the plan, so
// results do not depend on which wavefront ran which tile.
//
// Tiles are drawn from DRAW_LISTS counters (tile i belongs to list i mod
// DRAW_LISTS, a work-group draws from list blockIdx mod DRAW_LISTS): draws on
// one address serialise at about 10 ns, and 4096 wavefronts make more.  A
// wavefront starts with the tile of its own index, holds the index of its next
// tile when it starts one, and meanwhile reads that tile's descriptor and draws
// again.  With at most one tile per wavefront nothing is drawn.
//
// Bound by HBM and, below some 10 MB, by the launch and one round trip.
// MI355X, us, two launches of work-group tiles before | this: 43 + 27 problems
// bf16 1.8 MB 13.4 | 7.3; 100 + 10 f32 13.9 MB 23.5 | 7.5; 1000 + 50 bf16 67 MB
// 34.6 | 15.7; 22 + 7 f32 94 MB 108 | 18 (5.1 TB/s); 453 + 76 bf16 163 MB 102 |
// 30 (5.4 TB/s).  A work-group per tile on the same tables reached no more
// there and lost on large f32 batches.
#pragma once

#include "lift_batch.hpp"
#include "lift_gemv_rows.hpp"

namespace lift {

// A place in a list that is past any table's end.
constexpr unsigned NO_TILE = 0x1ffffff0u / DRAW_LISTS * DRAW_LISTS;

// A wave-uniform descriptor, loaded as one dword per lane.
struct TileWords {
    uint32_t w;
    __device__ __forceinline__ void load(const WaveTile *tiles, unsigned i)
    {
        constexpr int words = sizeof(WaveTile) / 4;
        w = reinterpret_cast<const uint32_t *>(tiles + i)[(threadIdx.x & 63) % words];
    }
    __device__ __forceinline__ uint32_t word(int k) const { return __builtin_amdgcn_readlane(w, k); }
    template <class P>
    __device__ __forceinline__ P *ptr(int k) const
    {
        return reinterpret_cast<P *>(((uint64_t)word(k + 1) << 32) | word(k));
    }
    __device__ __forceinline__ WaveTile get() const
    {
        WaveTile t;
        t.a = ptr<const void>(0);
        t.b = ptr<const void>(2);
        t.out = ptr<void>(4);
        t.pitch = (int64_t)(((uint64_t)word(7) << 32) | word(6));
        t.kind = (int32_t)word(8);
        t.n = (int32_t)word(9);
        t.rows = (int32_t)word(10);
        t.ntiles = (int32_t)word(11);
        t.slot = (int32_t)word(12);
        t.problem = (int32_t)word(13);
        t.alpha = bits_to_float(word(14));
        t.beta = bits_to_float(word(15));
        return t;
    }
};

// The wavefront's sum over n elements of x (and y), in every lane.
template <class T, int OP, int ACC, int U>
__device__ __forceinline__ typename BlockT<ACC>::type wave_reduce(const char *x, const char *y, int32_t n, int lane)
{
    constexpr int VB = 16, E = Elems<T, VB>::value;
    using V = typename Vec<VB>::type;
    const int32_t nvec = n / E, tail0 = nvec * E;
    // fewer than E elements past the last vector, read ahead
    const bool tail = tail0 + lane < n;
    float tx = 0.f, ty = 0.f;
    if (tail) {
        tx = load_elem<T>(x, tail0 + lane);
        if constexpr (OP == OP_DOT)
            ty = load_elem<T>(y, tail0 + lane);
    }
    LaneAcc<ACC, E> acc;
    int32_t base = 0;
    for (; base + 64 * U <= nvec; base += 64 * U) {
        V vx[U], vy[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t at = (int64_t)(base + lane + 64 * k) * VB;
            vx[k] = load_stream_any<T, VB>(x + at);
            if constexpr (OP == OP_DOT)
                vy[k] = load_stream_any<T, VB>(y + at);
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
    if (base < nvec) {  // the last, partial step: clamped loads, zeros past the end
        V vx[U], vy[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t at = (int64_t)min(base + lane + 64 * k, nvec - 1) * VB;
            vx[k] = load_stream_any<T, VB>(x + at);
            if constexpr (OP == OP_DOT)
                vy[k] = load_stream_any<T, VB>(y + at);
        }
        loads_in_flight();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool in = base + lane + 64 * k < nvec;
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
    if (tail)
        accumulate_scalar<T, OP, ACC, E>(acc, tx, ty);
    return wave_sum(acc.value());
}

template <int ACC, int E>
__device__ __forceinline__ RowPartT<ACC> lane_part(const RowAcc<ACC, E> &acc)
{
    if constexpr (ACC == ACC_F64)
        return (double)acc.value();
    else
        return acc.value();
}

// Rows of a gemv tile that L lanes x V vectors cover, 64 / L side by side and
// R such groups in flight (gemv_rows_kernel's arithmetic and layout, with
// every row read from where it starts).
template <class T, int ACC, int VB, int L, int V, int R, int WHOLE = V - 1>
__device__ __forceinline__ void wave_rows(const WaveTile &t, int lane)
{
    constexpr int E = Elems<T, VB>::value, G = 64 / L, B = V >= 8 ? 4 : V;   // B: vectors loaded together
    static_assert(V % B == 0 && R <= L, "whole batches of loads; lane i of a group stores row i");
    using VT = typename Vec<VB>::type;
    using D = RowPartT<ACC>;
    const int sub = lane % L, side = lane / L;
    const char *A = reinterpret_cast<const char *>(t.a);
    float *y = reinterpret_cast<float *>(t.out);

    LaneCols<T, ACC, VB, V, WHOLE> cols;
    cols.set(reinterpret_cast<const float *>(t.b), t.n, 0, sub, L);
    cols.mask();
    for (int32_t r0 = 0; r0 < t.rows; r0 += G * R) {   // wave-uniform
        const char *row[R];
#pragma unroll
        for (int i = 0; i < R; ++i)
            row[i] = A + (int64_t)min(r0 + i * G + side, t.rows - 1) * t.pitch;
        const int32_t mine = r0 + sub * G + side;      // the row this lane stores
        const bool stores = sub < R && mine < t.rows;
        const float yold = stores && t.beta != 0.f ? y[mine] : 0.f;
        RowAcc<ACC, E> acc[R];
#pragma unroll
        for (int k0 = 0; k0 < V; k0 += B) {
            VT v[R][B];
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int k = 0; k < B; ++k)
                    v[i][k] = load_stream_any<T, VB>(row[i] + cols.at(k0 + k));
            loads_in_flight();
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int k = 0; k < B; ++k)
                    cols.add(acc[i], k0 + k, v[i][k]);
        }
        D sum = {};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const D d = lanes_sum<L>(lane_part<ACC, E>(acc[i]));
            if (sub == i)
                sum = d;
        }
        if (stores)
            y[mine] = row_epilogue<ACC>(sum, t.alpha, t.beta, yold);
    }
}

// Rows longer than the registers hold of x: x from the cache, two rows at a
// time sharing it.
template <class T, int ACC>
__device__ __forceinline__ void wave_long_rows(const WaveTile &t, int lane)
{
    constexpr int VB = 16, E = Elems<T, VB>::value, R = 2, U = 4;
    using VT = typename Vec<VB>::type;
    using D = RowPartT<ACC>;
    const float *x = reinterpret_cast<const float *>(t.b);
    float *y = reinterpret_cast<float *>(t.out);
    const int32_t nvec = t.n / E, tail0 = nvec * E;
    const bool tail = tail0 + lane < t.n;
    const float tx = tail ? x[tail0 + lane] : 0.f;
    for (int32_t r0 = 0; r0 < t.rows; r0 += R) {
        const char *row[R];
        float ta[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            row[i] = reinterpret_cast<const char *>(t.a) + (int64_t)min(r0 + i, t.rows - 1) * t.pitch;
            ta[i] = tail ? load_elem<T>(row[i], tail0 + lane) : 0.f;
        }
        const bool stores = lane < R && r0 + lane < t.rows;
        const float yold = stores && t.beta != 0.f ? y[r0 + lane] : 0.f;
        RowAcc<ACC, E> acc[R];
        for (int32_t base = 0; base < nvec; base += 64 * U) {
            float xf[U][E];
            VT v[R][U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int32_t q = min(base + lane + 64 * k, nvec - 1);
                load_x_any<E>(x, (int64_t)q * E, xf[k]);
#pragma unroll
                for (int i = 0; i < R; ++i)
                    v[i][k] = load_stream_any<T, VB>(row[i] + (int64_t)q * VB);
            }
            loads_in_flight();
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const bool in = base + lane + 64 * k < nvec;
#pragma unroll
                for (int e = 0; e < E; ++e)
                    xf[k][e] = in ? xf[k][e] : 0.f;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    float f[E];
                    decode<T, VB>(v[i][k], f);
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        f[e] = in ? f[e] : 0.f;
                    acc[i].add(f, xf[k]);
                }
            }
        }
        D sum = {};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (tail)
                acc[i].add_scalar(ta[i], tx);
            const D d = lanes_sum<64>(lane_part<ACC, E>(acc[i]));
            if (lane == i)
                sum = d;
        }
        if (stores)
            y[r0 + lane] = row_epilogue<ACC>(sum, t.alpha, t.beta, yold);
    }
}

// A gemv tile by its row length (all wave-uniform).  Each instance takes the
// rows that the one before does not cover, so all but the last of its lanes'
// vectors are whole (or the WHOLE that it names), and keeps 3 to 8 loads in
// flight.
template <class T, int ACC>
__device__ __forceinline__ void wave_gemv(const WaveTile &t, int lane)
{
    constexpr int EB = T::bytes, E = 16 / EB;
    // the compensated sums' terms leave 16-bit storage fewer registers for x
    constexpr bool WIDE = EB == 4 || ACC != ACC_COMP;
    const int32_t vecs = (t.n + E - 1) / E;
    if (t.n < E) {
        if (t.n > 0) {
            wave_rows<T, ACC, EB, 8, 1, 4>(t, lane);
        } else {  // y = beta y
            float *y = reinterpret_cast<float *>(t.out);
            for (int32_t r = lane; r < t.rows; r += 64)
                y[r] = row_epilogue<ACC>(RowPartT<ACC>{}, t.alpha, t.beta, t.beta != 0.f ? y[r] : 0.f);
        }
    } else if (vecs <= 8) {
        wave_rows<T, ACC, 16, 8, 1, 4>(t, lane);
    } else if (vecs <= 16) {
        wave_rows<T, ACC, 16, 16, 1, 4>(t, lane);
    } else if (vecs <= 32) {
        wave_rows<T, ACC, 16, 32, 1, 4>(t, lane);
    } else if (vecs <= 64) {
        wave_rows<T, ACC, 16, 64, 1, 4>(t, lane);
    } else if (vecs <= 128) {
        wave_rows<T, ACC, 16, 64, 2, 2>(t, lane);
    } else if (vecs <= 192) {
        wave_rows<T, ACC, 16, 64, 3, EB == 4 ? 2 : 1>(t, lane);
    } else if (vecs <= 256) {
        wave_rows<T, ACC, 16, 64, 4, 1>(t, lane);
    } else if (vecs <= 320) {
        wave_rows<T, ACC, 16, 64, 5, 1>(t, lane);
    } else if (vecs <= 384) {
        wave_rows<T, ACC, 16, 64, 6, 1>(t, lane);
    } else if (WIDE && vecs <= 448) {
        if constexpr (WIDE)
            wave_rows<T, ACC, 16, 64, 7, 1>(t, lane);
    } else if (WIDE && vecs <= 512) {
        if constexpr (WIDE)
            wave_rows<T, ACC, 16, 64, 8, 1>(t, lane);
    } else if (EB == 4 && ACC == ACC_F32 && vecs <= 768) {   // more than 512: 8 vectors are whole
        if constexpr (EB == 4 && ACC == ACC_F32)
            wave_rows<T, ACC, 16, 64, 12, 1, 8>(t, lane);
    } else if (EB == 4 && ACC == ACC_F32 && vecs <= 1024) {   // more than 768: 12
        if constexpr (EB == 4 && ACC == ACC_F32)
            wave_rows<T, ACC, 16, 64, 16, 1, 12>(t, lane);
    } else {
        wave_long_rows<T, ACC>(t, lane);
    }
}

// Stamped instances, lane 0: the tile's start, what it is and who takes it.
__device__ __forceinline__ void stamp_wave_tile(const BatchWaveArgs &a, unsigned ti, const WaveTile &t)
{
    const uint32_t xcc = __builtin_amdgcn_s_getreg((20 << 0) | (0 << 6) | (3 << 11));  // XCC_ID[3:0]
    const uint32_t hw = __builtin_amdgcn_s_getreg((4 << 0) | (8 << 6) | (7 << 11));    // HW_ID[15:8]
    uint64_t *w = a.stamps + (int64_t)a.records[ti] * STAMPS_PER_TILE;
    w[0] = (uint64_t)wall_clock64();
    w[2] = ((uint64_t)(uint32_t)t.problem << 32) | (uint32_t)(t.kind == KIND_GEMV ? t.rows : t.n);
    w[3] = ((uint64_t)((xcc << 16) | hw) << 32) | (uint32_t)blockIdx.x;
}

// Puts lane 0's partial into a slot and counts it in on a counter; whether it
// is the last of `count`.
template <class ST>
__device__ __forceinline__ bool slot_last(char *slot, ST v, unsigned *counter, int32_t count, int lane)
{
    int last = 0;
    if (lane == 0) {
        store_coherent(slot, v);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);  // the partial's store has completed
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(count - 1);
        if (last)
            __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return __builtin_amdgcn_readfirstlane(last);
}

// A reduction tile's partial v (the same in every lane): the problem's result,
// or to its slot; the wavefront whose partial is the problem's last folds all
// of them in tile order.  A problem of more than TILE_GROUP tiles is folded
// group by group first, by the last wavefront of each group, whose sum takes
// the group's first slot: counting thousands in on one address and folding
// them with one wavefront took 45 us (a dot of 6.8 M bf16 by itself: 58 us).
template <int ACC>
__device__ __forceinline__ void finish_tile(const BatchWaveArgs &a, const WaveTile &t, typename BlockT<ACC>::type v, int lane)
{
    using ST = typename SlotT<ACC>::type;
    if (t.ntiles == 1) {
        if (lane == 0)
            write_result(t.out, a.result_f64, to_slot<ACC>(v));
        return;
    }
    char *slots = a.slots + (int64_t)(t.slot - t.rows) * WS_SLOT;   // rows: the tile's number in its problem
    const int32_t group = t.rows / TILE_GROUP, groups = (t.ntiles + TILE_GROUP - 1) / TILE_GROUP;
    const int32_t size = min(TILE_GROUP, t.ntiles - group * TILE_GROUP);
    char *first = slots + (int64_t)group * TILE_GROUP * WS_SLOT;
    unsigned *counter = groups == 1 ? &a.pcount[t.problem]
                                    : reinterpret_cast<unsigned *>(a.gcount + (int64_t)(t.slot / TILE_GROUP) * WS_GROUP_STRIDE);
    if (!slot_last<ST>(a.slots + (int64_t)t.slot * WS_SLOT, to_slot<ACC>(v), counter, size, lane))
        return;
    ST acc = zero_of<ST>();
    if (lane < size)
        acc = load_coherent<ST>(first + (int64_t)lane * WS_SLOT);
    acc = wave_sum(acc);
    if (groups > 1) {
        if (!slot_last<ST>(first, acc, &a.pcount[t.problem], groups, lane))
            return;
        acc = zero_of<ST>();
        for (int32_t i = lane; i < groups; i += 64)
            acc = merge(acc, load_coherent<ST>(slots + (int64_t)i * TILE_GROUP * WS_SLOT));
        acc = wave_sum(acc);
    }
    if (lane == 0)
        write_result(t.out, a.result_f64, acc);
}

// A work-group has drawn its last tile (one thread, all wavefronts done): the
// last one out resets the counters for the next run.
__device__ __forceinline__ void leave(const BatchWaveArgs &a)
{
    if (!arrive(a.done, a.groups))
        return;
    for (int l = 0; l < DRAW_LISTS; ++l)
        __hip_atomic_store(reinterpret_cast<unsigned *>(a.lists + l * WS_GROUP_STRIDE), 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T, int ACC, bool STAMP = false>
__global__ void __launch_bounds__(256, 4) batch_wave_kernel(BatchWaveArgs a)
{
    using BT = typename BlockT<ACC>::type;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned list = blockIdx.x % DRAW_LISTS;
    // among the list's wavefronts (the grid is a multiple of DRAW_LISTS): a
    // first one of every work-group, then a second, ..., so that few tiles
    // spread over the CUs
    const unsigned rank = wv * (gridDim.x / DRAW_LISTS) + blockIdx.x / DRAW_LISTS;
    const unsigned waves = 4 * (gridDim.x / DRAW_LISTS);
    unsigned *counter = reinterpret_cast<unsigned *>(a.lists + list * WS_GROUP_STRIDE);
    const auto draw = [&]() -> unsigned {   // lane 0 only; the caller broadcasts when it needs it
        return lane == 0 && a.dynamic
                   ? waves + __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   : NO_TILE;
    };
    // Of the list's tile `pos`; past the table's end: none left.  Indices stay
    // in 32 bits and are never clamped by a select: of `i < n ? i : n` on
    // uniform 64-bit values in such a loop the compiler (ROCm 7.2) has lost
    // the compare's result (s_cselect on an older SCC) and read past the table.
    const auto index = [&](unsigned pos) -> unsigned {
        return (unsigned)__builtin_amdgcn_readfirstlane(pos) * DRAW_LISTS + list;
    };
    const unsigned ntiles = a.ntiles;

    unsigned ti = index(rank);
    unsigned drawn = draw();
    TileWords words;
    if (ti < ntiles)
        words.load(a.tiles, ti);
    while (ti < ntiles) {
        const WaveTile t = words.get();
        const unsigned next = index(drawn);
        if (next < ntiles) {
            words.load(a.tiles, next);
            drawn = draw();
        }
        if constexpr (STAMP) {
            if (lane == 0)
                stamp_wave_tile(a, ti, t);
        }
        // opaque per tile: what the branches below derive from the lane would
        // otherwise be hoisted out of the loop and held in registers by all
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (t.kind == KIND_GEMV) {
            wave_gemv<T, ACC>(t, ln);
        } else {
            const char *x = reinterpret_cast<const char *>(t.a), *y = reinterpret_cast<const char *>(t.b);
            const BT v = t.kind == KIND_ASUM ? wave_reduce<T, OP_ASUM, ACC, 8>(x, nullptr, t.n, ln)
                                             : wave_reduce<T, OP_DOT, ACC, 4>(x, y, t.n, ln);
            finish_tile<ACC>(a, t, v, lane);
        }
        if constexpr (STAMP) {
            if (lane == 0)
                a.stamps[(int64_t)a.records[ti] * STAMPS_PER_TILE + 1] = (uint64_t)wall_clock64();
        }
        ti = next;
    }
    if (a.dynamic) {
        __syncthreads();
        if (threadIdx.x == 0)
            leave(a);
    }
}

template <class T>
const void *pick_batch_wave(int acc, bool stamped)
{
    if (stamped)
        return acc == ACC_F32 ? reinterpret_cast<const void *>(&batch_wave_kernel<T, ACC_F32, true>) : nullptr;
    switch (acc) {
    case ACC_F32: return reinterpret_cast<const void *>(&batch_wave_kernel<T, ACC_F32>);
    case ACC_COMP: return reinterpret_cast<const void *>(&batch_wave_kernel<T, ACC_COMP>);
    case ACC_F64: return reinterpret_cast<const void *>(&batch_wave_kernel<T, ACC_F64>);
    default: return nullptr;
    }
}

}  // namespace lift
