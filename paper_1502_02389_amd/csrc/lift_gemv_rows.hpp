// gemv for rows of any length, pitch and alignment: the launches of calls
// that leave the launch to the library.
//
// Three lowerings of map(scal(alpha) o dot(x)) over the rows, by row length:
//   gemv_rows_kernel : rows that one step of at most 64 lanes x 8 vectors
//                      covers.  L lanes (8 .. 64) share a row, 64 / L rows
//                      per wavefront at a time, R such groups of rows in
//                      flight, x held in registers over all rows.
//   gemv_rows_wg_kernel : longer rows that one step of a work-group covers,
//                      one row at a time, x held in registers.
//   gemv_panel_kernel: rows longer than that, or too few of them to fill the
//                      chip: a work-group takes R rows x a chunk of columns;
//                      the chunks of a row meet through a caller workspace.
//
// All of them read 16 bytes per lane from wherever a row starts.  gfx950
// serves a 16-byte load at any 4-byte boundary at the full streaming rate
// (512 MiB flat read: 74.4-75.0 us at byte offsets 0, 4, 8, 12) and at an odd
// 2-byte boundary in 35 % more time (100.5-101.0 us), so only 16-bit rows that
// start between two dwords need anything: their first column is taken as a
// scalar head and the vectors start at the second.  With an odd pitch every
// other row is such a row; the rows are dealt so that a lane only ever meets
// rows of one kind and its columns (and its part of x) stay the same.
// A row's last vector, if it is not whole, is read ending at the row's last
// column and the elements that the vector before it already holds are
// replaced by zeros, so every load lies inside its row.
#pragma once

#include "lift_gemv.hpp"

namespace lift {

// E consecutive binary32 values of x from element c on, at any alignment.
template <int E>
__device__ __forceinline__ void load_x_any(const float *x, int64_t c, float *o)
{
    if constexpr (E < 4) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            o[e] = x[c + e];
    } else {
#pragma unroll
        for (int h = 0; h < E / 4; ++h) {
            const u32x4 w = *reinterpret_cast<const u32x4_at4 *>(x + c + 4 * h);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o[4 * h + i] = bits_to_float(w[i]);
        }
    }
}

// y_i from the row's finished dot, y_i read before (`yold`).
template <int ACC>
__device__ __forceinline__ float row_epilogue(RowPartT<ACC> d, float alpha, float beta, float yold)
{
    if constexpr (ACC == ACC_F64) {
        const double by = beta == 0.f ? 0.0 : (double)beta * (double)yold;
        return (float)((double)alpha * d + by);
    } else {
        const float by = beta == 0.f ? 0.f : beta * yold;
        if constexpr (ACC == ACC_COMP)
            return fmaf(alpha, d.s + d.c, by);
        else
            return fmaf(alpha, d, by);
    }
}

// Scalar columns before a row's vectors: 1 where a 16-bit row starts between
// two dwords, else 0.
template <class T>
__device__ __forceinline__ int row_head(const void *A, int64_t lda, int64_t row)
{
    if constexpr (T::bytes == 2)
        return (int)(((reinterpret_cast<uintptr_t>(A) >> 1) + (uintptr_t)(row * lda)) & 1);
    else
        return 0;
}

// A lane's columns of every row it meets: V vectors of E columns, vector k
// from column head + (sub + L k) E on.  The row has more than L WHOLE vectors
// (by default all but a lane's last: V is the smallest that covers the row),
// so the first WHOLE of every lane are whole; a later one that would pass the
// row's last column is moved back to end there, and its leading elements that
// belong to the vector before (all, past the row) count as zeros.  Byte
// offsets are 32-bit (a row whose x the registers hold is short), which with a
// wave-uniform row leaves the address to the scalar unit.
template <class T, int ACC, int VB, int V, int WHOLE = V - 1>
struct LaneCols {
    static constexpr int E = Elems<T, VB>::value;
    uint32_t first, step;   // byte offset of vector 0 in a row, distance between vectors
    uint32_t end;           // of the last place where a vector fits
    float x[V][E];

    // vector k's byte offset, and how many of its leading elements to skip
    __device__ __forceinline__ uint32_t at(int k) const
    {
        return k < WHOLE ? first + k * step : min(first + k * step, end);
    }
    __device__ __forceinline__ int skip(int k) const { return (int)((first + k * step - at(k)) / T::bytes); }

    __device__ __forceinline__ void set(const float *xs, int64_t n, int head, int sub, int L)   // n >= E
    {
        first = (uint32_t)(head + sub * E) * T::bytes;
        step = (uint32_t)L * VB;
        end = (uint32_t)(n - E) * T::bytes;
#pragma unroll
        for (int k = 0; k < V; ++k)
            load_x_any<E>(xs, at(k) / T::bytes, x[k]);
    }
    // Zeros for the elements of x that are not the lane's.  Called once, after
    // the first rows' loads are issued, so that they do not wait for x
    // (300 x 9000 fp32, one row per work-group: 6.3 -> 5.0 us, with y read
    // ahead as well).
    __device__ __forceinline__ void mask()
    {
#pragma unroll
        for (int k = WHOLE; k < V; ++k)
#pragma unroll
            for (int e = 0; e < E; ++e)
                x[k][e] = e >= skip(k) ? x[k][e] : 0.f;
    }
    // The row's terms of vector k (loaded as v), into acc.
    __device__ __forceinline__ void add(RowAcc<ACC, E> &acc, int k, const typename Vec<VB>::type &v) const
    {
        float a[E];
        decode<T, VB>(v, a);
        if (k >= WHOLE) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                a[e] = e >= skip(k) ? a[e] : 0.f;
        }
        acc.add(a, x[k]);
    }
};

// Rows that 64 lanes x V vectors (or L < 64 lanes x one vector) cover.  A
// wavefront's block of rows is R x rs rows, rs = 64 / L rows side by side
// (with L = 64, two wavefronts take the even and the odd rows of a block
// where the rows' starts alternate); the R loads per vector are all in flight
// before any arithmetic.  After the butterfly every lane of a group holds
// the group's R sums: lane i of the group stores row i, so the rows' results
// leave in one store.
template <class T, int ACC, int VB, int L, int V, int R>
__global__ void __launch_bounds__(256) gemv_rows_kernel(GemvRowsArgs a)
{
    static_assert(R <= L, "lane i of a group stores row i");
    constexpr int E = Elems<T, VB>::value;
    constexpr int G = 64 / L;
    using VT = typename Vec<VB>::type;
    using D = RowPartT<ACC>;
    const int lane = threadIdx.x & 63, sub = lane % L;
    const int64_t wave = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int P = a.classes;
    const int rs = G > 1 ? G : P;
    const int ro = G > 1 ? lane / L : (int)(wave % P);
    const int64_t first = G > 1 ? wave : wave / P, stride = G > 1 ? nwaves : nwaves / P;
    const int head = VB == 16 ? row_head<T>(a.A, a.lda, ro) : 0;
    const int64_t pitch = a.lda * T::bytes;

    LaneCols<T, ACC, VB, V> cols;
    cols.set(a.x, a.n, head, sub, L);
    const bool heads = VB == 16 && T::bytes == 2 && a.heads;   // some row has a head column (uniform)
    const bool mine = heads && head && sub == 0;
    const float hx = mine ? a.x[0] : 0.f;

    int64_t u = first;
    if (u * rs * R >= a.m)
        return;
    int64_t myrow;   // the row this lane stores
    float yold;
    VT v[R][V];
    typename T::raw h[R] = {};
    const auto load_rows = [&] {
        const int64_t r0 = u * rs * R + ro;
        const char *row[R];
#pragma unroll
        for (int i = 0; i < R; ++i)
            row[i] = reinterpret_cast<const char *>(a.A) + min(r0 + (int64_t)i * rs, a.m - 1) * pitch;
        myrow = r0 + (int64_t)sub * rs;
        yold = sub < R && myrow < a.m && a.beta != 0.f ? a.y[myrow] : 0.f;
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int k = 0; k < V; ++k)
                v[i][k] = load_stream_any<T, VB>(row[i] + cols.at(k));
        if (mine) {  // one lane per row: a load by all of them costs as much as a vector
#pragma unroll
            for (int i = 0; i < R; ++i)
                h[i] = *reinterpret_cast<const typename T::raw *>(row[i]);
        }
        loads_in_flight();
    };
    load_rows();
    cols.mask();
    while (true) {
        D sum = {};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            RowAcc<ACC, E> acc;
#pragma unroll
            for (int k = 0; k < V; ++k)
                cols.add(acc, k, v[i][k]);
            if (heads)
                acc.add_scalar(decode_raw<T>(h[i]), hx);
            D d;
            if constexpr (ACC == ACC_F64)
                d = lanes_sum<L>((double)acc.value());
            else
                d = lanes_sum<L>(acc.value());
            if (sub == i)
                sum = d;
        }
        if (sub < R && myrow < a.m)
            a.y[myrow] = row_epilogue<ACC>(sum, a.alpha, a.beta, yold);
        u += stride;
        if (u * rs * R >= a.m)
            return;
        load_rows();
    }
}

// Rows that one step of a work-group covers: x in registers, one row at a
// time; the wave partials are parked in LDS and 16 rows finish together, as
// in gemv_xs_rows (two banks alternate, one barrier per 16 rows).  Work-group
// b takes rows b, b + G, ... (G even where the rows' starts alternate).
template <class T, int ACC, int V>
__global__ void __launch_bounds__(512) gemv_rows_wg_kernel(GemvRowsArgs a)
{
    constexpr int VB = 16, E = Elems<T, VB>::value, PARK = 16;
    using VT = typename Vec<VB>::type;
    using D = RowPartT<ACC>;
    __shared__ D lds[2][PARK][8];   // [bank][row][wave]
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, waves = blockDim.x >> 6;
    const int64_t step = gridDim.x;
    const int head = row_head<T>(a.A, a.lda, blockIdx.x);
    const int64_t pitch = a.lda * T::bytes;

    LaneCols<T, ACC, VB, V> cols;
    cols.set(a.x, a.n, head, t, blockDim.x);
    const bool mine = head && t == 0;
    const float hx = mine ? a.x[0] : 0.f;

    int j = 0;
    int64_t r = blockIdx.x;   // the grid never exceeds the row count
    float yold = 0.f;         // thread t: y of the parked row t, read with the row
    VT v[V];
    typename T::raw h = 0;
    const auto load_row = [&] {
        const char *row = reinterpret_cast<const char *>(a.A) + r * pitch;
#pragma unroll
        for (int k = 0; k < V; ++k)
            v[k] = load_stream_any<T, VB>(row + cols.at(k));
        if (mine)
            h = *reinterpret_cast<const typename T::raw *>(row);
        if (t == j % PARK && a.beta != 0.f)
            yold = a.y[r];
        loads_in_flight();
    };
    load_row();
    cols.mask();
    while (true) {  // uniform
        RowAcc<ACC, E> acc;
#pragma unroll
        for (int k = 0; k < V; ++k)
            cols.add(acc, k, v[k]);
        if (head)
            acc.add_scalar(decode_raw<T>(h), hx);
        const D w = wave_row_partial<ACC, E>(acc);
        const int slot = j % PARK, bank = (j / PARK) & 1;
        if (lane == 0)
            lds[bank][slot][wave] = w;
        if (slot == PARK - 1 || r + step >= a.m) {  // uniform: finish the parked rows
            __syncthreads();
            if (t <= slot) {
                const int64_t i = blockIdx.x + (int64_t)(j - slot + t) * step;
                D d = lds[bank][t][0];
                for (int q = 1; q < waves; ++q)
                    d = merge(d, lds[bank][t][q]);
                a.y[i] = row_epilogue<ACC>(d, a.alpha, a.beta, yold);
            }
        }
        r += step;
        ++j;
        if (r >= a.m)
            return;
        load_row();
    }
}

// R rows x a chunk of columns per work-group: work-group b takes row group
// b % groups and chunk b / groups, so the work-groups that run together share
// their part of x in the cache.  The R rows of a group start alike (they are
// `classes` apart) and share every x load.  One chunk: the rows are finished
// here.  More: the group's work-groups meet in its slots of the workspace
// (meet()) and one of them folds the partials in chunk order (lane t: chunks t,
// t + 64, ..., then the wave butterfly), so the result does not depend on the
// order of arrival.
template <class T, int ACC, int R, int U>
__global__ void __launch_bounds__(512) gemv_panel_kernel(GemvPanelArgs a)
{
    constexpr int VB = 16, E = Elems<T, VB>::value;
    using VT = typename Vec<VB>::type;
    using D = RowPartT<ACC>;
    __shared__ D lds[R][8];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, waves = blockDim.x >> 6;
    const int64_t B = blockDim.x;
    const int64_t group = blockIdx.x % a.groups, chunk = blockIdx.x / a.groups;
    const int P = a.rows.classes;
    const int64_t r0 = group % P + group / P * P * R;   // rows r0, r0 + P, ..., r0 + (R - 1) P
    const int64_t n = a.rows.n, m = a.rows.m, pitch = a.rows.lda * T::bytes;
    const int head = row_head<T>(a.rows.A, a.rows.lda, r0);
    const int64_t nv = (n - head) / E, tail0 = head + nv * E;
    const int64_t vbeg = chunk * a.chunk, vend = min(vbeg + a.chunk, nv);
    const bool last_chunk = chunk == a.chunks - 1;

    const char *row[R];
#pragma unroll
    for (int i = 0; i < R; ++i)
        row[i] = reinterpret_cast<const char *>(a.rows.A) + min(r0 + i * P, m - 1) * pitch;
    // the scalar columns: the head (chunk 0, lane 0) and the tail (last
    // chunk, lanes 1 ..), read ahead and added after the vectors
    const bool extra = (chunk == 0 && head && t == 0) || (last_chunk && t >= 1 && tail0 + t - 1 < n);
    const int64_t ecol = extra && t >= 1 ? tail0 + t - 1 : 0;
    typename T::raw er[R];
    float ex = 0.f;
    if (extra) {
        ex = a.rows.x[ecol];
#pragma unroll
        for (int i = 0; i < R; ++i)
            er[i] = reinterpret_cast<const typename T::raw *>(row[i])[ecol];
    }

    const bool row_lane = t < R && r0 + t * P < m;   // thread i finishes row i
    const float yold = row_lane && a.rows.beta != 0.f ? a.rows.y[r0 + t * P] : 0.f;

    RowAcc<ACC, E> acc[R];
    const int64_t step = B * U;
    const char *xs = reinterpret_cast<const char *>(a.rows.x + head);
    int64_t base = vbeg;
    for (; base + step <= vend; base += step) {
        float xf[U][E];
        VT v[R][U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            load_x_any<E>(reinterpret_cast<const float *>(xs), (base + t + k * B) * E, xf[k]);
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int k = 0; k < U; ++k)
                v[i][k] = load_stream_any<T, VB>(row[i] + head * T::bytes + (base + t + k * B) * VB);
        loads_in_flight();
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int k = 0; k < U; ++k) {
                float f[E];
                decode<T, VB>(v[i][k], f);
                acc[i].add(f, xf[k]);
            }
    }
    if (base < vend) {  // the last, partial step: clamped loads, zeros past the end
        float xf[U][E];
        VT v[R][U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t q = min(base + t + k * B, vend - 1);
            load_x_any<E>(reinterpret_cast<const float *>(xs), q * E, xf[k]);
#pragma unroll
            for (int i = 0; i < R; ++i)
                v[i][k] = load_stream_any<T, VB>(row[i] + head * T::bytes + q * VB);
        }
        loads_in_flight();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool in = base + t + k * B < vend;
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
    if (extra) {
#pragma unroll
        for (int i = 0; i < R; ++i)
            acc[i].add_scalar(decode_raw<T>(er[i]), ex);
    }

#pragma unroll
    for (int i = 0; i < R; ++i) {
        const D w = wave_row_partial<ACC, E>(acc[i]);
        if (lane == 0)
            lds[i][wave] = w;
    }
    __syncthreads();
    if (t >= 64)
        return;
    D d = zero_of<D>();
    if (t < R) {
        d = lds[t][0];
        for (int q = 1; q < waves; ++q)
            d = merge(d, lds[t][q]);
    }
    if (a.chunks == 1) {
        if (row_lane)
            a.rows.y[r0 + t * P] = row_epilogue<ACC>(d, a.rows.alpha, a.rows.beta, yold);
        return;
    }
    unsigned *pending = reinterpret_cast<unsigned *>(a.ws + WS_GROUPS + group * WS_GROUP_STRIDE);
    meet<1, D, R>(a.ws, pending, group * a.chunks * R, a.chunks, chunk, d, a.rounds, [&](D(&v)[R]) {
        D sum = zero_of<D>();
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const D s = lanes_sum<64>(v[i]);
            if (t == i)
                sum = s;
        }
        if (row_lane)
            a.rows.y[r0 + t * P] = row_epilogue<ACC>(sum, a.rows.alpha, a.rows.beta, yold);
    });
}

// Instances.  rows: (L, V) covering the row, R rows per group in flight.
template <class T, int ACC, int L, int V>
const void *gemv_rows_pick(int r)
{
    constexpr int RMAX = 8 / V;
    if (r == 1)
        return reinterpret_cast<const void *>(&gemv_rows_kernel<T, ACC, 16, L, V, 1>);
    if (r == RMAX)
        return reinterpret_cast<const void *>(&gemv_rows_kernel<T, ACC, 16, L, V, RMAX>);
    return nullptr;
}

template <class T, int ACC>
const void *gemv_rows_pick_shape(int vec_bytes, int lanes, int v, int r)
{
    if (vec_bytes == T::bytes)
        return lanes == 8 && v == 1 && r == 8
                   ? reinterpret_cast<const void *>(&gemv_rows_kernel<T, ACC, T::bytes, 8, 1, 8>) : nullptr;
    if (vec_bytes != 16)
        return nullptr;
    switch (lanes * 16 + v) {
    case 8 * 16 + 1: return gemv_rows_pick<T, ACC, 8, 1>(r);
    case 16 * 16 + 1: return gemv_rows_pick<T, ACC, 16, 1>(r);
    case 32 * 16 + 1: return gemv_rows_pick<T, ACC, 32, 1>(r);
    case 64 * 16 + 1: return gemv_rows_pick<T, ACC, 64, 1>(r);
    case 64 * 16 + 2: return gemv_rows_pick<T, ACC, 64, 2>(r);
    case 64 * 16 + 3: return gemv_rows_pick<T, ACC, 64, 3>(r);
    case 64 * 16 + 4: return gemv_rows_pick<T, ACC, 64, 4>(r);
    case 64 * 16 + 5: return gemv_rows_pick<T, ACC, 64, 5>(r);
    case 64 * 16 + 6: return gemv_rows_pick<T, ACC, 64, 6>(r);
    case 64 * 16 + 7: return gemv_rows_pick<T, ACC, 64, 7>(r);
    case 64 * 16 + 8: return gemv_rows_pick<T, ACC, 64, 8>(r);
    default: return nullptr;
    }
}

template <class T, int ACC>
const void *gemv_rows_wg_pick(int v)
{
    switch (v) {
    case 3: return reinterpret_cast<const void *>(&gemv_rows_wg_kernel<T, ACC, 3>);
    case 4: return reinterpret_cast<const void *>(&gemv_rows_wg_kernel<T, ACC, 4>);
    case 5: return reinterpret_cast<const void *>(&gemv_rows_wg_kernel<T, ACC, 5>);
    case 6: return reinterpret_cast<const void *>(&gemv_rows_wg_kernel<T, ACC, 6>);
    case 7: return reinterpret_cast<const void *>(&gemv_rows_wg_kernel<T, ACC, 7>);
    case 8: return reinterpret_cast<const void *>(&gemv_rows_wg_kernel<T, ACC, 8>);
    default: return nullptr;
    }
}

template <class T, int ACC>
const void *gemv_panel_pick(int r)
{
    switch (r) {
    case 1: return reinterpret_cast<const void *>(&gemv_panel_kernel<T, ACC, 1, 4>);
    case 2: return reinterpret_cast<const void *>(&gemv_panel_kernel<T, ACC, 2, 4>);
    case 4: return reinterpret_cast<const void *>(&gemv_panel_kernel<T, ACC, 4, 2>);
    default: return nullptr;
    }
}

template <class T>
const void *pick_gemv_rows(int acc, int vec_bytes, int lanes, int v, int r)
{
    switch (acc) {
    case ACC_F32: return gemv_rows_pick_shape<T, ACC_F32>(vec_bytes, lanes, v, r);
    case ACC_COMP: return gemv_rows_pick_shape<T, ACC_COMP>(vec_bytes, lanes, v, r);
    case ACC_F64: return gemv_rows_pick_shape<T, ACC_F64>(vec_bytes, lanes, v, r);
    default: return nullptr;
    }
}

template <class T>
const void *pick_gemv_rows_wg(int acc, int v)
{
    switch (acc) {
    case ACC_F32: return gemv_rows_wg_pick<T, ACC_F32>(v);
    case ACC_COMP: return gemv_rows_wg_pick<T, ACC_COMP>(v);
    case ACC_F64: return gemv_rows_wg_pick<T, ACC_F64>(v);
    default: return nullptr;
    }
}

template <class T>
const void *pick_gemv_panel(int acc, int r)
{
    switch (acc) {
    case ACC_F32: return gemv_panel_pick<T, ACC_F32>(r);
    case ACC_COMP: return gemv_panel_pick<T, ACC_COMP>(r);
    case ACC_F64: return gemv_panel_pick<T, ACC_F64>(r);
    default: return nullptr;
    }
}

}  // namespace lift
