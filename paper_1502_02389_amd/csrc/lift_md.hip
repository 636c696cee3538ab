// MD: the force on every particle from its neighbour list (Fig. 7):
//   md(ps, N, t) = map(lambda (p, ns): reduce(lambda (f, nId):
//                      updateF(f, nId, p, ps, t), 0, ns)) . zip(ps, N)
// with updateF adding the Lennard-Jones pair force of ps[nId] on p when
// their distance is below the cutoff t.
//
// The map over particles becomes groups of L lanes per particle (L = 1..16,
// 64 / L particles per wavefront); the reduce over the neighbour list is
// split over the group's lanes (split + partial reduce-seq per lane, then a
// DPP butterfly inside the group), which keeps thousands of wavefronts busy
// for the paper's 12288 particles.  Lane `sub` of a group reads index vectors
// sub, sub + L, ... of its particle's row (V indices per load, so L * V * 4
// contiguous bytes per group and step), keeps U index loads in flight, then
// gathers the U * V neighbour positions (16 bytes each; the position array
// is small and stays in cache) before any arithmetic.  Empty slots (indices
// outside [0, n)) load nothing and contribute zero.
//
// Per neighbour, in binary32: d = p - q, r2 = (dx dx + dy dy) + dz dz
// without contraction, and the cutoff test r2 < binary32(t^2).  That r2 is
// within about 5 ulps of the exact squared distance, so the test agrees
// with "distance < t" except for pairs whose squared distance lies within
// about 6 binary32 ulps of t^2; it is the same decision on every run and
// knob point.  Then 1/r2 by the hardware reciprocal, s6 = (sigma^2 / r2)^3,
// f = 24 eps / r2 * s6 * (2 s6 - 1) (zero outside the cutoff) and F += f d
// by fma.
#include "lift_device.hpp"
#include "lift_apps.hpp"
#include "lift_internal.hpp"

namespace lift {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

template <int V> struct IdxVec;
template <> struct IdxVec<1> { using type = int32_t; };
template <> struct IdxVec<2> { using type = i32x2; };
template <> struct IdxVec<4> { using type = i32x4; };

template <int V>
__device__ __forceinline__ int32_t lane_of(typename IdxVec<V>::type v, int e)
{
    if constexpr (V == 1)
        return v;
    else
        return v[e];
}

// Sum over the L lanes of an aligned group (the DPP steps of the wave
// butterfly that stay inside the group); every lane of the group gets it.
template <int L>
__device__ __forceinline__ float group_sum(float v)
{
    if constexpr (L >= 2)
        v += dpp<DPP_QUAD_XOR1>(v);
    if constexpr (L >= 4)
        v += dpp<DPP_QUAD_XOR2>(v);
    if constexpr (L >= 8)
        v += dpp<DPP_HALF_MIRROR>(v);
    if constexpr (L >= 16)
        v += dpp<DPP_ROW_MIRROR>(v);
    return v;
}

// One neighbour's term, added to the particle's force where `use`.
__device__ __forceinline__ void add_pair(const MdArgs &a, const f32x4 &p, const f32x4 &q, bool use, float &fx, float &fy,
                                         float &fz)
{
    const float dx = p[0] - q[0], dy = p[1] - q[1], dz = p[2] - q[2];
    const float r2 = (dx * dx + dy * dy) + dz * dz;
    const float r2inv = __builtin_amdgcn_rcpf(r2);
    const float s2 = a.sigma2 * r2inv;
    const float s6 = s2 * s2 * s2;
    const float fs = a.eps24 * r2inv * s6 * fmaf(2.f, s6, -1.f);  // 2 s6 is exact: one rounding either way
    const float fh = use && r2 < a.t2 ? fs : 0.f;
    fx = fmaf(fh, dx, fx);
    fy = fmaf(fh, dy, fy);
    fz = fmaf(fh, dz, fz);
}

// SORT: the first of several launches (see md_packed_kernel).  A wavefront
// most of whose first particle's neighbours (of the first 32) have indices more
// than n / 12 from its own leaves its particles to the passes, marked by their
// lists' length in the fourth component of their forces.  In random order five
// in six are that far; in a lattice's order only those beyond a periodic face.
template <int L, int V, int U, bool SORT = false>
__global__ void __launch_bounds__(1024) md_kernel(MdArgs a)
{
    using IV = typename IdxVec<V>::type;
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = gt / L;  // particle
    const int sub = (int)(gt % L);
    if (i >= a.n)  // whole groups leave together (L divides 64)
        return;
    if constexpr (SORT) {
        const int lane = threadIdx.x & 63;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)i), near = a.near;
        const uint32_t id = lane < 32 && lane < a.k ? (uint32_t)a.nbr[first * a.k + lane] : ~0u;
        const bool used = id < (uint32_t)a.n;
        const int far = __popcll(__ballot(used && id - (first - near) > 2 * near));
        if (2 * far > __popcll(__ballot(used))) {
            if (sub == 0)
                reinterpret_cast<f32x4 *>(a.force)[i] = f32x4{0.f, 0.f, 0.f, (float)a.k};
            return;
        }
    }
    const f32x4 *pos = reinterpret_cast<const f32x4 *>(a.pos);
    const f32x4 p = pos[i];
    const IV *row = reinterpret_cast<const IV *>(a.nbr + i * a.k);
    const int64_t kv = a.k / V;  // index vectors per row
    const uint32_t n = (uint32_t)a.n;

    float fx = 0.f, fy = 0.f, fz = 0.f;
    for (int64_t base = 0; base < kv; base += L * U) {
        IV iv[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            iv[u] = __builtin_nontemporal_load(row + min(base + sub + (int64_t)L * u, kv - 1));
        loads_in_flight();
        f32x4 q[U][V];
        bool use[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in_row = base + sub + (int64_t)L * u < kv;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const int32_t id = lane_of<V>(iv[u], e);
                use[u][e] = in_row && (uint32_t)id < n;
                q[u][e] = p;  // empty slots load nothing
                if (use[u][e])
                    q[u][e] = pos[id];
            }
        }
        loads_in_flight();
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e)
                add_pair(a, p, q[u][e], use[u][e], fx, fy, fz);
    }
    fx = group_sum<L>(fx);
    fy = group_sum<L>(fy);
    fz = group_sum<L>(fz);
    if (sub == 0) {
        f32x4 f = {fx, fy, fz, 0.f};
        reinterpret_cast<f32x4 *>(a.force)[i] = f;
    }
}

// MD in passes, for positions that do not fit one XCD's L2 and particles in
// no spatial order.  There the single-pass kernel waits for gathers that miss:
// a position is 16 bytes, the line it comes in 128 (2^20 particles in random
// order: 65.7 M misses, 8.4 GB for 0.57 GB of lists, positions and forces,
// 1090 us).  Each pass wants only the neighbours in one slice of the
// positions, which then stays in the L2, and adds to the force; a further pass
// costs 70 to 130 us there, most of it for reading the lists again, so three
// slices of 5.6 MB do best (one pass 1088, 2 slices 896, 3: 796, 4: 868, 6: 1136
// us).  Systems in a lattice's order pay 4 us per pass that finds no mark (2^20
// particles, 80 neighbours in lists of 128: 163 us, one pass of 8 lanes 150, of
// 16 lanes 170).
//
// A wavefront takes blocks of four marked particles (md_kernel's SORT form).
// It first packs the wanted neighbours of each list in LDS -- 64 lanes over
// the list, an index's place being the count of wanted ones before it, from a
// ballot -- and then 16 lanes per particle work through the packed list, so
// that the slots another pass wants cost a few instructions each instead of a
// pair's arithmetic.  It reads the marks of 64 of its blocks at once: with
// none marked a pass costs one round trip.
//
// A block's mark, in each of its particles' forces, is the number of leading
// indices of its lists that this pass has to read: each pass leaves the place
// of the last neighbour in a later slice, so padding and what is done are not
// read again, and the last pass leaves 0
// (2^20 particles, 80 neighbours in lists of 128: 803 us without, 795 with:
// the L1's outstanding requests bound a pass, not bytes, nor round trips --
// gathers for 64 packed indices at once instead of 32: 810).  Lists are far
// shorter than 2^24, which binary32 counts exactly.
template <int V>
__global__ void __launch_bounds__(256) md_packed_kernel(MdPackedArgs s)
{
    constexpr int L = 16, U = 2 / V, STEP = 128;   // indices per particle and step: 64 lanes x U x V
    constexpr int PITCH = STEP + 16;               // the four particles of a wave in different banks
    using IV = typename IdxVec<V>::type;
    __shared__ int32_t lds[4][4][PITCH];
    const MdArgs &a = s.md;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, sub = lane % L, grp = lane / L;
    int32_t(*list)[PITCH] = lds[wv];
    const int64_t wave = (int64_t)blockIdx.x * 4 + wv, nwaves = (int64_t)gridDim.x * 4;
    const int64_t nblocks = (a.n + 3) / 4;
    const f32x4 *pos = reinterpret_cast<const f32x4 *>(a.pos);
    f32x4 *force = reinterpret_cast<f32x4 *>(a.force);

    const auto block = [&](int64_t j) { return wave + j * nwaves; };   // the wave's j-th
    int64_t base = 0;          // of this wave's blocks base .. base + 63: `need` the mark (lane j: block
    int need = 0;              // base + j), `mask` which are to be done
    uint64_t mask = 0;
    const auto fill = [&] {
        const int64_t b = block(base + lane);
        need = b < nblocks ? (int)force[b * 4][3] : 0;
        mask = __ballot(need > 0);
    };
    int len = 0;                                 // the block's index vectors
    const auto next_block = [&]() -> int64_t {   // wave-uniform; -1: none left
        while (mask == 0) {
            base += 64;
            if (block(base) >= nblocks)
                return -1;
            fill();
        }
        const int j = __builtin_ctzll(mask);
        mask &= mask - 1;
        len = (__builtin_amdgcn_readlane(need, j) + V - 1) / V;
        return block(base + j);
    };

    IV iv[4][U];
    f32x4 p;
    const auto load = [&](int64_t blk, int step0) {   // the four particles' indices and positions
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const IV *row = reinterpret_cast<const IV *>(a.nbr + min(blk * 4 + g, a.n - 1) * a.k);
#pragma unroll
            for (int u = 0; u < U; ++u)
                iv[g][u] = __builtin_nontemporal_load(row + min(step0 + lane + 64 * u, len - 1));
        }
        p = pos[min(blk * 4 + grp, a.n - 1)];
    };

    fill();
    int64_t blk = next_block();
    if (blk < 0)
        return;
    int step0 = 0;
    float fx = 0.f, fy = 0.f, fz = 0.f;
    int later[4] = {0, 0, 0, 0};   // the marks this pass leaves
    load(blk, 0);
    while (true) {
        const f32x4 mine = p;
        const int64_t i = blk * 4 + grp;
        const uint32_t lo = s.lo, width = s.hi - s.lo, hi = s.hi, beyond = (uint32_t)a.n - s.hi;
        const int row = len;
        int count[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            count[g] = 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const int32_t id = lane_of<V>(iv[g][u], e);
                    const bool in_row = step0 + lane + 64 * u < row;
                    const bool want = in_row && (uint32_t)id - lo < width;
                    const uint64_t who = __ballot(want), rest = __ballot(in_row && (uint32_t)id - hi < beyond);
                    if (rest)
                        later[g] = max(later[g], (step0 + 64 * u + 63 - __builtin_clzll(rest)) * V + e + 1);
                    if (want)
                        list[g][__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)who, count[g]))] = id;
                    count[g] += __popcll(who);
                }
        }
        __builtin_amdgcn_wave_barrier();   // one wave writes and reads `list`: LDS keeps its order
        const int most = max(max(count[0], count[1]), max(count[2], count[3]));
        const int have = grp & 2 ? (grp & 1 ? count[3] : count[2]) : (grp & 1 ? count[1] : count[0]);
        const int32_t *from = list[grp] + sub;
        const bool row_done = step0 + 64 * U >= row;
        int64_t nblk = blk;
        int nstep = step0 + 64 * U;
        f32x4 prev = {0.f, 0.f, 0.f, 0.f};
        for (int r = 0; r < most || r == 0; r += 2 * L) {
            const bool v0 = r + sub < have, v1 = r + L + sub < have;
            f32x4 q0 = mine, q1 = mine;
            if (v0)
                q0 = pos[from[r]];
            if (v1)
                q1 = pos[from[r + L]];
            if (r == 0) {
                // the next step's indices, behind the first gathers
                if (row_done) {
                    if (sub == 0 && i < a.n)
                        prev = force[i];
                    nblk = next_block();
                    nstep = 0;
                }
                if (nblk >= 0)
                    load(nblk, nstep);
            }
            loads_in_flight();
            add_pair(a, mine, q0, v0, fx, fy, fz);
            add_pair(a, mine, q1, v1, fx, fy, fz);
        }
        __builtin_amdgcn_wave_barrier();
        if (row_done) {
            fx = group_sum<L>(fx);
            fy = group_sum<L>(fy);
            fz = group_sum<L>(fz);
            const int mark = max(max(later[0], later[1]), max(later[2], later[3]));   // one for the block
            if (sub == 0 && i < a.n)
                force[i] = f32x4{prev[0] + fx, prev[1] + fy, prev[2] + fz, (float)mark};
            fx = fy = fz = 0.f;
            later[0] = later[1] = later[2] = later[3] = 0;
            if (nblk < 0)
                return;
        }
        blk = nblk;
        step0 = nstep;
    }
}

// 8 lanes; 16 with two loads for rows that are not read 4 indices at a time.
const void *md_sort_kernel_table(int lanes, int v, int unroll)
{
    if (v == 4 && lanes == 8)
        switch (unroll) {
        case 2: return reinterpret_cast<const void *>(&md_kernel<8, 4, 2, true>);
        case 4: return reinterpret_cast<const void *>(&md_kernel<8, 4, 4, true>);
        }
    if (lanes == 16 && unroll == 2)
        switch (v) {
        case 1: return reinterpret_cast<const void *>(&md_kernel<16, 1, 2, true>);
        case 2: return reinterpret_cast<const void *>(&md_kernel<16, 2, 2, true>);
        }
    return nullptr;
}

const void *md_packed_kernel_table(int v)
{
    switch (v) {
    case 1: return reinterpret_cast<const void *>(&md_packed_kernel<1>);
    case 2: return reinterpret_cast<const void *>(&md_packed_kernel<2>);
    default: return nullptr;
    }
}

template <int L, int V>
static const void *md_pick_unroll(int unroll)
{
    switch (unroll) {
    case 1: return reinterpret_cast<const void *>(&md_kernel<L, V, 1>);
    case 2: return reinterpret_cast<const void *>(&md_kernel<L, V, 2>);
    case 4: return reinterpret_cast<const void *>(&md_kernel<L, V, 4>);
    default: return nullptr;
    }
}

template <int L>
static const void *md_pick_vec(int v, int unroll)
{
    switch (v) {
    case 1: return md_pick_unroll<L, 1>(unroll);
    case 2: return md_pick_unroll<L, 2>(unroll);
    case 4: return md_pick_unroll<L, 4>(unroll);
    default: return nullptr;
    }
}

const void *md_kernel_table(int lanes, int v, int unroll)
{
    switch (lanes) {
    case 1: return md_pick_vec<1>(v, unroll);
    case 2: return md_pick_vec<2>(v, unroll);
    case 4: return md_pick_vec<4>(v, unroll);
    case 8: return md_pick_vec<8>(v, unroll);
    case 16: return md_pick_vec<16>(v, unroll);
    default: return nullptr;
    }
}

}  // namespace lift
