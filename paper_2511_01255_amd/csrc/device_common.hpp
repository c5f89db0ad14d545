// device_common.hpp -- device helpers shared by the optimiser kernels:
// the per-individual DE draws and the (f descending, slot ascending) top-3.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

#include "philox.hpp"

namespace qpm {

// Donors r1, r2, r3 (distinct, != i) and jrand of individual i in
// generation g: one Philox call; word m < 3 gives k = floor(u (np-1-m) /
// 2^32) and r is the k-th index not yet excluded (exclusions applied in
// ascending order); word 3 gives jrand = floor(u D / 2^32).
__device__ __forceinline__ int4 de_draw(int64_t i, int64_t np, int64_t D, uint32_t g, uint32_t inst, uint32_t k0,
                                        uint32_t k1)
{
    const U4 o = philox10(0u, static_cast<uint32_t>(i), g, (inst << 8) | kTagDeIdx, k0, k1);
    int64_t r1 = bounded(o.x, static_cast<uint32_t>(np - 1));
    if (r1 >= i) ++r1;
    int64_t r2 = bounded(o.y, static_cast<uint32_t>(np - 2));
    {
        const int64_t lo = i < r1 ? i : r1, hi = i < r1 ? r1 : i;
        if (r2 >= lo) ++r2;
        if (r2 >= hi) ++r2;
    }
    int64_t r3 = bounded(o.z, static_cast<uint32_t>(np - 3));
    {
        int64_t e0 = i, e1 = r1, e2 = r2, t;
        if (e0 > e1) { t = e0; e0 = e1; e1 = t; }
        if (e1 > e2) { t = e1; e1 = e2; e2 = t; }
        if (e0 > e1) { t = e0; e0 = e1; e1 = t; }
        if (r3 >= e0) ++r3;
        if (r3 >= e1) ++r3;
        if (r3 >= e2) ++r3;
    }
    const int64_t jrand = bounded(o.w, static_cast<uint32_t>(D));
    return make_int4(static_cast<int>(r1), static_cast<int>(r2), static_cast<int>(r3), static_cast<int>(jrand));
}

template <typename T>
struct Top3 {
    T v[3];
    int i[3];
};

template <typename T>
__device__ __forceinline__ bool ahead(T va, int ia, T vb, int ib)
{
    return va > vb || (va == vb && ia < ib);
}

template <typename T>
__device__ __forceinline__ void top3_insert(Top3<T> &t, T v, int idx)
{
    if (ahead(v, idx, t.v[0], t.i[0])) {
        t.v[2] = t.v[1]; t.i[2] = t.i[1];
        t.v[1] = t.v[0]; t.i[1] = t.i[0];
        t.v[0] = v; t.i[0] = idx;
    } else if (ahead(v, idx, t.v[1], t.i[1])) {
        t.v[2] = t.v[1]; t.i[2] = t.i[1];
        t.v[1] = v; t.i[1] = idx;
    } else if (ahead(v, idx, t.v[2], t.i[2])) {
        t.v[2] = v; t.i[2] = idx;
    }
}

template <typename T>
__device__ __forceinline__ Top3<T> top3_empty()
{
    Top3<T> t;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        t.v[k] = -INFINITY;
        t.i[k] = INT_MAX;
    }
    return t;
}

// the value of the lane a DPP control names, or the lane's own where that lane
// does not exist
template <int CTRL>
__device__ __forceinline__ float dpp_take(float v)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_take(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int dpp_take(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ float lane63(float v)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ double lane63(double v)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}
__device__ __forceinline__ int lane63(int v) { return __builtin_amdgcn_readlane(v, 63); }

// op over the 64 lanes of a wave, in every lane: prefixes within the 16-lane
// rows, then across the rows (a lane without a source keeps its own value, so
// op must be idempotent)
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op)
{
    v = op(v, dpp_take<0x111>(v));  // row_shr 1, 2, 4, 8
    v = op(v, dpp_take<0x112>(v));
    v = op(v, dpp_take<0x114>(v));
    v = op(v, dpp_take<0x118>(v));
    v = op(v, dpp_take<0x142>(v));  // row_bcast 15, 31
    v = op(v, dpp_take<0x143>(v));
    return lane63(v);
}

// The three best of the 64 U (value, slot) pairs of a wave, f descending, slot
// ascending: their slots in lanes 0 .. 2 (INT_MAX where there are fewer), their
// values too with `vals`. Three rounds of a maximum and a minimum over the
// wave; values that are not a number never lead. The pairs are used up.
template <typename T, int U>
__device__ __forceinline__ int wave_best3(T (&v)[U], int (&ix)[U], int lane, T *vals = nullptr)
{
    int best = INT_MAX;
    T bv = static_cast<T>(-INFINITY);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T m = static_cast<T>(-INFINITY);
#pragma unroll
        for (int u = 0; u < U; ++u) m = v[u] > m ? v[u] : m;
        m = wave_reduce(m, [](T a, T b) { return b > a ? b : a; });
        int c = INT_MAX;
#pragma unroll
        for (int u = 0; u < U; ++u) c = v[u] == m ? min(c, ix[u]) : c;
        c = wave_reduce(c, [](int a, int b) { return min(a, b); });
        best = lane == k ? c : best;
        bv = lane == k ? m : bv;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool gone = ix[u] == c;
            v[u] = gone ? static_cast<T>(-INFINITY) : v[u];
            ix[u] = gone ? INT_MAX : ix[u];
        }
    }
    if (vals != nullptr) *vals = bv;
    return best;
}

// the same of the n <= 64 U candidates (cv[j], ci[j])
template <typename T, int U>
__device__ __forceinline__ int wave_best3_of(const T *__restrict__ cv, const int32_t *__restrict__ ci, int n, int lane)
{
    T v[U];
    int ix[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int j = lane + 64 * u, jj = j < n ? j : n - 1;
        const T fv = cv[jj];
        const int iv = ci[jj];
        v[u] = j < n ? fv : static_cast<T>(-INFINITY);
        ix[u] = j < n ? iv : INT_MAX;
    }
    return wave_best3<T, U>(v, ix, lane);
}

// The three best of the n candidates (f[j], idx ? idx[j] : j) over one
// workgroup of NT lanes (NT a multiple of 64, <= 1024). (f descending,
// slot ascending) is a strict total order, so the result is unique
// whatever the merge order. Loads are issued four at a time. Each wave's
// three and then the workgroup's come from wave_best3 (lists merged lane by
// lane took 3.4 us more in a kernel of one workgroup).
template <typename T, int NT>
__device__ void block_top3(const T *__restrict__ f, int64_t n, int32_t *__restrict__ out,
                           const int32_t *__restrict__ idx = nullptr)
{
    Top3<T> t = top3_empty<T>();
    for (int64_t base = threadIdx.x; base < n; base += 4 * NT) {
        T v[4];
        int ix[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + static_cast<int64_t>(u) * NT;
            const int64_t jj = j < n ? j : 0;
            const T fv = f[jj];
            const int iv = idx ? idx[jj] : static_cast<int>(jj);
            v[u] = j < n ? fv : static_cast<T>(-INFINITY);
            ix[u] = j < n ? iv : INT_MAX;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) top3_insert(t, v[u], ix[u]);
    }
    __shared__ T sv[3 * (NT / 64)];
    __shared__ int si[3 * (NT / 64)];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    T bv;
    const int b = wave_best3<T, 3>(t.v, t.i, lane, &bv);
    if (lane < 3) {
        sv[3 * wave + lane] = bv;
        si[3 * wave + lane] = b;
    }
    __syncthreads();
    if (wave == 0) {
        const int b3 = wave_best3_of<T, 1>(sv, si, 3 * (NT / 64), lane);
        if (lane < 3) out[lane] = b3;
    }
}

// The leaders from n <= 256 candidates (cv[j], ci[j]), by the first wave of a
// workgroup.
template <typename T>
__device__ __forceinline__ void merge_few_leaders(const T *__restrict__ cv, const int32_t *__restrict__ ci, int64_t n,
                                                  int32_t *__restrict__ out)
{
    if (threadIdx.x >= 64) return;
    const int lane = static_cast<int>(threadIdx.x), m = static_cast<int>(n);
    const int b = m <= 64 ? wave_best3_of<T, 1>(cv, ci, m, lane) : wave_best3_of<T, 4>(cv, ci, m, lane);
    if (lane < 3) out[lane] = b;
}

// The same of any number of candidates, by a workgroup of NT lanes
template <typename T, int NT>
__device__ __forceinline__ void merge_leaders(const T *__restrict__ cv, const int32_t *__restrict__ ci, int64_t n,
                                              int32_t *__restrict__ out)
{
    if (n > 256)
        block_top3<T, NT>(cv, n, out, ci);
    else
        merge_few_leaders<T>(cv, ci, n, out);
}

}  // namespace qpm
