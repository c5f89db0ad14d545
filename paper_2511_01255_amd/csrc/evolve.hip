// evolve.hip -- the optimiser steps around the fitness: initialisation, DE
// rand/1 mutation + binomial crossover (paper Sec. 2.2.1), the grey-wolf
// update of the omega wolves (paper Sec. 2.2.2), greedy selection and the
// leader (top-3) reduction (paper Sec. 3.2 steps 2-5).
//
// Layout: genes are float rows (row stride ldx, a multiple of 4) so that a
// lane moves one float4 (a gene quad) per row; a workgroup of 256 lanes
// covers 1024 genes of one individual, so the individual index -- and with
// it the donor / leader rows and the per-individual Philox draws -- is
// uniform across the workgroup and lives in scalar registers. The +-1 bits
// of a quad (4 bits) are merged across 8 neighbouring lanes with xor
// shuffles into one 32-gene word of the population-major layout.
//
// Binary32 arithmetic here is spelled out with explicit fmaf and the
// library is built with -ffp-contract=off, so trial and candidate genes are
// bit-for-bit what these formulas state.
#include <cfloat>
#include <climits>
#include <vector>

#include "common.hpp"
#include "device_common.hpp"
#include "genes.hpp"

namespace qpm {

// ------------------------------------------------------------ initialisation

__global__ __launch_bounds__(256) void init_kernel(int64_t D, int64_t ldx, uint32_t k0, uint32_t k1, uint32_t inst,
                                                   float *__restrict__ x, uint32_t *__restrict__ bits, int64_t ld)
{
    const int64_t i = blockIdx.x;
    const int64_t q = static_cast<int64_t>(blockIdx.y) * 256 + threadIdx.x;
    const int64_t j0 = 4 * q;
    const bool valid = j0 < D;
    uint32_t nib = 0;
    if (valid) {
        const U4 r = philox10(static_cast<uint32_t>(q), static_cast<uint32_t>(i), 0u, (inst << 8) | kTagInit, k0, k1);
        const float4 v = make_float4(sym24(r.x), sym24(r.y), sym24(r.z), sym24(r.w));
        store_quad(x + i * ldx, j0, D, v);
        nib = quad_nibble(v, j0, D);
    }
    store_word(nib, q, D, bits, ld, i);
}

// ------------------------------------------------------------ DE rand/1 + binomial crossover

// One draw per individual and generation, shared by every gene chunk.
__global__ __launch_bounds__(256) void de_draws_kernel(int64_t np, int64_t D, uint32_t k0, uint32_t k1,
                                                       const uint32_t *__restrict__ gen_dev, uint32_t gen_c,
                                                       uint32_t inst, int4 *__restrict__ draws)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= np) return;
    const uint32_t g = gen_dev ? gen_dev[0] : gen_c;
    draws[i] = de_draw(i, np, D, g, inst, k0, k1);
}

// Work split: a lane moves one gene quad (float4). A chunk is CW = 256 /
// IPW genes; one wave covers IPW individuals of a chunk (64 / IPW lanes
// each) and a 256-lane workgroup covers IPG = 4 IPW consecutive
// individuals per pass, R passes over R IPG consecutive individuals. The
// rows of pass r + 1 are loaded before the trials of pass r are stored, so
// two passes' reads are in flight per wave. Chunks are dealt to the eight
// XCDs round-robin (workgroup id mod 8 = XCD) and every XCD walks its
// chunks in order over all individuals, so while it works on a chunk that
// slice of the whole population (np x CW x 4 bytes, chosen <= 2 MB) stays in
// the XCD's L2 and the random donor rows hit it.
//
// The set-up of a workgroup (draws, flags, row offsets) is two dependent
// loads and two barriers before its first row is read, so the number of
// passes it is spread over sets the speed (see de_passes).
//
// Where a row lives: STAGED, the flags, if any (fbits: packed one bit per
// individual, np <= 65536), are copied to LDS first, so a donor's buffer
// costs an LDS read instead of a second dependent global load, and row
// offsets fit 32 bits. Otherwise the flags are read from global memory.
template <int IPW, int R, bool STAGED>
__global__ __launch_bounds__(256) void de_kernel(PopView pv, const int4 *__restrict__ draws,
                                                 const uint32_t *__restrict__ fbits, float F,
                                                 const float *__restrict__ F_tab, uint32_t cr_max,
                                                 uint32_t k0, uint32_t k1, const uint32_t *__restrict__ gen_dev,
                                                 uint32_t gen_c, uint32_t inst, uint32_t *__restrict__ bits,
                                                 int64_t ld, int groups, int chunks, int store_genes,
                                                 int64_t cols, int64_t rows, uint32_t *__restrict__ reset_cnt)
{
    extern __shared__ uint32_t sfb[];  // STAGED with flags: (np + 31) / 32 flag words
    const uint32_t b = blockIdx.x;
    const int k = static_cast<int>(b >> 3);
    const int gi = k % groups;
    const int c = static_cast<int>(b & 7u) + 8 * (k / groups);
    if (c >= chunks) return;
    const int64_t D = pv.D, np = pv.np;
    const uint32_t g = gen_dev ? gen_dev[0] : gen_c;
    const float Fg = F_tab ? F_tab[g] : F;  // a run's per-generation F
    // a run without stored trials: the list counter of the accepted trials
    // starts at 0 for this generation (the finish step appends to it)
    if (reset_cnt != nullptr && b == 0 && threadIdx.x == 0) reset_cnt[0] = 0u;
    // (the entry point passes no draws: each workgroup draws for its own);
    // the load is in flight while the flags are staged
    constexpr int IPB = 4 * IPW * R;
    int4 d = make_int4(0, 0, 0, 0);
    if (threadIdx.x < IPB) {
        const int64_t ip = min(static_cast<int64_t>(gi) * IPB + threadIdx.x, np - 1);
        d = draws ? draws[ip] : de_draw(ip, np, D, g, inst, k0, k1);
    }
    if constexpr (STAGED) {
        if (fbits != nullptr) {
            for (int w = threadIdx.x; w < static_cast<int>((np + 31) / 32); w += 256) sfb[w] = fbits[w];
            __syncthreads();
        }
        de_rows<IPW, R, uint32_t>(
            pv, gi, c, Fg, cr_max, g, inst, k0, k1, bits, ld, store_genes != 0, cols, rows, d,
            [&](int r) -> bool { return fbits != nullptr && ((sfb[r >> 5] >> (r & 31)) & 1u) != 0u; });
    } else {
        de_rows<IPW, R, uint64_t>(
            pv, gi, c, Fg, cr_max, g, inst, k0, k1, bits, ld, store_genes != 0, cols, rows, d,
            [&](int r) -> bool { return pv.flags != nullptr && pv.flags[r] != 0u; });
    }
}

// The accepted trials of a run whose DE step stored only their bits: the
// trial genes of every individual in list[0 .. cnt) are computed again,
// exactly as the DE kernel computed them (same draws, words and de_quad),
// from the population before the selection (fb_old: its packed flags), and
// written to the buffer that the selection made current. A work item is
// (chunk of 256 genes, listed individual) for one wave. Chunk c belongs to
// XCD c mod 8 (workgroup x runs on XCD x mod 8), and each XCD walks its
// items chunk by chunk, so the waves running together on an XCD read the
// same chunk of many rows and donor rows shared between accepted trials
// come from its L2. The grid is fixed; every wave loops until its XCD's
// items run out. With top3_out, workgroup 0 first merges the finish step's
// leader candidates (3 per group of 64) into the leaders, which saves the
// finish step a one-workgroup kernel (the grey-wolf step after this kernel
// reads them).
__global__ __launch_bounds__(256) void materialize_kernel(PopView pv, const int4 *__restrict__ draws,
                                                          const uint32_t *__restrict__ fb_old, float F,
                                                          const float *__restrict__ F_tab, uint32_t cr_max,
                                                          uint32_t k0, uint32_t k1, const uint32_t *__restrict__ gen,
                                                          uint32_t inst, const int32_t *__restrict__ list,
                                                          const uint32_t *__restrict__ cnt, const void *cand,
                                                          int64_t ngroups, int cand_f64, int32_t *top3_out)
{
    extern __shared__ uint32_t sfb[];  // (np + 31) / 32 old flag words
    if (top3_out != nullptr && blockIdx.x == 0) {
        // cand: 3 values per group (T) followed by 3 slots per group
        if (cand_f64) {
            const double *cv = static_cast<const double *>(cand);
            merge_leaders<double, 256>(cv, reinterpret_cast<const int32_t *>(cv + 3 * ngroups), 3 * ngroups, top3_out);
        } else {
            const float *cv = static_cast<const float *>(cand);
            merge_leaders<float, 256>(cv, reinterpret_cast<const int32_t *>(cv + 3 * ngroups), 3 * ngroups, top3_out);
        }
    }
    const int64_t np = pv.np, D = pv.D;
    for (int k = threadIdx.x; k < static_cast<int>((np + 31) / 32); k += 256) sfb[k] = fb_old[k];
    __syncthreads();
    const uint32_t g = gen[0];
    const float Fg = F_tab ? F_tab[g] : F;
    // np <= 65536 and D < 2^24 (checked by the launcher), so the item
    // counts fit 32 bits
    const uint32_t n_acc = static_cast<uint32_t>(min(static_cast<int64_t>(cnt[0]), np));
    const uint32_t chunks = static_cast<uint32_t>((D + 255) / 256);
    const uint32_t xcd = blockIdx.x & 7u;
    const uint32_t stride = (gridDim.x / 8) * 4;  // the waves of one XCD (the grid is a multiple of 8)
    const uint32_t my_chunks = chunks > xcd ? (chunks - xcd + 7) / 8 : 0;
    const int lane = threadIdx.x & 63;
    // the wave index is the same in all lanes: the item walk below is
    // scalar, and so are an item's individual, draws and row offsets
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t np32 = static_cast<uint32_t>(np), ldx24 = static_cast<uint32_t>(pv.ldx) & 0xFFFFFFu;
    auto row = [&](uint32_t rr, uint32_t flip) -> const float * {
        const uint32_t b = __builtin_amdgcn_readfirstlane((sfb[rr >> 5] >> (rr & 31u)) & 1u) ^ flip;
        return pv.x0 + static_cast<uint64_t>((rr + b * np32) & 0xFFFFFFu) * ldx24;
    };
    if (n_acc == 0 || my_chunks == 0) return;
    // item it = (chunk slot cq, list entry ir) with it = cq n_acc + ir,
    // stepped by `stride` without a division
    uint32_t it = (blockIdx.x >> 3) * 4 + wave;
    uint32_t cq = it / n_acc, ir = it - cq * n_acc;
    const uint32_t sq = stride / n_acc, sr = stride - sq * n_acc;
    for (; cq < my_chunks; cq += sq, ir += sr) {
        if (ir >= n_acc) {
            ir -= n_acc;
            ++cq;
            if (cq >= my_chunks) break;
        }
        const int64_t j0 = static_cast<int64_t>(xcd + 8 * cq) * 256 + 4 * lane;
        const int32_t iv = list[ir];
        if (iv < 0 || iv >= np || j0 >= D) continue;
        const uint32_t i = static_cast<uint32_t>(iv);
        const int4 dr = draws[i];
        const float4 xv = *reinterpret_cast<const float4 *>(row(i, 0u) + j0);
        const float4 a = *reinterpret_cast<const float4 *>(row(static_cast<uint32_t>(dr.x), 0u) + j0);
        const float4 bq = *reinterpret_cast<const float4 *>(row(static_cast<uint32_t>(dr.y), 0u) + j0);
        const float4 cv = *reinterpret_cast<const float4 *>(row(static_cast<uint32_t>(dr.z), 0u) + j0);
        const float4 uv = de_quad(xv, a, bq, cv, j0, dr.w, i, g, inst, k0, k1, Fg, cr_max);
        store_quad_nt(const_cast<float *>(row(i, 1u)), j0, D, uv);
    }
}

qpm_status launch_materialize(const PopView &pv, const int4 *draws, const uint32_t *fb_old, float F,
                              const float *F_tab, float CR, uint64_t seed, const uint32_t *gen, uint32_t inst,
                              const int32_t *list, const uint32_t *cnt, hipStream_t s, const void *cand,
                              int64_t ngroups, bool f64, int32_t *top3_out)
{
    QPM_REQUIRE(top3_out == nullptr || cand != nullptr, QPM_EINVAL, "merging leaders needs the candidates");
    QPM_REQUIRE(pv.np <= 65536 && pv.ldx < (int64_t(1) << 24) && pv.x1 == pv.x0 + pv.np * pv.ldx &&
                    pv.out0 == pv.x0 && pv.out1 == pv.x1,
                QPM_EINVAL, "materialising trials needs one allocation for both gene buffers");
    const size_t lds = sizeof(uint32_t) * static_cast<size_t>((pv.np + 31) / 32);
    materialize_kernel<<<2048, 256, lds, s>>>(pv, draws, fb_old, F, F_tab, cr_threshold(CR),
                                              static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), gen,
                                              inst, list, cnt, cand, ngroups, f64 ? 1 : 0, top3_out);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

// ------------------------------------------------------------ grey-wolf update

// row_of and out_row_of; merging, by offsets between the buffers (there, a
// choice between the pointers of `pv` would keep `pv` in memory)
template <int MERGE>
__device__ __forceinline__ const float *gwo_row(const PopView &pv, int64_t r)
{
    if constexpr (MERGE == 0) return row_of(pv, r);
    return pv.x0 + (r * pv.ldx + (pv.flags[r] != 0u ? pv.x1 - pv.x0 : 0));
}
template <int MERGE>
__device__ __forceinline__ float *gwo_out_row(const PopView &pv, int64_t r)
{
    if constexpr (MERGE == 0) return out_row_of(pv, r);
    return pv.out0 + (r * pv.ldx + (pv.flags[r] != 0u ? 0 : pv.out1 - pv.out0));
}

// Grid x = 8 ceil(np / 8): workgroup x runs on XCD x mod 8 (gridDim.x is a
// multiple of 8, so this holds for every y) and takes individual
// (x mod 8) ceil(np / 8) + x / 8. Each XCD thus owns a contiguous range of
// individuals and the 32-bit bit words of neighbouring individuals, which
// share cache lines, are written from one L2 instead of eight.
// `whole`: what the update leaves alone is written too (leader rows and genes
// past D as they are in x, 0 in the leaders' bit columns and in those past
// np), so that the caller needs no copy of x and no cleared words first: at
// 5000 x 6600 genes the copy and the clear took 54 us beside 62 for the step.
// MERGE (a run; T = MergeT<MERGE>): the leaders are not known yet; each
// workgroup takes them from the selection's candidates (ncand <= 256 values
// cand, then their slots) and the first one stores them. That is one wave's
// three reductions per workgroup instead of a kernel of one workgroup between
// the selection and this step (see merges_leaders).
template <int MERGE>
struct MergeT {
    using T = float;
};
template <>
struct MergeT<2> {
    using T = double;
};
template <int VARIANT, int MERGE>
__global__ __launch_bounds__(256) void gwo_kernel(PopView pv, int32_t *__restrict__ leaders, int4 lead_c,
                                                  const float *__restrict__ a_tab, float a_c, uint32_t k0, uint32_t k1,
                                                  const uint32_t *__restrict__ gen_dev, uint32_t gen_c, uint32_t inst,
                                                  uint32_t *__restrict__ bits, int64_t ld, int64_t per_xcd,
                                                  int whole, const void *__restrict__ cand, int ncand)
{
    const int64_t np = pv.np, D = pv.D;
    const int64_t i = static_cast<int64_t>(blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (i >= (whole ? ld : np)) return;
    const int64_t q = static_cast<int64_t>(blockIdx.y) * 256 + threadIdx.x;
    const int64_t j0 = 4 * q, cols = whole ? pv.ldx : D;
    // merging, the wolf's own genes are loaded before its leaders are known
    float4 own = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if constexpr (MERGE != 0) {
        if (j0 < D) own = *reinterpret_cast<const float4 *>(gwo_row<MERGE>(pv, i) + j0);
    }
    int64_t L0, L1, L2;
    if constexpr (MERGE != 0) {
        using T = typename MergeT<MERGE>::T;
        __shared__ int lead[3];
        if (threadIdx.x < 64) {
            const T *cv = static_cast<const T *>(cand);
            const int32_t *ci = reinterpret_cast<const int32_t *>(cv + ncand);
            const int lane = static_cast<int>(threadIdx.x);
            const int b = ncand <= 64 ? wave_best3_of<T, 1>(cv, ci, ncand, lane) : wave_best3_of<T, 4>(cv, ci, ncand, lane);
            if (lane < 3) {
                lead[lane] = b;
                if (blockIdx.x == 0 && blockIdx.y == 0) leaders[lane] = b;
            }
        }
        __syncthreads();
        L0 = __builtin_amdgcn_readfirstlane(lead[0]);
        L1 = __builtin_amdgcn_readfirstlane(lead[1]);
        L2 = __builtin_amdgcn_readfirstlane(lead[2]);
    } else {
        L0 = leaders ? leaders[0] : lead_c.x;
        L1 = leaders ? leaders[1] : lead_c.y;
        L2 = leaders ? leaders[2] : lead_c.z;
    }
    // leaders keep their positions; indices outside the population make
    // the launch a no-op instead of an out-of-bounds read
    const bool kept = i == L0 || i == L1 || i == L2 || i >= np;
    if (kept && !whole) return;
    if (L0 < 0 || L0 >= np || L1 < 0 || L1 >= np || L2 < 0 || L2 >= np) return;
    const uint32_t g = gen_dev ? gen_dev[0] : gen_c;
    const float a = a_tab ? a_tab[g] : a_c;
    const float two_a = 2.0f * a;

    uint32_t nib = 0;
    if (kept || j0 >= D) {
        if (i < np && j0 < cols)
            store_quad_nt(gwo_out_row<MERGE>(pv, i), j0, cols, *reinterpret_cast<const float4 *>(gwo_row<MERGE>(pv, i) + j0));
    } else {
        const float4 xv = MERGE != 0 ? own : *reinterpret_cast<const float4 *>(gwo_row<MERGE>(pv, i) + j0);
        const float4 X0 = *reinterpret_cast<const float4 *>(gwo_row<MERGE>(pv, L0) + j0);
        const float4 X1 = *reinterpret_cast<const float4 *>(gwo_row<MERGE>(pv, L1) + j0);
        const float4 X2 = *reinterpret_cast<const float4 *>(gwo_row<MERGE>(pv, L2) + j0);
        const float4 yv4 = gwo_quad<VARIANT>(xv, X0, X1, X2, static_cast<uint32_t>(q), static_cast<uint32_t>(i), g,
                                             inst, k0, k1, a, two_a);
        store_quad_nt(gwo_out_row<MERGE>(pv, i), j0, D, cols, yv4, xv);
        nib = quad_nibble(yv4, j0, D);
    }
    store_word(nib, q, D, bits, ld, i);
}

// The grey-wolf update of large populations: R consecutive individuals per
// workgroup (gwo_rows), grid x = 8 per_xcd groups of them (each XCD a contiguous
// range), y = 1024-gene chunk; arguments as gwo_kernel's.
template <int VARIANT, int R>
__global__ __launch_bounds__(256) void gwo_rows_kernel(PopView pv, const int32_t *__restrict__ leaders, int4 lead_c,
                                                       const float *__restrict__ a_tab, float a_c, uint32_t k0,
                                                       uint32_t k1, const uint32_t *__restrict__ gen_dev, uint32_t gen_c,
                                                       uint32_t inst, uint32_t *__restrict__ bits, int64_t ld,
                                                       int per_xcd, int whole)
{
    const int np = static_cast<int>(pv.np);
    const int i0 = R * (static_cast<int>(blockIdx.x & 7u) * per_xcd + static_cast<int>(blockIdx.x >> 3));
    if (i0 >= (whole ? static_cast<int>(ld) : np)) return;
    const int L0 = leaders ? leaders[0] : lead_c.x, L1 = leaders ? leaders[1] : lead_c.y,
              L2 = leaders ? leaders[2] : lead_c.z;
    if (L0 < 0 || L0 >= np || L1 < 0 || L1 >= np || L2 < 0 || L2 >= np) return;
    const uint32_t g = gen_dev ? gen_dev[0] : gen_c;
    gwo_rows<VARIANT, R>(pv, i0, static_cast<int64_t>(blockIdx.y) * 256 + threadIdx.x, L0, L1, L2,
                         a_tab ? a_tab[g] : a_c, g, inst, k0, k1, bits, ld, whole != 0);
}

// Improved discrete four-leader step (dgwo_quad), same grid as gwo_kernel.
// The new genes depend on the leaders' genes only, so the wolf's own row is
// not read. leaders: alpha, beta, delta (kept), then the fourth.
__global__ __launch_bounds__(256) void dgwo_kernel(PopView pv, const int32_t *__restrict__ leaders, int4 lead_c,
                                                   const float4 *__restrict__ par_tab, float4 par_c, uint32_t k0,
                                                   uint32_t k1, const uint32_t *__restrict__ gen_dev, uint32_t gen_c,
                                                   uint32_t inst, uint32_t *__restrict__ bits, int64_t ld,
                                                   int64_t per_xcd)
{
    const int64_t np = pv.np, D = pv.D;
    const int64_t i = static_cast<int64_t>(blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (i >= np) return;
    const int64_t L0 = leaders ? leaders[0] : lead_c.x, L1 = leaders ? leaders[1] : lead_c.y,
                  L2 = leaders ? leaders[2] : lead_c.z, L3 = leaders ? leaders[3] : lead_c.w;
    if (i == L0 || i == L1 || i == L2) return;
    if (L0 < 0 || L0 >= np || L1 < 0 || L1 >= np || L2 < 0 || L2 >= np || L3 < 0 || L3 >= np) return;
    const uint32_t g = gen_dev ? gen_dev[0] : gen_c;
    const float4 par = par_tab ? par_tab[g] : par_c;
    const int64_t q = static_cast<int64_t>(blockIdx.y) * 256 + threadIdx.x;
    const int64_t j0 = 4 * q;
    const bool valid = j0 < D;
    uint32_t nib = 0;
    if (valid) {
        const float4 X0 = *reinterpret_cast<const float4 *>(row_of(pv, L0) + j0);
        const float4 X1 = *reinterpret_cast<const float4 *>(row_of(pv, L1) + j0);
        const float4 X2 = *reinterpret_cast<const float4 *>(row_of(pv, L2) + j0);
        const float4 X3 = *reinterpret_cast<const float4 *>(row_of(pv, L3) + j0);
        const float4 yv4 = dgwo_quad(X0, X1, X2, X3, static_cast<uint32_t>(q), static_cast<uint32_t>(i), g, inst, k0,
                                     k1, par);
        store_quad_nt(out_row_of(pv, i), j0, D, yv4);
        nib = quad_nibble(yv4, j0, D);
    }
    store_word(nib, q, D, bits, ld, i);
}

// The fourth leader: the best genome (f descending, slot ascending) other
// than leaders[0..2], into leaders[3]. One workgroup; the order is total,
// so the result does not depend on the reduction order.
template <typename T>
__global__ __launch_bounds__(1024) void fourth_kernel(const T *__restrict__ f, int64_t np, int32_t *__restrict__ leaders)
{
    __shared__ T sv[16];
    __shared__ int si[16];
    const int64_t L0 = leaders[0], L1 = leaders[1], L2 = leaders[2];
    T bv = static_cast<T>(-INFINITY);
    int bi = INT_MAX;
    for (int64_t k = threadIdx.x; k < np; k += 1024) {
        if (k == L0 || k == L1 || k == L2) continue;
        const T v = f[k];
        if (v > bv || (v == bv && static_cast<int>(k) < bi)) {
            bv = v;
            bi = static_cast<int>(k);
        }
    }
    for (int o = 1; o < 64; o <<= 1) {
        const T ov = __shfl_xor(bv, o);
        const int oi = __shfl_xor(bi, o);
        if (ov > bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
        }
    }
    if ((threadIdx.x & 63) == 0) {
        sv[threadIdx.x >> 6] = bv;
        si[threadIdx.x >> 6] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w)
            if (sv[w] > bv || (sv[w] == bv && si[w] < bi)) {
                bv = sv[w];
                bi = si[w];
            }
        leaders[3] = bi;
    }
}

// ------------------------------------------------------------ top-3

template <typename T>
__global__ __launch_bounds__(1024) void top3_kernel(const T *__restrict__ f, int64_t np, int32_t *__restrict__ out)
{
    block_top3<T, 1024>(f, np, out);
}

// ------------------------------------------------------------ gather / pack

__global__ __launch_bounds__(256) void gather_kernel(PopView pv, const int32_t *__restrict__ rows,
                                                     float *__restrict__ out, int64_t ldo)
{
    const int64_t r = blockIdx.y;
    const int64_t src = rows ? rows[r] : r;
    const float *x = row_of(pv, src);
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; j < pv.D; j += 256 * gridDim.x)
        out[r * ldo + j] = x[j];
}

__global__ __launch_bounds__(256) void pack_pop_kernel(const float *__restrict__ x, int64_t D, int64_t ldx,
                                                       uint32_t *__restrict__ bits, int64_t ld)
{
    const int64_t i = blockIdx.x;
    const int64_t q = static_cast<int64_t>(blockIdx.y) * 256 + threadIdx.x;
    const int64_t j0 = 4 * q;
    const bool valid = j0 < D;
    uint32_t nib = 0;
    if (valid) nib = quad_nibble(*reinterpret_cast<const float4 *>(x + i * ldx + j0), j0, D);
    store_word(nib, q, D, bits, ld, i);
}

__global__ __launch_bounds__(256) void pack_row_kernel(const float *__restrict__ x, int64_t D,
                                                       uint32_t *__restrict__ bits)
{
    const int64_t w = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (32 * w >= D) return;
    uint32_t v = 0;
    for (int k = 0; k < 32; ++k) {
        const int64_t j = 32 * w + k;
        if (j < D && x[j] < 0.0f) v |= 1u << k;
    }
    bits[w] = v;
}

// ------------------------------------------------------------ launchers

// x = individual (fastest in dispatch order), y = 1024-gene chunk: all
// individuals of one chunk run before the next chunk, so the random donor
// rows of DE hit the caches (one chunk of the whole population is
// np x 4 KB) instead of streaming the population from HBM three times.
static dim3 quad_grid(int64_t D, int64_t rows)
{
    const int64_t quads = (D + 3) / 4;
    return dim3(static_cast<unsigned>(rows), static_cast<unsigned>((quads + 255) / 256));
}

// grid.x holds rows (< 2^31) and grid.y the 1024-gene chunks (<= 65535)
static qpm_status check_quad_grid(int64_t D, int64_t rows)
{
    QPM_REQUIRE(rows < (int64_t(1) << 31), QPM_ERANGE, "too many rows for one launch (%lld)", (long long)rows);
    QPM_REQUIRE((D + 1023) / 1024 <= 65535, QPM_ERANGE, "D = %lld exceeds 65535 chunks of 1024 genes",
                (long long)D);
    return QPM_OK;
}

qpm_status launch_init(int64_t np, int64_t D, int64_t ldx, uint64_t seed, uint32_t inst, float *x, uint32_t *bits,
                       int64_t ld, hipStream_t s)
{
    const qpm_status st = check_quad_grid(D, np);
    if (st != QPM_OK) return st;
    init_kernel<<<quad_grid(D, np), 256, 0, s>>>(D, ldx, static_cast<uint32_t>(seed),
                                                 static_cast<uint32_t>(seed >> 32), inst, x, bits, ld);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_de(const PopView &pv, float F, float CR, uint64_t seed, const uint32_t *gen_dev, uint32_t gen,
                     uint32_t inst, uint32_t *bits, int64_t ld, const int4 *draws, hipStream_t s,
                     int ipw_req, int passes, const uint32_t *fbits, const float *F_tab, bool store_genes,
                     uint32_t *reset_cnt, bool whole)
{
    QPM_REQUIRE(F_tab == nullptr || gen_dev != nullptr, QPM_EINVAL, "an F table needs the device generation");
    QPM_REQUIRE(store_genes || fbits != nullptr, QPM_EINVAL, "trials that are not stored need the packed flags");
    // flags (if any) staged in LDS: at most 65536 individuals, 8 KB
    // and 32-bit byte offsets of the rows over both buffers
    const bool staged = (pv.flags == nullptr || (fbits != nullptr && pv.np <= 65536)) && pv.x1 >= pv.x0 &&
                        pv.x1 - pv.x0 <= pv.np * pv.ldx && pv.out1 >= pv.out0 &&
                        pv.out1 - pv.out0 <= pv.np * pv.ldx && pv.np * pv.ldx < (int64_t(1) << 29);
    const size_t lds = fbits != nullptr && staged ? sizeof(uint32_t) * static_cast<size_t>((pv.np + 31) / 32) : 0;
    const uint32_t cr_max = cr_threshold(CR);
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    // individuals per wave so that one chunk of the population fits in 2 MB
    const int64_t row_bytes = 2 * 1024 * 1024 / pv.np;
    const int ipw_auto = row_bytes >= 1024 ? 1 : (row_bytes >= 512 ? 2 : 4);
    const int ipw = (ipw_req == 1 || ipw_req == 2 || ipw_req == 4) ? ipw_req : ipw_auto;
    const int64_t cw = 256 / ipw;
    // whole rows: the padding costs part of a chunk and of a row group, where
    // clearing u and its words first cost a pass (10000 x 4096: 21 us beside 87)
    const int64_t cols = whole ? pv.ldx : pv.D, rows = whole ? ld : pv.np;
    const int64_t chunks = (cols + cw - 1) / cw;
    const int R = (passes == 1 || passes == 2 || passes == 4)
                      ? passes
                      : de_passes((pv.np + 4 * ipw - 1) / (4 * ipw) * chunks);
    const int64_t groups = (rows + 4 * ipw * R - 1) / (4 * ipw * R);
    const int64_t blocks = 8 * ((chunks + 7) / 8) * groups;
    QPM_REQUIRE(blocks < (int64_t(1) << 31), QPM_ERANGE, "population too large for one DE launch");
    const int gr = static_cast<int>(groups), ch = static_cast<int>(chunks);
    const unsigned nb = static_cast<unsigned>(blocks);
#define QPM_DE(I, P)                                                                                            \
    if (staged)                                                                                                 \
        de_kernel<I, P, true><<<nb, 256, lds, s>>>(pv, draws, fbits, F, F_tab, cr_max, k0, k1, gen_dev, gen,     \
                                                   inst, bits, ld, gr, ch, store_genes ? 1 : 0, cols, rows,     \
                                                   reset_cnt);                                                  \
    else                                                                                                        \
        de_kernel<I, P, false><<<nb, 256, 0, s>>>(pv, draws, nullptr, F, F_tab, cr_max, k0, k1, gen_dev, gen,    \
                                                  inst, bits, ld, gr, ch, store_genes ? 1 : 0, cols, rows,      \
                                                  reset_cnt);
#define QPM_DE_R(I)                                                                                             \
    if (R == 1) { QPM_DE(I, 1) } else if (R == 2) { QPM_DE(I, 2) } else { QPM_DE(I, 4) }
    if (ipw == 1) {
        QPM_DE_R(1)
    } else if (ipw == 2) {
        QPM_DE_R(2)
    } else {
        QPM_DE_R(4)
    }
#undef QPM_DE_R
#undef QPM_DE
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_dgwo(const PopView &pv, const int32_t *leaders, const float4 *par_tab, float4 par,
                       uint64_t seed, const uint32_t *gen_dev, uint32_t gen, uint32_t inst, uint32_t *bits,
                       int64_t ld, hipStream_t s, int4 lead_c)
{
    const int64_t per_xcd = (pv.np + 7) / 8;
    const qpm_status st = check_quad_grid(pv.D, 8 * per_xcd);
    if (st != QPM_OK) return st;
    const dim3 grid(static_cast<unsigned>(8 * per_xcd), quad_grid(pv.D, pv.np).y);
    dgwo_kernel<<<grid, 256, 0, s>>>(pv, leaders, lead_c, par_tab, par, static_cast<uint32_t>(seed),
                                     static_cast<uint32_t>(seed >> 32), gen_dev, gen, inst, bits, ld, per_xcd);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_fourth(const void *f, int64_t np, bool f64, int32_t *leaders, hipStream_t s)
{
    if (f64)
        fourth_kernel<double><<<1, 1024, 0, s>>>(static_cast<const double *>(f), np, leaders);
    else
        fourth_kernel<float><<<1, 1024, 0, s>>>(static_cast<const float *>(f), np, leaders);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

// One wave's reductions in every workgroup against a kernel of one workgroup:
// the step merges the leaders itself up to kMergeGroups workgroups and 256
// candidates (np 5461). A generation, us, merged / by the kernel: 2000 x 500
// (1000 workgroups) 26.4 / 27.7, 1000 x 2000 (2000) 31.5 / 32.9, 4000 x 1000
// (4000) 38.7 / 38.6, 8000 x 1000 (8000) 55.9 / 53.9.
bool merges_leaders(int64_t np, int64_t D)
{
    return 3 * ((np + 63) / 64) <= 256 && np * ((D + 1023) / 1024) <= kMergeGroups;
}

qpm_status launch_gwo(const PopView &pv, int32_t *leaders, const float *a_tab, float a, uint64_t seed,
                      const uint32_t *gen_dev, uint32_t gen, uint32_t inst, int variant, uint32_t *bits, int64_t ld,
                      hipStream_t s, int4 lead_c, bool whole, const void *cand, bool cand_f64)
{
    const int64_t per_xcd = ((whole ? ld : pv.np) + 7) / 8, cols = whole ? pv.ldx : pv.D;
    const qpm_status st = check_quad_grid(cols, 8 * per_xcd);
    if (st != QPM_OK) return st;
    const dim3 grid(static_cast<unsigned>(8 * per_xcd), quad_grid(cols, pv.np).y);
    const int64_t ncand = 3 * ((pv.np + 63) / 64);
    QPM_REQUIRE(cand == nullptr || (leaders != nullptr && ncand <= 256), QPM_EINVAL,
                "merging leaders needs their buffer and at most 256 candidates");
    // 4 individuals per workgroup where their groups still fill the chip. The
    // entry point, us, 1 / 4: 8000 x 1000 17.8 / 17.6, 1500 x 5000 18.5 / 20.4,
    // 10^4 x 1024 22.5 / 21.7, 5000 x 2000 22.0 / 21.5, 6600 x 5000 69.3 / 67.3,
    // 10^4 x 4096 81.4 / 72.4, 5 x 10^4 x 900 86.9 / 76.8; 32 designs at once 193
    // x 10^6 genes 410 / 308, 19 x 10^6 42.3 / 38.7, 10 x 10^6 26.6 / 25.5, 3 x
    // 10^6 13.6 / 15.9.
    if (cand == nullptr && pv.np * pv.D >= kGwoRowsGenes && ld < (int64_t(1) << 30)) {
        const int rows_xcd = static_cast<int>(((whole ? ld : pv.np) + 31) / 32);
        const dim3 rgrid(static_cast<unsigned>(8 * rows_xcd), grid.y);
#define QPM_GWO_R(V)                                                                                              \
    gwo_rows_kernel<V, 4><<<rgrid, 256, 0, s>>>(pv, leaders, lead_c, a_tab, a, static_cast<uint32_t>(seed),       \
                                                static_cast<uint32_t>(seed >> 32), gen_dev, gen, inst, bits, ld,  \
                                                rows_xcd, whole ? 1 : 0)
        if (variant == 1)
            QPM_GWO_R(1);
        else
            QPM_GWO_R(0);
#undef QPM_GWO_R
        QPM_TRY_HIP(hipGetLastError());
        return QPM_OK;
    }
#define QPM_GWO(V, M)                                                                                             \
    gwo_kernel<V, M><<<grid, 256, 0, s>>>(pv, leaders, lead_c, a_tab, a, static_cast<uint32_t>(seed),             \
                                          static_cast<uint32_t>(seed >> 32), gen_dev, gen, inst, bits, ld,        \
                                          per_xcd, whole ? 1 : 0, cand, static_cast<int>(ncand))
#define QPM_GWO_M(M)                                                                                              \
    if (variant == 1)                                                                                             \
        QPM_GWO(1, M);                                                                                            \
    else                                                                                                          \
        QPM_GWO(0, M);
    if (cand == nullptr) {
        QPM_GWO_M(0)
    } else if (cand_f64) {
        QPM_GWO_M(2)
    } else {
        QPM_GWO_M(1)
    }
#undef QPM_GWO_M
#undef QPM_GWO
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_top3(const void *f, int64_t np, bool f64, int32_t *out3, hipStream_t s)
{
    if (f64)
        top3_kernel<double><<<1, 1024, 0, s>>>(static_cast<const double *>(f), np, out3);
    else
        top3_kernel<float><<<1, 1024, 0, s>>>(static_cast<const float *>(f), np, out3);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_gather(const PopView &pv, const int32_t *rows, int64_t nrows, float *out, int64_t ldo,
                         hipStream_t s)
{
    const int64_t blocks = (pv.D + 255) / 256;
    gather_kernel<<<dim3(static_cast<unsigned>(blocks < 64 ? blocks : 64), static_cast<unsigned>(nrows)), 256, 0,
                    s>>>(pv, rows, out, ldo);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_pack_pop(const float *x, int64_t np, int64_t D, int64_t ldx, uint32_t *bits, int64_t ld,
                           hipStream_t s)
{
    const qpm_status st = check_quad_grid(D, np);
    if (st != QPM_OK) return st;
    pack_pop_kernel<<<quad_grid(D, np), 256, 0, s>>>(x, D, ldx, bits, ld);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_draws(int64_t np, int64_t D, uint64_t seed, const uint32_t *gen_dev, uint32_t inst, int4 *draws,
                        hipStream_t s)
{
    de_draws_kernel<<<static_cast<unsigned>((np + 255) / 256), 256, 0, s>>>(
        np, D, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), gen_dev, 0u, inst, draws);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_pack_row(const float *x, int64_t D, uint32_t *bits, hipStream_t s)
{
    const int64_t W = words_for(D);
    pack_row_kernel<<<static_cast<unsigned>((W + 255) / 256), 256, 0, s>>>(x, D, bits);
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

}  // namespace qpm

using namespace qpm;

static qpm_status check_rows(const void *p, int64_t np, int64_t D, int64_t ldx, const char *name)
{
    QPM_REQUIRE(p != nullptr, QPM_EINVAL, "%s must not be NULL", name);
    QPM_REQUIRE(aligned16(p), QPM_EINVAL, "%s must be 16-byte aligned", name);
    QPM_REQUIRE(D >= 1 && D <= (int64_t(1) << 30), QPM_EINVAL, "D must be in [1, 2^30] (got %lld)", (long long)D);
    QPM_REQUIRE(ldx % 4 == 0 && ldx >= ((D + 3) / 4) * 4, QPM_EINVAL,
                "ldx (%lld) must be a multiple of 4 and >= D rounded up to 4", (long long)ldx);
    QPM_REQUIRE(np >= 1 && np <= (int64_t(1) << 31) - 1, QPM_EINVAL, "np out of range (%lld)", (long long)np);
    return QPM_OK;
}

static qpm_status check_bits(const uint32_t *bits, int64_t np, int64_t ld)
{
    QPM_REQUIRE(bits != nullptr, QPM_EINVAL, "bits must not be NULL");
    QPM_REQUIRE(ld >= np && ld % 64 == 0, QPM_EINVAL, "ld (%lld) must be >= np (%lld) and a multiple of 64",
                (long long)ld, (long long)np);
    return QPM_OK;
}

static bool overlaps(const void *a, size_t na, const void *b, size_t nb)
{
    const char *pa = static_cast<const char *>(a), *pb = static_cast<const char *>(b);
    return pa < pb + nb && pb < pa + na;
}

QPM_API qpm_status qpm_init_population(int64_t np, int64_t D, int64_t ldx, uint64_t seed, uint32_t inst, float *x,
                                       uint32_t *bits, int64_t ld, qpm_stream sv)
{
    clear_error();
    qpm_status st = check_rows(x, np, D, ldx, "x");
    if (st != QPM_OK) return st;
    st = check_bits(bits, np, ld);
    if (st != QPM_OK) return st;
    QPM_REQUIRE(inst < (1u << 24), QPM_EINVAL, "inst must be < 2^24");
    return launch_init(np, D, ldx, seed, inst, x, bits, ld, static_cast<hipStream_t>(sv));
}

static qpm_status de_step(const float *x, int64_t np, int64_t D, int64_t ldx, float F, float CR, uint64_t seed,
                          uint32_t generation, uint32_t inst, float *u, uint32_t *u_bits, int64_t ld, int ipw,
                          int passes, bool whole, qpm_stream sv)
{
    qpm_status st = check_rows(x, np, D, ldx, "x");
    if (st != QPM_OK) return st;
    st = check_rows(u, np, D, ldx, "u");
    if (st != QPM_OK) return st;
    st = check_bits(u_bits, np, ld);
    if (st != QPM_OK) return st;
    QPM_REQUIRE(np >= 4, QPM_EINVAL, "DE rand/1 needs np >= 4 (got %lld)", (long long)np);
    QPM_REQUIRE(F >= 0.0f && F <= 2.0f, QPM_EINVAL, "F must be in [0, 2] (got %g)", (double)F);
    QPM_REQUIRE(CR >= 0.0f && CR <= 1.0f, QPM_EINVAL, "CR must be in [0, 1] (got %g)", (double)CR);
    QPM_REQUIRE(inst < (1u << 24), QPM_EINVAL, "inst must be < 2^24");
    const size_t bytes = sizeof(float) * static_cast<size_t>(np) * static_cast<size_t>(ldx);
    QPM_REQUIRE(!overlaps(x, bytes, u, bytes), QPM_EINVAL, "x and u must not overlap");
    const PopView pv{x, x, nullptr, u, u, np, D, ldx};
    hipStream_t s = static_cast<hipStream_t>(sv);
    return launch_de(pv, F, CR, seed, nullptr, generation, inst, u_bits, ld, nullptr, s, ipw, passes,
                     nullptr, nullptr, true, nullptr, whole);
}

QPM_API qpm_status qpm_de_step(const float *x, int64_t np, int64_t D, int64_t ldx, float F, float CR,
                               uint64_t seed, uint32_t generation, uint32_t inst, float *u, uint32_t *u_bits,
                               int64_t ld, qpm_stream sv)
{
    clear_error();
    return de_step(x, np, D, ldx, F, CR, seed, generation, inst, u, u_bits, ld, 0, 0, false, sv);
}

QPM_API qpm_status qpm_de_step_whole(const float *x, int64_t np, int64_t D, int64_t ldx, float F, float CR,
                                     uint64_t seed, uint32_t generation, uint32_t inst, float *u, uint32_t *u_bits,
                                     int64_t ld, qpm_stream sv)
{
    clear_error();
    return de_step(x, np, D, ldx, F, CR, seed, generation, inst, u, u_bits, ld, 0, 0, true, sv);
}

QPM_API qpm_status qpm_de_step_shape(const float *x, int64_t np, int64_t D, int64_t ldx, float F, float CR,
                                     uint64_t seed, uint32_t generation, uint32_t inst, float *u, uint32_t *u_bits,
                                     int64_t ld, int32_t individuals_per_wave, int32_t passes, qpm_stream sv)
{
    clear_error();
    QPM_REQUIRE(individuals_per_wave == 0 || individuals_per_wave == 1 || individuals_per_wave == 2 ||
                    individuals_per_wave == 4,
                QPM_EINVAL, "individuals_per_wave must be 0, 1, 2 or 4 (got %d)", (int)individuals_per_wave);
    QPM_REQUIRE(passes == 1 || passes == 2 || passes == 4, QPM_EINVAL, "passes must be 1, 2 or 4 (got %d)",
                (int)passes);
    return de_step(x, np, D, ldx, F, CR, seed, generation, inst, u, u_bits, ld, individuals_per_wave, passes, false,
                   sv);
}

static qpm_status gwo_step(const float *x, int64_t np, int64_t D, int64_t ldx, const int32_t *leaders, float a,
                           uint64_t seed, uint32_t generation, uint32_t inst, int32_t variant, float *y,
                           uint32_t *y_bits, int64_t ld, bool whole, qpm_stream sv)
{
    qpm_status st = check_rows(x, np, D, ldx, "x");
    if (st != QPM_OK) return st;
    st = check_rows(y, np, D, ldx, "y");
    if (st != QPM_OK) return st;
    st = check_bits(y_bits, np, ld);
    if (st != QPM_OK) return st;
    QPM_REQUIRE(leaders != nullptr, QPM_EINVAL, "leaders must not be NULL");
    QPM_REQUIRE(np >= 4, QPM_EINVAL, "the grey-wolf step needs np >= 4 (got %lld)", (long long)np);
    QPM_REQUIRE(a == 0.0f || (a >= 0x1p-100f && a <= 1e30f), QPM_EINVAL,
                "a must be 0 or in [2^-100, 1e30] (got %g)", (double)a);
    QPM_REQUIRE(variant == 0 || variant == 1, QPM_EINVAL, "variant must be 0 or 1");
    QPM_REQUIRE(inst < (1u << 24), QPM_EINVAL, "inst must be < 2^24");
    const size_t bytes = sizeof(float) * static_cast<size_t>(np) * static_cast<size_t>(ldx);
    QPM_REQUIRE(!overlaps(x, bytes, y, bytes), QPM_EINVAL, "x and y must not overlap");
    hipStream_t s = static_cast<hipStream_t>(sv);
    const int32_t *L = leaders;  // host memory: validated here, passed by value
    for (int k = 0; k < 3; ++k)
        QPM_REQUIRE(L[k] >= 0 && L[k] < np, QPM_EINVAL, "leader %d (%d) is outside [0, np)", k, (int)L[k]);
    QPM_REQUIRE(L[0] != L[1] && L[0] != L[2] && L[1] != L[2], QPM_EINVAL, "leaders must be distinct");
    const PopView pv{x, x, nullptr, y, y, np, D, ldx};
    return launch_gwo(pv, nullptr, nullptr, a, seed, nullptr, generation, inst, variant, y_bits, ld, s,
                      make_int4(L[0], L[1], L[2], 0), whole);
}

QPM_API qpm_status qpm_gwo_step(const float *x, int64_t np, int64_t D, int64_t ldx, const int32_t *leaders,
                                float a, uint64_t seed, uint32_t generation, uint32_t inst, int32_t variant,
                                float *y, uint32_t *y_bits, int64_t ld, qpm_stream sv)
{
    clear_error();
    return gwo_step(x, np, D, ldx, leaders, a, seed, generation, inst, variant, y, y_bits, ld, false, sv);
}

QPM_API qpm_status qpm_gwo_step_whole(const float *x, int64_t np, int64_t D, int64_t ldx, const int32_t *leaders,
                                      float a, uint64_t seed, uint32_t generation, uint32_t inst, int32_t variant,
                                      float *y, uint32_t *y_bits, int64_t ld, qpm_stream sv)
{
    clear_error();
    return gwo_step(x, np, D, ldx, leaders, a, seed, generation, inst, variant, y, y_bits, ld, true, sv);
}

QPM_API qpm_status qpm_dgwo_step(const float *x, int64_t np, int64_t D, int64_t ldx, const int32_t *leaders,
                                 const float *params, uint64_t seed, uint32_t generation, uint32_t inst, float *y,
                                 uint32_t *y_bits, int64_t ld, qpm_stream sv)
{
    clear_error();
    qpm_status st = check_rows(x, np, D, ldx, "x");
    if (st != QPM_OK) return st;
    st = check_rows(y, np, D, ldx, "y");
    if (st != QPM_OK) return st;
    st = check_bits(y_bits, np, ld);
    if (st != QPM_OK) return st;
    QPM_REQUIRE(leaders != nullptr && params != nullptr, QPM_EINVAL, "leaders and params must not be NULL");
    QPM_REQUIRE(np >= 4, QPM_EINVAL, "the four-leader step needs np >= 4 (got %lld)", (long long)np);
    QPM_REQUIRE(inst < (1u << 24), QPM_EINVAL, "inst must be < 2^24");
    for (int k = 0; k < 4; ++k)
        QPM_REQUIRE(std::isfinite(params[k]), QPM_EINVAL, "params[%d] is not finite", k);
    const size_t bytes = sizeof(float) * static_cast<size_t>(np) * static_cast<size_t>(ldx);
    QPM_REQUIRE(!overlaps(x, bytes, y, bytes), QPM_EINVAL, "x and y must not overlap");
    hipStream_t s = static_cast<hipStream_t>(sv);
    const int32_t *L = leaders;  // host memory: validated here, passed by value
    for (int k = 0; k < 4; ++k)
        QPM_REQUIRE(L[k] >= 0 && L[k] < np, QPM_EINVAL, "leader %d (%d) is outside [0, np)", k, (int)L[k]);
    for (int a = 0; a < 4; ++a)
        for (int b = a + 1; b < 4; ++b) QPM_REQUIRE(L[a] != L[b], QPM_EINVAL, "leaders must be distinct");
    const PopView pv{x, x, nullptr, y, y, np, D, ldx};
    const float4 par = make_float4(params[0], params[1], params[2], params[3]);
    return launch_dgwo(pv, nullptr, nullptr, par, seed, nullptr, generation, inst, y_bits, ld, s,
                       make_int4(L[0], L[1], L[2], L[3]));
}
