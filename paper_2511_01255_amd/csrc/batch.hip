// batch.hip -- many independent designs of uneven length and phase
// mismatch optimised together: every step of a generation is one launch over
// all instances (an addition to the paper, whose runs optimise one crystal
// at a time).
//
// Layout: the per-domain tables of all instances are concatenated by whole
// 32-domain words (instance b starts at word row wofs_b), and so are the
// population-major bit rows; gene rows of instance b start at float offset
// xofs_b (row stride ldx_b). Per-individual arrays (fitness, flags, DE
// draws) are instance-major, np per instance. Small device tables map a
// workgroup to its (instance, segment) for the fitness and (instance,
// chunk) for DE, GWO and initialisation. Every instance uses the Philox
// instance number inst0 + b, so its random streams are those of a
// single-design run with that instance number.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "common.hpp"
#include "device_common.hpp"
#include "genes.hpp"
#include "scan.hpp"
#include "select.hpp"

namespace qpm {

struct InstDesc {
    int64_t n;     // domains (= genes)
    int64_t words; // W
    int64_t wofs;  // first word row of the instance
    int64_t xofs;  // float offset of row 0 in a gene buffer
    int64_t ldx;   // gene row stride
    double C[2];
};

struct FitSeg {
    int inst;  // instance
    int w0;    // first word (within the instance) of the workgroup
    int slot;  // partial slot
    int pad;
};

struct Tile {
    int inst;
    int chunk;
};

// ---------------------------------------------------------------- fitness

template <bool F32, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void batch_fit_kernel(const uint32_t *__restrict__ bits, int64_t ld,
                                                               const double4 *__restrict__ ph64,
                                                               const float4 *__restrict__ ph32, int wpw,
                                                               const InstDesc *__restrict__ inst,
                                                               const FitSeg *__restrict__ tab,
                                                               double *__restrict__ part, uint32_t *__restrict__ advance)
{
    if (advance != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) advance[0] += 1u;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const FitSeg fs = tab[blockIdx.y];
    const InstDesc id = inst[fs.inst];
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    const int w0 = fs.w0 + wave * wpw;
    const int w1 = min(static_cast<int>(id.words), w0 + wpw);
    Tri t{0, 0, 0, 0, 0, 0};
    const uint32_t *bp = bits + id.wofs * ld + i;
    if (w0 < w1) {
        uint32_t next = bp[static_cast<int64_t>(w0) * ld];
        for (int wd = w0; wd < w1; ++wd) {
            const uint32_t word = next;
            if (wd + 1 < w1) next = bp[static_cast<int64_t>(wd + 1) * ld];
            const int64_t dom = (id.wofs + wd) * 32;
            if constexpr (F32)
                scan_word_f32(t, word, ph64 + dom, ph32 + dom);
            else
                scan_word_f64(t, word, ph64 + dom);
        }
    }
    if constexpr (WAVES > 1) {
        __shared__ double sh[6][WAVES][64];
        sh[0][wave][lane] = t.ar;
        sh[1][wave][lane] = t.ai;
        sh[2][wave][lane] = t.br;
        sh[3][wave][lane] = t.bi;
        sh[4][wave][lane] = t.qr;
        sh[5][wave][lane] = t.qi;
        __syncthreads();
        if (wave != 0) return;
#pragma unroll 1
        for (int w = 1; w < WAVES; ++w) {
            const Tri u{sh[0][w][lane], sh[1][w][lane], sh[2][w][lane],
                        sh[3][w][lane], sh[4][w][lane], sh[5][w][lane]};
            tri_append(t, u);
        }
    }
    double *o = part + static_cast<int64_t>(fs.slot) * 6 * ld + i;
    o[0] = t.ar;
    o[ld] = t.ai;
    o[2 * ld] = t.br;
    o[3 * ld] = t.bi;
    o[4 * ld] = t.qr;
    o[5 * ld] = t.qi;
}

// The table kernel over (instance, segment) tiles: the sign-pattern tables
// and bit rows of instance b start at its word row wofs_b.
template <bool F32, int GW, bool STAGED>
__global__ __launch_bounds__(GW * 256) void batch_fit_tab_kernel(const uint32_t *__restrict__ bits, int64_t ld,
                                                                 const double2 *__restrict__ tab64,
                                                                 const int2 *__restrict__ tabq,
                                                                 const double *__restrict__ wsc, int wpw,
                                                                 int64_t np, const InstDesc *__restrict__ inst,
                                                                 const FitSeg *__restrict__ tab,
                                                                 double *__restrict__ part,
                                                                 uint32_t *__restrict__ advance)
{
    extern __shared__ __align__(16) unsigned char lds[];
    // a run's generation advance (this kernel does not read the counter)
    if (advance != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) advance[0] += 1u;
    const FitSeg fs = tab[blockIdx.y];
    const InstDesc id = inst[fs.inst];
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * GW + (threadIdx.x >> 8)) * 64 + (threadIdx.x & 63);
    Tri t;
    const int W = static_cast<int>(id.words);
    const double2 *t64 = tab64 + id.wofs * 8 * 48;
    const int2 *tq = tabq + id.wofs * 8 * 48;
    if constexpr (STAGED) {
        if (!tab_segment_staged<F32, GW>(t, bits + id.wofs * ld, ld, W, fs.w0, t64, tq, wsc + id.wofs, wpw, np, lds))
            return;
    } else {
        if (!tab_segment<F32, GW>(t, bits + id.wofs * ld, ld, W, fs.w0, t64, tq, wsc + id.wofs, wpw, np, lds)) return;
    }
    double *o = part + static_cast<int64_t>(fs.slot) * 6 * ld + i;
    o[0] = t.ar;
    o[ld] = t.ai;
    o[2 * ld] = t.br;
    o[3 * ld] = t.bi;
    o[4 * ld] = t.qr;
    o[5 * ld] = t.qi;
}

// The fitness of every genome from its instance's segment triples, over the
// whole batch at once: grid x = groups of 16 genomes, y = instance, 16 ranges
// per genome (combine_segments). Folded inside the one-workgroup-per-instance
// selection kernel instead, this took 20-26 us at 32 and 64 designs of up to
// 5 x 10^4 domains, against 6 us here.
template <typename T>
__global__ __launch_bounds__(256) void batch_combine_kernel(const double *__restrict__ part,
                                                            const int *__restrict__ slot_ofs, int64_t ld, int64_t np,
                                                            const InstDesc *__restrict__ inst, T *__restrict__ fit)
{
    __shared__ double sh[6 * 16 * 16];
    const int b = blockIdx.y;
    const int gl = threadIdx.x & 15, range = threadIdx.x >> 4;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 16 + gl;
    const int s0 = slot_ofs[b];
    const Tri t = combine_segments<16, 16>(part + static_cast<int64_t>(s0) * 6 * ld, slot_ofs[b + 1] - s0, ld, i,
                                           i < np, range, gl, sh);
    if (range == 0 && i < np) {
        const double sr = t.qr + inst[b].C[0], si = t.qi + inst[b].C[1];
        fit[static_cast<int64_t>(b) * np + i] = static_cast<T>(fma(sr, sr, si * si));
    }
}

// The end of an evaluation in a batched run, as finish_kernel: grid x = groups
// of 64 genomes, y = instance; 16 waves fold the group's segment triples,
// wave 0 then
//   mode 1 (initial): f_cur = f, leader candidates, DE draws of generation gen;
//   mode 2 (after DE): selects, leader candidates;
//   mode 3 (after GWO): selects with the leaders excluded, DE draws of the
//     next generation (gen, which the evaluation kernel before this one
//     advanced: it does not read the counter, so no cross-workgroup
//     ordering is needed here).
// The candidates (3 per group) are merged into the leaders by
// batch_leaders_kernel or the accepted-trial kernel after it. (With one
// workgroup per instance instead: 23-26 us at 32 designs of 256 genomes and
// up to 5 x 10^4 domains, against 8 us.)
template <typename T>
__global__ __launch_bounds__(1024) void batch_finish_kernel(int mode, const double *__restrict__ part,
                                                           const int *__restrict__ slot_ofs, int64_t ld, int64_t np,
                                                           const InstDesc *__restrict__ inst, T *__restrict__ f_cur,
                                                           uint32_t *__restrict__ flags,
                                                           const int32_t *__restrict__ leaders,
                                                           T *__restrict__ cand_v, int32_t *__restrict__ cand_i,
                                                           int4 *__restrict__ draws, const uint32_t *__restrict__ gen,
                                                           uint32_t k0, uint32_t k1, uint32_t inst0,
                                                           uint32_t *__restrict__ fbits, AcceptOut acc)
{
    __shared__ double sh[6 * 16 * 64];
    const int64_t b = blockIdx.y, grp = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int64_t i = grp * 64 + lane;
    const int s0 = slot_ofs[b];
    const Tri t = combine_segments<16, 64>(part + static_cast<int64_t>(s0) * 6 * ld, slot_ofs[b + 1] - s0, ld, i,
                                           i < np, static_cast<int>(threadIdx.x >> 6), lane, sh);
    if (threadIdx.x >= 64) return;
    const double sr = t.qr + inst[b].C[0], si = t.qi + inst[b].C[1];
    const double f = fma(sr, sr, si * si);
    const int64_t n = inst[b].n;
    const uint32_t instb = inst0 + static_cast<uint32_t>(b);
    const int64_t fw = 2 * static_cast<int64_t>(gridDim.x);  // packed flag words per instance
    T *fb = f_cur + b * np;
    int4 *db = draws + b * np;
    T *cv = mode <= 2 ? cand_v + b * 3 * gridDim.x : nullptr;
    int32_t *ci = cand_i + b * 3 * gridDim.x;
    if (mode == 1) {
        if (i < np) {
            fb[i] = static_cast<T>(f);
            db[i] = de_draw(i, np, n, gen[0], instb, k0, k1);
        }
        group_best3(i < np ? static_cast<T>(f) : static_cast<T>(-INFINITY), i < np ? static_cast<int>(i) : INT_MAX,
                    lane, cv + 3 * grp, ci + 3 * grp);
        return;
    }
    const AcceptOut accb = acc.list ? AcceptOut{acc.list + b * np, acc.cnt + b, acc.fbits_prev + b * fw} : AcceptOut{};
    select_group<T>(f, grp, lane, np, fb, flags + b * np, fbits + b * fw, mode == 3 ? leaders + 3 * b : nullptr, cv, ci,
                    mode == 3 ? db : nullptr, gen, n, k0, k1, instb, accb, 0u);
}

// the leaders of instance blockIdx.x from its groups' candidates (3 of each 64
// genomes: at most 192)
template <typename T>
__global__ __launch_bounds__(64) void batch_leaders_kernel(const T *__restrict__ cand_v,
                                                           const int32_t *__restrict__ cand_i, int64_t groups,
                                                           int32_t *__restrict__ leaders)
{
    const int64_t b = blockIdx.x;
    merge_few_leaders<T>(cand_v + b * 3 * groups, cand_i + b * 3 * groups, 3 * groups, leaders + 3 * b);
}

// ---------------------------------------------------------------- evolution

struct BatchPop {
    const float *x0, *x1;
    float *out0, *out1;
    const uint32_t *flags;  // instance-major, np per instance
    int64_t np;
};

__device__ __forceinline__ PopView view_of(const BatchPop &bp, const InstDesc &id, int b)
{
    return PopView{bp.x0 + id.xofs, bp.x1 + id.xofs, bp.flags + static_cast<int64_t>(b) * bp.np,
                   bp.out0 + id.xofs, bp.out1 + id.xofs, bp.np, id.n, id.ldx};
}

// initialisation: grid x = individual, y = tile (instance, 1024-gene chunk)
__global__ __launch_bounds__(256) void batch_init_kernel(int64_t np, const InstDesc *__restrict__ inst,
                                                         const Tile *__restrict__ tiles, uint32_t k0, uint32_t k1,
                                                         uint32_t inst0, float *__restrict__ x,
                                                         uint32_t *__restrict__ bits, int64_t ld)
{
    const Tile tl = tiles[blockIdx.y];
    const InstDesc id = inst[tl.inst];
    const int64_t i = blockIdx.x;
    const int64_t q = static_cast<int64_t>(tl.chunk) * 256 + threadIdx.x;
    const int64_t j0 = 4 * q;
    const bool valid = j0 < id.n;
    uint32_t nib = 0;
    if (valid) {
        const U4 r = philox10(static_cast<uint32_t>(q), static_cast<uint32_t>(i), 0u,
                              ((inst0 + static_cast<uint32_t>(tl.inst)) << 8) | kTagInit, k0, k1);
        const float4 v = make_float4(sym24(r.x), sym24(r.y), sym24(r.z), sym24(r.w));
        store_quad(x + id.xofs + i * id.ldx, j0, id.n, v);
        nib = quad_nibble(v, j0, id.n);
    }
    store_word(nib, q, id.n, bits + id.wofs * ld, ld, i);
}

// DE: tiles (instance, chunk of CW = 256 / IPW genes) dealt round-robin to
// the XCDs (workgroup id mod 8); a workgroup makes R passes over groups of
// 4 IPW consecutive individuals of one tile (de_rows). Each row's buffer flag
// comes from the instance's packed flags (np / 32 words, np <= 4096), copied
// to LDS first, instead of a dependent global load after the draw. Bound by
// the row reads (16 B per gene, a quarter of them from HBM): 32 designs of
// 26,000 domains on average, NP = 256, bits only: 219 us with 4 passes, 276 us
// with 1; 306-343 us with 1 pass when the row pointers sat in LDS (their
// loads then were flat ones, waited for all at once).
template <int IPW, int R, typename OFF>
__global__ __launch_bounds__(256) void batch_de_kernel(BatchPop bp, const InstDesc *__restrict__ inst,
                                                       const Tile *__restrict__ tiles, int ntiles, int groups,
                                                       const int4 *__restrict__ draws, float F, uint32_t cr_max,
                                                       uint32_t k0, uint32_t k1, const uint32_t *__restrict__ gen,
                                                       uint32_t inst0, uint32_t *__restrict__ bits, int64_t ld,
                                                       const uint32_t *__restrict__ fbits, int store_genes,
                                                       uint32_t *__restrict__ reset_cnt, int n_inst)
{
    // the accepted trials' counters start at 0 for this generation
    if (reset_cnt != nullptr && blockIdx.x == 0)
        for (int k = threadIdx.x; k < n_inst; k += 256) reset_cnt[k] = 0u;
    constexpr int IPB = 4 * IPW * R;
    const uint32_t blk = blockIdx.x;
    const int k = static_cast<int>(blk >> 3);
    const int gi = k % groups;
    const int ti = static_cast<int>(blk & 7u) + 8 * (k / groups);
    if (ti >= ntiles) return;
    const Tile tl = tiles[ti];
    const InstDesc id = inst[tl.inst];
    const int64_t np = bp.np;
    const int t = threadIdx.x;
    __shared__ uint32_t sfb[128];
    const int fw = 2 * static_cast<int>((np + 63) / 64);
    int4 d = make_int4(0, 0, 0, 0);
    if (t < IPB) d = draws[tl.inst * np + min(static_cast<int64_t>(gi) * IPB + t, np - 1)];
    if (t < fw) sfb[t] = fbits[static_cast<int64_t>(tl.inst) * fw + t];
    __syncthreads();
    const PopView pv = view_of(bp, id, tl.inst);
    de_rows<IPW, R, OFF>(pv, gi, tl.chunk, F, cr_max, gen[0], inst0 + static_cast<uint32_t>(tl.inst), k0, k1,
                         bits + id.wofs * ld, ld, store_genes != 0, pv.D, pv.np, d,
                         [&](int r) -> bool { return ((sfb[r >> 5] >> (r & 31)) & 1u) != 0u; });
}

// The accepted trials of a batched run whose DE step stored only bits: the
// entries list[0 .. cnt[b]) of instance b's list are slots whose trial genes
// are computed again exactly as batch_de_kernel computed them, from the rows
// before the selection (fb_old: the instance's packed flags before it), and
// written to the buffer the selection made current. Grid: x = shares of the
// list, y = tile (instance, 1024-gene chunk); a thread keeps one gene quad
// (and its Philox head) and walks its share of the list.
__global__ __launch_bounds__(256) void batch_materialize_kernel(BatchPop bp, const InstDesc *__restrict__ inst,
                                                                const Tile *__restrict__ tiles,
                                                                const int4 *__restrict__ draws,
                                                                const uint32_t *__restrict__ fb_old, float F,
                                                                uint32_t cr_max, uint32_t k0, uint32_t k1,
                                                                const uint32_t *__restrict__ gen, uint32_t inst0,
                                                                const int32_t *__restrict__ list,
                                                                const uint32_t *__restrict__ cnt,
                                                                const void *__restrict__ cand_v,
                                                                const int32_t *__restrict__ cand_i, int cand_f64,
                                                                int32_t *__restrict__ leaders)
{
    const Tile tl = tiles[blockIdx.y];
    // each instance's leaders from its groups' candidates, once
    if (blockIdx.x == 0 && tl.chunk == 0) {
        const int64_t n3 = 3 * ((bp.np + 63) / 64);
        if (cand_f64)
            merge_few_leaders<double>(static_cast<const double *>(cand_v) + tl.inst * n3, cand_i + tl.inst * n3, n3,
                                      leaders + 3 * tl.inst);
        else
            merge_few_leaders<float>(static_cast<const float *>(cand_v) + tl.inst * n3, cand_i + tl.inst * n3, n3,
                                     leaders + 3 * tl.inst);
    }
    const int64_t np = bp.np;
    const uint32_t n_acc = min(cnt[tl.inst], static_cast<uint32_t>(np));
    if (blockIdx.x >= n_acc) return;
    const InstDesc id = inst[tl.inst];
    const int64_t q = static_cast<int64_t>(tl.chunk) * 256 + threadIdx.x, j0 = 4 * q;
    if (j0 >= id.n) return;
    const uint32_t g = gen[0];
    const int64_t fw = 2 * ((np + 63) / 64);
    const uint32_t *fo = fb_old + tl.inst * fw;
    const int32_t *lb = list + tl.inst * np;
    const int4 *db = draws + tl.inst * np;
    const float *const x0 = bp.x0 + id.xofs + j0;
    float *const out0 = bp.out0 + id.xofs;
    const int64_t dx = bp.x1 - bp.x0, ldx = id.ldx;  // (the outputs are the same two buffers)
    auto src = [&](int32_t r) -> const float * {
        return x0 + (r * ldx + (((fo[r >> 5] >> (r & 31)) & 1u) != 0u ? dx : 0));
    };
    const PhiloxHead h = philox10_head(static_cast<uint32_t>(q), g,
                                       ((inst0 + static_cast<uint32_t>(tl.inst)) << 8) | kTagDeCr, k0, k1);
    for (uint32_t ir = blockIdx.x; ir < n_acc; ir += gridDim.x) {
        const int32_t i = lb[ir];
        if (i < 0 || i >= np) continue;
        const int4 dr = db[i];
        const bool old = ((fo[i >> 5] >> (i & 31)) & 1u) != 0u;
        const float4 v[4] = {*reinterpret_cast<const float4 *>(src(i)), *reinterpret_cast<const float4 *>(src(dr.x)),
                             *reinterpret_cast<const float4 *>(src(dr.y)),
                             *reinterpret_cast<const float4 *>(src(dr.z))};
        const float4 uv = de_quad_shared(h, philox10_individual(static_cast<uint32_t>(i), g, k0), v,
                                         dr.w - static_cast<int>(j0), k0, k1, F, cr_max);
        store_quad_nt(out0 + (i * ldx + (old ? 0 : dx)), j0, id.n, uv);
    }
}

// GWO: grid x = 8 ceil(np / 8) (individuals in contiguous ranges per XCD,
// as in the single-design kernel), y = tile (instance, 1024-gene chunk)
template <int VARIANT>
__global__ __launch_bounds__(256) void batch_gwo_kernel(BatchPop bp, const InstDesc *__restrict__ inst,
                                                        const Tile *__restrict__ tiles,
                                                        const int32_t *__restrict__ leaders,
                                                        const float *__restrict__ a_tab, uint32_t k0, uint32_t k1,
                                                        const uint32_t *__restrict__ gen, uint32_t inst0,
                                                        uint32_t *__restrict__ bits, int64_t ld, int64_t per_xcd)
{
    const int64_t np = bp.np;
    const int64_t i = static_cast<int64_t>(blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (i >= np) return;
    const Tile tl = tiles[blockIdx.y];
    const InstDesc id = inst[tl.inst];
    const int64_t D = id.n;
    const int64_t L0 = leaders[3 * tl.inst], L1 = leaders[3 * tl.inst + 1], L2 = leaders[3 * tl.inst + 2];
    if (i == L0 || i == L1 || i == L2) return;
    if (L0 < 0 || L0 >= np || L1 < 0 || L1 >= np || L2 < 0 || L2 >= np) return;
    const PopView pv = view_of(bp, id, tl.inst);
    const uint32_t g = gen[0];
    const float a = a_tab[g];
    const float two_a = 2.0f * a;
    const int64_t q = static_cast<int64_t>(tl.chunk) * 256 + threadIdx.x;
    const int64_t j0 = 4 * q;
    const bool valid = j0 < D;
    uint32_t nib = 0;
    if (valid) {
        const float4 xv = *reinterpret_cast<const float4 *>(row_of(pv, i) + j0);
        const float4 X0 = *reinterpret_cast<const float4 *>(row_of(pv, L0) + j0);
        const float4 X1 = *reinterpret_cast<const float4 *>(row_of(pv, L1) + j0);
        const float4 X2 = *reinterpret_cast<const float4 *>(row_of(pv, L2) + j0);
        const float4 yv = gwo_quad<VARIANT>(xv, X0, X1, X2, static_cast<uint32_t>(q), static_cast<uint32_t>(i), g,
                                            inst0 + static_cast<uint32_t>(tl.inst), k0, k1, a, two_a);
        store_quad_nt(out_row_of(pv, i), j0, D, yv);
        nib = quad_nibble(yv, j0, D);
    }
    store_word(nib, q, id.n, bits + id.wofs * ld, ld, i);
}

// The same for large batches (kGwoRowsGenes): R consecutive individuals per
// workgroup (gwo_rows), grid x = 8 per_xcd groups of them. 32 designs of up to
// 5 x 10^4 domains, NP = 256 (193 x 10^6 genes): 410 -> 308 us.
template <int VARIANT, int R>
__global__ __launch_bounds__(256) void batch_gwo_rows_kernel(BatchPop bp, const InstDesc *__restrict__ inst,
                                                        const Tile *__restrict__ tiles,
                                                        const int32_t *__restrict__ leaders,
                                                        const float *__restrict__ a_tab, uint32_t k0, uint32_t k1,
                                                        const uint32_t *__restrict__ gen, uint32_t inst0,
                                                        uint32_t *__restrict__ bits, int64_t ld, int per_xcd)
{
    const int np = static_cast<int>(bp.np);
    const int i0 = R * (static_cast<int>(blockIdx.x & 7u) * per_xcd + static_cast<int>(blockIdx.x >> 3));
    if (i0 >= np) return;
    const Tile tl = tiles[blockIdx.y];
    const InstDesc id = inst[tl.inst];
    const int L0 = leaders[3 * tl.inst], L1 = leaders[3 * tl.inst + 1], L2 = leaders[3 * tl.inst + 2];
    if (L0 < 0 || L0 >= np || L1 < 0 || L1 >= np || L2 < 0 || L2 >= np) return;
    const uint32_t g = gen[0];
    gwo_rows<VARIANT, R>(view_of(bp, id, tl.inst), i0, static_cast<int64_t>(tl.chunk) * 256 + threadIdx.x, L0, L1, L2,
                         a_tab[g], g, inst0 + static_cast<uint32_t>(tl.inst), k0, k1, bits + id.wofs * ld, ld, false);
}

// rows of instance b's current population -> dense out[np][ldo]
__global__ __launch_bounds__(256) void batch_gather_kernel(BatchPop bp, const InstDesc *__restrict__ inst, int b,
                                                           float *__restrict__ out, int64_t ldo)
{
    const InstDesc id = inst[b];
    const PopView pv = view_of(bp, id, b);
    const int64_t r = blockIdx.y;
    const float *x = row_of(pv, r);
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; j < id.n; j += 256 * gridDim.x)
        out[r * ldo + j] = x[j];
}

// ---------------------------------------------------------------- plans

struct BatchFitPlan {
    int waves = 16;  // per-domain kernel: waves per workgroup; table kernel: 4 segment waves
    int wpw = 8;
    int gw = 0;      // table kernel: genome groups of 64 per workgroup (0 = per-domain kernel)
    std::vector<FitSeg> segs;
    std::vector<int> slot_ofs;  // n_inst + 1
};

static BatchFitPlan make_fit_plan(const std::vector<InstDesc> &h, int waves, int wpw)
{
    BatchFitPlan p;
    p.waves = waves;
    p.wpw = wpw;
    p.slot_ofs.push_back(0);
    int slot = 0;
    const int per_wg = waves * wpw;
    for (size_t b = 0; b < h.size(); ++b) {
        for (int w0 = 0; w0 < h[b].words; w0 += per_wg) p.segs.push_back(FitSeg{static_cast<int>(b), w0, slot++, 0});
        p.slot_ofs.push_back(slot);
    }
    return p;
}

// the shape of a table plan without its tables
static BatchFitPlan tab_shape(int gw, int wpw)
{
    BatchFitPlan p;
    p.waves = 4;
    p.wpw = wpw;
    p.gw = gw;
    return p;
}

// the table plan: tiles of 4 wpw words, gw genome groups per workgroup
static BatchFitPlan make_tab_plan(const std::vector<InstDesc> &h, int gw, int wpw)
{
    BatchFitPlan p = make_fit_plan(h, 4, wpw);
    p.gw = gw;
    return p;
}

// Launch shape of the batched table kernel from the work, in waves' words (64-
// genome groups x words of all instances): as for single designs, small work
// takes small workgroups, large work long staged segments. Kernel + combine, us,
// shape / shape:
//   FP32  16 designs of 72 words, NP = 100 (1920): 1/2 8.6, 1/4 9.9
//         10 designs, NP = 400 (3122): 1/2 8.9, 4/4 12.0
//         64 designs, NP = 256 (188920): 4/8 62.8, 4/5 72.7;  32 (94204): 4/8 36.6, 4/5 41.9
//         39, NP = 125 (51122): 2/8 30.8, 2/5 32.0;  16, NP = 505 (46864): 4/8 26.9, 4/5 29.1
//   FP64  10 designs, NP = 400: 2/2 9.4, 4/2 10.1;  64, NP = 256: 4/12 71.4, 4/8 76.9, 4/2 94.7
//         32: 4/12 37.2, 4/2 50.2;  39, NP = 125: 2/6 35.7, 2/2 39.9;  16, NP = 505: 4/12 25.0, 4/2 30.3
static void default_tab_shape(int64_t np, int64_t words, bool f32, int *gw, int *wpw)
{
    const int64_t groups = (np + 63) / 64;
    const bool large = groups * words > 12000;
    const int most = large ? 4 : (f32 ? 1 : 2);
    *gw = groups >= 4 ? most : (groups >= 2 ? std::min(most, 2) : 1);
    *wpw = !large ? 2 : (f32 ? 8 : (*gw == 4 ? 12 : 6));
}

static void default_fit_shape(const std::vector<InstDesc> &h, int64_t np, int *waves, int *wpw)
{
    int64_t words = 0;
    for (const auto &d : h) words += d.words;
    const int64_t groups = (np + 63) / 64;
    // aim for ~8 waves per SIMD (8192 waves) over 256 CUs x 4 SIMDs
    int64_t w = (groups * words + 8191) / 8192;
    if (w < 1) w = 1;
    *waves = 16;
    *wpw = static_cast<int>(w);
}

}  // namespace qpm

using namespace qpm;

// ---------------------------------------------------------------- the batch design

// Device tables of an evaluation plan kept with the batch: they follow from
// the launch shape alone (not from np, ld or the stream).
struct EvalPlan {
    int waves = 0, wpw = 0, gw = 0;
    size_t nsegs = 0;
    FitSeg *segs = nullptr;
    int *slot_ofs = nullptr;
};
constexpr size_t kEvalPlans = 8;

struct qpm_batch_s {
    // shapes evaluated so far, at most kEvalPlans of them, each kept until the
    // batch is freed (so a launch never outlives its tables); the lock covers
    // the list
    std::mutex plan_mutex;
    std::vector<EvalPlan> plans;
    ScratchCache *scratch = nullptr;  // segment partials of the evaluations
    int32_t n_inst = 0;
    int64_t total_words = 0;
    int64_t total_genes_stride = 0;  // sum over instances of ldx
    std::vector<InstDesc> host;
    InstDesc *dev = nullptr;
    double4 *ph64 = nullptr;
    float4 *ph32 = nullptr;
    double2 *c64 = nullptr;
    double *Cdev = nullptr;
    double2 *tab64 = nullptr;  // sign-pattern tables, [8 total_words][3][16]
    int2 *tabq = nullptr;      // their fixed-point form at the word scales
    double *wsc = nullptr;     // [total_words] word scales (word_scales per instance)
};

static void free_batch(qpm_batch_s *b)
{
    if (!b) return;
    (void)hipFree(b->dev);
    (void)hipFree(b->ph64);
    (void)hipFree(b->ph32);
    (void)hipFree(b->c64);
    (void)hipFree(b->Cdev);
    (void)hipFree(b->tab64);
    (void)hipFree(b->tabq);
    (void)hipFree(b->wsc);
    for (auto &p : b->plans) {
        (void)hipFree(p.segs);
        (void)hipFree(p.slot_ofs);
    }
    scratch_cache_destroy(b->scratch);
    delete b;
}

QPM_API qpm_status qpm_precompute_phases_batched(const double *z, const int64_t *offsets, int32_t n_inst,
                                                 const double *dk1, const double *dk2, qpm_stream sv,
                                                 qpm_batch *out)
{
    clear_error();
    QPM_REQUIRE(z && offsets && dk1 && dk2 && out, QPM_EINVAL, "z, offsets, dk1, dk2 and out must not be NULL");
    QPM_REQUIRE(n_inst >= 1 && n_inst <= 65535, QPM_EINVAL, "n_inst must be in [1, 65535] (got %d)", (int)n_inst);
    QPM_REQUIRE(offsets[0] == 0, QPM_EINVAL, "offsets[0] must be 0");
    int64_t words = 0, genes = 0;
    for (int32_t b = 0; b < n_inst; ++b) {
        const int64_t n = offsets[b + 1] - offsets[b] - 1;
        QPM_REQUIRE(n >= 1 && n <= (int64_t(1) << 27), QPM_EINVAL,
                    "instance %d: needs 2 .. 2^27 + 1 boundaries (offsets must increase by >= 2)", (int)b);
        QPM_REQUIRE(std::isfinite(dk1[b]) && std::isfinite(dk2[b]), QPM_EINVAL, "instance %d: dk not finite",
                    (int)b);
        for (int64_t k = offsets[b]; k < offsets[b + 1]; ++k)
            QPM_REQUIRE(std::isfinite(z[k]), QPM_EINVAL, "instance %d: z[%lld] not finite", (int)b, (long long)k);
        for (int64_t k = offsets[b]; k + 1 < offsets[b + 1]; ++k)
            QPM_REQUIRE(z[k + 1] > z[k], QPM_EINVAL, "instance %d: z must be strictly increasing", (int)b);
        QPM_REQUIRE(z[offsets[b + 1] - 1] - z[offsets[b]] <= 1e100, QPM_EINVAL,
                    "instance %d: the crystal length must be at most 1e100", (int)b);
        words += words_for(n);
        genes += ((n + 63) / 64) * 64;
    }
    QPM_REQUIRE(words <= (int64_t(1) << 28), QPM_ERANGE, "batch too large (%lld words)", (long long)words);
    qpm_status st = check_device();
    if (st != QPM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(sv);
    auto *bt = new qpm_batch_s();
    bt->n_inst = n_inst;
    bt->total_words = words;
    bt->total_genes_stride = genes;
    int64_t wofs = 0, xofs = 0;
    for (int32_t b = 0; b < n_inst; ++b) {
        InstDesc d{};
        d.n = offsets[b + 1] - offsets[b] - 1;
        d.words = words_for(d.n);
        d.wofs = wofs;
        d.ldx = ((d.n + 63) / 64) * 64;
        d.xofs = xofs;  // in units of rows x ldx: scaled by np at run creation
        wofs += d.words;
        xofs += d.ldx;
        bt->host.push_back(d);
    }
    double *zdev = nullptr;
    hipError_t e = hipMalloc(&bt->ph64, sizeof(double4) * 32 * words);
    if (e == hipSuccess) e = hipMalloc(&bt->ph32, sizeof(float4) * 32 * words);
    if (e == hipSuccess) e = hipMalloc(&bt->c64, sizeof(double2) * 32 * words);
    if (e == hipSuccess) e = hipMalloc(&bt->Cdev, sizeof(double) * 2 * n_inst);
    if (e == hipSuccess) e = hipMalloc(&bt->tab64, sizeof(double2) * 48 * 8 * words);
    if (e == hipSuccess) e = hipMalloc(&bt->tabq, sizeof(int2) * 48 * 8 * words);
    if (e == hipSuccess) e = hipMalloc(&bt->wsc, sizeof(double) * words);
    std::vector<double> wsc(words);
    for (int32_t b = 0; b < n_inst; ++b) word_scales(z + offsets[b], bt->host[b].n, wsc.data() + bt->host[b].wofs);
    if (e == hipSuccess) e = hipMemcpyAsync(bt->wsc, wsc.data(), sizeof(double) * words, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMalloc(&bt->dev, sizeof(InstDesc) * n_inst);
    if (e == hipSuccess) e = hipMalloc(&zdev, sizeof(double) * offsets[n_inst]);
    if (e == hipSuccess) e = hipMemcpyAsync(zdev, z, sizeof(double) * offsets[n_inst], hipMemcpyHostToDevice, s);
    for (int32_t b = 0; b < n_inst && e == hipSuccess; ++b) {
        const InstDesc &d = bt->host[b];
        if (launch_phases(zdev + offsets[b], d.n, dk1[b], dk2[b], bt->ph64 + 32 * d.wofs, bt->ph32 + 32 * d.wofs,
                          bt->c64 + 32 * d.wofs, bt->Cdev + 2 * b, s) != QPM_OK)
            e = hipErrorLaunchFailure;
    }
    if (e == hipSuccess && launch_pattern_tables(bt->ph64, words, bt->wsc, bt->tab64, bt->tabq, s) != QPM_OK)
        e = hipErrorLaunchFailure;
    std::vector<double> C(2 * n_inst);
    if (e == hipSuccess) e = hipMemcpyAsync(C.data(), bt->Cdev, sizeof(double) * 2 * n_inst, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(zdev);
    if (e == hipSuccess) {
        for (int32_t b = 0; b < n_inst; ++b) {
            bt->host[b].C[0] = C[2 * b];
            bt->host[b].C[1] = C[2 * b + 1];
        }
        e = hipMemcpy(bt->dev, bt->host.data(), sizeof(InstDesc) * n_inst, hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        set_error("batched phase precompute failed: %s", hipGetErrorString(e));
        free_batch(bt);
        return e == hipErrorOutOfMemory ? QPM_ENOMEM : QPM_EHIP;
    }
    // the per-call scratch cache (without it every call allocates its own)
    bt->scratch = scratch_cache_create();
    bt->plans.reserve(kEvalPlans);
    *out = bt;
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_free(qpm_batch b)
{
    clear_error();
    if (!b) return QPM_OK;
    (void)hipDeviceSynchronize();
    free_batch(b);
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_info(qpm_batch b, int32_t *n_inst, int64_t *n_domains, double *C)
{
    clear_error();
    QPM_REQUIRE(b != nullptr, QPM_EINVAL, "batch is NULL");
    if (n_inst) *n_inst = b->n_inst;
    for (int32_t i = 0; i < b->n_inst; ++i) {
        if (n_domains) n_domains[i] = b->host[i].n;
        if (C) {
            C[2 * i] = b->host[i].C[0];
            C[2 * i + 1] = b->host[i].C[1];
        }
    }
    return QPM_OK;
}

// ---------------------------------------------------------------- batched fitness

static qpm_status launch_batch_fit(const qpm_batch_s &bt, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                   const BatchFitPlan &pl, size_t nsegs, const FitSeg *segs_dev, double *part,
                                   hipStream_t s, uint32_t *advance = nullptr)
{
    if (pl.gw > 0) {
        const dim3 grid(static_cast<unsigned>((np + 64 * pl.gw - 1) / (64 * pl.gw)),
                        static_cast<unsigned>(nsegs));
        const size_t lds = table_lds_bytes(4 * pl.wpw, p == QPM_PREC_F32, pl.gw, pl.wpw);
        const bool staged = pl.wpw > table_max_wpw(p == QPM_PREC_F32);
#define QPM_BT_KERNEL(F, G, ST)                                                                                    \
    batch_fit_tab_kernel<F, G, ST><<<grid, G * 256, lds, s>>>(bits, ld, bt.tab64, bt.tabq, bt.wsc, pl.wpw, np, bt.dev, \
                                                              segs_dev, part, advance)
#define QPM_BT_CASE(G)                                                                                             \
    case G:                                                                                                        \
        if (p == QPM_PREC_F32) {                                                                                   \
            if (staged)                                                                                            \
                QPM_BT_KERNEL(true, G, true);                                                                      \
            else                                                                                                   \
                QPM_BT_KERNEL(true, G, false);                                                                     \
        } else {                                                                                                   \
            if (staged)                                                                                            \
                QPM_BT_KERNEL(false, G, true);                                                                     \
            else                                                                                                   \
                QPM_BT_KERNEL(false, G, false);                                                                    \
        }                                                                                                          \
        break;
        switch (pl.gw) {
            QPM_BT_CASE(1)
            QPM_BT_CASE(2)
            QPM_BT_CASE(4)
        default: QPM_REQUIRE(false, QPM_EINVAL, "unsupported genome groups per workgroup %d", pl.gw);
        }
#undef QPM_BT_CASE
#undef QPM_BT_KERNEL
        QPM_TRY_HIP(hipGetLastError());
        return QPM_OK;
    }
    const dim3 grid(static_cast<unsigned>((np + 63) / 64), static_cast<unsigned>(nsegs));
#define QPM_BF_CASE(NW)                                                                                           \
    case NW:                                                                                                      \
        if (p == QPM_PREC_F32)                                                                                    \
            batch_fit_kernel<true, NW><<<grid, NW * 64, 0, s>>>(bits, ld, bt.ph64, bt.ph32, pl.wpw, bt.dev,       \
                                                                segs_dev, part, advance);                         \
        else                                                                                                      \
            batch_fit_kernel<false, NW><<<grid, NW * 64, 0, s>>>(bits, ld, bt.ph64, bt.ph32, pl.wpw, bt.dev,      \
                                                                 segs_dev, part, advance);                        \
        break;
    switch (pl.waves) {
        QPM_BF_CASE(4)
        QPM_BF_CASE(8)
        QPM_BF_CASE(16)
    default: QPM_REQUIRE(false, QPM_EINVAL, "unsupported waves per group %d", pl.waves);
    }
#undef QPM_BF_CASE
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

// device copies of a fitness plan's tables
struct FitPlanDev {
    FitSeg *segs = nullptr;
    int *slot_ofs = nullptr;
    double *part = nullptr;
};

static qpm_status upload_fit_plan(const BatchFitPlan &pl, int64_t ld, hipStream_t s, FitPlanDev *out)
{
    FitPlanDev d;
    hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&d.segs), sizeof(FitSeg) * pl.segs.size(), s);
    if (e == hipSuccess)
        e = hipMallocAsync(reinterpret_cast<void **>(&d.slot_ofs), sizeof(int) * pl.slot_ofs.size(), s);
    if (e == hipSuccess)
        e = hipMallocAsync(reinterpret_cast<void **>(&d.part), sizeof(double) * 6 * pl.segs.size() * ld, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(d.segs, pl.segs.data(), sizeof(FitSeg) * pl.segs.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(d.slot_ofs, pl.slot_ofs.data(), sizeof(int) * pl.slot_ofs.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);  // the host vectors must outlive the copies
    if (e != hipSuccess) {
        (void)hipFreeAsync(d.segs, s);
        (void)hipFreeAsync(d.slot_ofs, s);
        (void)hipFreeAsync(d.part, s);
        set_error("fitness plan upload failed: %s", hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? QPM_ENOMEM : QPM_EHIP;
    }
    *out = d;
    return QPM_OK;
}

static void free_fit_plan(FitPlanDev &d, hipStream_t s)
{
    (void)hipFreeAsync(d.segs, s);
    (void)hipFreeAsync(d.slot_ofs, s);
    (void)hipFreeAsync(d.part, s);
    d = FitPlanDev{};
}

static qpm_status launch_batch_combine(const qpm_batch_s &bt, qpm_prec p, const FitPlanDev &fp, int64_t ld,
                                       int64_t np, void *fit, hipStream_t s)
{
    const dim3 grid(static_cast<unsigned>((np + 15) / 16), static_cast<unsigned>(bt.n_inst));
    if (p == QPM_PREC_F64)
        batch_combine_kernel<double><<<grid, 256, 0, s>>>(fp.part, fp.slot_ofs, ld, np, bt.dev,
                                                          static_cast<double *>(fit));
    else
        batch_combine_kernel<float><<<grid, 256, 0, s>>>(fp.part, fp.slot_ofs, ld, np, bt.dev,
                                                         static_cast<float *>(fit));
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

static qpm_status batch_eval_plan(qpm_batch b, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                  void *fitness, const BatchFitPlan &pl, hipStream_t s);

QPM_API qpm_status qpm_batch_eval_fitness(qpm_batch b, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                          void *fitness, int32_t waves_per_group, int32_t words_per_wave,
                                          qpm_stream sv)
{
    clear_error();
    QPM_REQUIRE(b && bits && fitness, QPM_EINVAL, "batch, bits and fitness must not be NULL");
    QPM_REQUIRE(p == QPM_PREC_F32 || p == QPM_PREC_F64, QPM_EINVAL, "unknown precision %d", (int)p);
    QPM_REQUIRE(np >= 1 && np <= (int64_t(1) << 24), QPM_EINVAL, "np out of range (%lld)", (long long)np);
    QPM_REQUIRE(ld >= np && ld % 64 == 0, QPM_EINVAL, "ld (%lld) must be >= np and a multiple of 64", (long long)ld);
    QPM_REQUIRE(waves_per_group == 0 || waves_per_group == 4 || waves_per_group == 8 || waves_per_group == 16,
                QPM_EINVAL, "waves_per_group must be 0 (default), 4, 8 or 16");
    QPM_REQUIRE(words_per_wave >= 0, QPM_EINVAL, "words_per_wave must be >= 0");
    hipStream_t s = static_cast<hipStream_t>(sv);
    BatchFitPlan pl;
    if (waves_per_group == 0 && words_per_wave == 0) {
        int gw, wpw;
        default_tab_shape(np, b->total_words, p == QPM_PREC_F32, &gw, &wpw);
        pl = tab_shape(gw, wpw);
    } else {
        int waves, wpw;
        default_fit_shape(b->host, np, &waves, &wpw);
        if (waves_per_group) waves = waves_per_group;
        if (words_per_wave) wpw = words_per_wave;
        pl.waves = waves;
        pl.wpw = wpw;
    }
    return batch_eval_plan(b, p, bits, np, ld, fitness, pl, s);
}

QPM_API qpm_status qpm_batch_eval_fitness_table(qpm_batch b, qpm_prec p, const uint32_t *bits, int64_t np,
                                                int64_t ld, void *fitness, int32_t groups, int32_t wpw,
                                                qpm_stream sv)
{
    clear_error();
    QPM_REQUIRE(b && bits && fitness, QPM_EINVAL, "batch, bits and fitness must not be NULL");
    QPM_REQUIRE(p == QPM_PREC_F32 || p == QPM_PREC_F64, QPM_EINVAL, "unknown precision %d", (int)p);
    QPM_REQUIRE(np >= 1 && np <= (int64_t(1) << 24), QPM_EINVAL, "np out of range (%lld)", (long long)np);
    QPM_REQUIRE(ld >= np && ld % 64 == 0, QPM_EINVAL, "ld (%lld) must be >= np and a multiple of 64", (long long)ld);
    QPM_REQUIRE(groups == 1 || groups == 2 || groups == 4, QPM_EINVAL,
                "groups_per_workgroup must be 1, 2 or 4 (got %d)", (int)groups);
    QPM_REQUIRE(wpw >= 1 && wpw <= table_max_wpw(p == QPM_PREC_F32), QPM_EINVAL,
                "words_per_wave must be in [1, %d] (got %d)", table_max_wpw(p == QPM_PREC_F32), (int)wpw);
    return batch_eval_plan(b, p, bits, np, ld, fitness, tab_shape(groups, wpw), static_cast<hipStream_t>(sv));
}

// The plan of a shape from the batch's list, uploaded on its first use; false
// (nothing changed) when it is not there and cannot be added: the list is
// full, the stream is being captured, or memory is short.
static bool kept_plan(qpm_batch b, const BatchFitPlan &shape, hipStream_t s, EvalPlan *out)
{
    std::lock_guard<std::mutex> lock(b->plan_mutex);
    for (const EvalPlan &p : b->plans)
        if (p.waves == shape.waves && p.wpw == shape.wpw && p.gw == shape.gw) {
            *out = p;
            return true;
        }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    if (b->plans.size() >= kEvalPlans || hipStreamIsCapturing(s, &cap) != hipSuccess ||
        cap != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return false;
    }
    const BatchFitPlan pl = make_fit_plan(b->host, shape.waves, shape.wpw);
    EvalPlan p;
    p.waves = shape.waves;
    p.wpw = shape.wpw;
    p.gw = shape.gw;
    p.nsegs = pl.segs.size();
    if (p.nsegs > 65535) return false;
    hipError_t e = hipMalloc(&p.segs, sizeof(FitSeg) * pl.segs.size());
    if (e == hipSuccess) e = hipMalloc(&p.slot_ofs, sizeof(int) * pl.slot_ofs.size());
    // on the caller's stream and waited for: the tables are then ready on every stream
    if (e == hipSuccess)
        e = hipMemcpyAsync(p.segs, pl.segs.data(), sizeof(FitSeg) * pl.segs.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(p.slot_ofs, pl.slot_ofs.data(), sizeof(int) * pl.slot_ofs.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(p.segs);
        (void)hipFree(p.slot_ofs);
        (void)hipGetLastError();
        return false;
    }
    b->plans.push_back(p);
    *out = p;
    return true;
}

// An evaluation on the plan of a shape. The plan's tables stay with the batch
// and the partials in its scratch: building, uploading and freeing them per
// call, with a synchronisation, cost about 55 us of a 123 us call (64 designs
// of up to 5 x 10^4 domains, 256 genomes each).
static qpm_status batch_eval_plan(qpm_batch b, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                  void *fitness, const BatchFitPlan &shape, hipStream_t s)
{
    EvalPlan kp;
    if (kept_plan(b, shape, s, &kp)) {
        FitPlanDev fp;
        fp.segs = kp.segs;
        fp.slot_ofs = kp.slot_ofs;
        ScratchLease lease(b->scratch, s);
        void *ws = nullptr;
        qpm_status st = lease.begin(sizeof(double) * 6 * kp.nsegs * static_cast<size_t>(ld), &ws);
        if (st != QPM_OK) return st;
        fp.part = static_cast<double *>(ws);
        st = launch_batch_fit(*b, p, bits, np, ld, shape, kp.nsegs, fp.segs, fp.part, s);
        if (st == QPM_OK) st = launch_batch_combine(*b, p, fp, ld, np, fitness, s);
        const qpm_status se = lease.end();
        return st != QPM_OK ? st : se;
    }
    BatchFitPlan pl = make_fit_plan(b->host, shape.waves, shape.wpw);
    pl.gw = shape.gw;
    QPM_REQUIRE(pl.segs.size() <= 65535, QPM_ERANGE, "too many fitness segments (%zu)", pl.segs.size());
    FitPlanDev fp;
    qpm_status st = upload_fit_plan(pl, ld, s, &fp);
    if (st != QPM_OK) return st;
    st = launch_batch_fit(*b, p, bits, np, ld, pl, pl.segs.size(), fp.segs, fp.part, s);
    if (st == QPM_OK) st = launch_batch_combine(*b, p, fp, ld, np, fitness, s);
    free_fit_plan(fp, s);
    return st;
}

// ---------------------------------------------------------------- the batched run

struct qpm_batch_run_s {
    const qpm_batch_s *bt = nullptr;
    qpm_run_config cfg{};
    hipStream_t st = nullptr;
    int64_t ld = 0;
    float *buf[2] = {nullptr, nullptr};  // one allocation
    size_t gene_bytes = 0;               // of each buffer
    uint32_t *flags = nullptr;
    uint32_t *fbits = nullptr;  // flags packed one bit per individual, 2 ceil(np / 64) words per instance
    void *f_cur = nullptr;
    void *cand_v = nullptr;      // leader candidates, 3 per instance and group of 64
    int32_t *cand_i = nullptr;
    uint32_t *bits = nullptr;
    int32_t *leaders = nullptr;
    int4 *draws = nullptr;
    uint32_t *gen = nullptr;
    float *a_tab = nullptr;
    InstDesc *inst = nullptr;  // instance table with xofs scaled by np
    Tile *gtiles = nullptr;    // (instance, 1024-gene chunk)
    int n_gtiles = 0;
    Tile *dtiles[3] = {nullptr, nullptr, nullptr};  // (instance, DE chunk) for 1, 2, 4 individuals per wave
    int n_dtiles[3] = {0, 0, 0};
    int de_ipw = 1, de_passes = 1;
    // accepted-only trials (as in a single-design run): the DE step writes
    // bits only, the finish lists accepted slots, a kernel recomputes them
    bool lazy = false;
    int32_t *acc_list = nullptr;   // np entries per instance
    uint32_t *acc_cnt = nullptr;   // entries in use per instance
    uint32_t *fbits_prev = nullptr;
    BatchFitPlan fplan;
    FitPlanDev fdev;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int64_t done = 0;
    bool timing = false;
    hipEvent_t ev[QPM_K_COUNT + 1] = {};
    double ms[QPM_K_COUNT] = {};
    int64_t timed = 0;
    double tune_us = 0.0;

    bool f64() const { return cfg.prec == QPM_PREC_F64; }
    BatchPop pop() const { return BatchPop{buf[0], buf[1], buf[0], buf[1], flags, cfg.np}; }
};

static void release_batch_run(qpm_batch_run_s *r)
{
    if (!r) return;
    if (r->st) (void)hipStreamSynchronize(r->st);
    if (r->exec) (void)hipGraphExecDestroy(r->exec);
    if (r->graph) (void)hipGraphDestroy(r->graph);
    (void)hipFree(r->buf[0]);
    (void)hipFree(r->fbits);
    (void)hipFree(r->flags);
    (void)hipFree(r->f_cur);
    (void)hipFree(r->cand_v);
    (void)hipFree(r->cand_i);
    (void)hipFree(r->bits);
    (void)hipFree(r->leaders);
    (void)hipFree(r->draws);
    (void)hipFree(r->acc_list);
    (void)hipFree(r->acc_cnt);
    (void)hipFree(r->fbits_prev);
    (void)hipFree(r->gen);
    (void)hipFree(r->a_tab);
    (void)hipFree(r->inst);
    (void)hipFree(r->gtiles);
    for (auto *t : r->dtiles) (void)hipFree(t);
    if (r->st && r->fdev.segs) {
        free_fit_plan(r->fdev, r->st);
        (void)hipStreamSynchronize(r->st);
    }
    for (auto &e : r->ev)
        if (e) (void)hipEventDestroy(e);
    if (r->st) (void)hipStreamDestroy(r->st);
    delete r;
}

static qpm_status launch_batch_de(qpm_batch_run_s *r, int ipw, int passes)
{
    const qpm_run_config &c = r->cfg;
    const uint32_t k0 = static_cast<uint32_t>(c.seed), k1 = static_cast<uint32_t>(c.seed >> 32);
    const int64_t groups = (c.np + 4 * ipw * passes - 1) / (4 * ipw * passes);
    const Tile *tiles = ipw == 1 ? r->dtiles[0] : (ipw == 2 ? r->dtiles[1] : r->dtiles[2]);
    const int ntiles = ipw == 1 ? r->n_dtiles[0] : (ipw == 2 ? r->n_dtiles[1] : r->n_dtiles[2]);
    const int64_t blocks = 8 * ((ntiles + 7) / 8) * groups;
    QPM_REQUIRE(blocks < (int64_t(1) << 31), QPM_ERANGE, "batch too large for one DE launch");
    const unsigned nb = static_cast<unsigned>(blocks);
    const BatchPop bp = r->pop();
    const int gr = static_cast<int>(groups);
    uint32_t *reset = r->lazy ? r->acc_cnt : nullptr;
    // byte offsets of an instance's rows over both buffers fit 32 bits
    const bool near = 2 * r->gene_bytes < (size_t(1) << 32);
#define QPM_BDE(I, P)                                                                                           \
    {                                                                                                           \
        if (near)                                                                                               \
            batch_de_kernel<I, P, uint32_t><<<nb, 256, 0, r->st>>>(bp, r->inst, tiles, ntiles, gr, r->draws, c.F, \
                                                                   cr_threshold(c.CR), k0, k1, r->gen, c.inst,  \
                                                                   r->bits, r->ld, r->fbits, r->lazy ? 0 : 1, reset, \
                                                                   r->bt->n_inst);  \
        else                                                                                                    \
            batch_de_kernel<I, P, uint64_t><<<nb, 256, 0, r->st>>>(bp, r->inst, tiles, ntiles, gr, r->draws, c.F, \
                                                                   cr_threshold(c.CR), k0, k1, r->gen, c.inst,  \
                                                                   r->bits, r->ld, r->fbits, r->lazy ? 0 : 1, reset, \
                                                                   r->bt->n_inst);  \
    }
    if (ipw == 1) {
        if (passes == 1) QPM_BDE(1, 1) else if (passes == 2) QPM_BDE(1, 2) else QPM_BDE(1, 4)
    } else if (ipw == 2) {
        if (passes == 1) QPM_BDE(2, 1) else if (passes == 2) QPM_BDE(2, 2) else QPM_BDE(2, 4)
    } else {
        if (passes == 1) QPM_BDE(4, 1) else if (passes == 2) QPM_BDE(4, 2) else QPM_BDE(4, 4)
    }
#undef QPM_BDE
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

static qpm_status launch_batch_gwo(qpm_batch_run_s *r)
{
    const qpm_run_config &c = r->cfg;
    const uint32_t k0 = static_cast<uint32_t>(c.seed), k1 = static_cast<uint32_t>(c.seed >> 32);
    const bool rows = r->gene_bytes >= sizeof(float) * kGwoRowsGenes;
    const int64_t group = rows ? 32 : 8, per_xcd = (c.np + group - 1) / group;
    const dim3 grid(static_cast<unsigned>(8 * per_xcd), static_cast<unsigned>(r->n_gtiles));
    if (rows) {
        if (c.gwo_variant == 1)
            batch_gwo_rows_kernel<1, 4><<<grid, 256, 0, r->st>>>(r->pop(), r->inst, r->gtiles, r->leaders, r->a_tab, k0,
                                                                 k1, r->gen, c.inst, r->bits, r->ld,
                                                                 static_cast<int>(per_xcd));
        else
            batch_gwo_rows_kernel<0, 4><<<grid, 256, 0, r->st>>>(r->pop(), r->inst, r->gtiles, r->leaders, r->a_tab, k0,
                                                                 k1, r->gen, c.inst, r->bits, r->ld,
                                                                 static_cast<int>(per_xcd));
    } else if (c.gwo_variant == 1) {
        batch_gwo_kernel<1><<<grid, 256, 0, r->st>>>(r->pop(), r->inst, r->gtiles, r->leaders, r->a_tab, k0, k1, r->gen,
                                                    c.inst, r->bits, r->ld, per_xcd);
    } else {
        batch_gwo_kernel<0><<<grid, 256, 0, r->st>>>(r->pop(), r->inst, r->gtiles, r->leaders, r->a_tab, k0, k1, r->gen,
                                                    c.inst, r->bits, r->ld, per_xcd);
    }
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

// grid of the materialise kernels: list shares x tiles, about 16 workgroups
// per CU
static dim3 materialize_grid(const qpm_batch_run_s *r)
{
    const int64_t shares = std::min<int64_t>(r->cfg.np, std::max<int64_t>(1, 4096 / r->n_gtiles));
    return dim3(static_cast<unsigned>(shares), static_cast<unsigned>(r->n_gtiles));
}

// the evaluated genomes' fitness and their selection (batch_finish_kernel),
// and the leaders (modes 1 and 2) unless the accepted-trial kernel merges them
static qpm_status launch_batch_finish(qpm_batch_run_s *r, int mode, AcceptOut acc = AcceptOut{})
{
    const qpm_run_config &c = r->cfg;
    const uint32_t k0 = static_cast<uint32_t>(c.seed), k1 = static_cast<uint32_t>(c.seed >> 32);
    const int64_t groups = (c.np + 63) / 64;
    const dim3 grid(static_cast<unsigned>(groups), static_cast<unsigned>(r->bt->n_inst));
    const bool leaders = mode == 1 || (mode == 2 && acc.list == nullptr);
#define QPM_BFIN(T)                                                                                              \
    {                                                                                                            \
        batch_finish_kernel<T><<<grid, 1024, 0, r->st>>>(mode, r->fdev.part, r->fdev.slot_ofs, r->ld, c.np,      \
                                                         r->bt->dev, static_cast<T *>(r->f_cur), r->flags,       \
                                                         r->leaders, static_cast<T *>(r->cand_v), r->cand_i,     \
                                                         r->draws, r->gen, k0, k1, c.inst, r->fbits, acc);       \
        if (leaders)                                                                                             \
            batch_leaders_kernel<T><<<r->bt->n_inst, 64, 0, r->st>>>(static_cast<T *>(r->cand_v), r->cand_i,     \
                                                                     groups, r->leaders);                        \
    }
    if (r->f64())
        QPM_BFIN(double)
    else
        QPM_BFIN(float)
#undef QPM_BFIN
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

static qpm_status batch_generation(qpm_batch_run_s *r, hipEvent_t *ev = nullptr)
{
    const qpm_run_config &c = r->cfg;
    const qpm_prec p = static_cast<qpm_prec>(c.prec);
    auto mark = [&](int k) -> qpm_status {
        if (ev) QPM_TRY_HIP(hipEventRecord(ev[k], r->st));
        return QPM_OK;
    };
    qpm_status st;
#define QPM_STEP(k, call)                    \
    if ((st = mark(k)) != QPM_OK) return st; \
    if ((st = (call)) != QPM_OK) return st;
    QPM_STEP(QPM_K_DE, launch_batch_de(r, r->de_ipw, r->de_passes))
    const size_t nsegs = r->fplan.segs.size();
    QPM_STEP(QPM_K_FIT_DE, launch_batch_fit(*r->bt, p, r->bits, c.np, r->ld, r->fplan, nsegs, r->fdev.segs,
                                            r->fdev.part, r->st))
    QPM_STEP(QPM_K_FINISH_DE,
             launch_batch_finish(r, 2, r->lazy ? AcceptOut{r->acc_list, r->acc_cnt, r->fbits_prev} : AcceptOut{}))
    if (r->lazy) {  // the accepted trials' genes (timed with the finish)
        const uint32_t k0 = static_cast<uint32_t>(c.seed), k1 = static_cast<uint32_t>(c.seed >> 32);
        batch_materialize_kernel<<<materialize_grid(r), 256, 0, r->st>>>(r->pop(), r->inst, r->gtiles, r->draws,
                                                                         r->fbits_prev, c.F, cr_threshold(c.CR), k0,
                                                                         k1, r->gen, c.inst, r->acc_list, r->acc_cnt, r->cand_v,
                                                                         r->cand_i, r->f64() ? 1 : 0, r->leaders);
        QPM_TRY_HIP(hipGetLastError());
    }
    QPM_STEP(QPM_K_GWO, launch_batch_gwo(r))
    QPM_STEP(QPM_K_FIT_GWO, launch_batch_fit(*r->bt, p, r->bits, c.np, r->ld, r->fplan, nsegs, r->fdev.segs,
                                             r->fdev.part, r->st, r->gen))
    QPM_STEP(QPM_K_FINISH_GWO, launch_batch_finish(r, 3))
#undef QPM_STEP
    return mark(QPM_K_COUNT);
}

// time the batched table fitness for a few launch shapes on the current
// bits and keep the fastest (results are equal up to the summation order)
static qpm_status tune_fitness(qpm_batch_run_s *r)
{
    const qpm_run_config &c = r->cfg;
    const qpm_prec p = static_cast<qpm_prec>(c.prec);
    const std::string key = tune_key("batchtab", r->bt->total_words, c.np, c.prec, r->bt->n_inst);
    {
        int v0, v1;
        const int maxw = kTabPlanWords;
        if (tune_lookup(key, &v0, &v1, [&](int g, int w) { return (g == 1 || g == 2 || g == 4) && w >= 1 && w <= maxw; })) {
            r->fplan = make_tab_plan(r->bt->host, v0, v1);
            return QPM_OK;
        }
    }
    std::vector<std::pair<int, int>> cands;
    for (int g : {1, 2, 4})
        for (int w = 1; w <= table_max_wpw(p == QPM_PREC_F32); ++w) cands.push_back({g, w});
    for (int g : {2, 4})
        for (int w : {6, 8, 12}) cands.push_back({g, w});
    hipEvent_t e0, e1;
    QPM_TRY_HIP(hipEventCreate(&e0));
    QPM_TRY_HIP(hipEventCreate(&e1));
    float best = 1e30f;
    std::pair<int, int> pick{1, 1};
    default_tab_shape(c.np, r->bt->total_words, p == QPM_PREC_F32, &pick.first, &pick.second);
    for (auto cand : cands) {
        BatchFitPlan pl = make_tab_plan(r->bt->host, cand.first, cand.second);
        if (pl.segs.size() > 65535) continue;
        FitPlanDev fp;
        qpm_status st = upload_fit_plan(pl, r->ld, r->st, &fp);
        if (st != QPM_OK) return st;
        st = launch_batch_fit(*r->bt, p, r->bits, c.np, r->ld, pl, pl.segs.size(), fp.segs, fp.part,
                              r->st);  // warm-up
        float ms = 1e30f;
        for (int rep = 0; rep < 3 && st == QPM_OK; ++rep) {
            QPM_TRY_HIP(hipEventRecord(e0, r->st));
            st = launch_batch_fit(*r->bt, p, r->bits, c.np, r->ld, pl, pl.segs.size(), fp.segs, fp.part, r->st);
            QPM_TRY_HIP(hipEventRecord(e1, r->st));
            QPM_TRY_HIP(hipEventSynchronize(e1));
            float t = 0.0f;
            QPM_TRY_HIP(hipEventElapsedTime(&t, e0, e1));
            ms = std::min(ms, t);
        }
        free_fit_plan(fp, r->st);
        if (st != QPM_OK) return st;
        if (ms < best) {
            best = ms;
            pick = cand;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    QPM_TRY_HIP(hipStreamSynchronize(r->st));
    r->tune_us = best * 1000.0;
    r->fplan = make_tab_plan(r->bt->host, pick.first, pick.second);
    tune_store(key, pick.first, pick.second);
    return QPM_OK;
}

// one generation captured into r->graph / r->exec
static qpm_status capture_batch_generation(qpm_batch_run_s *r)
{
    hipError_t e = hipStreamBeginCapture(r->st, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        set_error("hipStreamBeginCapture failed: %s", hipGetErrorString(e));
        return QPM_EHIP;
    }
    qpm_status st = batch_generation(r);
    e = hipStreamEndCapture(r->st, &r->graph);
    if (st == QPM_OK && e != hipSuccess) {
        set_error("hipStreamEndCapture failed: %s", hipGetErrorString(e));
        st = QPM_EHIP;
    }
    if (st == QPM_OK && hipGraphInstantiate(&r->exec, r->graph, nullptr, nullptr, 0) != hipSuccess) {
        set_error("hipGraphInstantiate failed");
        st = QPM_EHIP;
    }
    return st;
}

// time the batched DE for every (individuals per wave, passes) shape on the
// initial population and keep the fastest (the shape never changes results)
static qpm_status tune_de(qpm_batch_run_s *r)
{
    const qpm_run_config &c = r->cfg;
    const std::string key = tune_key("batchde", r->bt->total_words, c.np, 0, r->bt->n_inst);
    int ipw = 0, passes = 0;
    const auto de_ok = [](int w, int pc) { return (w == 1 || w == 2 || w == 4) && (pc == 1 || pc == 2 || pc == 4); };
    if (!tune_lookup(key, &ipw, &passes, de_ok)) {
        hipEvent_t e0, e1;
        QPM_TRY_HIP(hipEventCreate(&e0));
        QPM_TRY_HIP(hipEventCreate(&e1));
        float best = 1e30f;
        qpm_status st = QPM_OK;
        for (int cand : {1, 2, 4})
            for (int pc : {1, 2, 4}) {
                st = launch_batch_de(r, cand, pc);  // warm-up
                float ms = 1e30f;
                for (int rep = 0; rep < 3 && st == QPM_OK; ++rep) {
                    QPM_TRY_HIP(hipEventRecord(e0, r->st));
                    st = launch_batch_de(r, cand, pc);
                    QPM_TRY_HIP(hipEventRecord(e1, r->st));
                    QPM_TRY_HIP(hipEventSynchronize(e1));
                    float t = 0.0f;
                    QPM_TRY_HIP(hipEventElapsedTime(&t, e0, e1));
                    ms = std::min(ms, t);
                }
                if (st != QPM_OK) break;
                if (ms < best) {
                    best = ms;
                    ipw = cand;
                    passes = pc;
                }
            }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        if (st != QPM_OK) return st;
        tune_store(key, ipw, passes);
    }
    r->de_ipw = ipw;
    r->de_passes = passes;
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_create(qpm_batch b, const qpm_run_config *cfg, int32_t tune, qpm_stream sv,
                                        qpm_batch_run_handle *out)
{
    clear_error();
    QPM_REQUIRE(b && cfg && out, QPM_EINVAL, "batch, cfg and out must not be NULL");
    const qpm_run_config c = *cfg;
    QPM_REQUIRE(c.np >= 4 && c.np <= 4096, QPM_EINVAL, "batched runs need 4 <= np <= 4096 (got %lld)",
                (long long)c.np);
    QPM_REQUIRE(c.generations >= 1 && c.generations <= (int64_t(1) << 31) - 2, QPM_EINVAL, "generations out of range");
    QPM_REQUIRE(c.F >= 0.0f && c.F <= 2.0f, QPM_EINVAL, "F must be in [0, 2]");
    QPM_REQUIRE(c.CR >= 0.0f && c.CR <= 1.0f, QPM_EINVAL, "CR must be in [0, 1]");
    QPM_REQUIRE(c.prec == QPM_PREC_F32 || c.prec == QPM_PREC_F64, QPM_EINVAL, "unknown precision %d", c.prec);
    QPM_REQUIRE(c.gwo_variant == 0 || c.gwo_variant == 1, c.gwo_variant == 2 ? QPM_ENOTSUP : QPM_EINVAL,
                "batched runs take gwo_variant 0 or 1 (got %d)", (int)c.gwo_variant);
    QPM_REQUIRE(c.control == QPM_CONTROL_FIXED, QPM_ENOTSUP, "batched runs use the fixed parameter control only");
    QPM_REQUIRE(c.algo == QPM_ALGO_HWSDA, c.algo == QPM_ALGO_DE || c.algo == QPM_ALGO_GWO ? QPM_ENOTSUP : QPM_EINVAL,
                "batched runs apply the hybrid optimiser only (algo %d)", (int)c.algo);
    QPM_REQUIRE(c.fused == 0 || c.fused == -1, c.fused == 1 ? QPM_ENOTSUP : QPM_EINVAL,
                "batched runs have no fused single-workgroup generations (fused %d)", (int)c.fused);
    QPM_REQUIRE(c.trials == QPM_TRIALS_AUTO || c.trials == QPM_TRIALS_STORE || c.trials == QPM_TRIALS_ACCEPTED,
                QPM_EINVAL, "unknown trial storage %d", c.trials);
    QPM_REQUIRE(static_cast<int64_t>(c.inst) + b->n_inst <= (int64_t(1) << 24), QPM_EINVAL,
                "inst + n_inst must be <= 2^24");
    qpm_status st = check_device();
    if (st != QPM_OK) return st;
    auto *r = new qpm_batch_run_s();
    r->bt = b;
    r->cfg = c;
    r->ld = ((c.np + 63) / 64) * 64;
    const int64_t n_inst = b->n_inst;
    // instance table with gene offsets for np rows per instance
    std::vector<InstDesc> h = b->host;
    int64_t xofs = 0;
    for (auto &d : h) {
        d.xofs = xofs;
        xofs += c.np * d.ldx;
    }
    const size_t gene_bytes = sizeof(float) * static_cast<size_t>(xofs);
    // tiles: GWO / init chunks of 1024 genes; DE chunks of 256 / ipw genes
    // for ipw = 1, 2, 4 (the shape is chosen by the default or the tuner)
    std::vector<Tile> gt, dt[3];
    const int64_t row_bytes = 2 * 1024 * 1024 / c.np;
    r->de_ipw = row_bytes >= 1024 ? 1 : (row_bytes >= 512 ? 2 : 4);
    for (int32_t i = 0; i < b->n_inst; ++i) {
        for (int64_t ch = 0; ch * 1024 < h[i].n; ++ch) gt.push_back(Tile{i, static_cast<int>(ch)});
        for (int v = 0; v < 3; ++v) {
            const int64_t cw = 256 >> v;
            for (int64_t ch = 0; ch * cw < h[i].n; ++ch) dt[v].push_back(Tile{i, static_cast<int>(ch)});
        }
    }
    r->de_passes = de_passes((c.np + 4 * r->de_ipw - 1) / (4 * r->de_ipw) *
                             static_cast<int64_t>(dt[r->de_ipw == 1 ? 0 : (r->de_ipw == 2 ? 1 : 2)].size()));
    // accepted-only trials: recomputing an accepted trial reads 20 B per
    // gene against 4 B per gene for storing every trial, so they pay below
    // about 20 % acceptance and for large populations; chosen automatically,
    // as for single runs, above 64 MB for both gene buffers (the 64-design
    // workload, NP = 256, 1.7 GB: a whole 500-generation run 0.909 s against
    // 0.946 s storing every trial)
    int64_t total_n = 0;
    for (const auto &d : h) total_n += d.n;
    r->lazy = c.trials == QPM_TRIALS_ACCEPTED ||
              (c.trials == QPM_TRIALS_AUTO && 2 * static_cast<int64_t>(sizeof(float)) * c.np * total_n >
                                                  (int64_t(64) << 20));
    if (r->lazy && n_inst * c.np >= (int64_t(1) << 31)) {  // (a limit of the accepted-only trials)
        if (c.trials == QPM_TRIALS_ACCEPTED) {
            set_error("accepted-only trials need n_inst * np < 2^31");
            release_batch_run(r);
            return QPM_EINVAL;
        }
        r->lazy = false;
    }
    if (gt.size() > 65535) {  // the GWO and init grids put these chunks on gridDim.y
        set_error("too many 1024-gene chunks over the batch (%zu > 65535)", gt.size());
        release_batch_run(r);
        return QPM_ERANGE;
    }
    r->n_gtiles = static_cast<int>(gt.size());
    for (int v = 0; v < 3; ++v) r->n_dtiles[v] = static_cast<int>(dt[v].size());
    const int64_t groups = (c.np + 63) / 64;  // of 64 genomes, per instance
    hipError_t e = hipStreamCreateWithFlags(&r->st, hipStreamNonBlocking);
    // both gene buffers in one allocation: row offsets count from the first
    if (e == hipSuccess) e = hipMalloc(&r->buf[0], 2 * gene_bytes);
    if (e == hipSuccess) r->buf[1] = r->buf[0] + xofs;
    r->gene_bytes = gene_bytes;
    if (e == hipSuccess) e = hipMalloc(&r->flags, sizeof(uint32_t) * n_inst * c.np);
    if (e == hipSuccess) e = hipMalloc(&r->fbits, sizeof(uint32_t) * n_inst * 2 * groups);
    if (e == hipSuccess) e = hipMalloc(&r->f_cur, (r->f64() ? 8 : 4) * n_inst * c.np);
    if (e == hipSuccess) e = hipMalloc(&r->cand_v, (r->f64() ? 8 : 4) * 3 * n_inst * groups);
    if (e == hipSuccess) e = hipMalloc(&r->cand_i, sizeof(int32_t) * 3 * n_inst * groups);
    if (e == hipSuccess) e = hipMalloc(&r->bits, sizeof(uint32_t) * b->total_words * r->ld);
    if (e == hipSuccess) e = hipMalloc(&r->leaders, sizeof(int32_t) * 3 * n_inst);
    if (e == hipSuccess) e = hipMalloc(&r->draws, sizeof(int4) * n_inst * c.np);
    if (e == hipSuccess && r->lazy) e = hipMalloc(&r->acc_list, sizeof(int32_t) * n_inst * c.np);
    if (e == hipSuccess && r->lazy) e = hipMalloc(&r->acc_cnt, sizeof(uint32_t) * n_inst);
    if (e == hipSuccess && r->lazy) e = hipMalloc(&r->fbits_prev, sizeof(uint32_t) * n_inst * 2 * groups);
    if (e == hipSuccess) e = hipMalloc(&r->gen, sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc(&r->a_tab, sizeof(float) * c.generations);
    if (e == hipSuccess) e = hipMalloc(&r->inst, sizeof(InstDesc) * n_inst);
    if (e == hipSuccess) e = hipMalloc(&r->gtiles, sizeof(Tile) * gt.size());
    for (int v = 0; v < 3; ++v)
        if (e == hipSuccess) e = hipMalloc(&r->dtiles[v], sizeof(Tile) * dt[v].size());
    if (e != hipSuccess) {
        set_error("batched run allocation failed: %s", hipGetErrorString(e));
        release_batch_run(r);
        return e == hipErrorOutOfMemory ? QPM_ENOMEM : QPM_EHIP;
    }
    std::vector<float> a(c.generations);
    for (int64_t g = 0; g < c.generations; ++g)
        a[g] = static_cast<float>(2.0 * (1.0 - static_cast<double>(g) / static_cast<double>(c.generations)));
    hipEvent_t ev = nullptr;
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(ev, static_cast<hipStream_t>(sv));
    if (e == hipSuccess) e = hipStreamWaitEvent(r->st, ev, 0);
    if (e == hipSuccess)
        e = hipMemcpyAsync(r->a_tab, a.data(), sizeof(float) * c.generations, hipMemcpyHostToDevice, r->st);
    if (e == hipSuccess) e = hipMemcpyAsync(r->inst, h.data(), sizeof(InstDesc) * n_inst, hipMemcpyHostToDevice, r->st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(r->gtiles, gt.data(), sizeof(Tile) * gt.size(), hipMemcpyHostToDevice, r->st);
    for (int v = 0; v < 3; ++v)
        if (e == hipSuccess)
            e = hipMemcpyAsync(r->dtiles[v], dt[v].data(), sizeof(Tile) * dt[v].size(), hipMemcpyHostToDevice,
                               r->st);
    if (e == hipSuccess) e = hipMemsetAsync(r->flags, 0, sizeof(uint32_t) * n_inst * c.np, r->st);
    if (e == hipSuccess) e = hipMemsetAsync(r->fbits, 0, sizeof(uint32_t) * n_inst * 2 * groups, r->st);
    if (e == hipSuccess) e = hipMemsetAsync(r->gen, 0, sizeof(uint32_t), r->st);
    if (e == hipSuccess) e = hipMemsetAsync(r->bits, 0, sizeof(uint32_t) * b->total_words * r->ld, r->st);
    if (e == hipSuccess) e = hipStreamSynchronize(r->st);
    if (ev) (void)hipEventDestroy(ev);
    if (e != hipSuccess) {
        set_error("batched run set-up failed: %s", hipGetErrorString(e));
        release_batch_run(r);
        return QPM_EHIP;
    }
    // step 1: initialise every instance
    {
        const dim3 grid(static_cast<unsigned>(c.np), static_cast<unsigned>(r->n_gtiles));
        batch_init_kernel<<<grid, 256, 0, r->st>>>(c.np, r->inst, r->gtiles, static_cast<uint32_t>(c.seed),
                                                  static_cast<uint32_t>(c.seed >> 32), c.inst, r->buf[0], r->bits,
                                                  r->ld);
        e = hipGetLastError();
        if (e != hipSuccess) {
            set_error("batched init launch failed: %s", hipGetErrorString(e));
            release_batch_run(r);
            return QPM_EHIP;
        }
    }
    if (tune) {
        st = tune_fitness(r);
    } else {
        int gw, wpw;
        default_tab_shape(c.np, b->total_words, c.prec == QPM_PREC_F32, &gw, &wpw);
        r->fplan = make_tab_plan(b->host, gw, wpw);
    }
    if (st == QPM_OK && r->fplan.segs.size() > 65535) {
        set_error("too many fitness segments (%zu)", r->fplan.segs.size());
        st = QPM_ERANGE;
    }
    if (st == QPM_OK) st = upload_fit_plan(r->fplan, r->ld, r->st, &r->fdev);
    const qpm_prec p = static_cast<qpm_prec>(c.prec);
    if (st == QPM_OK)
        st = launch_batch_fit(*b, p, r->bits, c.np, r->ld, r->fplan, r->fplan.segs.size(), r->fdev.segs, r->fdev.part,
                              r->st);
    if (st == QPM_OK) st = launch_batch_finish(r, 1);
    // the DE shape: the trial launches of the tuner write only the other
    // gene buffer and the bit rows, which the first generation overwrites
    if (st == QPM_OK && tune) st = tune_de(r);
    if (st == QPM_OK && c.use_graph) st = capture_batch_generation(r);
    if (st != QPM_OK) {
        release_batch_run(r);
        return st;
    }
    *out = r;
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_set_de_shape(qpm_batch_run_handle r, int32_t individuals_per_wave, int32_t passes)
{
    clear_error();
    QPM_REQUIRE(r != nullptr, QPM_EINVAL, "run is NULL");
    QPM_REQUIRE(individuals_per_wave == 1 || individuals_per_wave == 2 || individuals_per_wave == 4, QPM_EINVAL,
                "individuals_per_wave must be 1, 2 or 4 (got %d)", (int)individuals_per_wave);
    QPM_REQUIRE(passes == 1 || passes == 2 || passes == 4, QPM_EINVAL, "passes must be 1, 2 or 4 (got %d)",
                (int)passes);
    QPM_TRY_HIP(hipStreamSynchronize(r->st));
    r->de_ipw = individuals_per_wave;
    r->de_passes = passes;
    if (r->exec) {
        (void)hipGraphExecDestroy(r->exec);
        (void)hipGraphDestroy(r->graph);
        r->exec = nullptr;
        r->graph = nullptr;
        return capture_batch_generation(r);
    }
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_advance(qpm_batch_run_handle r, int64_t generations)
{
    clear_error();
    QPM_REQUIRE(r != nullptr, QPM_EINVAL, "run is NULL");
    QPM_REQUIRE(generations >= 0 && r->done + generations <= r->cfg.generations, QPM_EINVAL,
                "advancing %lld generations would pass the configured %lld (done %lld)", (long long)generations,
                (long long)r->cfg.generations, (long long)r->done);
    for (int64_t g = 0; g < generations; ++g) {
        if (r->timing) {
            qpm_status st = batch_generation(r, r->ev);
            if (st != QPM_OK) return st;
            QPM_TRY_HIP(hipEventSynchronize(r->ev[QPM_K_COUNT]));
            for (int k = 0; k < QPM_K_COUNT; ++k) {
                float t = 0.0f;
                QPM_TRY_HIP(hipEventElapsedTime(&t, r->ev[k], r->ev[k + 1]));
                r->ms[k] += t;
            }
            ++r->timed;
        } else if (r->exec) {
            QPM_TRY_HIP(hipGraphLaunch(r->exec, r->st));
        } else {
            qpm_status st = batch_generation(r);
            if (st != QPM_OK) return st;
        }
        ++r->done;
    }
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_set_timing(qpm_batch_run_handle r, int32_t enable)
{
    clear_error();
    QPM_REQUIRE(r != nullptr, QPM_EINVAL, "run is NULL");
    if (enable && !r->ev[0])
        for (auto &e : r->ev) QPM_TRY_HIP(hipEventCreate(&e));
    r->timing = enable != 0;
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_timing(qpm_batch_run_handle r, double *ms, int64_t *generations, int32_t reset)
{
    clear_error();
    QPM_REQUIRE(r != nullptr, QPM_EINVAL, "run is NULL");
    if (ms)
        for (int k = 0; k < QPM_K_COUNT; ++k) ms[k] = r->ms[k];
    if (generations) *generations = r->timed;
    if (reset) {
        for (double &v : r->ms) v = 0.0;
        r->timed = 0;
    }
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_read(qpm_batch_run_handle r, int32_t inst, float *x, int64_t ldx, void *fitness,
                                      int32_t *leaders, int32_t *fit_shape)
{
    clear_error();
    QPM_REQUIRE(r != nullptr, QPM_EINVAL, "run is NULL");
    QPM_REQUIRE(inst >= 0 && inst < r->bt->n_inst, QPM_EINVAL, "instance %d out of range", (int)inst);
    const InstDesc &d = r->bt->host[inst];
    if (x) {
        QPM_REQUIRE(ldx >= d.n, QPM_EINVAL, "ldx (%lld) must be >= the instance's N (%lld)", (long long)ldx,
                    (long long)d.n);
        const int64_t blocks = (d.n + 255) / 256;
        batch_gather_kernel<<<dim3(static_cast<unsigned>(blocks < 64 ? blocks : 64),
                                   static_cast<unsigned>(r->cfg.np)),
                              256, 0, r->st>>>(r->pop(), r->inst, inst, x, ldx);
        QPM_TRY_HIP(hipGetLastError());
    }
    const size_t es = r->f64() ? sizeof(double) : sizeof(float);
    if (fitness)
        QPM_TRY_HIP(hipMemcpyAsync(fitness, static_cast<char *>(r->f_cur) + es * r->cfg.np * inst, es * r->cfg.np,
                                   hipMemcpyDeviceToDevice, r->st));
    if (leaders)
        QPM_TRY_HIP(hipMemcpyAsync(leaders, r->leaders + 3 * inst, sizeof(int32_t) * 3, hipMemcpyDeviceToHost, r->st));
    QPM_TRY_HIP(hipStreamSynchronize(r->st));
    if (fit_shape) {
        fit_shape[0] = r->fplan.waves;
        fit_shape[1] = r->fplan.wpw;
    }
    return QPM_OK;
}

QPM_API qpm_status qpm_batch_run_destroy(qpm_batch_run_handle r)
{
    clear_error();
    release_batch_run(r);
    return QPM_OK;
}
