// objective.hip -- the multi-wavelength objective (the paper's
// multi-wavelength second-harmonic and coupled third-harmonic designs, its
// last section): K designs on one set of boundaries, one per wavelength,
// G_k = |sum d a| / L (SHG) or |d_eff| / L^2 (THG), and the paper's
// objective h = sum_k |G0 - G_k| + beta (max G - min G), maximised as -h.
//
// One bit stream serves the K designs: a workgroup (4 segment waves over
// one group of 64 genomes) loads its genomes' bit words into registers once,
// then for each design copies that design's sign-pattern tables of the
// workgroup's words to LDS and walks the words again from registers. SHG
// needs only the A row of each table (sum d a of a 4-domain block), THG
// the whole (A, B, Q) triple.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "device_common.hpp"
#include "scan.hpp"
#include "select.hpp"

namespace qpm {

namespace {

// table rows per 4-domain block (A only, or A, B, Q) and components of a
// segment partial
template <bool THG>
struct ObjShape {
    static constexpr int R = THG ? 3 : 1;
    static constexpr int NC = THG ? 6 : 2;
};

constexpr int kSegWaves = 4;

// LDS of the partials kernel: one design's tables, which the fold reuses; or
// those of two designs and two folds
template <bool F32, bool THG>
size_t obj_lds_bytes(int wpw, bool twice)
{
    const size_t tables = static_cast<size_t>(kSegWaves) * wpw * 8 * ObjShape<THG>::R * 16 * (F32 ? 8 : 16);
    const size_t fold = static_cast<size_t>(ObjShape<THG>::NC) * kSegWaves * 64 * sizeof(double);
    return twice ? 2 * (tables + fold) : (tables > fold ? tables : fold);
}

// where a grid of one segment writes its values itself (DIRECT)
struct ObjOut {
    double scale, G0, beta;
    void *fit;
    int f64;
    double *G;
    int64_t ldG;
    int gk_at;  // LDS offset of the G_k
};
struct ObjNoOut {};
template <bool DIRECT>
using ObjOutArg = std::conditional_t<DIRECT, ObjOut, ObjNoOut>;

// -(sum_k |G0 - G_k| + beta (max G - min G)) from gk[k stride]
__device__ __forceinline__ double obj_h(const double *gk, int stride, int K, double G0, double beta)
{
    double sum = 0.0, gmax = 0.0, gmin = 0.0;
    for (int k = 0; k < K; ++k) {
        const double Gk = gk[k * stride];
        sum += fabs(G0 - Gk);
        gmax = k == 0 ? Gk : fmax(gmax, Gk);
        gmin = k == 0 ? Gk : fmin(gmin, Gk);
    }
    return -(sum + beta * (gmax - gmin));
}

}  // namespace

// Grid: x = genome groups of 64, y = workgroup segments of 4 wpw words.
// part[(k gy + y) NC + c][ld] + i: the segment's (A, B, Q) (THG) or A (SHG)
// of design k for genome i, the 4 segment waves folded in order.
// TWICE: the tables of design k + 1 arrive in the other half of LDS while
// design k is walked, and its fold waits for the barrier that they need anyway
// (one per design instead of four), by a wave that changes from design to design.
// A workgroup's time is mostly these waits: 3000 x 5000, 5 SHG wavelengths FP32,
// 11.0 -> 9.7 us (4 words per wave).
// DIRECT (grids of one segment): the fold takes G_k, and the objective follows
// here instead of in a second launch; the G_k stand behind the other LDS.
template <bool F32, bool THG, bool TWICE, bool DIRECT>
__global__ __launch_bounds__(256) void obj_partials_kernel(ObjTabs tabs, int K, const uint32_t *__restrict__ bits,
                                                           int64_t ld, int W, int wpw, int gy, int64_t np,
                                                           double *__restrict__ part, uint32_t *__restrict__ advance,
                                                           ObjOutArg<DIRECT> out)
{
    if (advance != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) advance[0] += 1u;
    constexpr int R = ObjShape<THG>::R;
    constexpr int NC = ObjShape<THG>::NC;
    constexpr int ES = F32 ? 8 : 16;        // bytes per table entry (complex)
    constexpr int PPR = 16 * ES / 16;       // 16-byte pieces per block row of 16 entries
    constexpr int MAXW = table_max_wpw(F32);
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    const int wbase = static_cast<int>(blockIdx.y) * kSegWaves * wpw;
    const int nw = min(W - wbase, kSegWaves * wpw);  // >= 1 by the grid
    const bool live = i < np;
    const int w0 = wave * wpw, w1 = min(nw, w0 + wpw);
    const int64_t ic = i < ld ? i : ld - 1;
    const int n16 = nw * 8 * R * PPR;
    const int half = TWICE ? kSegWaves * wpw * 8 * R * 16 * ES : 0;  // bytes of one design's tables
    // design kd's table rows of words [wbase, wbase + nw) into LDS:
    // piece idx = ((word 8 + block) R + row) PPR + q
    auto issue = [&](int kd) {
        const unsigned char *src = F32 ? reinterpret_cast<const unsigned char *>(tabs.tq[kd])
                                       : reinterpret_cast<const unsigned char *>(tabs.t64[kd]);
        unsigned char *const to = lds + (kd & 1) * half;
        for (int r0 = 0; r0 * 256 < n16; ++r0) {
            const int idx = r0 * 256 + static_cast<int>(threadIdx.x);
            if (idx < n16) {
                const int q = idx % PPR, row = (idx / PPR) % R, blk = idx / (PPR * R);  // blk = word 8 + block
                const int64_t off =
                    ((static_cast<int64_t>(wbase) * 8 + blk) * 48 + row * 16) * ES + static_cast<int64_t>(q) * 16;
                __builtin_amdgcn_global_load_lds(
                    reinterpret_cast<const uint4 *>(src + off),
                    reinterpret_cast<__attribute__((address_space(3))) void *>(
                        reinterpret_cast<uintptr_t>(to + static_cast<size_t>(r0 * 256 + wave * 64) * 16)),
                    16, 0, 0);
            }
        }
    };
    // design kd's 4 segment waves in order, from LDS, by one wave
    auto fold = [&](int kd, const double *sh) {  // sh: [NC][4][64]
        if (!live) return;
        auto at = [&](int c, int s2) { return c < NC ? sh[(c * kSegWaves + s2) * 64 + lane] : 0.0; };
        Tri t{at(0, 0), at(1, 0), at(2, 0), at(3, 0), at(4, 0), at(5, 0)};
        for (int s2 = 1; s2 < kSegWaves; ++s2) {
            if (s2 * wpw >= nw) break;
            if constexpr (THG) {
                tri_append(t, Tri{at(0, s2), at(1, s2), at(2, s2), at(3, s2), at(4, s2), at(5, s2)});
            } else {
                t.ar += at(0, s2);
                t.ai += at(1, s2);
            }
        }
        if constexpr (DIRECT) {
            const double re = THG ? t.qr + tabs.C[kd][0] : t.ar, im = THG ? t.qi + tabs.C[kd][1] : t.ai;
            const double Gk = sqrt(fma(re, re, im * im)) * out.scale;
            reinterpret_cast<double *>(lds + out.gk_at)[kd * 64 + lane] = Gk;
            if (out.G) out.G[kd * out.ldG + i] = Gk;
        } else {
            double *p = part + ((static_cast<int64_t>(kd) * gy + blockIdx.y) * NC) * ld + i;
            const double comp[6] = {t.ar, t.ai, t.br, t.bi, t.qr, t.qi};
#pragma unroll
            for (int c = 0; c < NC; ++c) p[c * ld] = comp[c];
        }
    };
    issue(0);
    // the bit words of this wave's segment, loaded once for all K designs
    uint32_t wv[MAXW];
#pragma unroll
    for (int k = 0; k < MAXW; ++k) wv[k] = bits[static_cast<int64_t>(min(wbase + w0 + k, W - 1)) * ld + ic];
    for (int kd = 0; kd < K; ++kd) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        double *const folds = reinterpret_cast<double *>(lds + 2 * half);
        constexpr int kFold = NC * kSegWaves * 64;
        if constexpr (TWICE) {
            if (kd + 1 < K) issue(kd + 1);
            if (kd > 0 && wave == (kd - 1) % kSegWaves) fold(kd - 1, folds + ((kd - 1) & 1) * kFold);
        }
        const unsigned char *const from = lds + (kd & 1) * half;
        Tri t{0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < MAXW; ++k) {
            const int wr = w0 + k;
            if (wr >= w1) break;
            const uint32_t word = live ? wv[k] : 0u;
            if constexpr (F32) {
                word_tab_q<R>(t, word, reinterpret_cast<const int2 *>(from) + wr * 8 * R * 16,
                              tabs.wsc[kd][wbase + wr]);
            } else {
                const double2 *tb = reinterpret_cast<const double2 *>(from) + wr * 8 * R * 16;
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    const uint32_t pt = (word >> (4 * h)) & 15u;
                    const double2 A = tb[(h * R) * 16 + pt];
                    if constexpr (THG) {
                        const double2 B = tb[(h * R + 1) * 16 + pt], Q = tb[(h * R + 2) * 16 + pt];
                        t.qr = fma(-t.ai, B.y, fma(t.ar, B.x, t.qr + Q.x));
                        t.qi = fma(t.ai, B.x, fma(t.ar, B.y, t.qi + Q.y));
                        t.br += B.x;
                        t.bi += B.y;
                    }
                    t.ar += A.x;
                    t.ai += A.y;
                }
            }
        }
        if constexpr (!TWICE) __syncthreads();  // the fold takes the tables' place
        double *sh = TWICE ? folds + (kd & 1) * kFold : reinterpret_cast<double *>(lds);
        const double comp[6] = {t.ar, t.ai, t.br, t.bi, t.qr, t.qi};
#pragma unroll
        for (int c = 0; c < NC; ++c) sh[(c * kSegWaves + wave) * 64 + lane] = comp[c];
        if constexpr (!TWICE) {
            __syncthreads();
            if (wave == 0) fold(kd, sh);
            if (kd + 1 < K) {
                __syncthreads();
                issue(kd + 1);
            }
        } else if (kd + 1 == K) {
            __syncthreads();
            if (wave == kd % kSegWaves) fold(kd, sh);
        }
    }
    if constexpr (DIRECT) {
        __syncthreads();
        if (wave != 0 || !live) return;
        const double h = obj_h(reinterpret_cast<const double *>(lds + out.gk_at) + lane, 64, K, out.G0, out.beta);
        if (out.f64)
            static_cast<double *>(out.fit)[i] = h;
        else
            static_cast<float *>(out.fit)[i] = static_cast<float>(h);
    }
}

// -h of the NG genomes of a workgroup from the K designs' segment partials,
// for a workgroup of 256 threads or more (a multiple of NG). The segments of a
// design are split in NR ranges (combine_ranges) folded in order by one thread
// each; the (design, range) pairs of a genome are spread over the workgroup's threads, so
// their loads overlap (one design after the other, with 64 genomes per
// workgroup, took 12.6 us for 24 segments of 5 SHG designs at NP = 5000 and
// 37.7 us for 104 segments at NP = 1500, against 6.4 and 23.4 us), in batches
// of kb designs (kb NC NR NG doubles of LDS);
// then one thread per genome and design folds the ranges in order, and one
// per genome takes the objective. Valid in the first NG threads (gl =
// threadIdx.x). G (optional): G_k at G[k ldG + i]. sh: kb NR NC NG doubles, gk: K
// NG doubles. (With 4 ranges whatever the segments, one design of 78 segments
// took 10.9 us.)
template <bool THG, int NG, int NR>
__device__ double obj_value(const ObjTabs &tabs, int K, int kb, double scale, double G0, double beta,
                            const double *__restrict__ part, int gy, int64_t ld, int64_t i, bool valid, double *G,
                            int64_t ldG, double *sh, double *gk)
{
    constexpr int NC = ObjShape<THG>::NC;
    const int gl = static_cast<int>(threadIdx.x) % NG, slot = static_cast<int>(threadIdx.x) / NG;
    const int slots = static_cast<int>(blockDim.x) / NG;
    for (int k0 = 0; k0 < K; k0 += kb) {
        const int kn = min(kb, K - k0);
        for (int task = slot; task < NR * kn; task += slots) {
            const int kd = task / NR, r = task % NR;
            const int s0 = static_cast<int>((static_cast<int64_t>(gy) * r) / NR);
            const int s1 = static_cast<int>((static_cast<int64_t>(gy) * (r + 1)) / NR);
            const double *pk = part + static_cast<int64_t>(k0 + kd) * gy * NC * ld + i;
            double v[NC] = {};
            if (valid) {
                if constexpr (THG) {
                    Tri t{0, 0, 0, 0, 0, 0};
                    fold_segments<4>(t, pk - i, ld, i, s0, s1);
                    v[0] = t.ar;
                    v[1] = t.ai;
                    v[2] = t.br;
                    v[3] = t.bi;
                    v[4] = t.qr;
                    v[5] = t.qi;
                } else {
                    constexpr int U = NR == 4 ? 4 : 8;  // (in flight together, as in fold_segments)
                    for (int sg = s0; sg < s1; sg += U) {
                        double re[U], im[U];
#pragma unroll
                        for (int k = 0; k < U; ++k) {
                            const double *q = pk + static_cast<int64_t>(min(sg + k, s1 - 1)) * 2 * ld;
                            re[k] = q[0];
                            im[k] = q[ld];
                        }
#pragma unroll
                        for (int k = 0; k < U; ++k) {
                            if (sg + k < s1) {
                                v[0] += re[k];
                                v[1] += im[k];
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) sh[((kd * NC + c) * NR + r) * NG + gl] = v[c];
        }
        __syncthreads();
        for (int kd = slot; kd < kn; kd += slots) {
            auto at = [&](int c, int r) -> double { return sh[((kd * NC + c) * NR + r) * NG + gl]; };
            double re, im;
            if constexpr (THG) {
                Tri t{at(0, 0), at(1, 0), at(2, 0), at(3, 0), at(4, 0), at(5, 0)};
#pragma unroll
                for (int r = 1; r < NR; ++r)
                    tri_append(t, Tri{at(0, r), at(1, r), at(2, r), at(3, r), at(4, r), at(5, r)});
                re = t.qr + tabs.C[k0 + kd][0];
                im = t.qi + tabs.C[k0 + kd][1];
            } else {
                re = at(0, 0);
                im = at(1, 0);
#pragma unroll
                for (int r = 1; r < NR; ++r) {
                    re += at(0, r);
                    im += at(1, r);
                }
            }
            const double Gk = sqrt(fma(re, re, im * im)) * scale;
            gk[(k0 + kd) * NG + gl] = Gk;
            if (G && valid) G[(k0 + kd) * ldG + i] = Gk;
        }
        __syncthreads();
    }
    return slot == 0 ? obj_h(gk + gl, NG, K, G0, beta) : 0.0;
}

// designs folded together by obj_value, and its LDS
template <bool THG, int NG>
int obj_value_batch(int K, int gy)
{
    const int per = ObjShape<THG>::NC * combine_ranges(gy) * NG * static_cast<int>(sizeof(double));
    return std::min(K, std::max(1, (48 << 10) / per));
}
template <bool THG, int NG>
size_t obj_value_lds(int K, int gy)
{
    return sizeof(double) * NG *
           (static_cast<size_t>(ObjShape<THG>::NC) * combine_ranges(gy) * obj_value_batch<THG, NG>(K, gy) +
            static_cast<size_t>(K));
}

// 16 genomes per workgroup (a 128-byte line of each component) x 16 slots
constexpr int kObjGenomes = 16;
template <typename T, bool THG, int NR>
__global__ __launch_bounds__(256) void obj_values_kernel(ObjTabs tabs, int K, int kb, double scale, double G0,
                                                         double beta, const double *__restrict__ part, int gy,
                                                         int64_t ld, int64_t np, T *__restrict__ fit,
                                                         double *__restrict__ G, int64_t ldG)
{
    extern __shared__ double osh[];
    constexpr int NG = kObjGenomes;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * NG + threadIdx.x % NG;
    const bool valid = i < np;
    const double v = obj_value<THG, NG, NR>(tabs, K, kb, scale, G0, beta, part, gy, ld, i, valid, G, ldG, osh,
                                            osh + ObjShape<THG>::NC * NR * kb * NG);
    if (threadIdx.x < NG && valid) fit[i] = static_cast<T>(v);
}

// the run's finish step on the objective: as finish_kernel, with the
// fitness -h (64 genomes x 16 slots)
template <typename T, bool THG, int NR>
__global__ __launch_bounds__(1024) void obj_finish_kernel(ObjTabs tabs, int K, int kb, double scale, double G0,
                                                          double beta, const double *__restrict__ part, int gy,
                                                          int64_t ld, int64_t np, T *__restrict__ f_cur,
                                                          uint32_t *__restrict__ flags, uint32_t *__restrict__ fbits,
                                                          const int32_t *__restrict__ skip3, T *__restrict__ cand_v,
                                                          int32_t *__restrict__ cand_i, int4 *__restrict__ draws_next,
                                                          const uint32_t *__restrict__ gen, int64_t D, uint32_t k0,
                                                          uint32_t k1, uint32_t inst, AcceptOut acc, uint32_t next_off,
                                                          int replace_all)
{
    extern __shared__ double osh[];
    const int lane = threadIdx.x & 63;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    const double v = obj_value<THG, 64, NR>(tabs, K, kb, scale, G0, beta, part, gy, ld, i, i < np, nullptr, 0, osh,
                                            osh + ObjShape<THG>::NC * NR * kb * 64);
    if (threadIdx.x < 64)
        select_group<T>(v, blockIdx.x, lane, np, f_cur, flags, fbits, skip3, cand_v, cand_i, draws_next, gen, D, k0,
                        k1, inst, acc, next_off, replace_all != 0);
}

ObjPlan plan_objective_shape(const Objective &o, int wpw)
{
    ObjPlan pl;
    pl.wpw = wpw;
    pl.gy = static_cast<int>((o.words + 4 * pl.wpw - 1) / (4 * pl.wpw));
    return pl;
}

ObjPlan plan_objective(const Objective &o, qpm_prec p, int64_t np)
{
    // the most words per wave (fewest partials to write and fold) that still
    // leaves 400 workgroups, or 256 for 2 words, at most the register limit of
    // the word cache. Partials + values, us, by words per wave: 3000 x 5000, 5
    // SHG wavelengths FP32: 1 13.1 + 5.9, 2 10.4 + 4.4, 4 9.7 + 3.8, 5 10.6 +
    // 4.4; 13200 x 1500: 1 15.4 + 8.5, 2 12.7 + 8.2, 5 11.2 + 4.4 (THG, 3
    // designs: 1 18.3 + 9.6, 2 17.4 + 6.4, 5 19.4 + 4.0); 6000 x 1000 THG, 2
    // designs: 1 7.6 + 8.3, 2 8.1 + 4.6, 3 8.9 + 4.0; 1000 x 300: 1 4.9 + 3.2, 2
    // 5.4 + 2.9. Where 1 word would leave the longest folds (48 segments), several
    // designs take at least 2, and 3 where they are copied two at a time: 9000 x
    // 300, 5 SHG wavelengths FP32 1 6.3 + 8.9, 2 6.6 + 6.3, 3 7.2 + 5.2, 4 7.8 +
    // 5.0, FP64 1 6.8 + 8.7, 2 7.4 + 6.2; 12000 x 140, 3 THG designs FP32 1 7.4 +
    // 9.4, 2 8.9 + 5.7, 3 10.6 + 4.4; but one THG design, 9894 x 89: 1 4.2 + 5.1, 2
    // 4.9 + 5.2.
    const bool f32 = p == QPM_PREC_F32;
    const int64_t groups = (np + 63) / 64;
    const bool folds = o.K > 1 && combine_ranges(static_cast<int>((o.words + 3) / 4)) == kMaxRanges;
    const int least = !folds ? 1 : (f32 && o.kind != QPM_OBJ_THG ? 3 : 2);
    int wpw = table_max_wpw(f32);
    while (wpw > least && groups * ((o.words + 4 * wpw - 1) / (4 * wpw)) < (wpw > 2 ? 400 : 256)) --wpw;
    while (wpw < table_max_wpw(f32) && (o.words + 4 * wpw - 1) / (4 * wpw) > 65535) ++wpw;
    return plan_objective_shape(o, wpw);
}

size_t objective_partials_bytes(const Objective &o, const ObjPlan &pl, int64_t ld)
{
    const int nc = o.kind == QPM_OBJ_THG ? 6 : 2;
    return sizeof(double) * static_cast<size_t>(o.K) * pl.gy * nc * static_cast<size_t>(ld);
}

template <bool DIRECT>
static qpm_status launch_partials(const Objective &o, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                  const ObjPlan &pl, double *part, hipStream_t s, uint32_t *advance,
                                  ObjOutArg<DIRECT> out)
{
    QPM_REQUIRE(pl.gy <= 65535, QPM_ERANGE, "too many workgroup segments (%d)", pl.gy);
    const dim3 grid(static_cast<unsigned>((np + 63) / 64), static_cast<unsigned>(pl.gy));
    const int W = static_cast<int>(o.words);
    const bool f32 = p == QPM_PREC_F32, thg = o.kind == QPM_OBJ_THG;
    // two designs at a time where three workgroups per CU hold the whole grid
    // (their LDS leaves no more); beyond that and in FP64 and THG, whose tables
    // are 2 to 6 times as large, more workgroups hide more than the copies. us,
    // one / two at a time: 3000 x 5000, 5 wavelengths (474 workgroups of 4 words)
    // 11.0 / 9.7, 12000 x 80, 2 (32 of 3) 5.2 / 4.6, 3000 x 2000, 8 (384 of 2) 11.6
    // / 10.0; 20000 x 3000, 3 (1504 of 5) 13.8 / 16.2, 3000 x 50000, 2 19.2 / 25.5;
    // FP64 13200 x 1500, 5 12.2 / 16.8.
    const bool twice = f32 && !thg && o.K > 1 && static_cast<int64_t>(grid.x) * grid.y <= 768;
#define QPM_OP(F, H, T2)                                                                                          \
    do {                                                                                                          \
        const size_t lds = obj_lds_bytes<F, H>(pl.wpw, T2);                                                       \
        if constexpr (DIRECT) out.gk_at = static_cast<int>(lds);                                                  \
        obj_partials_kernel<F, H, T2, DIRECT><<<grid, 256, lds + (DIRECT ? o.K * 512 : 0), s>>>(                  \
            o.tabs, o.K, bits, ld, W, pl.wpw, pl.gy, np, part, advance, out);                                     \
    } while (0)
    if (f32 && thg)
        QPM_OP(true, true, false);
    else if (twice)
        QPM_OP(true, false, true);
    else if (f32)
        QPM_OP(true, false, false);
    else if (thg)
        QPM_OP(false, true, false);
    else
        QPM_OP(false, false, false);
#undef QPM_OP
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_objective_partials(const Objective &o, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                     const ObjPlan &pl, double *part, hipStream_t s, uint32_t *advance)
{
    return launch_partials<false>(o, p, bits, np, ld, pl, part, s, advance, ObjNoOut{});
}

qpm_status launch_objective_values(const Objective &o, const ObjPlan &pl, const double *part, int64_t ld, int64_t np,
                                   void *fitness, bool f64, double *G, int64_t ldG, hipStream_t s)
{
    const unsigned blocks = static_cast<unsigned>((np + kObjGenomes - 1) / kObjGenomes);
    const bool thg = o.kind == QPM_OBJ_THG;
    const bool many = combine_ranges(pl.gy) == kMaxRanges;
#define QPM_OV(T, H, N)                                                                                          \
    obj_values_kernel<T, H, N><<<blocks, 256, obj_value_lds<H, kObjGenomes>(o.K, pl.gy), s>>>(                   \
        o.tabs, o.K, obj_value_batch<H, kObjGenomes>(o.K, pl.gy), o.scale, o.G0, o.beta, part, pl.gy, ld, np,    \
        static_cast<T *>(fitness), G, ldG)
#define QPM_OV_N(T, H)                                                                                           \
    if (many)                                                                                                    \
        QPM_OV(T, H, kMaxRanges);                                                                                \
    else                                                                                                         \
        QPM_OV(T, H, 4);
    if (f64 && thg) {
        QPM_OV_N(double, true)
    } else if (f64) {
        QPM_OV_N(double, false)
    } else if (thg) {
        QPM_OV_N(float, true)
    } else {
        QPM_OV_N(float, false)
    }
#undef QPM_OV_N
#undef QPM_OV
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

qpm_status launch_objective_finish(const Objective &o, const ObjPlan &pl, const double *part, int64_t ld, int64_t np,
                                   void *f_cur, bool f64, uint32_t *flags, uint32_t *fbits, const int32_t *skip3,
                                   int32_t *top3_out, void *cand, int4 *draws_next, uint32_t *gen, int64_t D,
                                   uint64_t seed, uint32_t inst, hipStream_t s, AcceptOut acc, FinishMode mode)
{
    const unsigned blocks = static_cast<unsigned>((np + 63) / 64);
    QPM_REQUIRE(top3_out == nullptr || cand != nullptr, QPM_EINVAL, "leader candidates need a buffer");
    const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
    const int advance = draws_next != nullptr && !mode.gen_advanced;
    const uint32_t next_off = mode.gen_advanced ? 0u : 1u;
    const bool tail = (top3_out != nullptr && !mode.defer_leaders) || advance;
    int32_t *tail_top3 = mode.defer_leaders ? nullptr : top3_out;
    const bool thg = o.kind == QPM_OBJ_THG;
    const bool many = combine_ranges(pl.gy) == kMaxRanges;
    // cand: 3 values per workgroup (T) followed by 3 slots per workgroup
#define QPM_OF(T, H, N)                                                                                          \
    obj_finish_kernel<T, H, N><<<blocks, 1024, obj_value_lds<H, 64>(o.K, pl.gy), s>>>(                           \
        o.tabs, o.K, obj_value_batch<H, 64>(o.K, pl.gy), o.scale, o.G0, o.beta, part, pl.gy, ld, np,             \
        static_cast<T *>(f_cur), flags, fbits, skip3, cv, ci, draws_next, gen, D, k0, k1, inst, acc, next_off,   \
        mode.replace_all ? 1 : 0)
#define QPM_OF_N(T, H)                                                                                           \
    {                                                                                                            \
        T *cv = top3_out ? static_cast<T *>(cand) : nullptr;                                                     \
        int32_t *ci = cv ? reinterpret_cast<int32_t *>(cv + 3 * static_cast<size_t>(blocks)) : nullptr;         \
        if (many)                                                                                                \
            QPM_OF(T, H, kMaxRanges);                                                                            \
        else                                                                                                     \
            QPM_OF(T, H, 4);                                                                                     \
        if (tail) finish_tail_kernel<T><<<1, 256, 0, s>>>(cv, ci, blocks, tail_top3, gen, advance);              \
    }
    if (f64 && thg)
        QPM_OF_N(double, true)
    else if (f64)
        QPM_OF_N(double, false)
    else if (thg)
        QPM_OF_N(float, true)
    else
        QPM_OF_N(float, false)
#undef QPM_OF_N
#undef QPM_OF
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

}  // namespace qpm

using namespace qpm;

QPM_API qpm_status qpm_objective_create(const qpm_design *designs, int32_t K, int32_t kind, double G0, double beta,
                                        qpm_objective *out)
{
    clear_error();
    QPM_REQUIRE(designs != nullptr && out != nullptr, QPM_EINVAL, "designs and out must not be NULL");
    QPM_REQUIRE(K >= 1 && K <= kMaxObjectiveDesigns, QPM_EINVAL, "K must be in [1, %d] (got %d)",
                kMaxObjectiveDesigns, (int)K);
    QPM_REQUIRE(kind == QPM_OBJ_SHG || kind == QPM_OBJ_THG, QPM_EINVAL, "unknown objective kind %d", (int)kind);
    QPM_REQUIRE(std::isfinite(G0) && std::isfinite(beta), QPM_EINVAL, "G0 and beta must be finite");
    for (int k = 0; k < K; ++k) QPM_REQUIRE(designs[k] != nullptr, QPM_EINVAL, "design %d is NULL", k);
    const Design *d0 = designs[0];
    for (int k = 1; k < K; ++k) {
        const Design *dk = designs[k];
        QPM_REQUIRE(dk->n == d0->n && dk->z0 == d0->z0 && dk->zN == d0->zN && dk->zhash == d0->zhash, QPM_EINVAL,
                    "design %d has other boundaries than design 0", k);
        QPM_REQUIRE(dk->device == d0->device, QPM_EINVAL, "design %d lives on another device", k);
    }
    const double L = d0->zN - d0->z0;
    auto *o = new qpm_objective_s();
    o->K = K;
    o->kind = kind;
    o->G0 = G0;
    o->beta = beta;
    o->scale = kind == QPM_OBJ_SHG ? 1.0 / L : 1.0 / (L * L);
    o->n = d0->n;
    o->words = d0->words;
    for (int k = 0; k < K; ++k) {
        o->d[k] = designs[k];
        o->tabs.tq[k] = designs[k]->tabq;
        o->tabs.wsc[k] = designs[k]->wsc;
        o->tabs.t64[k] = designs[k]->tab64;
        o->tabs.C[k][0] = designs[k]->C[0];
        o->tabs.C[k][1] = designs[k]->C[1];
    }
    o->scratch = scratch_cache_create();
    *out = o;
    return QPM_OK;
}

QPM_API qpm_status qpm_objective_free(qpm_objective o)
{
    clear_error();
    if (o) scratch_cache_destroy(o->scratch);
    delete o;
    return QPM_OK;
}

static qpm_status eval_with_plan(qpm_objective o, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                 void *fitness, double *G, int64_t ldG, const ObjPlan &pl, hipStream_t s);

static qpm_status check_objective_args(qpm_objective o, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                       void *fitness, double *G, int64_t ldG)
{
    QPM_REQUIRE(o && bits && fitness, QPM_EINVAL, "objective, bits and fitness must not be NULL");
    QPM_REQUIRE(p == QPM_PREC_F32 || p == QPM_PREC_F64, QPM_EINVAL, "unknown precision %d", (int)p);
    QPM_REQUIRE(np >= 1, QPM_EINVAL, "np must be >= 1 (got %lld)", (long long)np);
    QPM_REQUIRE(ld >= np && ld % 64 == 0, QPM_EINVAL, "ld (%lld) must be >= np (%lld) and a multiple of 64",
                (long long)ld, (long long)np);
    QPM_REQUIRE((reinterpret_cast<uintptr_t>(bits) & 3u) == 0, QPM_EINVAL, "bits must be 4-byte aligned");
    QPM_REQUIRE(G == nullptr || ldG >= np, QPM_EINVAL, "ldG (%lld) must be >= np (%lld)", (long long)ldG,
                (long long)np);
    QPM_REQUIRE(np <= (int64_t(1) << 31) && o->words * ld <= (int64_t(1) << 40), QPM_ERANGE, "population too large");
    return QPM_OK;
}

QPM_API qpm_status qpm_eval_objective(qpm_objective o, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                      void *fitness, double *G, int64_t ldG, qpm_stream sv)
{
    clear_error();
    qpm_status st = check_objective_args(o, p, bits, np, ld, fitness, G, ldG);
    if (st != QPM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(sv);
    ObjPlan pl = plan_objective(*o, p, np);
    // Few words: one launch, which walks up to table_max_wpw words per wave and
    // writes the values itself, unless the longer walks of K THG designs cost more
    // than that launch. us per call back to back / with a wait after each, two
    // launches against one, NP = 100 (2000 is alike), by K x words per wave. SHG FP32:
    // 1 x 2 12.2 / 22.4 against 8.9 / 19.2, 8 x 3 12.2 / 26.4 against 9.6 / 25.2, 8 x 5
    // 12.3 / 26.3 against 11.8 / 27.6. THG: 3 x 2 12.0 / 25.1 against 8.9 / 24.3, 4 x 2
    // 12.1 / 26.5 against 10.7 / 26.4 (FP64 12.2 / 27.0 against 11.6 / 27.2), 2 x 3 12.3
    // / 23.8 against 8.9 / 23.7, 5 x 2 even (8 words, NP = 1000 FP64 13.3 against 14.4,
    // 5 words, NP = 5000 14.5 against 12.3); but 3 x 3 12.1 / 25.3 against 10.8 / 26.4,
    // 4 x 3 12.1 / 26.6 against 13.5 / 29.1, 6 x 2 13.8 / 29.8 against 15.1 / 30.7.
    const int wpw = static_cast<int>(std::min<int64_t>((o->words + 3) / 4, table_max_wpw(p == QPM_PREC_F32) + 1));
    if (wpw <= table_max_wpw(p == QPM_PREC_F32) && (o->kind != QPM_OBJ_THG || o->K * (wpw - 1) <= 5))
        pl = plan_objective_shape(*o, wpw);
    return eval_with_plan(o, p, bits, np, ld, fitness, G, ldG, pl, s);
}

QPM_API qpm_status qpm_eval_objective_shape(qpm_objective o, qpm_prec p, const uint32_t *bits, int64_t np,
                                            int64_t ld, void *fitness, double *G, int64_t ldG, int32_t wpw,
                                            qpm_stream sv)
{
    clear_error();
    qpm_status st = check_objective_args(o, p, bits, np, ld, fitness, G, ldG);
    if (st != QPM_OK) return st;
    QPM_REQUIRE(wpw >= 1 && wpw <= table_max_wpw(p == QPM_PREC_F32), QPM_EINVAL,
                "words_per_wave must be in [1, %d] (got %d)", table_max_wpw(p == QPM_PREC_F32), (int)wpw);
    const ObjPlan pl = plan_objective_shape(*o, wpw);
    QPM_REQUIRE(pl.gy <= 65535, QPM_ERANGE, "too many workgroup segments (%d)", pl.gy);
    return eval_with_plan(o, p, bits, np, ld, fitness, G, ldG, pl, static_cast<hipStream_t>(sv));
}

static qpm_status eval_with_plan(qpm_objective o, qpm_prec p, const uint32_t *bits, int64_t np, int64_t ld,
                                 void *fitness, double *G, int64_t ldG, const ObjPlan &pl, hipStream_t s)
{
    if (pl.gy == 1)
        return launch_partials<true>(*o, p, bits, np, ld, pl, nullptr, s, nullptr,
                                     ObjOut{o->scale, o->G0, o->beta, fitness, p == QPM_PREC_F64, G, ldG, 0});
    ScratchLease lease(o->scratch, s);
    void *ws = nullptr;
    qpm_status st = lease.begin(objective_partials_bytes(*o, pl, ld), &ws);
    if (st != QPM_OK) return st;
    double *part = static_cast<double *>(ws);
    st = launch_objective_partials(*o, p, bits, np, ld, pl, part, s);
    if (st == QPM_OK) st = launch_objective_values(*o, pl, part, ld, np, fitness, p == QPM_PREC_F64, G, ldG, s);
    const qpm_status se = lease.end();
    return st != QPM_OK ? st : se;
}
