// scan.hpp -- the per-domain walk of the d_eff double integral over one
// bit word of a genome, shared by the single-design and batched fitness
// kernels.
//
// Per genome, d_eff = sum_n d_n b_n P_{n-1} + C with P_n = sum_{m<=n} d_m a_m;
// a stretch of domains reduces to the triple (A, B, Q) = (sum d a, sum d b,
// sum d_n b_n (A before n)), and triples combine associatively:
// (A1,B1,Q1) + (A2,B2,Q2) = (A1+A2, B1+B2, Q1+Q2+A1 B2).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"

namespace qpm {

// +-1.0 from bit k of w (bit set -> -1), as a double and as a float
__device__ __forceinline__ double sign64(uint32_t w, int k)
{
    const uint32_t hi = ((w << (31 - k)) & 0x80000000u) | 0x3ff00000u;
    return __hiloint2double(static_cast<int>(hi), 0);
}
__device__ __forceinline__ float sign32(uint32_t w, int k)
{
    return __uint_as_float(((w << (31 - k)) & 0x80000000u) | 0x3f800000u);
}

struct Tri {
    double ar, ai, br, bi, qr, qi;
};

// t <- t (+) u   (t covers the domains before u)
__device__ __forceinline__ void tri_append(Tri &t, const Tri &u)
{
    t.qr = fma(t.ar, u.br, fma(-t.ai, u.bi, t.qr + u.qr));
    t.qi = fma(t.ar, u.bi, fma(t.ai, u.br, t.qi + u.qi));
    t.ar += u.ar;
    t.ai += u.ai;
    t.br += u.br;
    t.bi += u.bi;
}

// Segment triples of genome i are stored as part[s][6][ld] (A, B, Q real
// and imaginary parts). The gy segments are split into NR contiguous ranges,
// range r = [gy r / NR, gy (r+1) / NR) folded in order by one thread; the NR
// range triples are then folded in order. NR follows from gy alone
// (combine_ranges), so a genome's fitness has the same bits whichever of a single
// design's kernels combines it on a plan (the batched kernels take 16 ranges at
// any gy). What the fold waits for is the latency of a range's loads, one
// after the other: N = 5 x 10^4 (196 segments) took 18-19 us in 4 ranges for
// 256 or 1001 genomes, longer than the evaluation itself, and takes 6.6-7 us
// in 16 ranges with 8 segments (48 loads) in flight; 98 segments 10.7 and 5 us,
// 49 segments in the finish step of a run 9.3 with 8 in flight and 6.9 us with 4,
// 40 segments 4.0-5.9 and 4.8 us, 20 segments 3.8 and 4.7 us (the longer
// fold of the ranges and more code), so 4 ranges stay below 48 segments.
constexpr int kMaxRanges = 16;
__host__ __device__ inline int combine_ranges(int gy) { return gy >= 48 ? kMaxRanges : 4; }

// t <- the segments [s0, s1) of genome i in order, U at a time (every load of
// a batch goes out before the first is used; those past s1 repeat the last)
template <int U>
__device__ __forceinline__ void fold_segments(Tri &t, const double *__restrict__ part, int64_t ld, int64_t i, int s0,
                                              int s1)
{
    for (int sg = s0; sg < s1; sg += U) {
        double v[U][6];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const double *q = part + static_cast<int64_t>(min(sg + k, s1 - 1)) * 6 * ld + i;
#pragma unroll
            for (int c = 0; c < 6; ++c) v[k][c] = q[c * ld];
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (sg + k < s1) tri_append(t, Tri{v[k][0], v[k][1], v[k][2], v[k][3], v[k][4], v[k][5]});
    }
}

// A workgroup of NR x NG threads over NG genomes: thread (range, gl) folds
// the range's segments of genome i; the result is valid in range 0. sh: [6][NR][NG]
// doubles. Call from every thread (the workgroup synchronises).
template <int NR, int NG>
__device__ __forceinline__ Tri combine_segments(const double *__restrict__ part, int gy, int64_t ld, int64_t i,
                                                bool valid, int range, int gl, double *sh)
{
    const int s0 = static_cast<int>((static_cast<int64_t>(gy) * range) / NR);
    const int s1 = static_cast<int>((static_cast<int64_t>(gy) * (range + 1)) / NR);
    Tri t{0, 0, 0, 0, 0, 0};
    if (valid) {
        if constexpr (NR == 4) {
            if (s0 < s1) {
                const double *p = part + static_cast<int64_t>(s0) * 6 * ld + i;
                t = Tri{p[0], p[ld], p[2 * ld], p[3 * ld], p[4 * ld], p[5 * ld]};
#pragma unroll 4
                for (int sg = s0 + 1; sg < s1; ++sg) {
                    const double *q = part + static_cast<int64_t>(sg) * 6 * ld + i;
                    tri_append(t, Tri{q[0], q[ld], q[2 * ld], q[3 * ld], q[4 * ld], q[5 * ld]});
                }
            }
        } else if (gy <= 2 * NR) {
            fold_segments<2>(t, part, ld, i, s0, s1);
        } else if (gy <= 4 * NR) {
            fold_segments<4>(t, part, ld, i, s0, s1);
        } else {
            fold_segments<8>(t, part, ld, i, s0, s1);
        }
    }
    const double v[6] = {t.ar, t.ai, t.br, t.bi, t.qr, t.qi};
#pragma unroll
    for (int c = 0; c < 6; ++c) sh[(c * NR + range) * NG + gl] = v[c];
    __syncthreads();
    if (range == 0) {
#pragma unroll 4
        for (int r = 1; r < NR; ++r)
            if (static_cast<int64_t>(gy) * r / NR < static_cast<int64_t>(gy) * (r + 1) / NR)
                tri_append(t, Tri{sh[(0 * NR + r) * NG + gl], sh[(1 * NR + r) * NG + gl], sh[(2 * NR + r) * NG + gl],
                                  sh[(3 * NR + r) * NG + gl], sh[(4 * NR + r) * NG + gl],
                                  sh[(5 * NR + r) * NG + gl]});
    }
    return t;
}

__device__ __forceinline__ void store_fitness(void *fit, int out_f64, int64_t i, const Tri &t,
                                              const double *__restrict__ C)
{
    const double sr = t.qr + C[0], si = t.qi + C[1];
    const double f = fma(sr, sr, si * si);
    if (out_f64)
        static_cast<double *>(fit)[i] = f;
    else
        static_cast<float *>(fit)[i] = static_cast<float>(f);
}

// One word (32 domains) in FP64.
__device__ __forceinline__ void scan_word_f64(Tri &t, uint32_t word, const double4 *__restrict__ p)
{
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        const double4 c = p[k];  // {a.re, a.im, b.re, b.im}, wave-uniform
        const double s = sign64(word, k);
        const double tr = fma(c.z, t.ar, -(c.w * t.ai));
        const double ti = fma(c.z, t.ai, c.w * t.ar);
        t.qr = fma(s, tr, t.qr);
        t.qi = fma(s, ti, t.qi);
        t.ar = fma(s, c.x, t.ar);
        t.ai = fma(s, c.y, t.ai);
        t.br = fma(s, c.z, t.br);
        t.bi = fma(s, c.w, t.bi);
    }
}

// One word in the FP32 form of the per-domain walk: the word's sums A and B
// in FP64 (they multiply, and are carried into, the long prefix of the
// design, where FP32 rounding would accumulate coherently over periodic
// sign patterns), its own Q in FP32 from a float copy of the running A and
// the float b; the word's triple is folded into t in FP64.
__device__ __forceinline__ void scan_word_f32(Tri &t, uint32_t word, const double4 *__restrict__ p64,
                                              const float4 *__restrict__ p32)
{
    double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;
    float qr = 0.f, qi = 0.f;
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        const double4 c = p64[k];
        const float4 cf = p32[k];
        const double sd = sign64(word, k);
        const float s = sign32(word, k);
        const float fr = static_cast<float>(ar), fi = static_cast<float>(ai);
        const float tr = fmaf(cf.z, fr, -(cf.w * fi));
        const float ti = fmaf(cf.z, fi, cf.w * fr);
        qr = fmaf(s, tr, qr);
        qi = fmaf(s, ti, qi);
        ar = fma(sd, c.x, ar);
        ai = fma(sd, c.y, ai);
        br = fma(sd, c.z, br);
        bi = fma(sd, c.w, bi);
    }
    tri_append(t, Tri{ar, ai, br, bi, qr, qi});
}

// One word of the FP32 table walk. tb: the word's 8 blocks x R table rows x
// 16 patterns (row 0 A, then B and Q when R = 3): A and B are fixed-point
// integers at the word's scale 2^e and Q holds the float bits of Q 2^(2e);
// sc = 2^-e. A and B are summed exactly in 32-bit integers (the word scale
// keeps every partial sum below 2^31), the word's Q in FP32 from float
// copies of the running A and of B; the triple (only A when R = 1) is
// scaled back exactly and folded into t in FP64.
template <int R>
__device__ __forceinline__ void word_tab_q(Tri &t, uint32_t word, const int2 *__restrict__ tb, double sc)
{
    // the blocks' pattern offsets (8 bytes each) as the bytes of two words: two
    // instructions for four blocks, and each byte is taken by the add of the
    // table's address (5 SHG designs 3000 x 5000, where this is a third of the
    // walk: 14.4 -> 13.5 us; the full triple's walk does not change)
    uint32_t even = (word << 3) & 0x78787878u, odd = (word >> 1) & 0x78787878u;
    asm("" : "+v"(even), "+v"(odd));  // (or the compiler extracts each from the word again)
    auto entry = [&](int h, int row) -> int2 {
        const uint32_t off = (((h & 1) != 0 ? odd : even) >> (8 * (h >> 1))) & 0xFFu;
        return *reinterpret_cast<const int2 *>(reinterpret_cast<const char *>(tb) + off + (h * R + row) * 128);
    };
    const int2 A0 = entry(0, 0);
    int ar = A0.x, ai = A0.y;
    if constexpr (R == 1) {
#pragma unroll
        for (int h = 1; h < 8; ++h) {
            const int2 A = entry(h, 0);
            ar += A.x;
            ai += A.y;
        }
        t.ar += static_cast<double>(ar) * sc;
        t.ai += static_cast<double>(ai) * sc;
    } else {
        const int2 B0 = entry(0, 1), Q0 = entry(0, 2);
        int br = B0.x, bi = B0.y;
        float qr = __int_as_float(Q0.x), qi = __int_as_float(Q0.y);
#pragma unroll
        for (int h = 1; h < 8; ++h) {
            const int2 A = entry(h, 0), B = entry(h, 1), Q = entry(h, 2);
            const float fr = static_cast<float>(ar), fi = static_cast<float>(ai);
            const float bx = static_cast<float>(B.x), by = static_cast<float>(B.y);
            qr = fmaf(-fi, by, fmaf(fr, bx, qr + __int_as_float(Q.x)));
            qi = fmaf(fi, bx, fmaf(fr, by, qi + __int_as_float(Q.y)));
            ar += A.x;
            ai += A.y;
            br += B.x;
            bi += B.y;
        }
        const double sc2 = sc * sc;
        tri_append(t, Tri{static_cast<double>(ar) * sc, static_cast<double>(ai) * sc, static_cast<double>(br) * sc,
                          static_cast<double>(bi) * sc, static_cast<double>(qr) * sc2, static_cast<double>(qi) * sc2});
    }
}

// The 4 segment triples of each genome group of a table workgroup, in order,
// through LDS (the tables are no longer read): the workgroup's triple in t, and
// true, in the first segment wave of each group for live genomes.
template <int GW>
__device__ __forceinline__ bool fold_segment_waves(Tri &t, int wpw, int nw, int gsub, int ssub, int wave, int lane,
                                                   bool live, unsigned char *lds)
{
    constexpr int SW = 4;
    __syncthreads();
    double *sh = reinterpret_cast<double *>(lds);  // [6][GW * SW][64]
    constexpr int NWV = GW * SW;
    sh[(0 * NWV + wave) * 64 + lane] = t.ar;
    sh[(1 * NWV + wave) * 64 + lane] = t.ai;
    sh[(2 * NWV + wave) * 64 + lane] = t.br;
    sh[(3 * NWV + wave) * 64 + lane] = t.bi;
    sh[(4 * NWV + wave) * 64 + lane] = t.qr;
    sh[(5 * NWV + wave) * 64 + lane] = t.qi;
    __syncthreads();
    if (ssub != 0 || !live) return false;
#pragma unroll 1
    for (int s2 = 1; s2 < SW; ++s2) {
        if (s2 * wpw >= nw) break;
        const int v = gsub * SW + s2;
        tri_append(t, Tri{sh[(0 * NWV + v) * 64 + lane], sh[(1 * NWV + v) * 64 + lane], sh[(2 * NWV + v) * 64 + lane],
                          sh[(3 * NWV + v) * 64 + lane], sh[(4 * NWV + v) * 64 + lane],
                          sh[(5 * NWV + v) * 64 + lane]});
    }
    return true;
}

// One workgroup of the table kernels (GW genome groups of 64 x 4 segment
// waves, lane = genome) over the words [wbase, wbase + 4 wpw) of a design
// of W words: `bits` and the tables point at the design's word 0; the
// workgroup copies the tables of its words to `lds` (table_lds_bytes), each
// wave walks wpw words of its segment, and the 4 segment triples of each
// genome are folded in order. Returns true (with the workgroup's triple in
// t) in the first segment wave of each group for genomes i < np, where
// i = (blockIdx.x GW + group) 64 + lane. Every lane of the workgroup must
// call it (it synchronises the workgroup). FP32 walks the fixed-point
// tables tabq at the word scales wsc (word_tab_q), FP64 the tables tab64.
// SEGS (wbase 0): the GW groups of waves are not genome groups but the design's GW
// segments, over the same 64 genomes; their triples are folded in order too and
// the first wave of the workgroup holds the design's.
template <bool F32, int GW, bool SEGS = false>
__device__ __forceinline__ bool tab_segment(Tri &t, const uint32_t *__restrict__ bits, int64_t ld, int W, int wbase,
                                            const double2 *__restrict__ tab64, const int2 *__restrict__ tabq,
                                            const double *__restrict__ wsc, int wpw, int64_t np, unsigned char *lds)
{
    constexpr int SW = 4;
    constexpr int NT = GW * 256;
    constexpr int MAXW = table_max_wpw(F32);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int gsub = wave / SW, ssub = wave % SW;
    const int64_t i = (SEGS ? static_cast<int64_t>(blockIdx.x) : static_cast<int64_t>(blockIdx.x) * GW + gsub) * 64 + lane;
    const int nw = SEGS ? W : min(W - wbase, SW * wpw);  // >= 1 by the grid
    const int first = SEGS ? gsub * SW * wpw : 0;        // of this wave's segment
    // the tables of words [wbase, wbase + nw) go straight to LDS (16 bytes
    // per lane per load, no registers, no wait between loads)
    {
        const int n16 = nw * 8 * 48 * (F32 ? 8 : 16) / 16;
        const uint4 *src = F32 ? reinterpret_cast<const uint4 *>(tabq + static_cast<int64_t>(wbase) * 8 * 48)
                               : reinterpret_cast<const uint4 *>(tab64 + static_cast<int64_t>(wbase) * 8 * 48);
        for (int k = 0; k * NT < n16; ++k) {
            const int idx = k * NT + static_cast<int>(threadIdx.x);
            if (idx < n16)
                __builtin_amdgcn_global_load_lds(
                    src + idx, reinterpret_cast<__attribute__((address_space(3))) void *>(
                                   reinterpret_cast<uintptr_t>(lds + static_cast<size_t>(k * NT + wave * 64) * 16)),
                    16, 0, 0);
        }
    }
    // this wave's bit words, loaded while the tables arrive (clamped
    // addresses, so every load is in bounds and none is branched around)
    const bool live = i < np;
    const int w0 = first + ssub * wpw, w1 = min(nw, w0 + wpw);
    const int64_t ic = i < ld ? i : ld - 1;
    uint32_t wv[MAXW];
#pragma unroll
    for (int k = 0; k < MAXW; ++k) wv[k] = bits[static_cast<int64_t>(min(wbase + w0 + k, W - 1)) * ld + ic];
    // keep the loads here, issued together with the table copies (the
    // compiler would otherwise sink each one to its first use, one memory
    // latency per word)
#pragma unroll
    for (int k = 0; k < MAXW; ++k) asm volatile("" ::"v"(wv[k]));
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    t = Tri{0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < MAXW; ++k) {
        const int wr = w0 + k;
        if (wr >= w1) break;
        const uint32_t word = live ? wv[k] : 0u;
        if constexpr (F32) {
            word_tab_q<3>(t, word, reinterpret_cast<const int2 *>(lds) + wr * 8 * 48, wsc[wbase + wr]);
        } else {
            const double2 *tb = reinterpret_cast<const double2 *>(lds) + wr * 8 * 48;
#pragma unroll
            for (int h = 0; h < 8; ++h) {
                const uint32_t pt = (word >> (4 * h)) & 15u;
                const double2 A = tb[h * 48 + pt], B = tb[h * 48 + 16 + pt], Q = tb[h * 48 + 32 + pt];
                t.qr = fma(-t.ai, B.y, fma(t.ar, B.x, t.qr + Q.x));
                t.qi = fma(t.ai, B.x, fma(t.ar, B.y, t.qi + Q.y));
                t.ar += A.x;
                t.ai += A.y;
                t.br += B.x;
                t.bi += B.y;
            }
        }
    }
    const bool folded = fold_segment_waves<GW>(t, wpw, min(nw - first, SW * wpw), gsub, ssub, wave, lane, live, lds);
    if constexpr (!SEGS) {
        return folded;
    } else {
        double *sh = reinterpret_cast<double *>(lds);  // [GW][6][64]
        __syncthreads();
        if (gsub > 0 && folded) {
            const double v[6] = {t.ar, t.ai, t.br, t.bi, t.qr, t.qi};
#pragma unroll
            for (int c = 0; c < 6; ++c) sh[(gsub * 6 + c) * 64 + lane] = v[c];
        }
        __syncthreads();
        if (wave != 0 || !live) return false;
#pragma unroll
        for (int g = 1; g < GW; ++g) {
            const double *v = sh + g * 6 * 64 + lane;
            tri_append(t, Tri{v[0], v[64], v[128], v[192], v[256], v[320]});
        }
        return true;
    }
}

// Words per wave of one stage of the table kernels, and the bytes of a stage's
// tables (4 waves' words: 8 blocks x 48 entries each)
template <bool F32>
struct TabStage {
    static constexpr int kWords = F32 ? 2 : 1;
    static constexpr int kWordBytes = 8 * 48 * (F32 ? 8 : 16);
    static constexpr int kBytes = 4 * kWords * kWordBytes;
};

// tab_segment for longer segments than LDS holds the tables of (wpw >
// table_max_wpw): each wave walks its words in stages of kWords, and the tables
// of the next stage's words (and the wave's bit words) arrive in the other half
// of `lds` while one is walked, so only the first stage waits for memory and a
// workgroup leaves fewer segments to fold. Kernel + fold, us, against one stage:
// 49999 x 1001 FP64 18.1 + 6.8 -> 13.6 + 4.1, FP32 14.5 + 4.8 -> 13.4 + 4.3; 64
// designs of up to 5 x 10^4 domains, NP = 256, FP32 63.6 + 9.1 -> 56.2 + 6.6, FP64
// 76 + 19 -> 66 + 6. Short segments gain nothing and pay for the stages (2000 x
// 500 FP32: 4.1 -> 4.5).
template <bool F32, int GW>
__device__ __forceinline__ bool tab_segment_staged(Tri &t, const uint32_t *__restrict__ bits, int64_t ld, int W, int wbase,
                                            const double2 *__restrict__ tab64, const int2 *__restrict__ tabq,
                                            const double *__restrict__ wsc, int wpw, int64_t np, unsigned char *lds)
{
    constexpr int SW = 4;
    constexpr int NT = GW * 256;
    using Stage = TabStage<F32>;
    constexpr int WS = Stage::kWords;
    constexpr int PIECE = WS * Stage::kWordBytes / 16;  // 16-byte units of one wave's words
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int gsub = wave / SW, ssub = wave % SW;
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * GW + gsub) * 64 + lane;
    const int nw = min(W - wbase, SW * wpw);  // >= 1 by the grid
    const uint4 *const tabs =
        F32 ? reinterpret_cast<const uint4 *>(tabq) : reinterpret_cast<const uint4 *>(tab64);
    const bool live = i < np;
    const int w0 = ssub * wpw, w1 = min(nw, w0 + wpw);
    const int64_t ic = i < ld ? i : ld - 1;
    uint32_t next[WS];
    // stage k: words s wpw + k WS .. of every segment s, straight to LDS (16
    // bytes per lane per load, no registers, no wait between loads)
    auto issue = [&](int k) {
        unsigned char *const to = lds + (k & 1) * Stage::kBytes;
#pragma unroll
        for (int u = 0; u < (SW * PIECE + NT - 1) / NT; ++u) {
            const int idx = u * NT + static_cast<int>(threadIdx.x);
            const int s = idx / PIECE, in = idx % PIECE;
            const int w = s * wpw + k * WS + in / (PIECE / WS);  // the unit's word
            if (idx < SW * PIECE && w < min(nw, (s + 1) * wpw))
                __builtin_amdgcn_global_load_lds(
                    tabs + (static_cast<int64_t>(wbase + s * wpw + k * WS) * (PIECE / WS) + in),
                    reinterpret_cast<__attribute__((address_space(3))) void *>(
                        reinterpret_cast<uintptr_t>(to + static_cast<size_t>(u * NT + wave * 64) * 16)),
                    16, 0, 0);
        }
        // this wave's bit words (clamped addresses, so every load is in
        // bounds and none is branched around)
#pragma unroll
        for (int j = 0; j < WS; ++j) next[j] = bits[static_cast<int64_t>(min(wbase + w0 + k * WS + j, W - 1)) * ld + ic];
    };
    issue(0);
    t = Tri{0, 0, 0, 0, 0, 0};
    const int stages = (min(wpw, nw) + WS - 1) / WS;  // the same in every wave
#pragma unroll 1
    for (int k = 0; k < stages; ++k) {
        // this stage's loads have arrived in every wave, and every wave is
        // done with the half the next ones go to
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        uint32_t wv[WS];
#pragma unroll
        for (int j = 0; j < WS; ++j) wv[j] = live ? next[j] : 0u;
        if (k + 1 < stages) issue(k + 1);
        const unsigned char *const from = lds + (k & 1) * Stage::kBytes + ssub * (PIECE * 16);
#pragma unroll
        for (int j = 0; j < WS; ++j) {
            const int wr = w0 + k * WS + j;
            if (wr >= w1) break;
            const uint32_t word = wv[j];
            if constexpr (F32) {
                word_tab_q<3>(t, word, reinterpret_cast<const int2 *>(from) + j * 8 * 48, wsc[wbase + wr]);
            } else {
                const double2 *tb = reinterpret_cast<const double2 *>(from) + j * 8 * 48;
#pragma unroll
                for (int h = 0; h < 8; ++h) {
                    const uint32_t pt = (word >> (4 * h)) & 15u;
                    const double2 A = tb[h * 48 + pt], B = tb[h * 48 + 16 + pt], Q = tb[h * 48 + 32 + pt];
                    t.qr = fma(-t.ai, B.y, fma(t.ar, B.x, t.qr + Q.x));
                    t.qi = fma(t.ai, B.x, fma(t.ar, B.y, t.qi + Q.y));
                    t.ar += A.x;
                    t.ai += A.y;
                    t.br += B.x;
                    t.bi += B.y;
                }
            }
        }
    }
    return fold_segment_waves<GW>(t, wpw, nw, gsub, ssub, wave, lane, live, lds);
}

}  // namespace qpm
