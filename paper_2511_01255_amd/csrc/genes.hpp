// genes.hpp -- per-gene-quad arithmetic of the optimiser steps (paper Sec.
// 2.2.1 DE rand/1 + binomial crossover, Sec. 2.2.2 grey-wolf update), and
// the row / bit-word helpers, shared by the single-design and batched
// kernels. Binary32 arithmetic is spelled out with explicit fmaf and the
// library is built with -ffp-contract=off, so trial and candidate genes are
// bit-for-bit what these formulas state.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "philox.hpp"

namespace qpm {

__device__ __forceinline__ const float *row_of(const PopView &pv, int64_t r)
{
    const bool second = pv.flags != nullptr && pv.flags[r] != 0u;
    return (second ? pv.x1 : pv.x0) + r * pv.ldx;
}

__device__ __forceinline__ float *out_row_of(const PopView &pv, int64_t r)
{
    const bool second = pv.flags != nullptr && pv.flags[r] != 0u;
    return (second ? pv.out0 : pv.out1) + r * pv.ldx;
}

__device__ __forceinline__ float clamp1(float v) { return fminf(fmaxf(v, -1.0f), 1.0f); }

// clamp1 in one instruction (for a NaN both give -1: the median of three
// with a NaN is the minimum of the other two)
__device__ __forceinline__ float clamp1_med(float v) { return __builtin_amdgcn_fmed3f(v, -1.0f, 1.0f); }

// x / 3 correctly rounded, without a division: q0 = x RN(1/3), the exact
// remainder r = x - 3 q0 by FMA, one FMA correction, and the sign of x
// restored (only -0 would otherwise come out as +0). Checked against IEEE
// division for every finite binary32 input.
__device__ __forceinline__ float div3(float x)
{
    const float c = 0x1.555556p-2f;  // RN(1/3)
    const float q0 = x * c;
    const float r = fmaf(-q0, 3.0f, x);
    return copysignf(fmaf(r, c, q0), x);
}

// div3 for x != 0: the same three steps without the sign restore (checked
// against IEEE division for every nonzero finite binary32 input)
__device__ __forceinline__ float div3_nonzero(float x)
{
    const float c = 0x1.555556p-2f;
    const float q0 = x * c;
    const float r = fmaf(-q0, 3.0f, x);
    return fmaf(r, c, q0);
}

// n / d correctly rounded for d in [2^-60, 2^60] and |n| in [2^-60, 2^60]:
// the IEEE single-precision division sequence (reciprocal, one Newton step,
// quotient, two FMA remainder corrections) without its scaling and fix-up
// steps, which leave every operand and result unchanged in this range (no
// operand or quotient near the subnormal or overflow range, exponent gap
// far below 96, no special value), so the result is that of n / d.
__device__ __forceinline__ float div_in_range(float n, float d)
{
    const float r = __builtin_amdgcn_rcpf(d);
    const float e = fmaf(-d, r, 1.0f);
    const float r1 = fmaf(e, r, r);
    const float q = n * r1;
    const float rem = fmaf(-d, q, n);
    const float q1 = fmaf(rem, r1, q);
    const float rem2 = fmaf(-d, q1, n);
    return fmaf(rem2, r1, q1);
}

__device__ __forceinline__ void store_quad(float *dst, int64_t j0, int64_t D, float4 v)
{
    if (j0 + 3 < D) {
        *reinterpret_cast<float4 *>(dst + j0) = v;
    } else {
        dst[j0] = v.x;
        if (j0 + 1 < D) dst[j0 + 1] = v.y;
        if (j0 + 2 < D) dst[j0 + 2] = v.z;
    }
}

// store_quad with non-temporal full-quad stores: trial and candidate rows
// are not read again before the next step, so they should not displace the
// rows the donor reads are served from
__device__ __forceinline__ void store_quad_nt(float *dst, int64_t j0, int64_t D, float4 v)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    if (j0 + 3 < D) {
        const v4f w = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(w, reinterpret_cast<v4f *>(dst + j0));
    } else {
        dst[j0] = v.x;
        if (j0 + 1 < D) dst[j0 + 1] = v.y;
        if (j0 + 2 < D) dst[j0 + 2] = v.z;
    }
}

// the same for rows that are written up to cols >= D (a multiple of 4 where it
// is larger): genes from D on are those of `pad`
__device__ __forceinline__ void store_quad_nt(float *dst, int64_t j0, int64_t D, int64_t cols, float4 v, float4 pad)
{
    if (j0 + 3 < D) {
        store_quad_nt(dst, j0, D, v);
    } else {
        const float vs[4] = {v.x, v.y, v.z, v.w}, ps[4] = {pad.x, pad.y, pad.z, pad.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (j0 + e < cols) dst[j0 + e] = j0 + e < D ? vs[e] : ps[e];
    }
}

__device__ __forceinline__ uint32_t quad_nibble(float4 v, int64_t j0, int64_t D)
{
    uint32_t n = 0;
    n |= (v.x < 0.0f) ? 1u : 0u;
    n |= (j0 + 1 < D && v.y < 0.0f) ? 2u : 0u;
    n |= (j0 + 2 < D && v.z < 0.0f) ? 4u : 0u;
    n |= (j0 + 3 < D && v.w < 0.0f) ? 8u : 0u;
    return n;
}

// OR of the values of lanes l - 7 .. l, valid in lanes l = 7 (mod 8): three
// DPP row shifts (1, 2, 4) within the 16-lane row, no LDS traffic.
__device__ __forceinline__ uint32_t or8_into_last(uint32_t w)
{
    w |= static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(w), 0x111, 0xF, 0xF, true));
    w |= static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(w), 0x112, 0xF, 0xF, true));
    w |= static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(w), 0x114, 0xF, 0xF, true));
    return w;
}

// Merge the nibbles of 8 neighbouring lanes (gene quads 8w .. 8w+7) into
// word w and store it from the last lane of the group when the word holds
// genes (4 (8w) < D). Every lane of the wave must call this.
__device__ __forceinline__ void store_word(uint32_t nib, int64_t q, int64_t D, uint32_t *bits, int64_t ld, int64_t i)
{
    const uint32_t w = or8_into_last(nib << (4 * (threadIdx.x & 7)));
    if ((threadIdx.x & 7) == 7 && 4 * (q & ~int64_t(7)) < D) bits[(q >> 3) * ld + i] = w;
}

// DE for genes j0..j0+3 of individual i: v = clamp(fmaf(F, b - c, a)),
// u_j = v_j where ((w_j >> 8) 2^-24 <= CR) or j == jrand, else x_j, with
// the words w of Philox counter (j0 / 4, i, g, inst << 8 | DE_CR). The
// crossover test is taken on the raw word: w <= cr_max = cr_threshold(CR)
// holds exactly when (w >> 8) 2^-24 <= CR.
__device__ __forceinline__ float4 de_quad(float4 xv, float4 a, float4 b, float4 c, int64_t j0, int jrand, uint32_t i,
                                          uint32_t g, uint32_t inst, uint32_t k0, uint32_t k1, float F,
                                          uint32_t cr_max)
{
    const U4 r = philox10(static_cast<uint32_t>(j0 >> 2), i, g, (inst << 8) | kTagDeCr, k0, k1);
    const int rel = jrand - static_cast<int>(j0);  // D <= 2^30
    const float xs[4] = {xv.x, xv.y, xv.z, xv.w};
    const float as[4] = {a.x, a.y, a.z, a.w};
    const float bs[4] = {b.x, b.y, b.z, b.w};
    const float cs[4] = {c.x, c.y, c.z, c.w};
    const uint32_t rw[4] = {r.x, r.y, r.z, r.w};
    float us[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool take = (rw[e] <= cr_max) || (rel == e);
        const float v = clamp1(fmaf(F, bs[e] - cs[e], as[e]));
        us[e] = take ? v : xs[e];
    }
    return make_float4(us[0], us[1], us[2], us[3]);
}

// de_quad (the same trial, bit for bit) with the individual-free part of the
// Philox rounds taken from h = philox10_head(j0 / 4, g, inst << 8 | DE_CR)
// and pi = philox10_individual(i, g, k0)
__device__ __forceinline__ float4 de_quad_shared(const PhiloxHead &h, uint64_t pi, const float4 (&v)[4], int rel,
                                                 uint32_t k0, uint32_t k1, float F, uint32_t cr_max)
{
    U4 r = philox10_rest(h, pi, k0, k1);
    // jrand lies in one quad of a row: its word is made to pass there
    if (__any(static_cast<uint32_t>(rel) < 4u)) {
        if (rel == 0) r.x = 0u;
        if (rel == 1) r.y = 0u;
        if (rel == 2) r.z = 0u;
        if (rel == 3) r.w = 0u;
    }
    const float xs[4] = {v[0].x, v[0].y, v[0].z, v[0].w}, as[4] = {v[1].x, v[1].y, v[1].z, v[1].w};
    const float bs[4] = {v[2].x, v[2].y, v[2].z, v[2].w}, cs[4] = {v[3].x, v[3].y, v[3].z, v[3].w};
    const uint32_t rw[4] = {r.x, r.y, r.z, r.w};
    float us[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        us[e] = rw[e] <= cr_max ? clamp1_med(fmaf(F, bs[e] - cs[e], as[e])) : xs[e];
    }
    return make_float4(us[0], us[1], us[2], us[3]);
}

// bits 0 .. 3: a, b, c, d below zero (one compare and one add with carry
// each, where the compiler's select and shift-or take two more)
__device__ __forceinline__ uint32_t below_zero_nibble(float4 v)
{
    uint32_t n = 0;
    asm("v_cmp_gt_f32_e32 vcc, 0, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(n) : "v"(v.w) : "vcc");
    asm("v_cmp_gt_f32_e32 vcc, 0, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(n) : "v"(v.z) : "vcc");
    asm("v_cmp_gt_f32_e32 vcc, 0, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(n) : "v"(v.y) : "vcc");
    asm("v_cmp_gt_f32_e32 vcc, 0, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(n) : "v"(v.x) : "vcc");
    return n;
}

// DE trials of one workgroup (256 lanes): individuals gi IPB .. + IPB - 1 (IPB
// = 4 IPW R) of gene chunk c of CW = 256 / IPW genes; a wave covers IPW
// individuals at a time, 64 / IPW lanes each, a lane one gene quad. `second(r)`
// says which buffer holds row r (x0 or x1 = x0 + a constant; trials go to the
// other one), d holds (in lane t < IPB) the draws of individual min(gi IPB +
// t, np - 1). One lane per
// individual first works out where its target, donor and output rows begin
// (in bytes from x0 / out0, OFF = uint32_t below 4 GB); the passes then
// address them with one LDS read and one add per row, as global loads with a
// scalar base (pointers kept in LDS would make them flat loads, which the compiler waits
// for all together). The rows of pass r + 1 are in flight while pass r is
// computed. Rows past np and quads past D are computed on clamped addresses
// and not stored, so a pass is straight-line code. `cols` and `rows` are D and
// np, or ldx and ld where the caller wants whole rows: genes D .. cols - 1 and
// bit columns np .. rows - 1 are then written as 0.
template <int IPW, int R, typename OFF, typename Second>
__device__ __forceinline__ void de_rows(const PopView &pv, int gi, int c, float F, uint32_t cr_max, uint32_t g,
                                        uint32_t inst, uint32_t k0, uint32_t k1, uint32_t *__restrict__ bits,
                                        int64_t ld, bool store_genes, int64_t cols, int64_t rows, int4 d,
                                        Second second)
{
    constexpr int LPI = 64 / IPW;  // lanes per individual
    constexpr int WPC = LPI / 8;   // bit words per chunk and individual
    constexpr int IPG = 4 * IPW;   // individuals per pass
    constexpr int IPB = R * IPG;   // individuals per workgroup
    static_assert(IPB * WPC <= 256, "one bit word per thread at the end");
    struct alignas(4 * sizeof(OFF)) Rows {
        OFF o[4];  // target, donors
    };
    __shared__ uint32_t wsh[IPB][WPC];
    __shared__ Rows srow[IPB];
    __shared__ OFF sout[IPB];
    __shared__ int sjr[IPB];
    const int t = threadIdx.x;
    const int local = t / LPI, li = t % LPI;
    const int64_t np = pv.np, D = pv.D;
    const int64_t base = static_cast<int64_t>(gi) * IPB;
    if (t < IPB) {
        const int64_t ip = base + t < np ? base + t : np - 1;
        const OFF lq = static_cast<OFF>(4 * pv.ldx), bq = static_cast<OFF>(4 * (pv.x1 - pv.x0)),
                  bo = static_cast<OFF>(4 * (pv.out1 - pv.out0));
        auto src = [&](int r) -> OFF { return static_cast<OFF>(r) * lq + (second(r) ? bq : OFF(0)); };
        srow[t] = Rows{{src(static_cast<int>(ip)), src(d.x), src(d.y), src(d.z)}};
        sout[t] = static_cast<OFF>(ip) * lq + (second(static_cast<int>(ip)) ? OFF(0) : bo);
        sjr[t] = d.w;
    }
    const int64_t j0 = (static_cast<int64_t>(c) * LPI + li) * 4;
    const uint32_t q = static_cast<uint32_t>(j0 >> 2);
    const OFF qc = static_cast<OFF>(16 * (j0 < D ? static_cast<int64_t>(q) : (D - 1) >> 2));  // (in bounds)
    const uint32_t live = j0 + 3 < D ? 15u : (j0 < D ? (1u << (D - j0)) - 1u : 0u);
    const PhiloxHead h = philox10_head(q, g, (inst << 8) | kTagDeCr, k0, k1);
    const char *const xq = reinterpret_cast<const char *>(pv.x0);
    __syncthreads();
    float4 buf0[4], buf1[4];  // used alternately by the unrolled passes
    auto load = [&](int r, float4 (&v)[4]) {
        const Rows o = srow[r * IPG + local];
#pragma unroll
        for (int m = 0; m < 4; ++m) v[m] = *reinterpret_cast<const float4 *>(xq + (o.o[m] + qc));
    };
    load(0, buf0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float4(&cur)[4] = (r & 1) ? buf1 : buf0;
        if (r + 1 < R) load(r + 1, (r & 1) ? buf0 : buf1);
        const int li_r = r * IPG + local;
        const int64_t i = base + li_r;
        const float4 uv = de_quad_shared(h, philox10_individual(static_cast<uint32_t>(i), g, k0), cur,
                                         sjr[li_r] - static_cast<int>(j0), k0, k1, F, cr_max);
        if (store_genes && i < np && j0 < cols)
            store_quad_nt(reinterpret_cast<float *>(reinterpret_cast<char *>(pv.out0) + sout[li_r]), j0, D, cols, uv,
                          make_float4(0.0f, 0.0f, 0.0f, 0.0f));
        const uint32_t nib = below_zero_nibble(uv) & live;
        // merge the nibbles of 8 neighbouring lanes (32 genes) into one word
        const uint32_t w = or8_into_last(nib << (4 * (t & 7)));
        if ((t & 7) == 7) wsh[li_r][li >> 3] = w;
    }
    __syncthreads();
    // the IPB consecutive individuals of this workgroup share each bit row:
    // one contiguous store of IPB words per chunk word
    if (t < IPB * WPC) {
        const int wd = t / IPB, ii = t % IPB;
        const int64_t row = base + ii;
        const int64_t wg = static_cast<int64_t>(c) * WPC + wd;
        if (row < rows && wg * 32 < D) bits[wg * ld + row] = row < np ? wsh[ii][wd] : 0u;
    }
}

// Grey-wolf update of gene quad q of a non-leader: per gene e and leader k,
// word t = 3e + k of the counters (3q + t / 4, i, g, inst << 8 | GWO) gives
// r1 = lo16 2^-16 and C = 2 r2 = hi16 2^-15; A = fmaf(2a, r1, -a),
// D_k = |fmaf(C, X_k, -x)|, Y_k = fmaf(-A, D_k, X_k); then the weighted
// combination (variant 0) or the mean (variant 1), divided by 3, clamped.
template <int VARIANT>
__device__ __forceinline__ float4 gwo_quad_coef(float4 xv, float4 X0, float4 X1, float4 X2, const float (&A)[12],
                                                const float (&Cc)[12])
{
    const float xs[4] = {xv.x, xv.y, xv.z, xv.w};
    const float Xs[3][4] = {{X0.x, X0.y, X0.z, X0.w}, {X1.x, X1.y, X1.z, X1.w}, {X2.x, X2.y, X2.z, X2.w}};
    float ys[4], ss[4], ns[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float Y[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float Dk = fabsf(fmaf(Cc[3 * e + k], Xs[k][e], -xs[e]));
            Y[k] = fmaf(-A[3 * e + k], Dk, Xs[k][e]);
        }
        if constexpr (VARIANT == 1) {
            ys[e] = clamp1(div3((Y[0] + Y[1]) + Y[2]));
        } else {
            ss[e] = (fabsf(Y[0]) + fabsf(Y[1])) + fabsf(Y[2]);
            ns[e] = fmaf(fabsf(Y[2]), Y[2], fmaf(fabsf(Y[1]), Y[1], fabsf(Y[0]) * Y[0]));
        }
    }
    if constexpr (VARIANT == 0) {
        // |Y| <= 7, so s <= 21 and |num| <= 147: when every s and |num| of
        // the wave's quads is >= 2^-60, the division takes its short form
        // and, the quotient being nonzero, x / 3 needs no sign restore and
        // s == 0 cannot occur. Otherwise (tiny or zero weights) the full
        // IEEE division and the s == 0 case.
        const float lo = fminf(fminf(fminf(ss[0], fabsf(ns[0])), fminf(ss[1], fabsf(ns[1]))),
                               fminf(fminf(ss[2], fabsf(ns[2])), fminf(ss[3], fabsf(ns[3]))));
        if (__all(lo >= 0x1p-60f)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) ys[e] = clamp1(div3_nonzero(div_in_range(ns[e], ss[e])));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // evaluated unconditionally (no divergent branch); the 0/0
                // of s == 0 is selected away
                const float qv = div3(ns[e] / ss[e]);
                ys[e] = clamp1(ss[e] == 0.0f ? 0.0f : qv);
            }
        }
    }
    return make_float4(ys[0], ys[1], ys[2], ys[3]);
}

// A and C of a quad from its 12 words
__device__ __forceinline__ void gwo_word_coef(U4 wa, U4 wb, U4 wc, float a, float two_a, float (&A)[12],
                                              float (&Cc)[12])
{
    const float two_a_s = two_a * 0x1p-16f;
    const uint32_t wrd[12] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w, wc.x, wc.y, wc.z, wc.w};
#pragma unroll
    for (int t = 0; t < 12; ++t) {
        // A = fmaf(2a, lo16 2^-16, -a) with the power of two moved onto
        // 2a: the product is the same real number (both scalings are
        // exact for a = 0 or a >= 2^-100), so A is the same float
        A[t] = fmaf(two_a_s, static_cast<float>(wrd[t] & 0xFFFFu), -a);
        Cc[t] = static_cast<float>(wrd[t] >> 16) * 0x1p-15f;  // = 2 r2, exactly
    }
}

// A and C of gene quad q of individual i
__device__ __forceinline__ void gwo_coef(uint32_t q, uint32_t i, uint32_t g, uint32_t inst, uint32_t k0, uint32_t k1,
                                         float a, float two_a, float (&A)[12], float (&Cc)[12])
{
    const uint32_t c3 = (inst << 8) | kTagGwo;
    const uint32_t cq = 3u * q;
    gwo_word_coef(philox10(cq, i, g, c3, k0, k1), philox10(cq + 1u, i, g, c3, k0, k1),
                  philox10(cq + 2u, i, g, c3, k0, k1), a, two_a, A, Cc);
}

template <int VARIANT>
__device__ __forceinline__ float4 gwo_quad(float4 xv, float4 X0, float4 X1, float4 X2, uint32_t q, uint32_t i,
                                           uint32_t g, uint32_t inst, uint32_t k0, uint32_t k1, float a, float two_a)
{
    float A[12], Cc[12];
    gwo_coef(q, i, g, inst, k0, k1, a, two_a, A, Cc);
    return gwo_quad_coef<VARIANT>(xv, X0, X1, X2, A, Cc);
}

// four words at any word address
typedef uint32_t uint4u __attribute__((ext_vector_type(4), aligned(4)));

// The grey-wolf candidates of R consecutive individuals i0 .. i0 + R - 1 (i0 a
// multiple of R) of gene quad q per thread, as gwo_quad: a thread keeps its
// quad's leader genes and the individual-free part of its Philox calls for all R,
// loads the next row while it computes one, and stores R bit words at once.
// Leaders L0 .. L2 (in [0, np)) and their words are left alone; with `whole`
// rows are written up to ldx and columns up to ld as gwo_kernel says.
template <int VARIANT, int R>
__device__ __forceinline__ void gwo_rows(const PopView &pv, int i0, int64_t q, int L0, int L1, int L2, float a,
                                         uint32_t g, uint32_t inst, uint32_t k0, uint32_t k1,
                                         uint32_t *__restrict__ bits, int64_t ld, bool whole)
{
    const int np = static_cast<int>(pv.np);
    const int64_t D = pv.D, j0 = 4 * q, cols = whole ? pv.ldx : D;
    const int64_t jc = j0 < cols ? j0 : (cols - 1) / 4 * 4;  // (in bounds)
    // rows by offsets between the buffers: as a choice between the pointers of
    // `pv`, the compiler keeps `pv` in memory
    const int64_t dx = pv.x1 - pv.x0, dout = pv.out1 - pv.out0;
    auto flag = [&](int r) -> bool { return pv.flags != nullptr && pv.flags[r] != 0u; };
    auto quad_of = [&](int r, bool second) -> float4 {
        return *reinterpret_cast<const float4 *>(pv.x0 + (r * pv.ldx + (second ? dx : 0) + jc));
    };
    bool second[R];
#pragma unroll
    for (int r = 0; r < R; ++r) second[r] = flag(min(i0 + r, np - 1));
    float4 next = quad_of(min(i0, np - 1), second[0]);
    const float4 X0 = quad_of(L0, flag(L0)), X1 = quad_of(L1, flag(L1)), X2 = quad_of(L2, flag(L2));
    const float two_a = 2.0f * a;
    const uint32_t c3 = (inst << 8) | kTagGwo, cq = 3u * static_cast<uint32_t>(q);
    const PhiloxHead ha = philox10_head(cq, g, c3, k0, k1), hb = philox10_head(cq + 1u, g, c3, k0, k1),
                     hc = philox10_head(cq + 2u, g, c3, k0, k1);
    uint32_t w[R];
    bool plain = true;  // every individual moves (the same in every lane)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = i0 + r;
        const float4 xv = next;
        if (r + 1 < R) next = quad_of(min(i + 1, np - 1), second[r + 1 < R ? r + 1 : r]);
        float *const out = pv.out0 + (i * pv.ldx + (second[r] ? 0 : dout));
        uint32_t nib = 0;
        if (i < np && i != L0 && i != L1 && i != L2) {
            const uint64_t pi = philox10_individual(static_cast<uint32_t>(i), g, k0);
            float A[12], Cc[12];
            gwo_word_coef(philox10_rest(ha, pi, k0, k1), philox10_rest(hb, pi, k0, k1), philox10_rest(hc, pi, k0, k1),
                          a, two_a, A, Cc);
            const float4 yv = gwo_quad_coef<VARIANT>(xv, X0, X1, X2, A, Cc);
            if (j0 < cols) store_quad_nt(out, j0, D, cols, yv, xv);
            nib = j0 < D ? quad_nibble(yv, j0, D) : 0u;
        } else {
            plain = false;
            if (whole && i < np && j0 < cols) store_quad_nt(out, j0, cols, xv);
        }
        w[r] = or8_into_last(nib << (4 * (threadIdx.x & 7)));
    }
    if ((threadIdx.x & 7) == 7 && 4 * (q & ~int64_t(7)) < D) {
        uint32_t *const b = bits + ((q >> 3) * ld + i0);
        if (plain || whole) {
            static_assert(R == 4, "the individuals' words are one 16-byte store");
            *reinterpret_cast<uint4u *>(b) = uint4u{w[0], w[1], w[2], w[3]};
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = i0 + r;
                if (i < np && i != L0 && i != L1 && i != L2) b[r] = w[r];
            }
        }
    }
}

// Improved discrete four-leader step (paper Sec. 3.1.2, as read here: the
// paper gives no formula) for the 4 genes of quad q of wolf i: one Philox
// word per gene (counter (q, i, g, inst << 8 | 5), word e); X0..X3 the
// leaders' genes (state +1 when >= 0); par = {t, 1 - 2 eps, eps, lambda}.
//   n = leaders in state +1; dist = n / 4; maj = 1, 0, 1/2 for n > 2, < 2, = 2;
//   p = fmaf(t, maj - dist, dist); p' = fmaf(1 - 2 eps, p, eps);
//   social learning when (w >> 16 & 0x3FFF) 2^-14 < lambda: the state of
//   leader w >> 30; else +1 when (w & 0xFFFF) 2^-16 < p', else -1.
__device__ __forceinline__ float4 dgwo_quad(float4 X0, float4 X1, float4 X2, float4 X3, uint32_t q, uint32_t i,
                                            uint32_t g, uint32_t inst, uint32_t k0, uint32_t k1, float4 par)
{
    const U4 w4 = philox10(q, i, g, (inst << 8) | kTagDgwo, k0, k1);
    const uint32_t ws[4] = {w4.x, w4.y, w4.z, w4.w};
    const float Xs[4][4] = {{X0.x, X0.y, X0.z, X0.w}, {X1.x, X1.y, X1.z, X1.w}, {X2.x, X2.y, X2.z, X2.w},
                            {X3.x, X3.y, X3.z, X3.w}};
    float ys[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t w = ws[e];
        uint32_t plus = 0;  // bit k: leader k in state +1
        int n = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t pk = Xs[k][e] < 0.0f ? 0u : 1u;
            plus |= pk << k;
            n += static_cast<int>(pk);
        }
        const float dist = static_cast<float>(n) * 0.25f;
        const float maj = n > 2 ? 1.0f : (n < 2 ? 0.0f : 0.5f);
        const float p = fmaf(par.x, maj - dist, dist);
        const float p2 = fmaf(par.y, p, par.z);
        const float us = static_cast<float>((w >> 16) & 0x3FFFu) * 0x1p-14f;
        const float up = static_cast<float>(w & 0xFFFFu) * 0x1p-16f;
        const bool st = us < par.w ? ((plus >> (w >> 30)) & 1u) != 0u : up < p2;
        ys[e] = st ? 1.0f : -1.0f;
    }
    return make_float4(ys[0], ys[1], ys[2], ys[3]);
}

}  // namespace qpm
