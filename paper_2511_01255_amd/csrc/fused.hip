// fused.hip -- whole HWSDA generations (paper Sec. 3.2, steps 2-6) in one
// workgroup for populations small enough to live in LDS (the plain
// configuration: N = 256 domains, NP = 32). A run's generation is otherwise
// six or seven launches of a few microseconds each; here one launch runs
// any number of generations with workgroup barriers between the steps.
//
// LDS holds both gene buffers (a per-row pair of offsets says which holds the
// current row), the fitness (as doubles), the trial / candidate bits, the
// donors, the leaders and, when they fit, the design's FP64 sign-pattern
// tables. The arithmetic of every step is the multi-kernel path's (de_draw,
// the DE trial, gwo_quad; the FP64 table walk), so in FP64 trials, candidates
// and decisions are those of the oracle. An FP32 run takes the same FP64 walk
// and rounds each fitness to binary32, the precision its fitness is held and
// compared in (on one CU the FP64 walk costs what an FP32 one would).
//
// One compute unit's vector issue bounds a generation, and half of it would be
// Philox rounds. Those depend on the generation's number only, so a kernel of
// the whole chip makes them first (fused_words_kernel): the donors, the genes
// DE takes from the mutant, and the grey-wolf coefficients A and C. The
// generations read them back (98 bytes per gene quad, at up to 115 GB/s for one
// compute unit) ahead of their use (a launch of few generations makes them itself). At 256 x 32, FP64: 9.8 -> 5.8 us per
// generation, of which the two optimiser steps' vector instructions are half
// and the two evaluations 2 us.
//
// Thread mapping: the optimiser steps walk (individual, gene quad) pairs,
// each individual padded to a whole number of 32-gene words, so eight
// neighbouring lanes always hold one bit word; the fitness gives each
// genome eight lanes of a DPP row, which walk consecutive shares of its
// 4-domain blocks and fold their triples in order with row shifts; the
// leaders come from each individual's rank, counted by 16 lanes. Each
// genome's selection is taken by the first lane of its evaluation right after
// the fold, so an evaluation and its selection need one barrier.
#include <algorithm>

#include "common.hpp"
#include "device_common.hpp"
#include "genes.hpp"
#include "scan.hpp"

namespace qpm {

namespace {

constexpr int kFusedThreads = 1024;

struct FusedArgs {
    float *x0;              // run buffer 0 (rows written back here)
    const float *x1;        // run buffer 1
    uint32_t *flags;        // per-row buffer flags (cleared on exit)
    uint32_t *fbits;        // packed flags (cleared on exit), nfb words
    void *f_cur;            // current fitness, double or float (read, written back)
    int f32;                // the run's fitness is binary32
    int32_t *leaders;       // leaders of the last generation (written)
    uint32_t *gen;          // generation counter (advanced by gens)
    const float *a_tab;     // a_g
    const float *F_tab;     // F_g
    const double2 *tab64;   // the design's FP64 sign-pattern tables
    const double *C;        // C (re, im)
    int64_t np, D, ldx;
    int W;                  // bit words per genome
    int nfb;                // packed flag words
    int gens;               // generations to run
    int algo;               // qpm_algo
    uint32_t cr_max, k0, k1, inst;
    unsigned char *words;   // the random numbers of the launch's generations (FusedWords)
};

// What fused_words_kernel leaves of one generation's random numbers. A pair
// (individual, gene quad) is a slot k = individual Qpad + quad; thread t of the
// generation kernel walks slots t, t + 1024, ... (its rounds).
//   donors[i]  8 r1 | 8 r2 << 10 | 8 r3 << 20
//   take[t]    bit 4 r + e: round r of thread t takes the mutant's gene e
//   coef       six planes of float4 per slot: A[0..11], C[0..11]
constexpr int kFusedMaxRounds = 8;
struct FusedWords {
    int slots;  // slots rounded up to whole rounds
    size_t take, coef, stride;
};

__host__ __device__ inline FusedWords fused_words(int64_t np, int W)
{
    FusedWords w;
    w.slots = static_cast<int>((np * 8 * W + kFusedThreads - 1) / kFusedThreads * kFusedThreads);
    w.take = (sizeof(uint32_t) * static_cast<size_t>(np) + 15) / 16 * 16;
    w.coef = w.take + sizeof(uint32_t) * kFusedThreads;
    w.stride = w.coef + 6 * sizeof(float4) * static_cast<size_t>(w.slots);
    return w;
}

// LDS layout (bytes), shared by the kernel and the launcher
struct FusedLayout {
    int64_t D4, Q, Qpad;  // gene stride, quads, quads padded to whole words
    // cur (int2 per row, at 0): the byte offsets of its current row and of its
    // row in the other buffer
    size_t dr, fs, bw, sl, buf, tab, total;
};

__host__ __device__ inline FusedLayout fused_layout(int64_t np, int64_t D, int W, bool tab_lds)
{
    FusedLayout L;
    L.D4 = (D + 3) / 4 * 4;
    L.Q = (D + 3) / 4;
    L.Qpad = static_cast<int64_t>(W) * 8;
    size_t o = static_cast<size_t>(np) * sizeof(int2);
    L.dr = o;
    o += static_cast<size_t>(np) * sizeof(uint32_t);
    o = (o + 7) / 8 * 8;
    L.fs = o;
    o += static_cast<size_t>(np) * sizeof(double);
    L.bw = o;
    o += static_cast<size_t>(np) * W * sizeof(uint32_t);
    o = (o + 15) / 16 * 16;
    L.sl = o;
    o += 8 * sizeof(int32_t);
    L.buf = o;
    o += 2 * static_cast<size_t>(np) * L.D4 * sizeof(float);
    L.tab = o;
    if (tab_lds) o += static_cast<size_t>(W) * 8 * 48 * sizeof(double2);
    L.total = o;
    return L;
}

// the donors of individual i in generation g, packed
__device__ __forceinline__ uint32_t fused_donors(const FusedArgs &a, int i, uint32_t g)
{
    const int4 d = de_draw(i, a.np, a.D, g, a.inst, a.k0, a.k1);
    return static_cast<uint32_t>(8 * d.x) | static_cast<uint32_t>(8 * d.y) << 10 | static_cast<uint32_t>(8 * d.z) << 20;
}

// which genes of quad q individual i takes from the mutant (bits 0 .. 3)
__device__ __forceinline__ uint32_t fused_take(const FusedArgs &a, uint32_t i, uint32_t q, uint32_t g)
{
    const U4 u = philox10(q, i, g, (a.inst << 8) | kTagDeCr, a.k0, a.k1);
    const int rel = de_draw(i, a.np, a.D, g, a.inst, a.k0, a.k1).w - 4 * static_cast<int>(q);
    return (u.x <= a.cr_max || rel == 0 ? 1u : 0u) | (u.y <= a.cr_max || rel == 1 ? 2u : 0u) |
           (u.z <= a.cr_max || rel == 2 ? 4u : 0u) | (u.w <= a.cr_max || rel == 3 ? 8u : 0u);
}

// The random numbers of generations gen[0] + blockIdx.y. Grid: 4 workgroups
// (together the threads of the generation kernel) x generations.
__global__ __launch_bounds__(256) void fused_words_kernel(FusedArgs a)
{
    const FusedWords w = fused_words(a.np, a.W);
    unsigned char *base = a.words + blockIdx.y * w.stride;
    const uint32_t g = a.gen[0] + blockIdx.y;
    const int t = static_cast<int>(blockIdx.x) * 256 + static_cast<int>(threadIdx.x);
    const int np = static_cast<int>(a.np), D = static_cast<int>(a.D), Q = (D + 3) / 4, Qpad = 8 * a.W;
    const bool has_de = a.algo != QPM_ALGO_GWO, has_gwo = a.algo != QPM_ALGO_DE;
    if (has_de && t < np) reinterpret_cast<uint32_t *>(base)[t] = fused_donors(a, t, g);
    float4 *coef = reinterpret_cast<float4 *>(base + w.coef);
    const float ag = a.a_tab[g], two_a = 2.0f * ag;
    uint32_t take = 0;
    for (int k = t, r = 0; k < np * Qpad; k += kFusedThreads, ++r) {
        const uint32_t i = static_cast<uint32_t>(k / Qpad), q = static_cast<uint32_t>(k % Qpad);
        if (static_cast<int>(q) >= Q) continue;
        if (has_de) take |= fused_take(a, i, q, g) << (4 * r);
        if (has_gwo) {
            float A[12], Cc[12];
            gwo_coef(q, i, g, a.inst, a.k0, a.k1, ag, two_a, A, Cc);
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                coef[m * w.slots + k] = make_float4(A[4 * m], A[4 * m + 1], A[4 * m + 2], A[4 * m + 3]);
                coef[(3 + m) * w.slots + k] = make_float4(Cc[4 * m], Cc[4 * m + 1], Cc[4 * m + 2], Cc[4 * m + 3]);
            }
        }
    }
    if (has_de) reinterpret_cast<uint32_t *>(base + w.take)[t] = take;
}

// lanes per genome of the fitness walk (np <= 64, so np T <= 1024), within one
// DPP row. Fewer lanes walk more blocks each, more lanes fold more often: a
// fold level costs two blocks' vector instructions (an evaluation at 256 x 32:
// 2300 cycles with 8 lanes, 2550 with 16)
constexpr int kFusedLanes = 8;

// the value of lane l + OFF (OFF in {1, 2, 4}) of the same 16-lane row, by
// DPP row shifts (lanes past the row's end read 0; they are not used)
template <int OFF>
__device__ __forceinline__ double row_down(double v)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x100 + OFF, 0xF, 0xF, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), 0x100 + OFF, 0xF, 0xF, true));
}

// The triple of the lanes [s, s + 2 OFF) in lanes whose s is a multiple of
// 2 OFF, from those of [s, s + OFF) and [s + OFF, s + 2 OFF). Other lanes are
// left with sums that are not used (no branch around them).
template <int OFF>
__device__ __forceinline__ void fold_level(Tri &t)
{
    tri_append(t, Tri{row_down<OFF>(t.ar), row_down<OFF>(t.ai), row_down<OFF>(t.br), row_down<OFF>(t.bi),
                      row_down<OFF>(t.qr), row_down<OFF>(t.qi)});
}

// How the evaluated genomes replace the current ones (paper Sec. 3.2 steps 4
// and 5): SEL_GREEDY keeps a genome whose fitness is strictly higher;
// SEL_GREEDY_OMEGA does so for every genome but the three leaders; SEL_MOVE
// (the grey-wolf optimiser alone) moves every genome but the leaders.
enum { SEL_GREEDY = 0, SEL_GREEDY_OMEGA = 1, SEL_MOVE = 2 };

// The fitness of every genome of the bit words, then its selection, by the
// genome's first lane once its triples are folded (no other thread reads
// fs or cur meanwhile). The table entries of kFusedAhead blocks are read
// before the first is used: a lane has few blocks (4 at 256 domains), and
// one after another each pays two LDS latencies.
constexpr int kFusedAhead = 4;
template <bool TAB_LDS>
__device__ __forceinline__ void fused_fitness(const FusedArgs &a, const FusedLayout &L, unsigned char *lds,
                                              const double2 *__restrict__ tabs, double Cr, double Ci, int sel,
                                              int4 lead)
{
    const uint32_t *bw = reinterpret_cast<const uint32_t *>(lds + L.bw);
    double *fs = reinterpret_cast<double *>(lds + L.fs);
    int2 *cur = reinterpret_cast<int2 *>(lds);
    constexpr int T = kFusedLanes;
    const int tid = static_cast<int>(threadIdx.x), np = static_cast<int>(a.np);
    const int i = tid / T;
    const int s = tid % T;
    const int NB = 8 * a.W;
    const int bpt = (NB + T - 1) / T;
    if (tid - (tid & 63) >= np * T) return;  // (whole waves: the fold below is within a wave)
    const double f_old = fs[min(i, np - 1)];
    const int2 c_old = cur[min(i, np - 1)];
    Tri t{0, 0, 0, 0, 0, 0};
    if (i < np) {
        const int b0 = s * bpt, b1 = min(NB, b0 + bpt);
        int b = b0;
        auto load = [&](int bk, double2 &A, double2 &B, double2 &Q) {
            const uint32_t p = (bw[i * a.W + (bk >> 3)] >> (4 * (bk & 7))) & 15u;
            const double2 *e = tabs + (bk * 48 + static_cast<int>(p));
            A = e[0];
            B = e[16];
            Q = e[32];
        };
        auto append = [&](const double2 &A, const double2 &B, const double2 &Q) {
            t.qr = fma(-t.ai, B.y, fma(t.ar, B.x, t.qr + Q.x));
            t.qi = fma(t.ai, B.x, fma(t.ar, B.y, t.qi + Q.y));
            t.ar += A.x;
            t.ai += A.y;
            t.br += B.x;
            t.bi += B.y;
        };
        for (; b + kFusedAhead <= b1; b += kFusedAhead) {
            double2 A[kFusedAhead], B[kFusedAhead], Q[kFusedAhead];
#pragma unroll
            for (int k = 0; k < kFusedAhead; ++k) load(b + k, A[k], B[k], Q[k]);
#pragma unroll
            for (int k = 0; k < kFusedAhead; ++k) append(A[k], B[k], Q[k]);
        }
        for (; b < b1; ++b) {
            double2 A, B, Q;
            load(b, A, B, Q);
            append(A, B, Q);
        }
    }
    // fold the T triples of each genome in block order
    static_assert(T == 8, "a genome's lanes lie in one DPP row, folded in three levels");
    fold_level<1>(t);
    fold_level<2>(t);
    fold_level<4>(t);
    if (i < np && s == 0) {
        const double sr = t.qr + Cr, si = t.qi + Ci;
        double fnew = fma(sr, sr, si * si);
        // an FP32 run holds its fitness in binary32 (compared as such)
        if (a.f32) fnew = static_cast<double>(static_cast<float>(fnew));
        const bool leader = i == lead.x || i == lead.y || i == lead.z;
        const bool take = sel == SEL_GREEDY ? fnew > f_old : (!leader && (sel == SEL_MOVE || fnew > f_old));
        if (take) {
            fs[i] = fnew;
            cur[i] = make_int2(c_old.y, c_old.x);
        }
    }
}

// The three best of fs[0..np) (f descending, slot ascending): their slots in
// sl[0..2] and the byte offsets of their rows in sl[4..6]. 16 lanes per individual
// count the individuals ahead of it over a share of the population each
// (np <= 64: at most four, read together), the counts are summed across the
// DPP row, and the individuals of rank 0, 1, 2 write themselves. The order is
// strict and total, so the ranks are distinct. Called by every thread; ends
// with a barrier.
__device__ __forceinline__ void fused_leaders(const double *fs, const int2 *cur, int np, int32_t *sl)
{
    const int tid = static_cast<int>(threadIdx.x);
    const int i = tid >> 4, part = tid & 15;
    if (tid - (tid & 63) < np * 16) {
        const int ic = min(i, np - 1);
        const double fi = fs[ic];
        const int row = cur[ic].x;
        double fj[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) fj[k] = fs[min(part + 16 * k, np - 1)];
        int ahead = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = part + 16 * k;
            ahead += static_cast<int>(j < np) & (static_cast<int>(fj[k] > fi) |
                                                 (static_cast<int>(fj[k] == fi) & static_cast<int>(j < i)));
        }
        ahead += __builtin_amdgcn_update_dpp(0, ahead, 0x101, 0xF, 0xF, false);
        ahead += __builtin_amdgcn_update_dpp(0, ahead, 0x102, 0xF, 0xF, false);
        ahead += __builtin_amdgcn_update_dpp(0, ahead, 0x104, 0xF, 0xF, false);
        ahead += __builtin_amdgcn_update_dpp(0, ahead, 0x108, 0xF, 0xF, false);
        if (i < np && part == 0 && ahead < 3) {
            sl[ahead] = i;
            sl[4 + ahead] = row;
        }
    }
    __syncthreads();
}

// OWN: the kernel makes its random numbers itself, where they are used
template <int VARIANT, bool TAB_LDS, bool OWN>
__global__ __launch_bounds__(kFusedThreads) void fused_gen_kernel(FusedArgs a)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const FusedLayout L = fused_layout(a.np, a.D, a.W, TAB_LDS);
    const FusedWords fw = fused_words(a.np, a.W);
    int2 *cur = reinterpret_cast<int2 *>(lds);
    uint32_t *dr = reinterpret_cast<uint32_t *>(lds + L.dr);
    double *fs = reinterpret_cast<double *>(lds + L.fs);
    uint32_t *bw = reinterpret_cast<uint32_t *>(lds + L.bw);
    int32_t *sl = reinterpret_cast<int32_t *>(lds + L.sl);
    const double2 *tabs = TAB_LDS ? reinterpret_cast<const double2 *>(lds + L.tab) : a.tab64;
    const int tid = static_cast<int>(threadIdx.x);
    const int np = static_cast<int>(a.np), D = static_cast<int>(a.D), Q = static_cast<int>(L.Q),
              Qpad = static_cast<int>(L.Qpad);
    const int row_bytes = 4 * static_cast<int>(L.D4), buf0 = static_cast<int>(L.buf), buf1 = buf0 + np * row_bytes;
    auto quad = [&](int offset) -> float4 & { return *reinterpret_cast<float4 *>(lds + offset); };

    // load the population (current rows through the run's flags) into
    // buffer 0, the fitness, and the tables
    for (int k = tid; k < np * Q; k += kFusedThreads) {
        const int r = k / Q, q = k % Q;
        const float *src = (a.flags[r] ? a.x1 : a.x0) + r * a.ldx;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (4 * q + 3 < D) {
            v = *reinterpret_cast<const float4 *>(src + 4 * q);
        } else {
            v.x = src[4 * q];
            if (4 * q + 1 < D) v.y = src[4 * q + 1];
            if (4 * q + 2 < D) v.z = src[4 * q + 2];
        }
        quad(buf0 + r * row_bytes + 16 * q) = v;
    }
    if (tid < np) {
        fs[tid] = a.f32 ? static_cast<double>(static_cast<const float *>(a.f_cur)[tid])
                        : static_cast<const double *>(a.f_cur)[tid];
        cur[tid] = make_int2(buf0 + tid * row_bytes, buf1 + tid * row_bytes);
    }
    if constexpr (TAB_LDS) {
        double2 *dst = reinterpret_cast<double2 *>(lds + L.tab);
        for (int k = tid; k < a.W * 8 * 48; k += kFusedThreads) dst[k] = a.tab64[k];
    }
    const bool has_de = a.algo != QPM_ALGO_GWO, has_gwo = a.algo != QPM_ALGO_DE;
    const unsigned char *words = a.words;
    uint32_t g = a.gen[0];
    const double Cr = a.C[0], Ci = a.C[1];
    float Fg = a.F_tab[g];
    // one optimiser step over every (individual, quad) pair: slot tid + 1024
    // rd in round rd, its pair followed without divisions; results go to the
    // other buffer and the bit words. All threads run the same rounds.
    const int rounds = fw.slots / kFusedThreads;
    const int i_first = tid / Qpad, q_first = tid % Qpad;
    const int di = kFusedThreads / Qpad, dq = kFusedThreads % Qpad;
    const uint32_t tail = D % 4 ? (1u << (D % 4)) - 1u : 15u;  // bits of the last quad
    auto next_pair = [&](int &i, int &q) {
        i += di;
        q += dq;
        if (q >= Qpad) {
            q -= Qpad;
            ++i;
        }
    };
    auto store_bits = [&](uint32_t nib, int rd, int i) {
        const uint32_t w = or8_into_last(nib << (4 * (tid & 7)));
        if ((tid & 7) == 7 && i < np) bw[(rd * kFusedThreads + tid) >> 3] = w;  // word i W + q / 8
    };
    // the random numbers are loaded well before their use, so the memory's
    // latency passes under other steps: the coefficients a round of the step
    // (or the steps between) ahead, the rest a generation ahead
    auto coef = [&](const unsigned char *base, int rd, float4 (&v)[6]) {
        const float4 *p = reinterpret_cast<const float4 *>(base + fw.coef) + (rd * kFusedThreads + tid);
#pragma unroll
        for (int m = 0; m < 6; ++m) v[m] = p[m * fw.slots];
    };
    const int donor = min(tid, np - 1);
    uint32_t d_next = 0, take = 0, take_next = 0;
    float4 v[6] = {};
    if constexpr (OWN) {
        if (has_de && tid < np) dr[tid] = fused_donors(a, tid, g);
    } else {
        if (has_de) {
            if (tid < np) dr[tid] = reinterpret_cast<const uint32_t *>(words)[tid];
            take = reinterpret_cast<const uint32_t *>(words + fw.take)[tid];
        }
        if (has_gwo) coef(words, 0, v);
    }
    __syncthreads();

    for (int it = 0; it < a.gens; ++it, ++g) {
        const bool more = it + 1 < a.gens;
        const unsigned char *words_next = more ? words + fw.stride : words;
        const float F_next = a.F_tab[more ? g + 1 : g];
        const float ag = OWN ? a.a_tab[g] : 0.0f;
        if (has_de) {
            // (by every thread: a load in a branch makes its uses wait for
            // every later load too)
            if constexpr (OWN) {
                if (more && tid < np) d_next = fused_donors(a, tid, g + 1);
            } else {
                d_next = reinterpret_cast<const uint32_t *>(words_next)[donor];
                take_next = reinterpret_cast<const uint32_t *>(words_next + fw.take)[tid];
            }
            // DE trials, evaluation, greedy selection
            for (int rd = 0, i = i_first, q = q_first; rd < rounds; ++rd) {
                uint32_t nib = 0;
                if (i < np && q < Q) {
                    if constexpr (OWN) take = fused_take(a, i, q, g) << (4 * rd);
                    const uint32_t d = dr[i];
                    const int2 ci = cur[i];
                    auto row = [&](uint32_t at) -> int { return *reinterpret_cast<const int *>(lds + at); };
                    const float4 xv = quad(ci.x + 16 * q);
                    const float4 r1 = quad(row(d & 1023u) + 16 * q);
                    const float4 r2 = quad(row((d >> 10) & 1023u) + 16 * q);
                    const float4 r3 = quad(row(d >> 20) + 16 * q);
                    // (the masks are hidden from the compiler, which would
                    // turn the selects into branches around the loads)
                    auto pick = [&](uint32_t e, float m, float x) -> float {
                        int32_t k = static_cast<int32_t>(take << (31u - (4u * rd + e))) >> 31;
                        asm("" : "+v"(k));
                        return __int_as_float((k & __float_as_int(m)) | (~k & __float_as_int(x)));
                    };
                    const float4 uv = make_float4(pick(0u, clamp1_med(fmaf(Fg, r2.x - r3.x, r1.x)), xv.x),
                                                  pick(1u, clamp1_med(fmaf(Fg, r2.y - r3.y, r1.y)), xv.y),
                                                  pick(2u, clamp1_med(fmaf(Fg, r2.z - r3.z, r1.z)), xv.z),
                                                  pick(3u, clamp1_med(fmaf(Fg, r2.w - r3.w, r1.w)), xv.w));
                    quad(ci.y + 16 * q) = uv;
                    nib = below_zero_nibble(uv) & (q == Q - 1 ? tail : 15u);
                }
                store_bits(nib, rd, i);
                next_pair(i, q);
            }
            __syncthreads();
            fused_fitness<TAB_LDS>(a, L, lds, tabs, Cr, Ci, SEL_GREEDY, make_int4(-1, -1, -1, -1));
            // DE alone: the draws of the next generation (read by its DE step)
            if (!has_gwo && tid < np) dr[tid] = d_next;
            __syncthreads();
        }
        // leaders: the three best (f descending, slot ascending)
        fused_leaders(fs, cur, np, sl);
        if (has_gwo) {
            // grey-wolf candidates of the omega wolves, evaluation, selection
            const int L0 = sl[0], L1 = sl[1], L2 = sl[2], o0 = sl[4], o1 = sl[5], o2 = sl[6];
            // the loads of d_next and take_next end here, where they have had
            // an evaluation's time, and not after the coefficients' below
            asm volatile("" : "+v"(d_next), "+v"(take_next));
            for (int rd = 0, i = i_first, q = q_first; rd < rounds; ++rd) {
                uint32_t nib = 0;
                if (i < np && q < Q && i != L0 && i != L1 && i != L2) {
                    const int2 ci = cur[i];
                    float A[12], Cc[12];
                    if constexpr (OWN) {
                        gwo_coef(q, i, g, a.inst, a.k0, a.k1, ag, 2.0f * ag, A, Cc);
                    } else {
#pragma unroll
                        for (int m = 0; m < 3; ++m) {
                            const float4 va = v[m], vc = v[3 + m];
                            A[4 * m] = va.x, A[4 * m + 1] = va.y, A[4 * m + 2] = va.z, A[4 * m + 3] = va.w;
                            Cc[4 * m] = vc.x, Cc[4 * m + 1] = vc.y, Cc[4 * m + 2] = vc.z, Cc[4 * m + 3] = vc.w;
                        }
                    }
                    const float4 yv = gwo_quad_coef<VARIANT>(quad(ci.x + 16 * q), quad(o0 + 16 * q),
                                                             quad(o1 + 16 * q), quad(o2 + 16 * q), A, Cc);
                    quad(ci.y + 16 * q) = yv;
                    nib = below_zero_nibble(yv) & (q == Q - 1 ? tail : 15u);
                }
                if constexpr (!OWN) coef(rd + 1 < rounds ? words : words_next, rd + 1 < rounds ? rd + 1 : 0, v);
                store_bits(nib, rd, i);
                next_pair(i, q);
            }
            __syncthreads();
            // evaluation and selection (leaders kept); the DE draws of the
            // next generation
            fused_fitness<TAB_LDS>(a, L, lds, tabs, Cr, Ci, has_de ? SEL_GREEDY_OMEGA : SEL_MOVE,
                                   make_int4(L0, L1, L2, -1));
            if (has_de && tid < np) dr[tid] = d_next;
            __syncthreads();
            // the leaders of the next generation (and those reported)
            if (!has_de) fused_leaders(fs, cur, np, sl);
        }
        if constexpr (!OWN) {
            words = words_next;
            take = take_next;
        }
        Fg = F_next;
    }

    // write back: every row to buffer 0 with its flag cleared
    for (int k = tid; k < np * Q; k += kFusedThreads) {
        const int r = k / Q, q = k % Q;
        const float4 x = quad(cur[r].x + 16 * q);
        float *dst = a.x0 + r * a.ldx + 4 * q;
        if (4 * q + 3 < D) {
            *reinterpret_cast<float4 *>(dst) = x;
        } else {
            dst[0] = x.x;
            if (4 * q + 1 < D) dst[1] = x.y;
            if (4 * q + 2 < D) dst[2] = x.z;
        }
    }
    if (tid < np) {
        if (a.f32)
            static_cast<float *>(a.f_cur)[tid] = static_cast<float>(fs[tid]);  // (exact: fs holds binary32 values)
        else
            static_cast<double *>(a.f_cur)[tid] = fs[tid];
        a.flags[tid] = 0u;
    }
    for (int k = tid; k < a.nfb; k += kFusedThreads) a.fbits[k] = 0u;
    if (tid < 3) a.leaders[tid] = sl[tid];
    if (tid == 0) a.gen[0] = g;
}

}  // namespace

bool fused_eligible(int64_t np, int64_t D)
{
    if (np < 4 || np > 64 || D < 1) return false;
    const int W = static_cast<int>((D + 31) / 32);
    // (20480 genes at most in each buffer, and at most 64 x 7 padding quads:
    // 6 rounds)
    return fused_layout(np, D, W, false).total <= kFusedMaxLds;
}

size_t fused_words_bytes(int64_t np, int64_t D, int gens)
{
    return fused_words(np, static_cast<int>((D + 31) / 32)).stride * static_cast<size_t>(gens);
}

qpm_status launch_fused_generations(const FusedRun &fr, int gens, hipStream_t s)
{
    QPM_REQUIRE(fused_eligible(fr.np, fr.D), QPM_EINVAL, "population does not fit the fused generation kernel");
    QPM_REQUIRE(fr.variant == 0 || fr.variant == 1, QPM_EINVAL, "fused generations take gwo_variant 0 or 1");
    FusedArgs a;
    a.x0 = fr.x0;
    a.x1 = fr.x1;
    a.flags = fr.flags;
    a.fbits = fr.fbits;
    a.f_cur = fr.f_cur;
    a.f32 = fr.f32;
    a.leaders = fr.leaders;
    a.gen = fr.gen;
    a.a_tab = fr.a_tab;
    a.F_tab = fr.F_tab;
    a.tab64 = fr.tab64;
    a.C = fr.C;
    a.np = fr.np;
    a.D = fr.D;
    a.ldx = fr.ldx;
    a.W = static_cast<int>((fr.D + 31) / 32);
    a.nfb = static_cast<int>(2 * ((fr.np + 63) / 64));
    a.gens = gens;
    a.algo = fr.algo;
    a.cr_max = cr_threshold(fr.CR);
    a.k0 = static_cast<uint32_t>(fr.seed);
    a.k1 = static_cast<uint32_t>(fr.seed >> 32);
    a.inst = fr.inst;
    a.words = static_cast<unsigned char *>(fr.words);
    QPM_REQUIRE(fr.words != nullptr && gens >= 1 && gens <= fr.words_gens && gens <= 65535, QPM_EINVAL,
                "the workspace holds the random numbers of %d generations (got %d)", fr.words_gens, gens);
    const FusedWords fw = fused_words(fr.np, a.W);
    QPM_REQUIRE(fw.slots <= kFusedMaxRounds * kFusedThreads, QPM_EINVAL, "too many gene quads for one workgroup");
    // A launch for the random numbers costs about 2.5 us, making them in one
    // workgroup 0.7 us a generation and round. us per generation, with the launch /
    // without, HWSDA FP64: 100 x 16 (1 round) one generation 11.6 / 9.2, three 6.0 /
    // 5.7; 256 x 32 (2) one 16.0 / 14.8, two 11.1 / 11.6; 1000 x 16 (4) one 29.1 /
    // 28.1; 300 x 64 (5) one 32.4 / 33.0. DE alone, 100 x 16: 9.9 / 7.4, 4.2 / 3.7.
    const int rounds = fw.slots / kFusedThreads;
    const bool own = gens * rounds <= (gens == 1 ? 4 : 3);
    if (!own) {
        fused_words_kernel<<<dim3(kFusedThreads / 256, static_cast<unsigned>(gens)), 256, 0, s>>>(a);
        QPM_TRY_HIP(hipGetLastError());
    }
    const bool tab_lds = fused_layout(fr.np, fr.D, a.W, true).total <= kFusedMaxLds;
    const size_t lds = fused_layout(fr.np, fr.D, a.W, tab_lds).total;
#define QPM_FUSED_OWN(V, T, O)                                                                                   \
    {                                                                                                            \
        QPM_TRY_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&fused_gen_kernel<V, T, O>),              \
                                        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));     \
        fused_gen_kernel<V, T, O><<<1, kFusedThreads, lds, s>>>(a);                                              \
    }
#define QPM_FUSED(V, T)                                                                                          \
    {                                                                                                            \
        if (own) QPM_FUSED_OWN(V, T, true) else QPM_FUSED_OWN(V, T, false)                                       \
    }
    if (fr.variant == 1) {
        if (tab_lds) QPM_FUSED(1, true) else QPM_FUSED(1, false)
    } else {
        if (tab_lds) QPM_FUSED(0, true) else QPM_FUSED(0, false)
    }
#undef QPM_FUSED
#undef QPM_FUSED_OWN
    QPM_TRY_HIP(hipGetLastError());
    return QPM_OK;
}

}  // namespace qpm
