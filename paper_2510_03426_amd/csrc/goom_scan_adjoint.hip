// Adjoints of the prefix scan with the gradients of the factors, for states and factors of up to 128 rows and columns: the backward
// pass walked as what it is, Lam_t = G_t / P_t + K_t, K_{t-1} = M_t^T Lam_t (K_{T-1} = 0), instead of as a scan of stacked matrices.
//
// Three kernels, all this one: chunk vectors (what a chunk's own G adds to the K that leaves it, from K = 0), carries (K at every
// chunk's end, from the chunk products A_c = M_last .. M_first, which the plain chain kernels form: K <- A_c^T K + V_c), and the
// gradients (every chunk again from its K; M_t is read once for K_{t-1} and for
//     dL / d Re M'_t[i, j] = M_t[i, j] sum_k Lam_t[i, k] P_{t-1}[j, k]).
// A chain that fills the chip by its batch alone is one chunk.
//
// A workgroup owns a chunk, wave w the columns 16 w .. of the state in the matrix instruction's layout (goom_chain_kernel.h) as
// mantissas with one power of two a column, however far the states have grown.  Rows have none: entries of a column that lie further
// apart than a mantissa reaches, entries that a chunk product has no room for (in float all of its columns are on one power of two)
// and log-magnitudes past the whole numbers used here are looked for on the way (8 to 12 % of a pass); an item in which any are found is
// left to goom_scan_adjoint_wide.hip.
//   Lam:  G_t / P_t joins a column on the larger power of two of the two; Lam goes to LDS for the other waves.
//   K:    M_t column by column on powers of two of its own (they are rows of M_t^T), through LDS; Lam is the B operand as it stands.
//   sum:  wave w takes the columns j = 16 w .. of M_t; row j of P_{t-1}, straight from memory, on the largest of its entries times
//         Lam's column's power of two; a row of Lam that lies far below 1 on its own power of two.
//
// Bound by instruction issue: at 64 x 64 a step's two products are 4096 cycles of matrix instructions a wave, and the conversions of
// M, P and G and the exponents of G / P, K and the gradients some 1300 vector instructions (which do not overlap with them on this
// chip).  64 chains of 128 complex64 64 x 64: 1759 -> 444 us against the scan of the stacked 128 x 128 factors, whose operands alone were
// written and read as 2 GB (products 68, vectors 145, carries 27, gradients 265, 10 for three launches that find no flag); 65 536 steps in one chain 13.1 -> 5.5 ms;
// 16 x 60 of 100 x 100 1476 -> 704 us; complex128, 16 x 128 of 64 x 64: 1459 -> 439 us.  Row exponents of Lam: 3 % of a step.  Loads behind a branch, which
// the optimiser makes of any selection around one, cost threefold: hence entries that are loaded first and selected afterwards.
#include "goom_chain_kernel.h"

namespace {

using namespace goom_chain;

template <typename R> struct C2;
template <> struct C2<float> { typedef float2 type; };
template <> struct C2<double> { typedef double2 type; };

template <typename R> struct AdjointArgs {
    typedef typename C2<R>::type c2;
    const c2 *M, *P, *S0;        // factors [batch][T][d][d], states [batch][T][d][m], NULL or the initial state [batch][d][m]
    const R *G;                  // gradients with respect to the states' log-magnitudes
    R *gM, *gS0;                 // gS0: NULL or [batch][d][m]
    const unsigned char *totals; // factored chunk products [batch][C]
    long long tot_stride;
    int tot_cols;
    size_t tot_mant;
    unsigned char *vecs;         // factored d x m matrices [batch][C]: chunk vectors, replaced by the K that enters each chunk
    long long vec_stride;
    int vec_cols;
    size_t vec_mant;
    int *wide;                   // [batch][C][2]: whether magnitudes lie too far apart for the walk (see Reach)
    long long T, L, C;
    int d, m;
};

enum { kVectors, kCarries, kGradients };

// Exponents are whole numbers throughout; kNone stands for "no entry" (a zero), far below any that occurs, and log-magnitudes are
// held within +-3.4e8, so that sums of three exponents stay whole numbers: a zero then needs no comparison of its own, it is an
// entry times 2^kNone.
constexpr int kNone = -500000000;

// What the walk's mantissas hold for certain.  A product of two matrices loses nothing as long as the non-zero entries of Lam (and K) lie within
// 2^kLam of their column's largest and those of M, P and the chunk products within 1 / kOtherLeast (every term is then a normal number), and exponents stay
// inside +-kFar.  A workgroup that meets what leaves that says so, and goom_scan_adjoint_wide.hip writes that item's gradients again.
template <typename R> struct Reach;
template <> struct Reach<float> {
    static constexpr int kLam = 80;
    static constexpr float kLamLeast = 0x1p-80f, kOtherLeast = 0x1p-40f;
};
template <> struct Reach<double> {
    static constexpr int kLam = 700;
    static constexpr double kLamLeast = 0x1p-700, kOtherLeast = 0x1p-300;
};
constexpr int kFar = 450000000, kNothing = 1000000000; // kNothing: the least exponent of no entry at all
constexpr double kFarLog = 3.1e8;                      // kFar, of a log-magnitude

template <typename R> struct Num;
template <> struct Num<float> {
    __device__ static float bound(float re) { return __builtin_amdgcn_fmed3f(re, -3.4e8f, 3.4e8f); }
    __device__ static int whole(float re) { return (int)__builtin_ceilf(re * 1.44269502162933349609375f); } // about re log2(e), not below
    // 2^(re log2(e) - n), re within its bounds (see Comp<float>::exp2_shifted)
    __device__ static float exp2(float re, int n)
    {
#pragma clang fp contract(off)
        const float kHi = 1.44269502162933349609375f, kLo = 1.925963033500011e-8f;
        const float p_hi = re * kHi;
        float p_lo = __builtin_fmaf(re, kHi, -p_hi);
        p_lo = __builtin_fmaf(re, kLo, p_lo);
        const float y = __builtin_amdgcn_exp2f(p_hi - (float)n);
        return __builtin_fmaf(y, p_lo * 0.693147182464599609375f, y);
    }
    __device__ static int exponent(float x) { return __builtin_amdgcn_frexp_expf(x); }
    __device__ static float mantissa(float x) { return __builtin_amdgcn_frexp_mantf(x); }
    __device__ static float larger(float a, float b) { return __builtin_fmaxf(a, b); }
    __device__ static float with_sign(float x, unsigned bits, int at) { return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, x) ^ (bits << (31 - at) & 0x80000000u)); }
};
template <> struct Num<double> {
    __device__ static double bound(double re) { return __builtin_fmin(__builtin_fmax(re, -3.4e8), 3.4e8); }
    __device__ static int whole(double re) { return (int)__builtin_ceil(re * kLog2e); }
    __device__ static double exp2(double re, int n)
    {
        const double t = __builtin_fma(re, kLog2e, -(double)n), k = __builtin_rint(t);
        return __builtin_ldexp(Comp<double>::exp2_small(t - k), (int)k);
    }
    __device__ static int exponent(double x) { return __builtin_amdgcn_frexp_exp(x); }
    __device__ static double mantissa(double x) { return __builtin_amdgcn_frexp_mant(x); }
    __device__ static double larger(double a, double b) { return __builtin_fmax(a, b); }
    __device__ static double with_sign(double x, unsigned bits, int at)
    {
        return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, x) ^ ((unsigned long long)(bits << (31 - at) & 0x80000000u) << 32));
    }
};
__device__ inline int imax(int x, int y) { return x > y ? x : y; }
__device__ inline int imin(int x, int y) { return x < y ? x : y; }
__device__ inline int column_max(int x) { return Comp<float>::xor32_imax(Comp<float>::xor16_imax(x)); } // over the four lanes of a column

// DP: rows and columns in whole tiles of sixteen
template <typename R, int DP> struct Tiles {
    static constexpr bool kOne = sizeof(R) == 8 && DP > 80;  // one tile serves Lam and M in turn
    static constexpr bool kReload = sizeof(R) == 8 && DP > 48; // M's entries are read again for the gradients instead of kept in registers
    static constexpr int kLam = DP + (sizeof(R) == 4 ? 4 : 2); // row strides, against bank conflicts
    static constexpr int kM = sizeof(R) == 4 ? DP + 4 : DP % 32 == 16 ? DP : DP + 16;
    static constexpr int kAll = kOne ? DP * (kLam > kM ? kLam : kM) : DP * (kLam + kM);
    static constexpr size_t kBytes = (size_t)kAll * sizeof(R) + 2 * DP * sizeof(int);
    static_assert(kLam * sizeof(R) % 16 == 0, "rows of Lam are read in pieces of 16 bytes");
};
// four entries of a row of Lam: rows of an odd number lie 16 bytes from a multiple of 32 in double
template <typename R> struct RowPiece;
template <> struct RowPiece<float> { typedef f4 type; };
template <> struct RowPiece<double> { typedef double type __attribute__((ext_vector_type(4), aligned(16))); };

// FULL: d = m = DP, no entry to leave out.  Comparisons, selections and addresses are a seventh of a step's vector instructions then, and registers that
// are short at 128.  Before / now: 64 x 128 of 64 x 64 499 -> 444 us, of 32 x 32 143 -> 128; 64 x 40 of 128 x 128 1268 -> 947; complex128, 16 x 30 of 128 x
// 128 2199 -> 1572.  (Loading a step ahead instead of at its start took no more off.)
template <typename R, int DP, int MODE, bool FULL> __global__ __launch_bounds__(DP * 4, sizeof(R) == 4 || DP > 64 ? 2 : 1) void scan_adjoint_kernel(AdjointArgs<R> a)
{
    typedef Comp<R> N;
    typedef typename N::vec4 vec4;
    typedef typename C2<R>::type c2;
    typedef Num<R> X2;
    typedef Tiles<R, DP> TL;
    constexpr int KT = DP / 16;
    constexpr bool EARLY = FULL && sizeof(R) == 4 && DP <= 64; // all that a step reads is loaded at its start: as far as the registers go
    extern __shared__ __align__(32) unsigned char smem[];
    R *lam = reinterpret_cast<R *>(smem);                // [DP][kLam] Lam_t's mantissas
    R *mt = TL::kOne ? lam : lam + DP * TL::kLam;        // [DP][kM] M_t, column j times 2^-mexp[j]
    int *lexp = reinterpret_cast<int *>(reinterpret_cast<R *>(smem) + TL::kAll); // Lam's column exponents
    int *mexp = lexp + DP;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15, col = 16 * w + c;
    const int d = FULL ? DP : a.d, m = FULL ? DP : a.m;
    const long long per = MODE == kVectors ? a.C - 1 : MODE == kCarries ? 1 : a.C;
    const long long b = blockIdx.x / per, chunk = MODE == kVectors ? blockIdx.x % per + 1 : MODE == kCarries ? a.C - 1 : blockIdx.x % per;

    vec4 S[KT];               // K, then Lam: entry (16 it + row_of(g, v), col), times 2^e
    int e = kNone;            // (a column of zeros)
    int low = kNothing;       // least exponent of K's non-zero entries that this lane holds
    unsigned long long lost = 0; // lanes in which something may not have fitted
    // (noted at once: the scheduler otherwise puts it off and keeps what it is formed from)
    auto note = [&](bool c) {
        lost |= __builtin_amdgcn_ballot_w64(c);
        asm("" : "+s"(lost));
    };
    typedef Reach<R> Rc;
#pragma unroll
    for (int it = 0; it < KT; ++it) S[it] = vec4{0, 0, 0, 0};

    // Entry (16 it + row_of(g, v), col) of a matrix with `rows` rows and `cols` columns: one base for the wave and an offset for the lane
    // formed where it is used (the optimiser otherwise keeps them, and the comparisons' results, for the whole loop, and spills),
    // and the first entry where there is none, so that no load is behind a branch.
    auto row_at = [&](int it, int v) { return 16 * it + N::row_of(g, v); };
    const int lim_m = col < m ? d : 0, lim_d = col < d ? d : 0; // rows of a d x m, of a d x d matrix that this lane's column has
    auto inside = [](int i, int lim) { return FULL || i < lim; };
    auto opaque = [](unsigned x) {
        asm volatile("" : "+v"(x));
        return x;
    };
    auto opaque_int = [](int x) {
        if (!FULL) asm volatile("" : "+s"(x));
        return x;
    };
    // both formed here, entry by entry (the scheduler otherwise puts one of them off and keeps what it is formed from)
    auto now = [](int &x, int &y) { asm("" : "+v"(x), "+v"(y)); };
    auto at_byte = [](const auto *base, unsigned byte) { return *reinterpret_cast<decltype(base)>(reinterpret_cast<const unsigned char *>(base) + byte); };

    auto vec_at = [&](long long q) { return a.vecs + (b * a.C + q) * a.vec_stride; };
    // (written and read whole, by the same lanes: what lies past the matrix is zero)
    const bool owns = FULL || 16 * w < a.vec_cols;
    auto load_vec = [&](long long q, vec4 (&V)[KT], int &ev) {
        const unsigned char *src = vec_at(q);
        const int at = owns ? col : 0;
#pragma unroll
        for (int it = 0; it < KT; ++it)
#pragma unroll
            for (int v = 0; v < 4; ++v) V[it][v] = reinterpret_cast<const R *>(src)[(unsigned)(row_at(it, v) * a.vec_cols + at)];
        const double ex = reinterpret_cast<const double *>(src + a.vec_mant)[at];
        ev = owns ? (int)ex : kNone;
#pragma unroll
        for (int it = 0; it < KT; ++it)
#pragma unroll
            for (int v = 0; v < 4; ++v) V[it][v] = owns ? V[it][v] : (R)0;
    };
    auto store_vec = [&](long long q) {
        unsigned char *dst = vec_at(q);
        if (owns) {
#pragma unroll
            for (int it = 0; it < KT; ++it)
#pragma unroll
                for (int v = 0; v < 4; ++v) reinterpret_cast<R *>(dst)[(unsigned)(row_at(it, v) * a.vec_cols + col)] = S[it][v];
            if (g == 0) reinterpret_cast<double *>(dst + a.vec_mant)[col] = (double)e;
        }
    };
    auto least = [&](const vec4 (&V)[KT], int ev) {
        int l = kNothing;
#pragma unroll
        for (int it = 0; it < KT; ++it)
#pragma unroll
            for (int v = 0; v < 4; ++v) l = imin(l, V[it][v] != (R)0 ? X2::exponent(V[it][v]) + ev : kNothing);
        return l;
    };
    // S 2^e + V 2^ev, on the larger of the two
    auto add_scaled = [&](const vec4 (&V)[KT], int ev) {
        const int top = imax(e, ev);
        note((low < imax(top - Rc::kLam, -kFar)) || (top > kFar));
#pragma unroll
        for (int it = 0; it < KT; ++it)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const R x = N::ldexp_(V[it][v], ev - top);
                note((N::abs_(x) < Rc::kLamLeast) && (V[it][v] != (R)0));
                S[it][v] = N::ldexp_(S[it][v], e - top) + x;
            }
        e = top;
    };
    // K = (matrix in mt)^T Lam
    auto propagate = [&]() {
        vec4 acc[KT];
#pragma unroll
        for (int jt = 0; jt < KT; ++jt) acc[jt] = vec4{0, 0, 0, 0};
#pragma unroll
        for (int it = 0; it < KT; ++it)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const R *row = &mt[row_at(it, v) * TL::kM + c];
                const R s = S[it][v];
#pragma unroll
                for (int jt = 0; jt < KT; ++jt) acc[jt] = N::mfma(row[16 * jt], s, acc[jt]);
            }
        int top = 2 * kNone;
        low = kNothing;
#pragma unroll
        for (int jt = 0; jt < KT; ++jt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const R x = acc[jt][v];
                const int ex = X2::exponent(x) + mexp[row_at(jt, v)];
                top = imax(top, x != (R)0 ? ex : 2 * kNone);
                low = imin(low, x != (R)0 ? ex : kNothing); // (kept until K has its gradient's other part)
                now(top, low);
            }
        top = column_max(top);
        low = low < kNothing ? low + e : kNothing;
#pragma unroll
        for (int jt = 0; jt < KT; ++jt)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[jt][v] = N::ldexp_(acc[jt][v], mexp[row_at(jt, v)] - top);
        e = imax(e + top, kNone); // (nothing there: e below kNone)
    };

    if constexpr (MODE == kCarries) {
        for (long long q = a.C - 1; q >= 0; --q) {
            vec4 V[KT];
            int ev;
            if (q > 0) {
                const unsigned char *tp = a.totals + (b * a.C + q) * a.tot_stride;
                const double cex = reinterpret_cast<const double *>(tp + a.tot_mant)[col < d ? col : 0]; // (in double every column on its own power of two, in float all on one)
                vec4 A[KT];
#pragma unroll
                for (int it = 0; it < KT; ++it)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        A[it][v] = reinterpret_cast<const R *>(tp)[inside(row_at(it, v), lim_d) ? (unsigned)(row_at(it, v) * a.tot_cols + col) : 0u];
                load_vec(q, V, ev);
                __syncthreads();
#pragma unroll
                for (int it = 0; it < KT; ++it)
#pragma unroll
                    for (int v = 0; v < 4; ++v) mt[row_at(it, v) * TL::kM + col] = inside(row_at(it, v), lim_d) ? A[it][v] : (R)0;
                if (g == 0) mexp[col] = col < d ? (int)__builtin_fmin(__builtin_fmax(cex, -1.0e9), 1.0e9) : 0; // (past kFar: noted with the vectors)
                __syncthreads();
                store_vec(q); // K as it enters this chunk, in its vector's place (each lane in the places it read)
                propagate();
                add_scaled(V, ev);
            } else {
                store_vec(0);
            }
        }
    } else {
        const long long lo = chunk * a.L, hi = lo + a.L < a.T ? lo + a.L : a.T;
        if (MODE == kVectors) {
            // the carries' other operand (a zero may be an entry that the product's common exponent had no room for)
            const unsigned char *total = a.totals + (b * a.C + chunk) * a.tot_stride;
            const R *tp = reinterpret_cast<const R *>(total);
            note(!(__builtin_fabs(reinterpret_cast<const double *>(total + a.tot_mant)[col < d ? col : 0]) <= (double)kFar));
#pragma unroll
            for (int it = 0; it < KT; ++it)
#pragma unroll
                for (int v = 0; v < 4; ++v) note((inside(row_at(it, v), lim_d)) && !(N::abs_(tp[inside(row_at(it, v), lim_d) ? (unsigned)(row_at(it, v) * a.tot_cols + col) : 0u]) >= Rc::kOtherLeast));
        }
        if (MODE == kGradients && a.C > 1) {
            load_vec(chunk, S, e);
            low = least(S, e);
        }
        for (long long t = hi - 1; t >= lo; --t) {
            const size_t step = (size_t)(b * a.T + t);
            const bool onward = MODE != kGradients || t > lo || (chunk == 0 && a.gS0); // is K_{t-1} of any use
            [[maybe_unused]] c2 mraw[EARLY ? KT : 1][4], praw[EARLY ? KT : 1][4]; // EARLY: M_t, and row col of P_{t-1}
            // ---- Lam = K + G / P
            {
                const c2 *Pt = a.P + step * d * m;
                const R *Gt = a.G + step * d * m;
                c2 pv[KT][4];
                R gv[KT][4];
                int nb = kNone;
                const unsigned first = opaque((unsigned)(N::row_of(g, 0) * m + col));
                const int rows = FULL ? DP : (int)opaque((unsigned)lim_m), cols = opaque_int(m);
#pragma unroll
                for (int it = 0; it < KT; ++it)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const unsigned at = inside(row_at(it, v), rows) ? first + (unsigned)((row_at(it, v) - N::row_of(g, 0)) * cols) : 0u;
                        pv[it][v] = at_byte(Pt, at * (unsigned)sizeof(c2));
                        gv[it][v] = at_byte(Gt, at * (unsigned)sizeof(R));
                    }
                if constexpr (EARLY) {
                    const c2 *Mt = a.M + step * DP * DP + N::row_of(g, 0) * DP + col;
                    const c2 *prev = (t > 0 ? Pt - (size_t)DP * DP : a.S0 ? a.S0 + (size_t)b * DP * DP : Pt) + col * DP + 4 * g;
#pragma unroll
                    for (int it = 0; it < KT; ++it)
#pragma unroll
                        for (int v = 0; v < 4; ++v) mraw[it][v] = Mt[(row_at(it, v) - N::row_of(g, 0)) * DP];
                    if (MODE == kGradients) {
#pragma unroll
                        for (int it = 0; it < KT; ++it)
#pragma unroll
                            for (int v = 0; v < 4; ++v) praw[it][v] = prev[16 * it + v];
                    }
                }
                __builtin_amdgcn_sched_barrier(0); // (all loads of a matrix in flight at once)
#pragma unroll
                for (int it = 0; it < KT; ++it)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const c2 p = pv[it][v];
                        const R x = N::apply_sign(gv[it][v], p.y), re = X2::bound(-p.x);
                        const bool in = (inside(row_at(it, v), rows)) & __builtin_isfinite(p.x) & (x != (R)0);
                        const int up = X2::whole(re) + X2::exponent(x);
                        pv[it][v].x = re;
                        gv[it][v] = in ? x : (R)0;
                        nb = imax(nb, in ? up : kNone);
                        if (MODE == kGradients) note((inside(row_at(it, v), rows)) && __builtin_isfinite(p.x) && (N::abs_(re) > (R)kFarLog));
                    }
                const int top = imax(e, column_max(nb));
                note((low < imax(top - Rc::kLam, -kFar)) || (top > kFar));
#pragma unroll
                for (int it = 0; it < KT; ++it)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const R x = gv[it][v], f = X2::mantissa(x) * X2::exp2(pv[it][v].x, top - X2::exponent(x));
                        note((N::abs_(f) < Rc::kLamLeast) && (x != (R)0));
                        S[it][v] = N::ldexp_(S[it][v], e - top) + (x != (R)0 ? f : (R)0);
                    }
                e = top;
                if (MODE == kGradients) {
#pragma unroll
                    for (int it = 0; it < KT; ++it)
#pragma unroll
                        for (int v = 0; v < 4; ++v) lam[row_at(it, v) * TL::kLam + col] = S[it][v];
                    if (g == 0) lexp[col] = e;
                }
            }
            // ---- M_t, entry (16 it + row_of(g, v), col) = my 2^mn
            const c2 *Mt = a.M + step * d * d;
            const unsigned mfirst = opaque((unsigned)(N::row_of(g, 0) * d + col));
            const int dd = opaque_int(d), mrows = FULL ? DP : (int)opaque((unsigned)lim_d);
            auto fetch_m = [&](int it, int v) {
                return at_byte(Mt, (inside(row_at(it, v), mrows) ? mfirst + (unsigned)((row_at(it, v) - N::row_of(g, 0)) * dd) : 0u) * (unsigned)sizeof(c2));
            };
            R my[KT][4];
            int mn[KT][4];
            auto split = [&](c2 x, bool in, R &y, int &n) { // y 2^n
                const R re = X2::bound(in ? x.x : N::neg_inf());
                n = X2::whole(re);
                y = N::apply_sign(X2::exp2(re, n), x.y);
            };
            auto put_m = [&]() {
                c2 x[KT][4];
#pragma unroll
                for (int it = 0; it < KT; ++it)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (EARLY)
                            x[it][v] = mraw[it][v];
                        else
                            x[it][v] = fetch_m(it, v);
                    }
                if (!EARLY) __builtin_amdgcn_sched_barrier(0);
                int sh = kNone;
                // a column's power of two: none for a column of zeros, whose entries would come out as ones
                auto column_shift = [](int x) {
                    x = column_max(x);
                    return x > -kFar ? x : 0;
                };
                if constexpr (TL::kReload) {
                    R most = -3.4e8;
#pragma unroll
                    for (int it = 0; it < KT; ++it)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            x[it][v].x = inside(row_at(it, v), mrows) ? x[it][v].x : N::neg_inf();
                            most = X2::larger(most, X2::bound(x[it][v].x));
                        }
                    sh = column_shift(X2::whole(most));
#pragma unroll
                    for (int it = 0; it < KT; ++it)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const R y = X2::exp2(X2::bound(x[it][v].x), sh);
                            note(onward && (x[it][v].x > N::neg_inf()) && (y < Rc::kOtherLeast));
                            mt[row_at(it, v) * TL::kM + col] = N::apply_sign(y, x[it][v].y);
                        }
                } else {
#pragma unroll
                    for (int it = 0; it < KT; ++it)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            split(x[it][v], inside(row_at(it, v), mrows), my[it][v], mn[it][v]);
                            sh = imax(sh, mn[it][v]);
                        }
                    sh = column_shift(sh);
#pragma unroll
                    for (int it = 0; it < KT; ++it)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const R y = N::ldexp_(my[it][v], mn[it][v] - sh);
                            note(onward && (inside(row_at(it, v), mrows)) && (x[it][v].x > N::neg_inf()) && (N::abs_(y) < Rc::kOtherLeast));
                            mt[row_at(it, v) * TL::kM + col] = y;
                        }
                }
                if (g == 0) mexp[col] = sh;
                note(onward && (sh > kFar));
            };
            if (!TL::kOne) put_m();
            __syncthreads();
            // ---- gradients of M_t
            if constexpr (MODE == kGradients) {
                const c2 *prev = t > 0 ? a.P + (step - 1) * d * m : a.S0 ? a.S0 + (size_t)b * d * m : nullptr;
                const c2 *src = prev ? prev : a.P + step * d * m; // (no S0: the identity, and nothing of what is read)
                vec4 pb[KT]; // row col of P_{t-1}, columns 16 kt + 4 g + v
                int nj = 2 * kNone;
                const unsigned pfirst = opaque((unsigned)(col * m + 4 * g));
                unsigned pneg = 0; // signs, a bit an entry
                const bool have = prev != nullptr;
                const int klim = FULL ? DP : (int)opaque((unsigned)(col < d ? m : 0));
                c2 raw[KT][4];
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (EARLY)
                            raw[kt][v] = praw[kt][v];
                        else
                            raw[kt][v] = at_byte(src, (inside(16 * kt + 4 * g + v, klim) ? pfirst + (unsigned)(16 * kt + v) : 0u) * (unsigned)sizeof(c2));
                    }
                if (!EARLY) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int k = 16 * kt + 4 * g + v;
                        const c2 x = raw[kt][v];
                        const R re = have ? x.x : k == col ? (R)0 : N::neg_inf();
                        pb[kt][v] = X2::bound(inside(k, klim) ? re : N::neg_inf());
                        pneg |= (unsigned)(have & N::is_negative(x.y)) << (4 * kt + v);
                        nj = imax(nj, X2::whole(pb[kt][v]) + lexp[k]);
                    }
                nj = column_max(nj);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        // (a zero, or a column of Lam without entries, is half a billion powers of two away; P itself was looked at as P_t)
                        const int far = nj - lexp[16 * kt + 4 * g + v];
                        const R y = X2::exp2(pb[kt][v], far);
                        note((y < Rc::kOtherLeast) && (pb[kt][v] > (R)-kFarLog) && (far < kFar));
                        pb[kt][v] = X2::with_sign(y, pneg, 4 * kt + v);
                    }
                R *out = a.gM + step * d * d;
#pragma unroll
                for (int it = 0; it < KT; ++it) {
                    R y[4];
                    int n0[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (TL::kReload) {
                            split(fetch_m(it, v), true, y[v], n0[v]); // (nothing past the matrix is stored)
                        } else {
                            n0[v] = mn[it][v];
                            y[v] = my[it][v];
                        }
                    }
                    vec4 la[KT];
                    R big = 0;
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt) {
                        la[kt] = *reinterpret_cast<const typename RowPiece<R>::type *>(&lam[(16 * it + c) * TL::kLam + 16 * kt + 4 * g]);
#pragma unroll
                        for (int v = 0; v < 4; ++v) big = X2::larger(big, N::abs_(la[kt][v]));
                    }
                    // rows 16 it + c whose largest entry is small, on a power of two of their own
                    big = N::xor16_32_max(big);
                    const bool far = __builtin_amdgcn_ballot_w64(big < (R)1.0e-9 && big > (R)0) != 0;
                    int r = 0;
                    if (far) {
                        r = X2::exponent(big);
#pragma unroll
                        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                            for (int v = 0; v < 4; ++v) la[kt][v] = N::ldexp_(la[kt][v], -r);
                    }
                    vec4 X = vec4{0, 0, 0, 0};
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int v = 0; v < 4; ++v) X = N::mfma(la[kt][v], pb[kt][v], X);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int ri = far ? __shfl(r, N::row_of(g, v), 64) : 0;
                        const R val = N::ldexp_(X[v] * y[v], n0[v] + nj + ri);
                        if (inside(row_at(it, v), mrows))
                            *reinterpret_cast<R *>(reinterpret_cast<unsigned char *>(out) + (mfirst + (unsigned)((row_at(it, v) - N::row_of(g, 0)) * dd)) * (unsigned)sizeof(R)) = val;
                    }
                }
            }
            if (TL::kOne) { // M takes Lam's place
                __syncthreads();
                put_m();
                __syncthreads();
            }
            if (onward) propagate();
            __syncthreads();
        }
        if (MODE == kVectors) store_vec(chunk);
        if (MODE == kGradients && chunk == 0 && a.S0) {
            const c2 *S0 = a.S0 + (size_t)b * d * m;
            R *out = a.gS0 ? a.gS0 + (size_t)b * d * m : nullptr;
#pragma unroll
            for (int it = 0; it < KT; ++it)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool in = inside(row_at(it, v), lim_m);
                    const c2 x = S0[in ? (unsigned)(row_at(it, v) * m + col) : 0u];
                    const R re = X2::bound(x.x);
                    const int n0 = X2::whole(re);
                    note(in && __builtin_isfinite(x.x) && N::abs_(re) > (R)kFarLog);
                    if (in && out) out[(unsigned)(row_at(it, v) * m + col)] = N::apply_sign(N::ldexp_(S[it][v] * X2::exp2(re, n0), n0 + e), x.y);
                }
        }
    }
    // a word a workgroup (the carries' where the first chunk's vector would have been)
    __syncthreads();
    if (threadIdx.x == 0) lexp[0] = 0;
    __syncthreads();
    if (lost) lexp[0] = 1;
    __syncthreads();
    if (threadIdx.x == 0) {
        int *out = a.wide + (b * a.C + (MODE == kCarries ? 0 : chunk)) * 2;
        if (MODE != kGradients || a.C == 1) out[0] = lexp[0];
        if (MODE == kGradients) out[1] = lexp[0];
    }
}

template <typename R, int DP, int MODE, bool FULL> int launch_mode(goom_ctx *ctx, const AdjointArgs<R> &a, long long grid, const char *label)
{
    const void *kern = reinterpret_cast<const void *>(scan_adjoint_kernel<R, DP, MODE, FULL>);
    const size_t lds = Tiles<R, DP>::kBytes;
    if (int st = goom::check_hip(ctx, hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds), "hipFuncSetAttribute(scan_adjoint_kernel)")) return st;
    goom::prof_begin(ctx, label);
    hipLaunchKernelGGL((scan_adjoint_kernel<R, DP, MODE, FULL>), dim3((unsigned)grid), dim3(DP * 4), lds, ctx->stream, a);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch scan_adjoint_kernel");
}

template <typename R, int DP, bool FULL> int launch_phase(goom_ctx *ctx, const AdjointArgs<R> &a, long long batch, int phase)
{
    if (phase == 0) {
        if (int st = launch_mode<R, DP, kVectors, FULL>(ctx, a, batch * (a.C - 1), "scan_adjoint_chunk_vectors")) return st;
        return launch_mode<R, DP, kCarries, FULL>(ctx, a, batch, "scan_adjoint_carries");
    }
    return launch_mode<R, DP, kGradients, FULL>(ctx, a, batch * a.C, "scan_adjoint_gradients");
}

template <typename R, int DP> int launch_dp(goom_ctx *ctx, const AdjointArgs<R> &a, long long batch, int phase)
{
    if constexpr (DP == 16 || DP == 32 || DP == 64 || DP == 128) { // (the sizes that are common)
        if (a.d == DP && a.m == DP) return launch_phase<R, DP, true>(ctx, a, batch, phase);
    }
    return launch_phase<R, DP, false>(ctx, a, batch, phase);
}

template <typename R> int launch_t(goom_ctx *ctx, const goom::ScanAdjointLaunch &l, int phase)
{
    typedef typename C2<R>::type c2;
    AdjointArgs<R> a;
    a.M = static_cast<const c2 *>(l.M);
    a.P = static_cast<const c2 *>(l.P);
    a.S0 = static_cast<const c2 *>(l.S0);
    a.G = static_cast<const R *>(l.G);
    a.gM = static_cast<R *>(l.gM);
    a.gS0 = static_cast<R *>(l.gS0);
    a.totals = static_cast<const unsigned char *>(l.totals);
    a.tot_stride = (long long)l.tot.stride;
    a.tot_cols = l.tot.cols_padded;
    a.tot_mant = l.tot.mant_bytes;
    a.vecs = static_cast<unsigned char *>(l.vecs);
    a.vec_stride = (long long)l.vec.stride;
    a.vec_cols = l.vec.cols_padded;
    a.vec_mant = l.vec.mant_bytes;
    a.wide = l.wide;
    a.T = l.T;
    a.L = l.L;
    a.C = l.C;
    a.d = l.d;
    a.m = l.m;
    switch (((l.d > l.m ? l.d : l.m) + 15) / 16) {
    case 1: return launch_dp<R, 16>(ctx, a, l.batch, phase);
    case 2: return launch_dp<R, 32>(ctx, a, l.batch, phase);
    case 3: return launch_dp<R, 48>(ctx, a, l.batch, phase);
    case 4: return launch_dp<R, 64>(ctx, a, l.batch, phase);
    case 5: return launch_dp<R, 80>(ctx, a, l.batch, phase);
    case 6: return launch_dp<R, 96>(ctx, a, l.batch, phase);
    case 7: return launch_dp<R, 112>(ctx, a, l.batch, phase);
    default: return launch_dp<R, 128>(ctx, a, l.batch, phase);
    }
}

} // namespace

namespace goom {

int launch_scan_adjoint(goom_ctx *ctx, const ScanAdjointLaunch &l, int phase)
{
    return l.dtype == GOOM_C64 ? launch_t<float>(ctx, l, phase) : launch_t<double>(ctx, l, phase);
}

} // namespace goom
