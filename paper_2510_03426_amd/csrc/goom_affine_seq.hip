// Linear recurrence with bias, h_t = A_t h_{t-1} + b_t over GOOMs (paper Section 4.3), float components, d = 32, for
// batches of many sequences: one workgroup walks one whole sequence, step after step, and reads every matrix once.
//
// With a hundred sequences or more there is no need to cut a sequence into chunks (whose products cost a matrix-matrix
// product per step and a second pass over the matrices): a workgroup keeps a dozen of its sequence's matrices in
// flight, which is enough outstanding memory traffic per compute unit, and a step is a matrix-vector product.  The
// work of a step falls into a part that does not depend on the running vector and a chain that does, and the
// waves of the workgroup are split accordingly, so that the first fills the waits of the second; two more waves bring the
// biases in and the states out:
//
//   * matrix waves scale the matrices, one step ahead: a lane loads four adjacent entries of a row (eight lanes a row,
//     eight rows a wave), the row's lanes agree on its power-of-two shift n_i, and (+-) 2^(log2|A_ij| - n_i) goes to
//     LDS with n_i; what the chain needs of the row's bias (a whole-number exponent at or above its log2
//     magnitude, its log-magnitude, its sign bit) lies there too;
//   * chain waves run the chain: the vector lives in LDS as float mantissas with one whole-number exponent per group of
//     eight entries (the rows one wave produces); a lane reads four scaled entries of its row and its four entries of
//     the vector, brings these to the largest group exponent G, and the row's eight lanes add up their products: entry
//     i of A_t h is that sum times 2^(n_i + G).  The bias b_i joins on the new exponent of the wave's eight rows (the
//     largest of the eight sums' and the eight bias terms' exponents), the wave writes eight mantissas and that exponent.
//
// The adjoint recurrence is walked the same way, backwards over the forward pass's matrices as they are stored, and writes the
// gradients: while the chain applies A_t^T to lam_t, the matrix waves that still hold A_t's entries form
// lam_t[i] A_t[i, j] h_{t-1}[j] from them and store it, others scale the next matrix, and two more waves bring h_{t-1} to LDS and write the
// bias's gradient.  A pass of its own over the matrices for the gradients took almost as long as the walk: 128 x 4096 x 32,
// 1336 + 1212 us, in one walk 1567 to 1633.
//
// One workgroup barrier ends a step (285 ns, adjoint 380: the chain's dependent instructions and LDS reads; longer rings and contiguous loads
// change nothing): scaled matrices, mantissas and exponents alternate between two sets of LDS words.
// The state of step t - 1 leaves during step t: as a GOOM, and / or as the scaled exponential of Section 4.3, eq. 27
// with its log-scaling constant.  Nothing but A_t, b_t (read once) and the outputs (written once) touches HBM; the chain
// waves touch no memory but LDS.
#include "goom_chain_fast.h"
#include <type_traits>

namespace goom_chain {

namespace {

constexpr int kSeqDepth = 8;          // steps written out per round of the chain waves' loop
constexpr int kSeqRing = 12;          // matrices of a sequence in flight (more change nothing)
constexpr int kSeqRingAdj = 8;        // ... for each of the two sets of matrix waves of the adjoint recurrence
constexpr int kSeqNone = -(1 << 28);  // exponent of a group of zeros
constexpr int kSeqExpLimit = 1 << 27; // whole-number exponents are kept inside +- this
constexpr int kSeqD = 32;
constexpr int kSeqCol = 34; // (eight lanes that write a column's entries and eight that read it fall on few of the same banks, and pairs are aligned)
// waves: four (adjoint recurrence: eight) for the matrices, four for the chain, two for what enters and leaves beside them
constexpr int kSeqThreads = 10 * 64, kSeqThreadsAdj = 14 * 64;

struct SeqArgs {
    const unsigned char *A;    // [batch, T, 32, 32] complex64
    const unsigned char *bias; // [batch, T, 32] complex64
    const unsigned char *h0;   // NULL (zero) or [batch, 32] complex64
    unsigned char *out_goom;   // NULL or [batch, T, 32] complex64
    float *out_scaled;         // NULL or [batch, T, 32]
    float *out_logscale;       // NULL or [batch, T]
    long long T;
    // adjoint recurrence (step s of it belongs to time t = T - 1 - s): bias is then G_t / h_t times 2^(c_t), in order of s
    const int *scale;                 // [batch, T], in order of s: the whole numbers c_t
    const unsigned char *states;      // [batch, T, 32] (float mantissa, int exponent) pairs, in order of t: the entries of h_{t-1} 2^(-c_t)
    const unsigned char *fwd_bias;    // [batch, T, 32] complex64: the forward pass's bias
    float *grad_A;                    // [batch, T, 32, 32]
    float *grad_bias;                 // NULL or [batch, T, 32]
};

struct SeqShared {
    alignas(16) float sv[2][kSeqD * kSeqCol]; // scaled, signed entries of a step's matrix, by rows of 32 (adjoint recurrence: by columns, kSeqCol words each)
    int nrow[2][kSeqD];             // the rows' shifts n_i
    alignas(16) int ngroup[2][4];   // adjoint recurrence: one shift for the eight rows of a wave
    alignas(16) int4 rec[2][kSeqD]; // per row: its bias's whole-number exponent, log-magnitude (float bits) and sign bit
    alignas(16) float m[2][kSeqD];  // mantissas of the vector
    alignas(16) int2 hp[2][kSeqD];  // adjoint recurrence: the entries of h_{t-1} 2^(-c_t), mantissa (float bits) and whole-number exponent
    int q[2];                       // adjoint recurrence: c_s - c_{s-1}
    alignas(16) int f[2][4];    // exponent of entries 8 w .. 8 w + 7 (the rows chain wave w produces)
};

// Workgroup barrier that orders LDS traffic only: the matrices in flight from HBM stay in flight across it (the
// general barrier would wait for every outstanding load, and with it for the whole ring of prefetched steps).
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The rings of prefetched steps: loads the compiler does not track (it would make every step wait for the loads issued in it,
// to copy what they fetched to the registers of the step that consumes it), issued and awaited by hand.  A load's registers
// pass through the wait before their first use, so nothing reads them earlier; a wave's vector-memory loads return in the
// order of issue, stores among them (a wait counts both).
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ inline void load_matrix_part(f4 &x, f4 &y, const unsigned char *p)
{
    asm volatile("global_load_dwordx4 %0, %2, off\n\tglobal_load_dwordx4 %1, %2, off offset:16" : "=&v"(x), "=&v"(y) : "v"(p) : "memory");
}
// what was issued a ring's length ago has landed once at most NEWER younger loads and stores are outstanding
template <int NEWER> __device__ inline void wait_matrix_part(f4 &x, f4 &y) { asm volatile("s_waitcnt vmcnt(%2)" : "+v"(x), "+v"(y) : "n"(NEWER) : "memory"); }

template <int I, int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

constexpr float kSeqHi = 1.44269502162933349609375f; // float nearest log2(e)
constexpr float kSeqLo = 1.925963033500011e-8f;      // log2(e) - kSeqHi

// whole-number exponent at or above log2 of a magnitude given by its natural logarithm; kSeqNone for a zero
__device__ inline int exponent_above(float re)
{
    const float e = __builtin_amdgcn_fmed3f(__builtin_ceilf(re * kSeqHi), -(float)kSeqExpLimit, (float)kSeqExpLimit);
    return re > -__builtin_huge_valf() ? (int)e : kSeqNone;
}
// (+-) 2^(re log2(e) - f) for a whole number f, the product with log2(e) carried in two floats
__device__ inline float scaled_term(float re, float im, int f)
{
    float x = __builtin_fmaf(re, kSeqHi, -(float)f);
    x = __builtin_fmaf(re, kSeqLo, x);
    return Comp<float>::apply_sign(__builtin_amdgcn_exp2f(x), im);
}

// log2 of a magnitude, given by its natural logarithm, as a whole number and what is left of it: between -1.5 and -0.5 (-inf for a zero), where
// it is rounded to the nearest 2^-24 or so.  The hardware exponential cuts off what a smaller argument has below that, always downwards:
// between -0.5 and 0.5 the adjoint lost 1.5e-6 of its size in 512 steps that way, here 3e-7.
struct WholeFrac {
    int whole;
    float frac;
};
__device__ inline WholeFrac whole_frac(float re)
{
    const float k = __builtin_amdgcn_fmed3f(__builtin_rintf(__builtin_fmaf(re, kSeqHi, 1.0f)), -(float)kSeqExpLimit, (float)kSeqExpLimit);
    return WholeFrac{(int)k, __builtin_fmaf(re, kSeqLo, __builtin_fmaf(re, kSeqHi, -k))};
}
// the parity of round(im / pi) as a sign bit
__device__ inline int sign_bit(float im) { return __builtin_bit_cast(int, __builtin_fmaf(im, 0.318309886183790671538f, 12582912.0f)) << 31; }
__device__ inline float with_sign(float v, int bit) { return __builtin_bit_cast(float, __builtin_bit_cast(int, v) | bit); }
typedef float f4a __attribute__((ext_vector_type(4), aligned(4))); // (a gradient's array may start at any float)

// ---- the matrices, one step ahead of the chain
// ADJ: the adjoint recurrence, read from the forward pass's matrices: step s applies the transpose of matrix T - s times
// 2^(c_s - c_{s-1}) (a zero matrix for s = 0; the chain applies the power to its sums).  The matrix is loaded and scaled as it is stored, row by row (the same contiguous loads
// as in the forward pass); the chain reads it by columns, and the shift of a stored row j goes with entry j of the vector.  An entry
// stays in registers one step longer, as a signed mantissa in [0.7, 1.42] and a whole-number exponent of its own: with the adjoint's
// entry and the earlier state's in the same form its gradient is two products and one change of exponent, whatever the three
// magnitudes are.  One more matrix, A_0, is read for its gradient alone.
// SETS: sets of four waves that take turns; set P has the matrices of steps j = P mod SETS and SETS steps of the chain's time for each.  With
// one set the gradients held the adjoint walk up (128 x 4096: 1706 us, with two 1567); without them one is enough (1175 / 1180).
template <bool ADJ, int SETS, int P, int DEPTH> __device__ __forceinline__ void seq_matrix_waves(const SeqArgs &a, SeqShared &s, int wave, int lane)
{
    static_assert(SETS == (ADJ ? 2 : 1) && SETS * DEPTH % 2 == 0, "a step's place in a round says which LDS set it has");
    typedef Comp<float> C;
    constexpr int D = kSeqD, ROUND = SETS * DEPTH;
    const long long T = a.T;
    const size_t item = blockIdx.x;
    const int row = 8 * wave + (lane >> 3); // eight lanes a row
    const int cq = lane & 7;                // the lane's columns: 4 cq .. 4 cq + 3
    const unsigned char *Ap = a.A + item * (size_t)T * (D * D * 8) + (size_t)(row * D + 4 * cq) * 8;
    [[maybe_unused]] float *gp = ADJ ? a.grad_A + item * (size_t)T * (D * D) + (size_t)(row * D + 4 * cq) : nullptr;

    // slot (j / SETS) mod DEPTH: the lane's four entries of the matrix of step j
    f4 ra[DEPTH], rb[DEPTH];
    // Loads issued after a slot's own until its turn comes again, and (adjoint recurrence) gradients stored: one for every slot loaded
    // from the start on, where they are zeros that the set's first gradient replaces (T is at least 2), so that the number is the same all the way.
    constexpr int kNewer = 2 * (DEPTH - 1) + (ADJ ? DEPTH : 0);
    auto load_slot = [&](auto sc, long long j) { // factor of step j (past the end: the last one again)
        constexpr int k = decltype(sc)::value;
        const long long src = !ADJ ? (j < T ? j : T - 1) : j <= 0 ? T - 1 : j < T ? T - j : 0; // (adjoint recurrence, step T: A_0, for its gradient)
        load_matrix_part(ra[k], rb[k], Ap + (size_t)src * (D * D * 8));
    };
    auto wait_slot = [&](auto sc) {
        constexpr int k = decltype(sc)::value;
        wait_matrix_part<kNewer>(ra[k], rb[k]);
    };
    auto store_zeros = [&]() { // to the place of this set's first gradient (by the wave that writes it: its stores stay in order); in asm, that it stays
        const f4 z = {0.0f, 0.0f, 0.0f, 0.0f};
        asm volatile("global_store_dwordx4 %0, %1, off" : : "v"(gp + (size_t)(T - 2 + P) * (D * D)), "v"(z) : "memory");
    };
    static_for<0, DEPTH>([&](auto sc) {
        load_slot(sc, SETS * decltype(sc)::value + P);
        if constexpr (ADJ) store_zeros();
    });

    // adjoint recurrence: the entries scaled last, mantissas and exponents
    [[maybe_unused]] float held[4];
    [[maybe_unused]] int heldx[4];
    // the lane's four entries scaled by a power of two (in the forward pass, the row's) and signed, to LDS set `set`
    auto scale_rows = [&](auto sc, int set, [[maybe_unused]] auto first) {
        constexpr int k = decltype(sc)::value;
        const f4 x = ra[k], y = rb[k];
        const float re[4] = {x[0], x[2], y[0], y[2]};
        const float im[4] = {x[1], x[3], y[1], y[3]};
        if constexpr (ADJ) {
            int n;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const WholeFrac w = whole_frac(re[e]); // (a zero: exponent -kSeqExpLimit, mantissa 2^-inf = 0; a NaN stays one)
                heldx[e] = w.whole;
                held[e] = with_sign(__builtin_amdgcn_exp2f(w.frac), sign_bit(im[e]));
            }
            // one shift for the wave's eight rows: they are the group of entries that share an exponent in the vector
            n = C::imax(C::imax(heldx[0], heldx[1]), C::imax(heldx[2], heldx[3]));
            n = C::imax(n, C::dpp<0xB1>(n));
            n = C::imax(n, C::dpp<0x4E>(n));
            n = C::imax(n, C::dpp<0x141>(n));
            n = C::imax(n, C::dpp<0x140>(n));
            n = C::xor16_imax(n);
            n = C::xor32_imax(n);
            constexpr bool kZero = decltype(first)::value;
#pragma unroll
            for (int e = 0; e < 4; ++e) s.sv[set][(4 * cq + e) * kSeqCol + row] = kZero ? 0.0f : __builtin_ldexpf(held[e], heldx[e] - n);
            // (rows of zeros are down at -kSeqExpLimit and do not set the scale of the vector)
            if (lane == 0) s.ngroup[set][wave] = kZero ? -kSeqExpLimit : n;
        } else {
            int key = C::key_of(vmax_raw(vmax_raw(re[0], re[1]), vmax_raw(re[2], re[3])) * kSeqHi);
            key = C::imax(key, C::dpp<0xB1>(key));
            key = C::imax(key, C::dpp<0x4E>(key));
            key = C::imax(key, C::dpp<0x141>(key));
            const float mx = C::of_key(key);
            const bool zero_row = !(mx > -1.0e30f);
            const float nf = zero_row ? 0.0f : __builtin_amdgcn_fmed3f(__builtin_ceilf(mx), -(float)kSeqExpLimit, (float)kSeqExpLimit);
            const float nsub = zero_row ? __builtin_huge_valf() : nf;
            f4 sv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float xx = __builtin_fmaf(re[e], kSeqHi, -nsub);
                xx = __builtin_fmaf(re[e], kSeqLo, xx);
                sv[e] = with_sign(__builtin_amdgcn_exp2f(xx), sign_bit(im[e])); // 2^-inf = 0 covers zero entries and zero rows
            }
            *reinterpret_cast<f4 *>(&s.sv[set][row * D + 4 * cq]) = sv;
            if (cq == 0) s.nrow[set][row] = (int)nf;
        }
    };
    // adjoint recurrence, while the chain takes step t: the gradient of matrix T - t, whose entries are still held, from the adjoint
    // of step t - 1 (what the chain reads) and the state before it
    auto write_gradient = [&](long long t) {
        constexpr int par = P; // t mod 2
        const float mi = s.m[par ^ 1][row];
        const int fi = s.f[par ^ 1][wave];
        const int4 h01 = *reinterpret_cast<const int4 *>(&s.hp[par][4 * cq]), h23 = *reinterpret_cast<const int4 *>(&s.hp[par][4 * cq + 2]);
        const int hm[4] = {h01.x, h01.z, h23.x, h23.z}, he[4] = {h01.y, h01.w, h23.y, h23.w};
        f4a o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = __builtin_ldexpf(held[e] * (mi * __builtin_bit_cast(float, hm[e])), heldx[e] + fi + he[e]);
            o[e] = v;
        }
        // a NaN passes no gradient on, nor does an infinity beside a zero (one look at all four)
        const float any = (o[0] + o[1]) + (o[2] + o[3]);
        if (__builtin_amdgcn_ballot_w64(any != any) != 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = o[e] == o[e] ? o[e] : 0.0f;
        }
        *reinterpret_cast<f4a *>(gp + (size_t)(T - t) * (D * D)) = o;
    };

    // the factor of step 0, before the chain's first step
    if constexpr (P == 0) {
        wait_slot(std::integral_constant<int, 0>{});
        scale_rows(std::integral_constant<int, 0>{}, 0, std::true_type{});
        load_slot(std::integral_constant<int, 0>{}, ROUND);
    }
    lds_barrier();

    // While the chain takes step t, the set whose turn it is scales the matrix of step t + 1; in the adjoint recurrence the other one forms the gradient
    // of this step's matrix.  u = t mod ROUND picks the ring's registers and the LDS set at compile time.
    auto step = [&](auto uc, auto prefetch, long long t) {
        constexpr int u = decltype(uc)::value;
        constexpr bool kPrefetch = decltype(prefetch)::value; // false after the last full round: the rest of the sequence has landed
        constexpr int slot = (u + 1) / SETS % DEPTH;
        typedef std::integral_constant<int, slot> S;
        if constexpr ((u + 1) % SETS == P) {
            if constexpr (kPrefetch) wait_slot(S{});
            scale_rows(S{}, (u + 1) & 1, std::false_type{}); // (past the end: not read by the chain)
            // the registers are free: the set's matrix a round on (every round issues its loads)
            if constexpr (kPrefetch) load_slot(S{}, t + 1 + ROUND);
        } else {
            if (u > 0 || t > 0)
                write_gradient(t);
            else
                store_zeros();
        }
        lds_barrier();
    };
    long long tb = 0;
    for (; tb + ROUND <= T; tb += ROUND) static_for<0, ROUND>([&](auto uc) { step(uc, std::true_type{}, tb + decltype(uc)::value); });
    // Everything still in flight lands before the last, partial round: from here on the compiler is free to reuse a ring register
    // that no step reads any more, and a load still on its way would overwrite whatever it put there.
    static_for<0, DEPTH>([&](auto sc) { // (every register of the ring passes a wait for all of them)
        constexpr int k = decltype(sc)::value;
        wait_matrix_part<0>(ra[k], rb[k]);
    });
    const int rest = (int)(T - tb); // (the same for the whole workgroup)
    static_for<0, ROUND - 1>([&](auto uc) {
        if (rest > decltype(uc)::value) step(uc, std::false_type{}, tb + decltype(uc)::value);
    });
    if constexpr (ADJ) {
        if ((T & 1) == P) write_gradient(T); // A_0
    }
}

// ---- the chain
// ADJ: the step's matrix lies in LDS by columns, its rows scaled by one shift for every eight, and is applied transposed: entry i of the product is
// the sum over j of (entry (j, i)) (entry j of the vector) 2^(n_g(j)), so n_g joins the exponent of group g of the vector.
template <bool ADJ> __device__ __forceinline__ void seq_chain_waves(const SeqArgs &a, SeqShared &s, int kw, int lane)
{
    typedef Comp<float> C;
    constexpr int D = kSeqD;
    const long long T = a.T;
    const size_t item = blockIdx.x;
    const int row = 8 * kw + (lane >> 3);
    const int cq = lane & 7;
    const int src_group = cq >> 1; // the group the lane's four entries of the vector belong to
    const float kNegInf = -__builtin_huge_valf();

    // the starting vector goes to the set of LDS words that step 0 reads
    if (kw == 0) {
        const int ent = lane & 31;
        float2 v = float2{kNegInf, 0.0f};
        if (a.h0) v = *reinterpret_cast<const float2 *>(a.h0 + (item * D + ent) * 8);
        int f = exponent_above(v.x);
        f = C::imax(f, C::dpp<0xB1>(f));
        f = C::imax(f, C::dpp<0x4E>(f));
        f = C::imax(f, C::dpp<0x141>(f)); // the eight entries of a group sit in eight adjacent lanes
        s.m[1][ent] = v.x > kNegInf ? scaled_term(v.x, v.y, f) : 0.0f;
        if ((lane & 7) == 0) s.f[1][ent >> 3] = f;
    }
    lds_barrier();

    auto step = [&](auto uc, auto, long long) {
        constexpr int u = decltype(uc)::value;
        constexpr int rs = (u + 1) & 1, ws = u & 1; // sets of the vector read and written (tb is a multiple of the depth, which is even)
        constexpr int ms = u & 1;                   // set of the scaled matrix
        const int4 rec = s.rec[ms][row]; // the row's bias: exponent, log-magnitude, sign
        const int eb = rec.x;
        const float bre = __builtin_bit_cast(float, rec.y);
        const f4 hm = *reinterpret_cast<const f4 *>(&s.m[rs][4 * cq]);
        int fsrc = s.f[rs][src_group];
        int4 fa = *reinterpret_cast<const int4 *>(&s.f[rs][0]);
        f4 sv;
        int n;
        if constexpr (ADJ) {
            // ---- row i of A^T h: the lane's entries j = 4 cq .. 4 cq + 3 of column i; the rows' shift joins the exponent of their group of the
            // vector
            const float2 s01 = *reinterpret_cast<const float2 *>(&s.sv[ms][row * kSeqCol + 4 * cq]);
            const float2 s23 = *reinterpret_cast<const float2 *>(&s.sv[ms][row * kSeqCol + 4 * cq + 2]);
            sv = f4{s01.x, s01.y, s23.x, s23.y};
            const int4 na = *reinterpret_cast<const int4 *>(&s.ngroup[ms][0]);
            fa = int4{fa.x + na.x, fa.y + na.y, fa.z + na.z, fa.w + na.w};
            fsrc += s.ngroup[ms][src_group];
            n = s.q[ms]; // from the scale of the step before to this one's
        } else {
            // ---- row i of A_t h_{t-1}
            sv = *reinterpret_cast<const f4 *>(&s.sv[ms][row * D + 4 * cq]);
            n = s.nrow[ms][row];
        }
        // the eight lanes' products on the exponent n + G
        const int G = C::imax(C::imax(fa.x, fa.y), C::imax(fa.z, fa.w));
        float part = sv[0] * hm[0];
        part = __builtin_fmaf(sv[1], hm[1], part);
        part = __builtin_fmaf(sv[2], hm[2], part);
        part = __builtin_fmaf(sv[3], hm[3], part);
        part = __builtin_ldexpf(part, fsrc - G); // (between -2^30 and 0: the hardware's change of exponent gives a zero far down)
        part = add_dpp<0xB1>(part);
        part = add_dpp<0x4E>(part);
        part = add_dpp<0x141>(part);
        // ---- new exponent of the wave's eight entries: the largest among the eight sums and the eight bias terms
        int ep;
        (void)__builtin_frexpf(part, &ep);
        int F = C::imax(part != 0.0f ? ep + n + G : kSeqNone, eb);
        F = C::imax(F, C::dpp<0x140>(F)); // the other row in these sixteen lanes
        F = C::xor16_imax(F);
        F = C::xor32_imax(F);
        F = F < kSeqNone ? kSeqNone : (F > 2 * kSeqExpLimit ? 2 * kSeqExpLimit : F); // (float log-magnitudes resolve nothing out there)
        const int up = n + G - F; // at most 0 for a non-zero sum
        float mant = __builtin_ldexpf(part, up > -300 ? (up < 300 ? up : 300) : -300);
        float xb = __builtin_fmaf(bre, kSeqHi, -(float)F); // the bias on that exponent (a zero bias, log-magnitude -inf, adds 2^-inf = 0)
        xb = __builtin_fmaf(bre, kSeqLo, xb);
        mant += __builtin_bit_cast(float, __builtin_bit_cast(int, __builtin_amdgcn_exp2f(xb)) | rec.z);
        const bool none = __builtin_amdgcn_ballot_w64(mant != 0.0f) == 0; // a group of zeros carries no exponent
        if (cq == 0) s.m[ws][row] = mant;
        if (lane == 0) s.f[ws][kw] = none ? kSeqNone : F;
        lds_barrier();
    };
    long long tb = 0;
    for (; tb + kSeqDepth <= T; tb += kSeqDepth) {
        step(std::integral_constant<int, 0>{}, std::true_type{}, tb);
        step(std::integral_constant<int, 1>{}, std::true_type{}, tb + 1);
        step(std::integral_constant<int, 2>{}, std::true_type{}, tb + 2);
        step(std::integral_constant<int, 3>{}, std::true_type{}, tb + 3);
        step(std::integral_constant<int, 4>{}, std::true_type{}, tb + 4);
        step(std::integral_constant<int, 5>{}, std::true_type{}, tb + 5);
        step(std::integral_constant<int, 6>{}, std::true_type{}, tb + 6);
        step(std::integral_constant<int, 7>{}, std::true_type{}, tb + 7);
    }
    const int rest = (int)(T - tb);
    if (rest > 0) step(std::integral_constant<int, 0>{}, std::false_type{}, tb);
    if (rest > 1) step(std::integral_constant<int, 1>{}, std::false_type{}, tb + 1);
    if (rest > 2) step(std::integral_constant<int, 2>{}, std::false_type{}, tb + 2);
    if (rest > 3) step(std::integral_constant<int, 3>{}, std::false_type{}, tb + 3);
    if (rest > 4) step(std::integral_constant<int, 4>{}, std::false_type{}, tb + 4);
    if (rest > 5) step(std::integral_constant<int, 5>{}, std::false_type{}, tb + 5);
    if (rest > 6) step(std::integral_constant<int, 6>{}, std::false_type{}, tb + 6);
}

// ---- the states out.  While the chain takes step t it reads the state of step t - 1 from LDS and stores it, so that
// neither the chain nor the matrix waves ever wait for a logarithm or a store.
__device__ __forceinline__ void seq_output_wave(const SeqArgs &a, SeqShared &s, int lane)
{
    typedef Comp<float> C;
    constexpr int D = kSeqD;
    const long long T = a.T;
    const size_t item = blockIdx.x;
    const int ent = lane & 31; // the entry this lane handles (the upper half of the wave repeats the lower and stores nothing)
    unsigned char *og = a.out_goom ? a.out_goom + item * (size_t)T * (D * 8) + (size_t)ent * 8 : nullptr;
    float *os = a.out_scaled ? a.out_scaled + item * (size_t)T * D + ent : nullptr;
    float *ol = a.out_logscale ? a.out_logscale + item * (size_t)T : nullptr;
    const float kNegInf = -__builtin_huge_valf();
    // the state held in LDS set `set` (that of step t)
    auto write_state = [&](int set, long long t) {
        const float m = s.m[set][ent];
        const int f = s.f[set][ent >> 3];
        if (og) {
            float2 o;
            o.x = C::out_re_f(m, (float)f); // (-inf for a zero)
            o.y = m < 0.0f ? C::pi() : 0.0f;
            if (lane < D) *reinterpret_cast<float2 *>(og + (size_t)t * (D * 8)) = o;
        }
        if (os || ol) {
            // scaled exponentiation (Section 4.3, eq. 27): with c the log of the largest magnitude, exp(z_i - c + 2) is the entry over the
            // largest entry, times e^2; the exponents only enter c
            const int4 fa = *reinterpret_cast<const int4 *>(&s.f[set][0]);
            const int g = C::imax(C::imax(fa.x, fa.y), C::imax(fa.z, fa.w));
            const int down = f - g;
            const float v = __builtin_ldexpf(m, down > -300 ? down : -300);
            float am = __builtin_fabsf(v);
            am = C::group_allmax<32>(am, am);
            if (os && lane < D) os[(size_t)t * D] = am == 0.0f ? 0.0f : v * (7.38905609893065022723f * __builtin_amdgcn_rcpf(am)); // (a NaN anywhere: am is one)
            if (ol && lane == 0) ol[t] = am == 0.0f ? kNegInf : (float)(((double)C::log2_abs(am) + (double)g) * 0.693147180559945309417);
        }
    };

    lds_barrier(); // the set-up of the other waves
    for (long long t = 0; t < T; ++t) {
        if (t > 0) write_state((int)((t + 1) & 1), t - 1);
        lds_barrier();
    }
    write_state((int)((T - 1) & 1), T - 1);
}

// ---- what enters and leaves beside the matrices, one 8-byte word a lane and step; a round of kSeqDepth steps loads the words of the
// next one.  While the chain takes step t:
//   kSideBias    forward pass: puts the bias of step t + 1 into LDS (not through the matrix waves' rings: registers)
//   kSideStates  adjoint recurrence: does so too and adds the state that goes with the next step's gradient (matrix T - t - 1)
//                and what the next step's scale is above this one's
//   kSideGrad    adjoint recurrence: writes the gradient of the forward bias of time T - t, lam b, from the adjoint of step t - 1
enum SideWork { kSideBias, kSideStates, kSideGrad };
template <SideWork WORK> __device__ __forceinline__ void seq_side_wave(const SeqArgs &a, SeqShared &s, int lane)
{
    constexpr int D = kSeqD, N = kSeqDepth;
    const long long T = a.T;
    const size_t item = blockIdx.x;
    const int ent = lane & 31;
    const bool low = lane < D;                            // (kSideBias, kSideGrad: the upper half repeats the lower and stores nothing)
    const bool state_lane = WORK == kSideStates && low;   // ... kSideStates: it has the bias
    const bool bias_lane = WORK == kSideBias ? low : !low;
    const bool from_end = WORK == kSideGrad || state_lane; // words in order of t, and t falls
    const unsigned char *wp = (WORK == kSideGrad ? a.fwd_bias : state_lane ? a.states : a.bias) + item * (size_t)T * (D * 8) + (size_t)ent * 8;
    const int *scp = WORK == kSideBias ? nullptr : a.scale + item * (size_t)T;
    float *gb = WORK == kSideGrad && a.grad_bias ? a.grad_bias + item * (size_t)T * D + ent : nullptr;
    struct Word {
        float2 x;
        int c;
    };
    // word j: the bias of step j; the state or the forward bias of time T - j (j from 1 on); the scale of step j, or of that time's step j - 1
    auto load = [&](long long j) {
        const long long step = j < T ? j : T - 1, back = T - (j < 1 ? 1 : j < T ? j : T);
        Word w;
        w.x = *reinterpret_cast<const float2 *>(wp + (size_t)(from_end ? back : step) * (D * 8));
        w.c = WORK == kSideBias ? 0 : scp[WORK == kSideStates ? step : T - 1 - back];
        return w;
    };
    Word now = load(0);
    auto put = [&](int set, const Word &w) {
        if (WORK == kSideGrad) return;
        if (bias_lane) s.rec[set][ent] = int4{exponent_above(w.x.x), __builtin_bit_cast(int, w.x.x), sign_bit(w.x.y), 0};
        if (state_lane) s.hp[set][ent] = int2{__builtin_bit_cast(int, w.x.x), __builtin_bit_cast(int, w.x.y)};
        if (WORK == kSideStates && lane == 0) s.q[set] = w.c - now.c;
    };
    // the gradient of the bias of time T - t, to which `now` belongs
    auto write_bias = [&](long long t) {
        if (WORK != kSideGrad || !gb) return;
        const int par = (int)(t & 1);
        const WholeFrac b = whole_frac(now.x.x);
        const float v = __builtin_ldexpf(s.m[par ^ 1][ent] * with_sign(__builtin_amdgcn_exp2f(b.frac), sign_bit(now.x.y)), s.f[par ^ 1][ent >> 3] + b.whole - now.c);
        if (low) gb[(size_t)(T - t) * D] = v == v ? v : 0.0f;
    };
    put(0, now);
    Word cur[N], next[N];
#pragma unroll
    for (int u = 0; u < N; ++u) cur[u] = load(1 + u);
    lds_barrier(); // the set-up of the other waves
    for (long long tb = 0; tb < T; tb += N) {
#pragma unroll
        for (int u = 0; u < N; ++u) next[u] = load(tb + N + 1 + u);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const long long t = tb + u;
            if (t >= T) break; // (the same for the whole workgroup)
            if (t > 0) write_bias(t);
            put((u + 1) & 1, cur[u]);
            now = cur[u];
            lds_barrier();
        }
#pragma unroll
        for (int u = 0; u < N; ++u) cur[u] = next[u];
    }
    write_bias(T);
}

// All kinds of waves pass the same barriers: one after their set-up, one at the end of every step.
template <bool ADJ> __global__ __launch_bounds__(ADJ ? kSeqThreadsAdj : kSeqThreads) void affine_seq_kernel(SeqArgs a)
{
    __shared__ __align__(16) SeqShared s;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (ADJ) {
        if (wave < 4)
            seq_matrix_waves<true, 2, 0, kSeqRingAdj>(a, s, wave, lane);
        else if (wave < 8)
            seq_matrix_waves<true, 2, 1, kSeqRingAdj>(a, s, wave - 4, lane);
        else if (wave < 12)
            seq_chain_waves<true>(a, s, wave - 8, lane);
        else if (wave == 12)
            seq_side_wave<kSideStates>(a, s, lane);
        else
            seq_side_wave<kSideGrad>(a, s, lane);
    } else {
        if (wave < 4)
            seq_matrix_waves<false, 1, 0, kSeqRing>(a, s, wave, lane);
        else if (wave < 8)
            seq_chain_waves<false>(a, s, wave - 4, lane);
        else if (wave == 8)
            seq_output_wave(a, s, lane);
        else
            seq_side_wave<kSideBias>(a, s, lane);
    }
}

// What the adjoint recurrence walks over, 32 lanes a step (s = T - 1 - t): c_t, the whole number nearest the largest log2 magnitude of
// h_t; G_t / h_t times 2^(c_t) as GOOMs (zero where either is; all operands then have magnitudes of ordinary size, and a power of two
// comes off exactly again); h_{t-1} 2^(-c_t) as mantissas and exponents.
__global__ __launch_bounds__(256) void seq_adjoint_prepare_kernel(const float2 *__restrict__ H, const float2 *__restrict__ h0, const float *__restrict__ G,
                                                                  int *__restrict__ scale, float2 *__restrict__ bias, int2 *__restrict__ states, long long T,
                                                                  long long nsteps)
{
    constexpr int D = kSeqD;
    constexpr double kLog2e = 1.44269504088896340736, kLn2 = 0.693147180559945309417;
    const float kNegInf = -__builtin_huge_valf();
    const long long step = ((long long)blockIdx.x * 256 + threadIdx.x) / D; // b T + t
    const int i = threadIdx.x % D;
    if (step >= nsteps) return; // (half a wave at a time)
    const long long b = step / T, t = step - b * T, s = T - 1 - t;
    const float2 h = H[step * D + i];
    float top = h.x > kNegInf ? h.x : kNegInf; // (a NaN does not count)
    top = Comp<float>::group_allmax<32>(top, top);
    const bool finite = top > kNegInf && top < -kNegInf;
    const int c = finite ? (int)__builtin_rint(__builtin_fmin(__builtin_fmax((double)top * kLog2e, -(double)kSeqExpLimit), (double)kSeqExpLimit)) : 0;
    if (i == 0) scale[b * T + s] = c;
    const float g = G[step * D + i];
    const bool live = g != 0.0f && h.x > kNegInf;
    float2 o;
    o.x = live ? (float)((double)__builtin_logf(__builtin_fabsf(g)) - ((double)h.x - c * kLn2)) : kNegInf;
    o.y = live && (g < 0.0f) != (sign_bit(h.y) != 0) ? Comp<float>::pi() : 0.0f;
    bias[(b * T + s) * D + i] = o;
    float2 p = float2{kNegInf, 0.0f};
    if (t > 0) p = H[(step - 1) * D + i];
    else if (h0) p = h0[b * D + i];
    const double x = (double)p.x * kLog2e - c;
    const double k = __builtin_fmin(__builtin_fmax(__builtin_rint(x), -(double)kSeqExpLimit), (double)kSeqExpLimit);
    const float m = p.x > kNegInf ? __builtin_amdgcn_exp2f((float)(x - k)) : 0.0f; // (a NaN counts as zero)
    states[step * D + i] = int2{__builtin_bit_cast(int, with_sign(m, sign_bit(p.y))), (int)k};
}

} // namespace

// every sequence of the batch by one workgroup, start to end; the caller has checked pointers and sizes
int launch_affine_seq(goom_ctx *ctx, const void *A, const void *bias, const void *h0, void *H, void *scaled, void *logscale, long long T, long long batch)
{
    if (T <= 0 || batch <= 0) return GOOM_OK;
    if (batch > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many sequences for one launch (%lld)", batch);
    SeqArgs args = {};
    args.A = static_cast<const unsigned char *>(A);
    args.bias = static_cast<const unsigned char *>(bias);
    args.h0 = static_cast<const unsigned char *>(h0);
    args.out_goom = static_cast<unsigned char *>(H);
    args.out_scaled = static_cast<float *>(scaled);
    args.out_logscale = static_cast<float *>(logscale);
    args.T = T;
    goom::prof_begin(ctx, "affine_sequential_walk");
    hipLaunchKernelGGL(affine_seq_kernel<false>, dim3((unsigned)batch), dim3(kSeqThreads), 0, ctx->stream, args);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch affine_seq_kernel");
}

// The adjoint recurrence of every sequence and the gradients of its matrices and biases
int launch_affine_seq_adjoint(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *G, int *scale, void *adj_bias,
                              void *states, void *grad_A, void *grad_bias, long long T, long long batch)
{
    if (T < 2 || batch <= 0) return goom::fail(ctx, GOOM_EINVAL, "the adjoint walk takes sequences of two steps and more");
    if (batch * T > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    const long long nsteps = batch * T, per_block = 256 / kSeqD;
    goom::prof_begin(ctx, "affine_backward_prepare_operands");
    hipLaunchKernelGGL(seq_adjoint_prepare_kernel, dim3((unsigned)((nsteps + per_block - 1) / per_block)), dim3(256), 0, ctx->stream,
                       static_cast<const float2 *>(H), static_cast<const float2 *>(h0), static_cast<const float *>(G), scale, static_cast<float2 *>(adj_bias),
                       static_cast<int2 *>(states), T, nsteps);
    goom::prof_end(ctx);
    if (int st = goom::check_hip(ctx, hipGetLastError(), "launch seq_adjoint_prepare_kernel")) return st;
    SeqArgs args = {};
    args.A = static_cast<const unsigned char *>(A);
    args.bias = static_cast<const unsigned char *>(adj_bias);
    args.T = T;
    args.scale = scale;
    args.states = static_cast<const unsigned char *>(states);
    args.fwd_bias = static_cast<const unsigned char *>(bias);
    args.grad_A = static_cast<float *>(grad_A);
    args.grad_bias = static_cast<float *>(grad_bias);
    goom::prof_begin(ctx, "affine_sequential_adjoint");
    hipLaunchKernelGGL(affine_seq_kernel<true>, dim3((unsigned)batch), dim3(kSeqThreadsAdj), 0, ctx->stream, args);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch affine_seq_kernel");
}

} // namespace goom_chain
