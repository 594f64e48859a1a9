// Adjoint of the recurrence h_t = A_t h_{t-1} + b_t (paper Section 4.3 with the derivatives of Section 3.1 in the limit eps -> 0):
// lam_t = G_t / h_t + A_{t+1}^T lam_{t+1}, and the gradients lam_t[i] A_t[i, j] h_{t-1}[j], lam_t[i] b_t[i] as reals.
//
// A step x <- A_t^T x needs the matrix that the gradient of step t needs, with x = lam_t at hand: one read of A_t serves both, where a
// transposed and rescaled copy of all matrices, a scan over it and a pass for the gradients read them four times and wrote them once.
// What bounds the kernel is then memory (A read, gradients written), or the latency of a step where few chains run.
//   * As in goom_vec.hip a workgroup owns a chain, a wave a band of rows, sixteen lanes a row.  The transposed product is a sum over
//     rows: a lane adds up its rows' entries of each of its columns, the four rows of a pass meet by lane swaps, the waves'
//     sums in LDS, each on a power of two of its own; after one barrier the lane that owns a row adds the waves' sums and G_t / h_t, and
//     hands mantissa and exponent to the row's sixteen lanes through LDS words of its wave.
//   * lam is kept as mantissa and exponent per entry with a double base, so no scaling of h or A comes before: adjoints of e^-1000 and
//     below are ordinary numbers here.
//   * Entries of one row, of lam and of h may lie further apart than the component type reaches (diagonal and triangular matrices, states
//     in units of their own), while lam_i A_ij h_j is an ordinary number.  So the exponents of lam_i, of the row and of h_j meet as whole numbers
//     before the gradient is formed, and the product takes one power of two a row and a wave only while nothing that is summed lies more
//     than 2^-40 (2^-320) below it; a wave that finds more gives every term an exponent of its own and every column the largest of them.
//     Looking for it costs 5 to 10 % of a step (128 x 500 matrices of float d = 64: 1160 -> 1280 us; of double d = 24: 900 -> 1140 us), the rare way twice a step's time.
//   * The same kernel walks the factored chunk products backwards (FACT): mu <- P_c^T mu + v_c.
#include "goom_vec.h"

namespace goom_chain {

namespace {

template <typename V> __device__ inline V sum_groups(V v); // over lanes l, l ^ 16, l ^ 32, l ^ 48
template <> __device__ inline float sum_groups(float v)
{
    // (the halves go through variables of their own: a bit cast of a vector's element 1 reads element 0 here)
    u2 r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    unsigned lo = r[0], hi = r[1];
    v = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
    r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    lo = r[0];
    hi = r[1];
    return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}
template <> __device__ inline double sum_groups(double v)
{
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

struct AdjointArgs {
    const unsigned char *left; // GOOM matrices [batch][T][d][d], or factored chunk products (FACT)
    long long left_batch_stride, left_step_stride;
    long long T, chunk_len, first_chunk, chunks; // chunks first_chunk .. first_chunk + chunks - 1 of every batch item
    int d, left_cols;                            // left_cols: padded columns of the factored products
    const void *bias, *h0, *H, *G;               // GOOMs [batch][T][d], NULL or [batch][d], [batch][T][d]; reals [batch][T][d]
    const unsigned char *init;                   // NULL (zero), or the vectors that enter the chunks: [batch][init_per_item] from chunk 0 on
    long long init_per_item, vec_stride;         // bytes of a vector: DP mantissas of the component type, then its exponent
    unsigned char *out_total;                    // the vector that leaves the chunk, as column d of its factored product
    long long total_stride, totals_per_item;
    unsigned char *out_vecs;                     // FACT: the vector before every step, and (step chunks) the last one
    void *gA, *gb, *gh0;                         // gradients (gb, gh0: may be NULL)
};

// whole powers of two that are added up as integers (three of them stay inside 32 bits); what they are clamped at is far beyond any result
__device__ inline int whole(float v) { return (int)__builtin_amdgcn_fmed3f(v, -5.0e8f, 5.0e8f); }
__device__ inline int whole(double v) { return (int)(v > -5.0e8 ? (v < 5.0e8 ? v : 5.0e8) : -5.0e8); }

// Keys of log-magnitudes whose largest belongs to the lowest finite one (if any is negative): the bit pattern of a negative number grows as
// it falls, and the step added takes -inf, the one above all of them, round to the bottom.  kNoDepth is the key of no entry (a NaN).
constexpr unsigned kNoDepth = 1u;
__device__ inline unsigned depth_key(float v) { return __builtin_bit_cast(unsigned, v) + 0x00800000u; }
__device__ inline unsigned depth_key(double v) { return (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32) + 0x00100000u; }
template <typename R> __device__ inline R depth_of(unsigned key);
template <> __device__ inline float depth_of<float>(unsigned key) { return __builtin_bit_cast(float, key - 0x00800000u); }
template <> __device__ inline double depth_of<double>(unsigned key) { return __builtin_bit_cast(double, (unsigned long long)(key - 0x00100000u) << 32); }

// A wave-uniform byte offset that the optimiser sees as new in every step: each entry's address stays one scalar base and a 32-bit lane
// offset.  (Followed from step to step they became a 64-bit pointer in vector registers for every entry: 128 registers at d = 128, and
// spills whose reloads waited for the gradients' stores; 128 x 200 matrices of float d = 128: 1790 -> 1480 us with all that is below.)
__device__ inline long long opaque(long long v)
{
    asm volatile("" : "+s"(v));
    return v;
}

__device__ inline float round_(float v) { return __builtin_rintf(v); }
__device__ inline double round_(double v) { return __builtin_rint(v); }

// Steps s = 0 .. len - 1 of a chunk take matrix t1 - 1 - s.
template <typename R, int DP, int NW, bool FACT, bool FULL, bool GRAD, int PD>
__global__ __launch_bounds__(NW * 64) void vec_adjoint_kernel(AdjointArgs a)
{
    typedef typename std::conditional<FACT || sizeof(R) == 8, double, float>::type V;
    typedef R R2 __attribute__((ext_vector_type(2)));
    constexpr int K = DP / 16, RW = DP / NW, Q = RW / 4;
    static_assert(Q >= 1 && Q <= 16 && 4 * Q * NW == DP, "a lane finishes at most one row");
    constexpr bool EARLY = !FACT && DP <= 32;
    // The largest factors with gradients: the next factor is loaded once this one's registers are done with.  (Held beside them registers
    // are spilled, and a reload waits for the gradients' stores: 18 us a step of float d = 128 where 7.4 are taken now.)
    constexpr bool LATE = GRAD && DP == 128;
    // A term of the product is a row's mantissa times an entry on its row's power of two, a gradient also has a state's entry on the
    // largest one's: each may lie this far below 1 before the type's smallest normal number is in sight.
    constexpr V kSpread = sizeof(V) == 4 ? (V)40 : (V)320;
    typedef V V2 __attribute__((ext_vector_type(2)));
    __shared__ __align__(16) V2 part[2][NW][DP]; // the waves' sums of every column: mantissa and exponent
    __shared__ V partn[2][NW], lm[DP], lx[DP];
    constexpr V kHighest = sizeof(V) == 4 ? (V)120 : (V)1000; // largest power of two of lam_i times a row's times h's that is formed as a number

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15, d = a.d;
    // (in scalar registers: the grid has fewer than 2^31 workgroups)
    const int item_of = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (unsigned)a.chunks));
    const long long item = item_of, chunk = a.first_chunk + (int)(blockIdx.x - (unsigned)item_of * (unsigned)a.chunks);
    const long long t0 = chunk * a.chunk_len;
    long long len = a.T - t0;
    if (len > a.chunk_len) len = a.chunk_len;
    if (len <= 0) return; // the whole workgroup
    const long long tlast = t0 + len - 1;

    const unsigned char *left0 = a.left + item * a.left_batch_stride;
    const int row0 = wave * RW + g;
    const int orow = row0 + 4 * (c < Q ? c : 0);
    const bool owner = c < Q, row_ok = orow < d;
    const size_t orow_in = (size_t)(row_ok ? orow : 0);

    // entries beyond the matrix: the last row and column stand in (their vector entries are zero, or their sums dropped)
    constexpr unsigned kEntry = FACT ? sizeof(R) : sizeof(R2);
    const unsigned row_bytes = FACT ? (unsigned)a.left_cols * (unsigned)sizeof(R) : (unsigned)(FULL ? DP : d) * (unsigned)sizeof(R2);
    unsigned row_at[FULL ? 1 : Q], col_at[FULL ? 1 : K];
    if constexpr (FULL) {
        row_at[0] = (unsigned)row0 * row_bytes;
        col_at[0] = (unsigned)c * kEntry;
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) row_at[q] = (unsigned)(row0 + 4 * q < d ? row0 + 4 * q : d - 1) * row_bytes;
#pragma unroll
        for (int k = 0; k < K; ++k) col_at[k] = (unsigned)(c + 16 * k < d ? c + 16 * k : d - 1) * kEntry;
    }
    // entry (q, k) of the matrix at `base`, whose entries take kEntry / SHRINK bytes
    auto place = [&](auto *base, int q, int k, auto shrink) {
        constexpr unsigned kShrink = decltype(shrink)::value;
        unsigned at = FULL ? row_at[0] + col_at[0] : row_at[FULL ? 0 : q] + col_at[FULL ? 0 : k];
        asm volatile("" : "+v"(at)); // (see opaque)
        return base + (FULL ? (4 * q * DP + 16 * k) * (int)(kEntry / kShrink) : 0) + at / kShrink;
    };
    typedef std::integral_constant<unsigned, 1> whole_size;
    typedef std::integral_constant<unsigned, 2> half_size; // (a real's place is half a GOOM's)
    auto col_in = [&](int k) { return FULL || c + 16 * k < d ? c + 16 * k : d - 1; };

    struct Matrix {
        R2 z[FACT ? 1 : Q][FACT ? 1 : K];
        R w[FACT ? Q : 1][FACT ? K : 1];
    };
    struct Rest {
        R2 h;          // h_{t-1}, the owner's row
        R gv;          // G_{t-1}, the owner's row
        R2 b;          // b_t, the owner's row
        R2 hc[GRAD && EARLY ? K : 1]; // h_{t-1}, the lane's columns (larger factors: loaded while the factor is converted)
        R bias_m;      // FACT: v_c
        double bias_e, common;
    };
    auto load = [&](long long s, Matrix &m) {
        const long long t = tlast - (s < len ? s : len - 1);
        const unsigned char *src = left0 + opaque(t * a.left_step_stride);
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (FACT)
                    m.w[q][k] = *reinterpret_cast<const R *>(place(src, q, k, whole_size()));
                else
                    m.z[q][k] = *reinterpret_cast<const R2 *>(place(src, q, k, whole_size()));
            }
    };
    const R2 *H = reinterpret_cast<const R2 *>(a.H) + (size_t)item * a.T * d;
    const R *G = reinterpret_cast<const R *>(a.G) + (size_t)item * a.T * d;
    const R2 *B = reinterpret_cast<const R2 *>(a.bias) + (size_t)item * a.T * d;
    const R2 *h0 = a.h0 ? reinterpret_cast<const R2 *>(a.h0) + (size_t)item * d : nullptr;
    auto load_columns = [&](long long t, auto &hc) {
        const R2 *hp = t > 0 ? H + (size_t)(t - 1) * d : h0 ? h0 : H; // (no h0: loaded and not used)
#pragma unroll
        for (int k = 0; k < K; ++k) hc[k] = hp[col_in(k)];
    };
    auto load_rest = [&](long long s, Rest &r) {
        const long long t = tlast - (s < len ? s : len - 1);
        if constexpr (FACT) {
            const unsigned char *src = left0 + t * a.left_step_stride;
            const double *ep = reinterpret_cast<const double *>(src + (size_t)DP * a.left_cols * sizeof(R));
            r.common = ep[0];
            r.bias_m = reinterpret_cast<const R *>(src)[orow_in * a.left_cols + d];
            r.bias_e = ep[d];
        } else {
            const size_t tp = (size_t)(t > 0 ? t - 1 : 0);
            r.h = H[tp * d + orow_in];
            r.gv = G[tp * d + orow_in];
            if constexpr (GRAD) {
                r.b = B[(size_t)t * d + orow_in];
                if constexpr (EARLY) load_columns(t, r.hc);
            }
        }
    };

    V sv[Q][K], sn[Q]; // the factor's entries on their rows' powers of two
    bool far = false;  // some entry of the wave's rows, not zero, lies more than kSpread below its row's
    auto convert = [&](const Matrix &m) {
        bool small = false;
        if constexpr (!FACT) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                V u = m.z[q][0][0];
#pragma unroll
                for (int k = 1; k < K; ++k) u = raw_max(u, (V)m.z[q][k][0]);
                u = max16(u);
                sn[q] = u > (V)kNone ? Comp<V>::ceil_(u * (V)kLog2e) : (V)0;
#pragma unroll
                for (int k = 0; k < K; ++k) sv[q][k] = scaled_entry((V)m.z[q][k][0], (V)m.z[q][k][1], sn[q]);
                unsigned key = kNoDepth;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const unsigned o = depth_key(m.z[q][k][0]);
                    key = o > key ? o : key;
                }
                small = small || depth_of<R>(key) < u - kSpread * (V)kLn2;
                if (K >= 8) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                sn[q] = (V)0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    sv[q][k] = (V)m.w[q][k];
                    if constexpr (sizeof(R) == 8) small = small || (Comp<V>::abs_(sv[q][k]) < (V)4.681778573893022e-97 && sv[q][k] != (V)0); // 2^-320
                }
            }
        }
        far = __builtin_amdgcn_ballot_w64(small) != 0;
    };

    double base = 0.0;    // the vector's entries: m 2^(x + base)
    V om = (V)0, ox = (V)kNone; // the owner's entry
    V vm[Q], vx[Q];       // the lane's rows' entries
    // own entry (y 2^yx) 2^base plus (bm 2^be) 2^base, and its way to the row's lanes
    auto take = [&](V y, V yx, V bm, V be) {
        const V pe = y != (V)0 ? Comp<V>::exponent_of(y) + yx : (V)kNone;
        ox = be > pe ? be : pe;
        om = Comp<V>::ldexp_(y, (int)Comp<V>::clamp_shift(yx - ox)) + Comp<V>::ldexp_(bm, (int)Comp<V>::clamp_shift(be - ox));
        if (!row_ok) {
            om = (V)0;
            ox = (V)kNone;
        }
        if (owner) {
            lm[orow] = om;
            lx[orow] = ox;
        }
        // (a band's words are written and read by one wave, whose LDS operations complete in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            vm[q] = lm[row0 + 4 * q];
            vx[q] = lx[row0 + 4 * q];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // G / h on the current base; an entry that is exactly zero passes no gradient, and an infinite one divides it away
    auto source = [&](R gv, R2 h, V &bm, V &be) {
        bm = (V)0;
        be = (V)kNone;
        if (gv != (R)0 && !((double)h[0] < -1.0e300) && h[0] != -Comp<R>::neg_inf()) {
            const V e = Comp<V>::exponent_of((V)gv);
            const double x = -__builtin_fma((double)h[0], kLog2e, base);
            const double xe = __builtin_rint(x);
            V f;
            if constexpr (sizeof(V) == 4)
                f = __builtin_amdgcn_exp2f((float)(x - xe));
            else
                f = Comp<double>::exp2_small(x - xe);
            bm = Comp<V>::apply_sign(Comp<V>::ldexp_((V)gv, -(int)e) * f, (V)h[1]);
            be = e + (V)xe;
        }
    };
    // m 2^x of a log-magnitude re added to the owner's entry: the owner's entry times exp(re)
    auto times_exp = [&](R2 z) {
        double x = __builtin_fma((double)z[0], kLog2e, base + (double)ox);
        x = x > -4000.0 ? x : -4000.0; // (NaN too becomes a zero: the log-magnitude of no number)
        x = x < 4000.0 ? x : 4000.0;
        const double xe = __builtin_rint(x);
        const double f = sizeof(V) == 4 ? (double)__builtin_amdgcn_exp2f((float)(x - xe)) : Comp<double>::exp2_small(x - xe);
        const double v = __builtin_ldexp((double)om * f, (int)xe);
        const bool live = om != (V)0 && !((double)z[0] < -1.0e300);
        return (R)(live ? (Comp<V>::is_negative((V)z[1]) ? -v : v) : 0.0);
    };

    // ---- the vector that enters, with the last step's G / h
    {
        V y = (V)0;
        if (a.init) {
            const unsigned char *ip = a.init + (item * a.init_per_item + chunk) * a.vec_stride;
            y = (V) reinterpret_cast<const R *>(ip)[orow];
            base = *reinterpret_cast<const double *>(ip + (size_t)DP * sizeof(R));
            if (!(__builtin_fabs(base) < 1.0e15)) base = 0.0;
        }
        V bm = (V)0, be = (V)kNone;
        if constexpr (!FACT) {
            const R2 h = H[(size_t)tlast * d + orow_in];
            const R gv = G[(size_t)tlast * d + orow_in];
            // a zero vector takes the scale of what is added to it (its own base says nothing)
            if (!a.init) base = 0.0;
            source(gv, h, bm, be);
        }
        take(y, (V)0, bm, be);
    }
    // FACT: vectors [batch][T + 1], the one that enters chunk j at j; GRAD / GOOM walks: nothing
    auto store_vec = [&](long long j) {
        // mantissas relative to the vector's largest exponent: through LDS, each wave its own rows
        unsigned char *dst = a.out_vecs + (item * (a.T + 1) + j) * a.vec_stride;
        // the largest exponent over all rows needs every wave's: kept in partn by the caller
        V top = (V)kNone;
#pragma unroll
        for (int w = 0; w < NW; ++w) top = raw_max(top, partn[0][w]);
        const bool none = !(top > (V)(0.5f * kNone));
        if (none) top = (V)0;
        if (owner) reinterpret_cast<R *>(dst)[orow] = (R)Comp<V>::ldexp_(om, (int)Comp<V>::clamp_shift(ox - top));
        if (threadIdx.x == 0) *reinterpret_cast<double *>(dst + (size_t)DP * sizeof(R)) = none ? 0.0 : base + (double)top;
    };
    auto publish_top = [&]() { // each wave's largest exponent, for store_vec
        V top = (V)kNone;
#pragma unroll
        for (int q = 0; q < Q; ++q) top = raw_max(top, vx[q]);
        top = Comp<V>::xor16_32_max(top);
        __syncthreads();
        if (lane == 0) partn[0][wave] = top;
        __syncthreads();
    };
    if (FACT && a.out_vecs && tlast + 1 == a.T) { // the zero vector enters the last chunk (a group's last one: the next group's walk has it)
        publish_top();
        store_vec(tlast + 1);
        __syncthreads();
    }

    auto step = [&](long long s, Matrix &mat, Rest &next) {
        const Rest r = next;
        load_rest(s + 1, next); // in flight for the whole step
        const bool live = s < len; // (the whole workgroup; a step past the end is computed and dropped)
        const long long t = tlast - (live ? s : len - 1);
        [[maybe_unused]] R2 hcol[GRAD ? K : 1];
        if constexpr (GRAD && !EARLY) load_columns(t, hcol);
        if constexpr (GRAD && EARLY) {
#pragma unroll
            for (int k = 0; k < K; ++k) hcol[k] = r.hc[k];
        }
        if constexpr (!EARLY) {
            convert(mat);
            if (Q * K >= 16) __builtin_amdgcn_sched_barrier(0);
            if constexpr (!LATE) load(s + PD, mat);
            if (Q * K >= 16) __builtin_amdgcn_sched_barrier(0);
        }
        // ---- A_t^T x: this wave's rows, on the power of two nw
        V nw = (V)kNone;
        float lowest = -kNone;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            nw = raw_max(nw, vm[q] != (V)0 ? vx[q] + sn[q] : (V)kNone);
            lowest = __builtin_fminf(lowest, vm[q] != (V)0 ? (float)(vx[q] + sn[q]) : -kNone);
        }
        nw = Comp<V>::xor16_32_max(nw);
        // h_{t-1} on the power of two of its largest entry
        [[maybe_unused]] V htop = (V)0;
        bool wide = false;
        if constexpr (GRAD) {
            V u = hcol[0][0];
            unsigned key = kNoDepth;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                u = raw_max(u, (V)hcol[k][0]);
                const unsigned o = depth_key(hcol[k][0]);
                key = o > key ? o : key;
            }
            u = max16(u);
            htop = u > (V)kNone ? Comp<V>::ceil_(u * (V)kLog2e) : (V)0;
            wide = depth_of<R>(key) < u - kSpread * (V)kLn2 || base + (double)(htop + nw) > (double)kHighest;
        }
        const bool apart = far || __builtin_amdgcn_ballot_w64(lowest < (float)nw - (float)kSpread || wide) != 0; // (a row with an entry far below it, or rows far apart)
        const int buf = (int)(s & 1);
        [[maybe_unused]] unsigned char *gA = nullptr;
        if constexpr (GRAD) {
            gA = reinterpret_cast<unsigned char *>(a.gA) + opaque((item * a.T + t) * (long long)((size_t)d * d * sizeof(R)));
            if (a.gb && live && owner && row_ok) reinterpret_cast<R *>(a.gb)[(size_t)(item * a.T + t) * d + orow] = times_exp(r.b);
        }
        // an entry of h_{t-1} as hh 2^hx
        [[maybe_unused]] auto entry = [&](const R2 &z, V &hh, int &hx) {
            const V n = (V)z[0] > (V)kNone ? round_((V)z[0] * (V)kLog2e) : (V)0;
            hh = t == 0 && !h0 ? (V)0 : scaled_entry((V)z[0], (V)z[1], n);
            hx = whole(n);
        };
        V p[K];
        [[maybe_unused]] V hh[K]; // h_{t-1} on the power of two of its largest entry
#pragma unroll
        for (int k = 0; k < K; ++k) {
            p[k] = (V)0;
            if constexpr (GRAD) hh[k] = t == 0 && !h0 ? (V)0 : scaled_entry((V)hcol[k][0], (V)hcol[k][1], htop);
        }
        // (lanes beyond the last column write its value once more)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const V w = Comp<V>::ldexp_(vm[q], (int)Comp<V>::clamp_shift(vx[q] + sn[q] - nw));
#pragma unroll
            for (int k = 0; k < K; ++k) p[k] = p[k] + w * sv[q][k];
            if constexpr (GRAD) {
                const V f = Comp<V>::ldexp_(vm[q], whole(base + (double)(htop + (vx[q] + sn[q]))));
                if (live && (FULL || row0 + 4 * q < d)) {
#pragma unroll
                    for (int k = 0; k < K; ++k) *reinterpret_cast<R *>(place(gA, q, k, half_size())) = (R)(f * hh[k] * sv[q][k]);
                }
            }
            if (K >= 8) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (LATE) {
            __builtin_amdgcn_sched_barrier(0);
            load(s + PD, mat);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) p[k] = sum_groups(p[k]);
        if (g == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) part[buf][wave][c + 16 * k] = V2{p[k], nw};
        }
        if constexpr (EARLY) {
            convert(mat);
            load(s + PD + 1, mat);
        }
        if (apart) {
            // What was formed above is replaced.  (After it, not instead of it: the question is settled while that work goes on.  The factor's
            // registers are the next one's by now: it is read again, a column at a time, which keeps this rare path out of the common
            // one's registers.)
            const unsigned char *src = left0 + t * a.left_step_stride;
            const R2 *hp = t > 0 ? H + (size_t)(t - 1) * d : h0 ? h0 : H;
#pragma unroll 1
            for (int k = 0; k < K; ++k) {
                const int col = c + 16 * k < d ? c + 16 * k : d - 1;
                [[maybe_unused]] V hh = (V)0;
                [[maybe_unused]] int hx = 0;
                if constexpr (GRAD) entry(hp[col], hh, hx);
                V term[Q], ex[Q], ctop = (V)kNone, sum = (V)0;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const unsigned at = (unsigned)(row0 + 4 * q < d ? row0 + 4 * q : d - 1) * row_bytes + (unsigned)col * kEntry;
                    V m, n;
                    if constexpr (FACT) {
                        const V w = (V) * reinterpret_cast<const R *>(src + at);
                        n = Comp<V>::exponent_of(w);
                        m = Comp<V>::ldexp_(w, -(int)n);
                    } else {
                        const R2 z = *reinterpret_cast<const R2 *>(src + at);
                        n = (V)z[0] > (V)kNone ? round_((V)z[0] * (V)kLog2e) : (V)kNone;
                        m = scaled_entry((V)z[0], (V)z[1], n);
                    }
                    term[q] = vm[q] * m;
                    ex[q] = term[q] != (V)0 ? vx[q] + n : (V)kNone;
                    ctop = raw_max(ctop, ex[q]);
                    if constexpr (GRAD) {
                        if (live && row0 + 4 * q < d)
                            *reinterpret_cast<R *>(gA + (at >> 1)) = (R)Comp<V>::ldexp_(term[q] * hh, whole(base + (double)vx[q]) + whole(n) + hx);
                    }
                }
                ctop = Comp<V>::xor16_32_max(ctop);
#pragma unroll
                for (int q = 0; q < Q; ++q) sum = sum + Comp<V>::ldexp_(term[q], (int)Comp<V>::clamp_shift(ex[q] - ctop));
                sum = sum_groups(sum);
                if (g == 0) part[buf][wave][c + 16 * k] = V2{sum, ctop};
            }
        }
        if (lane == 0) partn[buf][wave] = nw;
        __syncthreads();
        V2 pv[NW];
        V top = (V)kNone, ctop = (V)kNone; // the largest power of two of any wave; of the owner's column
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            pv[w] = part[buf][w][orow];
            top = raw_max(top, partn[buf][w]);
            ctop = pv[w][0] != (V)0 && pv[w][1] > ctop ? pv[w][1] : ctop;
        }
        const bool none = !(top > (V)(0.5f * kNone));
        if (none) top = (V)0;
        if (!(ctop > (V)(0.5f * kNone))) ctop = top;
        V y = (V)0; // the owner's column: y 2^(ctop - top) on the new base
#pragma unroll
        for (int w = 0; w < NW; ++w) y = y + Comp<V>::ldexp_(pv[w][0], (int)Comp<V>::clamp_shift(pv[w][1] - ctop));
        if (live) {
            base = none ? 0.0 : base + (FACT ? r.common : 0.0) + (double)top;
            V bm = (V)0, be = (V)kNone;
            if constexpr (FACT) {
                bm = (V)r.bias_m;
                if (bm != (V)0) {
                    const V e = Comp<V>::exponent_of(bm);
                    bm = Comp<V>::ldexp_(bm, -(int)e);
                    be = e + (V)(r.bias_e - base);
                }
            } else if (t > t0) { // (the entry before the chunk's first step gets its G / h in the chunk that it belongs to)
                source(r.gv, r.h, bm, be);
            }
            take(y, ctop - top, bm, be);
        }
        if (FACT && a.out_vecs) {
            publish_top();
            if (live) store_vec(t);
            __syncthreads();
        }
    };

    Matrix ring[PD];
    Rest rest;
    if constexpr (EARLY) {
        load(0, ring[0]);
        convert(ring[0]);
    }
#pragma unroll
    for (int i = 0; i < PD; ++i) load(i + (EARLY ? 1 : 0), ring[i]);
    load_rest(0, rest);
    for (long long s = 0; s < len; s += PD) {
#pragma unroll
        for (int i = 0; i < PD; ++i) step(s + i, ring[i], rest);
    }
    if (a.out_total) { // the chunk's vector as column d of its factored product
        publish_top();
        V top = (V)kNone;
#pragma unroll
        for (int w = 0; w < NW; ++w) top = raw_max(top, partn[0][w]);
        const bool none = !(top > (V)(0.5f * kNone));
        if (none) top = (V)0;
        unsigned char *dst = a.out_total + (item * a.totals_per_item + chunk - a.first_chunk) * a.total_stride;
        if (owner) reinterpret_cast<R *>(dst)[(size_t)orow * a.left_cols + d] = (R)Comp<V>::ldexp_(om, (int)Comp<V>::clamp_shift(ox - top));
        if (threadIdx.x == 0) reinterpret_cast<double *>(dst + (size_t)DP * a.left_cols * sizeof(R))[d] = none ? 0.0 : base + (double)top;
    }
    if constexpr (GRAD) {
        if (a.gh0 && chunk == 0 && owner && row_ok) reinterpret_cast<R *>(a.gh0)[(size_t)item * d + orow] = times_exp(h0[orow]);
    }
}

template <typename R, int DP, int NW, bool FACT, bool FULL, bool GRAD, int PD> int launch_one(goom_ctx *ctx, const AdjointArgs &a, long long grid, const char *label)
{
    if (grid <= 0) return GOOM_OK;
    if (grid > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many chains for one launch (%lld)", grid);
    goom::prof_begin(ctx, label);
    hipLaunchKernelGGL((vec_adjoint_kernel<R, DP, NW, FACT, FULL, GRAD, PD>), dim3((unsigned)grid), dim3(NW * 64), 0, ctx->stream, a);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch vec_adjoint_kernel");
}

template <typename R, int DP, int NW, int PD> int goom_walk(goom_ctx *ctx, const AdjointArgs &a, bool grad, long long grid, const char *label)
{
    if (a.d == DP)
        return grad ? launch_one<R, DP, NW, false, true, true, PD>(ctx, a, grid, label) : launch_one<R, DP, NW, false, true, false, PD>(ctx, a, grid, label);
    return grad ? launch_one<R, DP, NW, false, false, true, PD>(ctx, a, grid, label) : launch_one<R, DP, NW, false, false, false, PD>(ctx, a, grid, label);
}

template <typename R> int walk(goom_ctx *ctx, const AdjointArgs &a, int dp, bool fact, bool grad, long long grid, const char *label)
{
    constexpr bool f32 = sizeof(R) == 4;
    if (fact) {
        switch (dp) {
        case 16: return launch_one<R, 16, 1, true, false, false, 2>(ctx, a, grid, label);
        case 32: return launch_one<R, 32, 2, true, false, false, 2>(ctx, a, grid, label);
        case 64: return launch_one<R, 64, 8, true, false, false, 2>(ctx, a, grid, label);
        default: return launch_one<R, 128, 8, true, false, false, 1>(ctx, a, grid, label);
        }
    }
    switch (dp) {
    case 16: return goom_walk<R, 16, 1, 2>(ctx, a, grad, grid, label);
    case 32: return goom_walk<R, 32, f32 ? 2 : 4, 2>(ctx, a, grad, grid, label);
    case 64: return goom_walk<R, 64, f32 ? 4 : 8, f32 ? 2 : 1>(ctx, a, grad, grid, label);
    default: return goom_walk<R, 128, 8, 1>(ctx, a, grad, grid, label);
    }
}

} // namespace

// The adjoint pass of a recurrence over `chunks` chunks of chunk_len steps.  totals: factored products of chunks 1 .. chunks - 1
// (their column d is written here), vecs: room for batch * chunks vectors of adjoint_vec_stride bytes; neither is used with one chunk.
// group: 0, or that many chunk products make a group: gtot then holds the products of groups 1 .. (column d written here), gvecs has room for a
// vector a group.
size_t adjoint_vec_stride(int dp, int dtype) { return goom::align_up((size_t)dp * (dtype == GOOM_C64 ? 4 : 8) + 8, 256); }

int launch_affine_adjoint(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *G, void *gA, void *gb, void *gh0,
                          long long T, int d, long long batch, int dtype, int dp, long long chunk_len, long long chunks, void *totals,
                          long long total_stride, int total_cols, void *vecs, long long group, void *gtot, void *gvecs)
{
    const bool f32 = dtype == GOOM_C64;
    const size_t cb = f32 ? 8 : 16;
    AdjointArgs a;
    a.left = static_cast<const unsigned char *>(A);
    a.left_step_stride = (long long)(d * (size_t)d * cb);
    a.left_batch_stride = T * a.left_step_stride;
    a.T = T;
    a.chunk_len = chunk_len;
    a.d = d;
    a.left_cols = total_cols;
    a.bias = bias;
    a.h0 = h0;
    a.H = H;
    a.G = G;
    a.init = nullptr;
    a.init_per_item = chunks;
    a.vec_stride = (long long)adjoint_vec_stride(dp, dtype);
    a.out_total = nullptr;
    a.total_stride = total_stride;
    a.totals_per_item = chunks - 1;
    a.out_vecs = nullptr;
    a.gA = gA;
    a.gb = gb;
    a.gh0 = gh0;
    auto run = [&](const AdjointArgs &w, bool fact, bool grad, long long grid, const char *label) {
        return f32 ? walk<float>(ctx, w, dp, fact, grad, grid, label) : walk<double>(ctx, w, dp, fact, grad, grid, label);
    };
    if (chunks > 1) {
        AdjointArgs v = a; // the vectors that leave chunks 1 .. chunks - 1 when nothing enters
        v.first_chunk = 1;
        v.chunks = chunks - 1;
        v.out_total = static_cast<unsigned char *>(totals);
        if (int s = run(v, false, false, batch * (chunks - 1), "affine_adjoint_chunk_vectors")) return s;
        AdjointArgs f = a; // the vectors that enter chunks chunks - 1 .. 0: one chain over the products, in reverse
        f.left = static_cast<const unsigned char *>(totals);
        f.left_step_stride = total_stride;
        f.left_batch_stride = (chunks - 1) * total_stride;
        f.T = chunks - 1;
        f.chunk_len = chunks - 1;
        f.first_chunk = 0;
        f.chunks = 1;
        f.out_vecs = static_cast<unsigned char *>(vecs);
        if (group) {
            const long long groups = (f.T + group - 1) / group;
            AdjointArgs u = f; // the vectors that leave groups 1 .. groups - 1 when nothing enters
            u.chunk_len = group;
            u.first_chunk = 1;
            u.chunks = groups - 1;
            u.out_vecs = nullptr;
            u.out_total = static_cast<unsigned char *>(gtot);
            u.totals_per_item = groups - 1;
            if (int s = run(u, true, false, batch * (groups - 1), "affine_adjoint_group_vectors")) return s;
            u = f; // the vectors that enter the groups
            u.left = static_cast<const unsigned char *>(gtot);
            u.left_batch_stride = (groups - 1) * total_stride;
            u.T = u.chunk_len = groups - 1;
            u.out_vecs = static_cast<unsigned char *>(gvecs);
            if (int s = run(u, true, false, batch, "affine_adjoint_carries")) return s;
            f.chunk_len = group; // and every group again, from there
            f.chunks = groups;
            f.init = static_cast<const unsigned char *>(gvecs);
            f.init_per_item = groups;
        }
        if (int s = run(f, true, false, batch * f.chunks, "affine_adjoint_carries")) return s;
        a.init = static_cast<const unsigned char *>(vecs);
    }
    a.first_chunk = 0;
    a.chunks = chunks;
    return run(a, false, true, batch * chunks, "affine_adjoint_gradients");
}

} // namespace goom_chain
