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
//   * lam is kept as mantissa and exponent per entry with a double base, so no scaling of h or A comes before: values e^-1000 and
//     below are ordinary numbers here.
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

// Steps s = 0 .. len - 1 of a chunk take matrix t1 - 1 - s.
template <typename R, int DP, int NW, bool FACT, bool FULL, bool GRAD, int PD>
__global__ __launch_bounds__(NW * 64) void vec_adjoint_kernel(AdjointArgs a)
{
    typedef typename std::conditional<FACT || sizeof(R) == 8, double, float>::type V;
    typedef R R2 __attribute__((ext_vector_type(2)));
    constexpr int K = DP / 16, RW = DP / NW, Q = RW / 4;
    static_assert(Q >= 1 && Q <= 16 && 4 * Q * NW == DP, "a lane finishes at most one row");
    constexpr bool EARLY = !FACT && DP <= 32;
    // The largest factors with gradients: the next factor is loaded once this one's registers are done with.  (Held beside them, 82
    // registers are spilled, and a reload waits for the gradients' stores: 18 us a step.)
    constexpr bool LATE = GRAD && DP == 128;
    __shared__ V part[2][NW][DP], partn[2][NW], lm[DP], lx[DP];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15, d = a.d;
    const long long item = (long long)blockIdx.x / a.chunks, chunk = a.first_chunk + (long long)blockIdx.x % a.chunks;
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
    auto offset_of = [&](int q, int k) {
        if constexpr (FULL)
            return row_at[0] + col_at[0] + (unsigned)(4 * q) * (unsigned)(DP * kEntry) + (unsigned)(16 * k) * kEntry;
        else
            return row_at[q] + col_at[k];
    };
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
        const unsigned char *src = left0 + t * a.left_step_stride;
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (FACT)
                    m.w[q][k] = *reinterpret_cast<const R *>(src + offset_of(q, k));
                else
                    m.z[q][k] = *reinterpret_cast<const R2 *>(src + offset_of(q, k));
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
    auto convert = [&](const Matrix &m) {
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
                if (K >= 8) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                sn[q] = (V)0;
#pragma unroll
                for (int k = 0; k < K; ++k) sv[q][k] = (V)m.w[q][k];
            }
        }
    };

    double base = 0.0;    // the vector's entries: m 2^(x + base)
    V om = (V)0, ox = (V)kNone; // the owner's entry
    V vm[Q], vx[Q];       // the lane's rows' entries
    // own entry y 2^base plus (bm 2^be) 2^base, and its way to the row's lanes
    auto take = [&](V y, V bm, V be) {
        const V pe = y != (V)0 ? Comp<V>::exponent_of(y) : (V)kNone;
        ox = be > pe ? be : pe;
        om = Comp<V>::ldexp_(y, (int)Comp<V>::clamp_shift(-ox)) + Comp<V>::ldexp_(bm, (int)Comp<V>::clamp_shift(be - ox));
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
    // G / h on the current base; an entry that is exactly zero passes no gradient
    auto source = [&](R gv, R2 h, V &bm, V &be) {
        bm = (V)0;
        be = (V)kNone;
        if (gv != (R)0 && !((double)h[0] < -1.0e300)) {
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
        take(y, bm, be);
    }
    // FACT: vectors [batch][chunk_len + 1], the one that enters chunk j at j; GRAD / GOOM walks: nothing
    auto store_vec = [&](long long j) {
        // mantissas relative to the vector's largest exponent: through LDS, each wave its own rows
        unsigned char *dst = a.out_vecs + (item * (a.chunk_len + 1) + j) * a.vec_stride;
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
    if (FACT && a.out_vecs) { // the zero vector enters the last chunk
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
#pragma unroll
        for (int q = 0; q < Q; ++q) nw = raw_max(nw, vm[q] != (V)0 ? vx[q] + sn[q] : (V)kNone);
        nw = Comp<V>::xor16_32_max(nw);
        V p[K];
#pragma unroll
        for (int k = 0; k < K; ++k) p[k] = (V)0;
        [[maybe_unused]] V hh[K];
        [[maybe_unused]] double htop = 0.0;
        if constexpr (GRAD) {
            V u = hcol[0][0];
#pragma unroll
            for (int k = 1; k < K; ++k) u = raw_max(u, (V)hcol[k][0]);
            u = max16(u);
            const V hn = u > (V)kNone ? Comp<V>::ceil_(u * (V)kLog2e) : (V)0;
            htop = (double)hn;
            const bool none = t == 0 && !h0;
#pragma unroll
            for (int k = 0; k < K; ++k) hh[k] = none ? (V)0 : scaled_entry((V)hcol[k][0], (V)hcol[k][1], hn);
        }
        [[maybe_unused]] unsigned char *gA = nullptr;
        if constexpr (GRAD) gA = reinterpret_cast<unsigned char *>(a.gA) + (size_t)(item * a.T + t) * d * d * sizeof(R);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const V w = Comp<V>::ldexp_(vm[q], (int)Comp<V>::clamp_shift(vx[q] + sn[q] - nw));
            [[maybe_unused]] V f = (V)0;
            if constexpr (GRAD) {
                double e = base + htop + (double)(vx[q] + sn[q]);
                e = e > -4000.0 ? e : -4000.0;
                e = e < 4000.0 ? e : 4000.0;
                f = Comp<V>::ldexp_(vm[q], (int)e);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) p[k] = p[k] + w * sv[q][k];
            if constexpr (GRAD) {
                // a real's place is half a GOOM's; lanes beyond the last column write its value once more
                if (live && (FULL || row0 + 4 * q < d)) {
#pragma unroll
                    for (int k = 0; k < K; ++k) *reinterpret_cast<R *>(gA + (offset_of(q, k) >> 1)) = (R)(f * hh[k] * sv[q][k]);
                }
            }
            if (K >= 8) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (GRAD) {
            if (a.gb && live && owner && row_ok) reinterpret_cast<R *>(a.gb)[(size_t)(item * a.T + t) * d + orow] = times_exp(r.b);
        }
        if constexpr (LATE) {
            __builtin_amdgcn_sched_barrier(0);
            load(s + PD, mat);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) p[k] = sum_groups(p[k]);
        const int buf = (int)(s & 1);
        if (g == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) part[buf][wave][c + 16 * k] = p[k];
            if (c == 0) partn[buf][wave] = nw;
        }
        if constexpr (EARLY) {
            convert(mat);
            load(s + PD + 1, mat);
        }
        __syncthreads();
        V top = (V)kNone;
#pragma unroll
        for (int w = 0; w < NW; ++w) top = raw_max(top, partn[buf][w]);
        const bool none = !(top > (V)(0.5f * kNone));
        if (none) top = (V)0;
        V y = (V)0;
#pragma unroll
        for (int w = 0; w < NW; ++w) y = y + Comp<V>::ldexp_(part[buf][w][orow], (int)Comp<V>::clamp_shift(partn[buf][w] - top));
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
            take(y, bm, be);
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
size_t adjoint_vec_stride(int dp, int dtype) { return goom::align_up((size_t)dp * (dtype == GOOM_C64 ? 4 : 8) + 8, 256); }

int launch_affine_adjoint(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *G, void *gA, void *gb, void *gh0,
                          long long T, int d, long long batch, int dtype, int dp, long long chunk_len, long long chunks, void *totals,
                          long long total_stride, int total_cols, void *vecs)
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
        if (int s = run(f, true, false, batch, "affine_adjoint_carries")) return s;
        a.init = static_cast<const unsigned char *>(vecs);
    }
    a.first_chunk = 0;
    a.chunks = chunks;
    return run(a, false, true, batch * chunks, "affine_adjoint_gradients");
}

} // namespace goom_chain
