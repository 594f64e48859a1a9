// Chains with a state of one column: h <- A_t h (+ b_t), for every size up to 128, both component types, GOOM or
// factored left factors (the recurrence's carries and states, vector initial states, largest exponents).
//
// A matrix-vector product reads its matrix once and does two operations per entry, so with GOOM factors what bounds it
// is the matrices' way from memory, and with factored ones (the serial middle phase, one chain per batch item) the
// latency of a step.  The matrix instruction has nothing to offer here (one column of sixteen would be used, behind a
// tile in LDS that every entry has to pass), so:
//   * a workgroup of NW waves owns one chain, a wave a band of rows.  Sixteen lanes share a row and hold every sixteenth
//     entry of it, so that a load instruction covers whole 128-byte (256-byte) pieces of four rows whatever the
//     size or its alignment, and a row's shift and sum are four lane permutations on the vector ALU;
//   * the entries of the next PD factors are in flight in registers while a step is computed;
//   * a row's result goes to LDS as mantissa and exponent of its own, and one barrier later every wave reads the
//     vector and brings it onto the largest exponent itself (the buffers alternate, so one barrier a step is enough);
//   * the bias joins a row on the larger of the two exponents: no case of a bias too large for the vector's scale;
//   * one factor for all steps (SAME) is converted once and stays in registers.
// Carries (factored matrices) are multiplied and added in double for float components too.
// Measured against the general chain kernel with one column (16 x 4096 x 64 float, 63 carries a sequence): see launch_vec.
#include "goom_chain_kernel.h"

#include <type_traits>

namespace goom_chain {

namespace {

template <int CTRL> __device__ inline float dpp_of(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ inline double dpp_of(double v)
{
    const u2 b = __builtin_bit_cast(u2, v);
    u2 r;
    r[0] = (unsigned)__builtin_amdgcn_mov_dpp((int)b[0], CTRL, 0xF, 0xF, true);
    r[1] = (unsigned)__builtin_amdgcn_mov_dpp((int)b[1], CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, r);
}
__device__ inline float raw_max(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ inline double raw_max(double a, double b) { return __builtin_fmax(a, b); }
// sum / maximum over the sixteen lanes of a row (in every one of them)
template <typename V> __device__ inline V sum16(V v)
{
    v += dpp_of<0xB1>(v);
    v += dpp_of<0x4E>(v);
    v += dpp_of<0x141>(v);
    v += dpp_of<0x140>(v);
    return v;
}
template <typename V> __device__ inline V max16(V v)
{
    v = raw_max(v, dpp_of<0xB1>(v));
    v = raw_max(v, dpp_of<0x4E>(v));
    v = raw_max(v, dpp_of<0x141>(v));
    v = raw_max(v, dpp_of<0x140>(v));
    return v;
}

// (+-) 2^(re log2(e) - n), one rounding of a small argument; -inf gives zero, NaN stays NaN
__device__ inline float scaled_entry(float re, float im, float n)
{
    const float kHi = 1.44269502162933349609375f; // float nearest log2(e)
    const float kLo = 1.925963033500011e-8f;      // log2(e) - kHi
    float t = __builtin_fmaf(re, kHi, -n);
    t = __builtin_fmaf(re, kLo, t);
    return Comp<float>::apply_sign(__builtin_amdgcn_exp2f(t), im);
}
__device__ inline double scaled_entry(double re, double im, double n)
{
    const double t = __builtin_fma(re, kLog2e, -n);
    const double k = __builtin_rint(t);
    const double y = __builtin_ldexp(Comp<double>::exp2_small(t - k), (int)(k < -4000.0 ? -4000.0 : k));
    return Comp<double>::apply_sign(t < -1200.0 ? 0.0 : y, im);
}

constexpr float kNone = -1.0e30f; // stands for the exponent of zero

template <typename R, typename IO, int DP, int NW, bool FACT, bool FULL, bool SAME, int PD>
__global__ __launch_bounds__(NW * 64) void vec_walk_kernel(ChainArgs a)
{
    typedef typename std::conditional<FACT || sizeof(R) == 8, double, float>::type V; // the vector and the sums
    typedef IO IO2 __attribute__((ext_vector_type(2)));
    constexpr int K = DP / 16;  // entries of a row per lane
    constexpr int RW = DP / NW; // rows of a wave
    constexpr int Q = RW / 4;   // passes of four rows
    static_assert(Q >= 1 && Q <= 16 && 4 * Q * NW == DP, "a lane finishes at most one row");
    __shared__ V vm[2][DP], vx[2][DP];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int n_rows = a.n, d = a.d;
    const long long item = (long long)blockIdx.x / a.chunks_launched, chunk = (long long)blockIdx.x % a.chunks_launched;
    const long long chain = item * a.chunks_per_item + chunk;
    const long long t0 = chunk * a.chunk_len;
    long long len = a.steps - t0;
    if (len > a.chunk_len) len = a.chunk_len;
    if (len <= 0) return; // the whole workgroup

    const unsigned char *left0 = a.left + item * a.left_batch_stride + t0 * a.left_step_stride;
    const int lfc = a.left_fact_cols;
    const int row0 = wave * RW + g;           // row of pass q: row0 + 4 q
    const int orow = row0 + 4 * (c < Q ? c : 0); // the row this lane finishes (lanes c >= Q repeat one and store nothing)
    const bool owner = c < Q;
    const bool row_ok = orow < n_rows;
    const size_t bias_row = (size_t)(row_ok ? orow : 0);
    const bool bias_goom = a.bias_mode == 1, bias_fact = a.bias_mode == 2;

    // entry (q, k) of this lane: row row0 + 4 q, column c + 16 k
    auto entry_ok = [&](int q, int k) { return FULL || (row0 + 4 * q < n_rows && c + 16 * k < d); };

    struct Raw {
        IO2 z[FACT || SAME ? 1 : Q][FACT || SAME ? 1 : K];
        R w[FACT && !SAME ? Q : 1][FACT && !SAME ? K : 1];
        IO2 bias;      // GOOM bias of the lane's row
        R bias_m;      // factored bias: mantissa ...
        double bias_e; // ... and exponent
        double common; // the factored matrix's exponent
        float shift;   // io_shift
    };
    auto load_goom = [&](long long t, int q, int k) {
        const IO2 *src = reinterpret_cast<const IO2 *>(left0 + t * a.left_step_stride);
        const int idx = entry_ok(q, k) ? (row0 + 4 * q) * (FULL ? DP : d) + c + 16 * k : 0;
        return src[idx];
    };
    auto load_fact = [&](long long t, int q, int k) {
        const R *src = reinterpret_cast<const R *>(left0 + t * a.left_step_stride);
        return src[(size_t)((row0 + 4 * q) * lfc + (entry_ok(q, k) ? c + 16 * k : 0))]; // (DP rows are there)
    };
    auto load = [&](long long t, Raw &r) {
        if constexpr (!SAME) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (FACT)
                        r.w[q][k] = load_fact(t, q, k);
                    else
                        r.z[q][k] = load_goom(t, q, k);
                }
        }
        if (FACT) {
            const unsigned char *src = left0 + t * a.left_step_stride;
            const double *ep = reinterpret_cast<const double *>(src + (size_t)DP * lfc * sizeof(R));
            if (!SAME) r.common = ep[0];
            if (bias_fact) {
                r.bias_m = reinterpret_cast<const R *>(src)[bias_row * lfc + d];
                r.bias_e = ep[d];
            }
        }
        if (bias_goom) {
            r.bias = reinterpret_cast<const IO2 *>(a.bias)[(size_t)(item * a.steps + t0 + t) * d + bias_row];
            if (a.io_shift) r.shift = a.io_shift[item * a.steps + t0 + t];
        }
    };

    // ---- one factor's entries, scaled by their rows' powers of two
    V same_s[SAME ? Q : 1][SAME ? K : 1], same_n[SAME ? Q : 1];
    double same_common = 0.0;
    auto row_shift_of = [&](const IO2 (&z)[K], int q) { // a whole number near the row's largest log2|A_ij|
        V u = -__builtin_huge_val();
#pragma unroll
        for (int k = 0; k < K; ++k) u = raw_max(u, entry_ok(q, k) ? (V)z[k][0] : (V)-__builtin_huge_val());
        u = max16(u);
        return u > (V)kNone ? Comp<V>::ceil_(u * (V)kLog2e) : (V)0; // (+inf stays: its row comes out as NaN)
    };
    if constexpr (SAME) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if constexpr (FACT) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const R w = load_fact(0, q, k);
                    same_s[q][k] = entry_ok(q, k) ? (V)w : (V)0;
                }
                same_n[q] = (V)0;
            } else {
                IO2 z[K];
#pragma unroll
                for (int k = 0; k < K; ++k) z[k] = load_goom(0, q, k);
                same_n[q] = row_shift_of(z, q);
                // the one conversion's rounding is the same at every step and adds up along the chain: made in double, rounded once
#pragma unroll
                for (int k = 0; k < K; ++k)
                    same_s[q][k] = entry_ok(q, k) ? (V)scaled_entry((double)z[k][0], (double)z[k][1], (double)same_n[q]) : (V)0;
            }
        }
        if (FACT) same_common = *reinterpret_cast<const double *>(left0 + (size_t)DP * lfc * sizeof(R));
    }

    // ---- initial vector: this lane's columns c + 16 k, mantissas times 2^eh
    V hm[K];
    double eh = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) hm[k] = (V)0;
    if (a.init_mode == 0) {
        if (c == 0) hm[0] = (V)1; // the identity's only column
    } else if (a.init_mode == 1) {
        long long iidx = chain;
        if (a.init_group > 0) {
            long long grp = chunk / a.init_group;
            if (grp >= a.init_ngroups) grp = a.init_ngroups - 1;
            iidx = (item * a.init_ngroups + grp) * (a.init_group + 1) + (chunk - grp * a.init_group);
        }
        const unsigned char *ip = a.init + iidx * a.init_stride;
        const bool f64 = sizeof(R) == 8 || a.fact_f64;
        bool nz = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = c + 16 * k;
            if (j < d) {
                hm[k] = f64 ? (V) reinterpret_cast<const double *>(ip)[(size_t)j * a.fact_cols] : (V) reinterpret_cast<const float *>(ip)[(size_t)j * a.fact_cols];
                nz = nz || hm[k] != (V)0;
            }
        }
        eh = *reinterpret_cast<const double *>(ip + (size_t)DP * a.fact_cols * (f64 ? 8 : 4));
        if (__builtin_amdgcn_ballot_w64(nz) == 0) eh = 0.0; // a zero vector has no exponent
    } else if (a.init_mode == 2) {
        const IO2 *gp = reinterpret_cast<const IO2 *>(a.init + item * a.init_stride);
        double u = -__builtin_huge_val();
        IO2 z[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int j = c + 16 * k;
            z[k] = gp[j < d ? j : 0];
            if (j >= d) z[k][0] = -__builtin_huge_val();
            u = raw_max(u, (double)z[k][0]);
        }
        u = max16(u);
        eh = u > -1.0e300 ? __builtin_ceil(u * kLog2e) : 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) hm[k] = (V)scaled_entry((double)z[k][0], (double)z[k][1], eh);
    }

    unsigned char *fact_steps = a.out_fact_steps ? a.out_fact_steps + chain * (a.chunk_len + 1) * a.fact_stride : nullptr;
    // the vector as column `col` of a factored matrix, with its own exponent
    auto store_fact = [&](unsigned char *dst, int col, bool f64) {
        if (wave == 0 && g == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const size_t at = (size_t)(c + 16 * k) * a.fact_cols + col;
                if (f64)
                    reinterpret_cast<double *>(dst)[at] = (double)hm[k];
                else
                    reinterpret_cast<float *>(dst)[at] = (float)hm[k];
            }
            if (c == 0) reinterpret_cast<double *>(dst + (size_t)DP * a.fact_cols * (f64 ? 8 : 4))[col] = eh;
        }
    };
    if (fact_steps) store_fact(fact_steps, 0, sizeof(R) == 8);

    IO *scaled = reinterpret_cast<IO *>(a.out_scaled);
    IO *logscale = reinterpret_cast<IO *>(a.out_logscale);
    const bool last_only = a.out_goom_last_only != 0;

    auto step = [&](long long t, Raw &r) {
        // ---- the lane's row of A_t h, as part 2^(n + base)
        V part = (V)0, n = (V)0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            V p = (V)0, nq = (V)0;
            if constexpr (SAME) {
#pragma unroll
                for (int k = 0; k < K; ++k) p = p + same_s[q][k] * hm[k];
                nq = same_n[q];
            } else if constexpr (FACT) {
#pragma unroll
                for (int k = 0; k < K; ++k) p = p + (entry_ok(q, k) ? (V)r.w[q][k] : (V)0) * hm[k];
            } else {
                nq = row_shift_of(r.z[q], q);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const V s = scaled_entry((V)r.z[q][k][0], (V)r.z[q][k][1], nq);
                    p = p + (entry_ok(q, k) ? s : (V)0) * hm[k];
                }
            }
            p = sum16(p);
            part = c == q ? p : part;
            n = c == q ? nq : n;
        }
        // ---- the bias on the same base; the sum on the larger exponent
        const double base = eh + (FACT ? (SAME ? same_common : r.common) : 0.0);
        V bm = (V)0, be = (V)kNone;
        double cs = 0.0; // rescaled bias and states, in powers of two
        if (bias_goom) {
            if (a.io_shift) cs = (double)r.shift * kLog2e;
            const double x = __builtin_fma((double)r.bias[0], kLog2e, -(cs + base));
            if (!(x < (double)kNone)) { // (NaN goes on)
                const double xe = __builtin_rint(x); // (the double series wants at most half a unit)
                be = (V)xe;
                if constexpr (sizeof(V) == 4)
                    bm = Comp<float>::apply_sign(__builtin_amdgcn_exp2f((float)(x - xe)), (float)r.bias[1]);
                else
                    bm = Comp<double>::apply_sign(Comp<double>::exp2_small(x - xe), (double)r.bias[1]);
            }
        } else if (bias_fact) {
            bm = (V)r.bias_m;
            if (bm != (V)0) {
                const V e = Comp<V>::exponent_of(bm);
                bm = Comp<V>::ldexp_(bm, -(int)e);
                be = e + (V)(r.bias_e - base);
            }
        }
        const V pe = part != (V)0 ? Comp<V>::exponent_of(part) + n : (V)kNone;
        const V ex = be > pe ? be : pe;
        V m = Comp<V>::ldexp_(part, (int)Comp<V>::clamp_shift(n - ex)) + Comp<V>::ldexp_(bm, (int)Comp<V>::clamp_shift(be - ex));
        const int buf = (int)(t & 1);
        if (owner) {
            vm[buf][orow] = row_ok ? m : (V)0;
            vx[buf][orow] = row_ok ? ex : (V)kNone;
        }
        if (a.out_goom && owner && row_ok && (!last_only || t == len - 1)) {
            const size_t at = (size_t)(last_only ? chain : item * a.steps + t0 + t) * n_rows + orow;
            IO re;
            if constexpr (sizeof(V) == 4 && sizeof(IO) == 4)
                re = Comp<float>::out_re_f(m, (float)((double)ex + base + cs));
            else
                re = (IO)Comp<double>::out_re((double)m, (double)ex, base + cs);
            reinterpret_cast<IO2 *>(a.out_goom)[at] = IO2{re, m < (V)0 ? Comp<IO>::pi() : (IO)0};
        }
        // ---- everyone reads the vector and brings it onto its largest exponent
        if (NW > 1) {
            __syncthreads();
        } else { // a wave's LDS operations complete in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        V xs[K], xm = (V)kNone;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            hm[k] = vm[buf][c + 16 * k];
            xs[k] = vx[buf][c + 16 * k];
            xm = raw_max(xm, xs[k]);
        }
        xm = max16(xm);
        const bool none = !(xm > (V)(0.5f * kNone));
        if (none) xm = (V)0;
#pragma unroll
        for (int k = 0; k < K; ++k) hm[k] = Comp<V>::ldexp_(hm[k], (int)Comp<V>::clamp_shift(xs[k] - xm));
        eh = none ? 0.0 : base + (double)xm;
        if (fact_steps) store_fact(fact_steps + (t + 1) * a.fact_stride, 0, sizeof(R) == 8);
        if (scaled) {
            // exp(z - c + 2), c the log of the largest magnitude: the mantissa over the largest one, times e^2
            V am = (V)0;
#pragma unroll
            for (int k = 0; k < K; ++k) am = raw_max(am, Comp<V>::abs_(hm[k]));
            am = max16(am);
            if (wave == (NW - 1) && g == 3) { // (not the wave that has carries to store)
                const size_t at = (size_t)(item * a.steps + t0 + t);
                const V f = am > (V)0 ? (V)7.38905609893065022723 / am : (V)0;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (c + 16 * k < d) scaled[at * d + c + 16 * k] = (IO)(am > (V)0 ? hm[k] * f : (V)0);
                if (logscale && c == 0) logscale[at] = am > (V)0 ? (IO)(((double)Comp<V>::log2_abs(am) + eh) * kLn2) : (IO)-__builtin_huge_val();
            }
        }
    };

    Raw ring[PD];
#pragma unroll
    for (int i = 0; i < PD; ++i) load(i < len ? i : len - 1, ring[i]);
    for (long long t = 0; t < len; t += PD) {
#pragma unroll
        for (int i = 0; i < PD; ++i) {
            if (t + i < len) { // (the whole workgroup)
                step(t + i, ring[i]);
                load(t + i + PD < len ? t + i + PD : len - 1, ring[i]);
            }
        }
    }
    if (a.out_fact_final) store_fact(a.out_fact_final + chain * a.fact_stride, a.bias_mode == 1 ? a.bias_col : 0, sizeof(R) == 8 || a.fact_f64);
}

template <typename R, typename IO, int DP, int NW, bool FACT, bool FULL, bool SAME, int PD>
int launch_vec(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    if (grid <= 0) return GOOM_OK;
    if (grid > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many chains for one launch (%lld)", grid);
    goom::prof_begin(ctx, label);
    hipLaunchKernelGGL((vec_walk_kernel<R, IO, DP, NW, FACT, FULL, SAME, PD>), dim3((unsigned)grid), dim3(NW * 64), 0, ctx->stream, args);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch vec_walk_kernel");
}

template <typename R, int DP, int NW, int PD> int goom_factors(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    if (args.left_step_stride == 0 && args.steps > 1) return launch_vec<R, R, DP, NW, false, false, true, 2>(ctx, args, grid, label);
    if (args.n == DP && args.d == DP) return launch_vec<R, R, DP, NW, false, true, false, PD>(ctx, args, grid, label);
    return launch_vec<R, R, DP, NW, false, false, false, PD>(ctx, args, grid, label);
}

template <typename R, int DP, int NW, int PD> int factored(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    if (args.left_same) return launch_vec<R, R, DP, NW, true, false, true, 2>(ctx, args, grid, label);
    return launch_vec<R, R, DP, NW, true, false, false, PD>(ctx, args, grid, label);
}

} // namespace

int dispatch_vec(goom_ctx *ctx, const ChainArgs &args, int dp, int f64, int left_fact, long long grid, const char *label)
{
    if (left_fact) {
        switch (dp) {
        case 16: return f64 ? factored<double, 16, 1, 4>(ctx, args, grid, label) : factored<float, 16, 1, 4>(ctx, args, grid, label);
        case 32: return f64 ? factored<double, 32, 2, 4>(ctx, args, grid, label) : factored<float, 32, 1, 4>(ctx, args, grid, label);
        case 64: return f64 ? factored<double, 64, 8, 4>(ctx, args, grid, label) : factored<float, 64, 4, 4>(ctx, args, grid, label);
        default: return f64 ? factored<double, 128, 8, 2>(ctx, args, grid, label) : factored<float, 128, 8, 2>(ctx, args, grid, label);
        }
    }
    switch (dp) {
    case 16: return f64 ? goom_factors<double, 16, 1, 2>(ctx, args, grid, label) : goom_factors<float, 16, 1, 2>(ctx, args, grid, label);
    case 32: return f64 ? goom_factors<double, 32, 2, 2>(ctx, args, grid, label) : goom_factors<float, 32, 1, 2>(ctx, args, grid, label);
    case 64: return f64 ? goom_factors<double, 64, 4, 2>(ctx, args, grid, label) : goom_factors<float, 64, 2, 2>(ctx, args, grid, label);
    default: return f64 ? goom_factors<double, 128, 8, 1>(ctx, args, grid, label) : goom_factors<float, 128, 8, 2>(ctx, args, grid, label);
    }
}

} // namespace goom_chain
