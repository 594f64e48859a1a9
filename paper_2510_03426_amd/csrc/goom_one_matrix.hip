// The recurrence h <- A h + b_t with one matrix for all steps (paper Section 4.3, the state-space layer): every chunk of a sequence walked from
// its incoming vector, or from zero.
//
// The chunks of an item share the matrix, so sixteen of them are the sixteen columns of a matrix product: a workgroup takes sixteen chunks of
// an item, wave w the rows 16 w .. 16 w + 15 of A, converted once and held as the left operand of the matrix instruction for all steps.  The
// state (DP x 16) passes through LDS between two steps, one barrier a step: a wave writes its rows on an exponent of their own per
// column, every wave brings what it reads onto the column's largest (as in goom_carry.hip).  A row's sum and its bias meet on the larger
// exponent of the two, and leave as a GOOM from there.
//
// Bound by a step's own instructions, 1.1 us at d = 64 (480 vector instructions of a wave that has its matrix core to itself, half of them the
// four entries' bias and logarithm; 16 matrix instructions).  Float 64 x 1000 steps of d = 64, a pass over all: one wave a chain 44 us (chunks of
// 64), now 29 (of 16); the recurrence 179 -> 135 us and its backward pass 330 -> 258; complex128 607 -> 171, 758 -> 325; 256 x 512 x 64 float 269 ->
// 145; 128 x 4096 x 32 296 -> 264, complex128 1361 -> 366; one sequence of 16384 x 64 346 -> 186.
#include "goom_vec.h"

namespace goom_chain {

namespace {

struct OneMatrixArgs {
    const unsigned char *prepared; // per item: A's mantissas [DP][prepared_cols] (float or double), its rows' powers of two (double)
    long long prepared_stride;
    int prepared_cols, prepared_f64;
    const unsigned char *bias;     // GOOMs [batch][T][d]
    const float *io_shift;         // SHIFT: [batch][T]
    long long T, L, C;             // steps, steps a chunk, chunks an item
    long long launched;            // of them, this launch
    int d, groups;                 // groups of sixteen chunks an item
    const unsigned char *init;     // NULL: zero; else factored vectors [batch][C], or in groups (see ChainArgs)
    long long init_stride, init_group, init_ngroups;
    int fact_cols, fact_f64;
    unsigned char *out_goom;       // [batch][T][d], or NULL
    void *out_scaled, *out_logscale;
    unsigned char *out_fact;       // the chunks' last vectors as column `fact_col` of factored matrices [batch][C], or NULL
    long long fact_stride;
    int fact_col;
};

// natural log of |x| 2^(w + E), w a whole number (see goom_vec.hip: the logarithm of a mantissa)
__device__ inline float log_of(float x, float w, double E)
{
#pragma clang fp contract(off)
    const float kLn2Hi = 0.693147182464599609375f;
    const float kLn2Lo = -1.90465429995776806e-9f;
    const float e = Comp<float>::exponent_of(x);
    const float l2 = __builtin_amdgcn_logf(__builtin_fabsf(__builtin_ldexpf(x, -(int)e))); // (-inf of a zero)
    const float s = (float)(E + (double)(w + e));
    return __builtin_fmaf(s, kLn2Hi, __builtin_fmaf(s, kLn2Lo, l2 * kLn2Hi));
}
__device__ inline double log_of(double x, double w, double E) { return Comp<double>::out_re(x, w, E); }

// FULL: d = DP.  (All conditions of a step are masks: a branch around an entry costs more than the entry.)
template <typename R, int DP, bool FULL, bool SHIFT, int PD> __global__ __launch_bounds__(DP * 4) void one_matrix_walk_kernel(OneMatrixArgs a)
{
    typedef typename Comp<R>::vec4 vec4;
    typedef R R2 __attribute__((ext_vector_type(2)));
    constexpr int KT = DP / 16;
    constexpr int LDC = DP + Comp<R>::kPad;
    constexpr int LDX = KT + (KT > 4 ? 4 : 0);
    constexpr R kLast = (R)(sizeof(R) == 4 ? 149 : 1074);
    __shared__ __align__(16) R state[2][16 * LDC];
    __shared__ __align__(16) R expo[2][16 * LDX];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const R kNegInf = Comp<R>::neg_inf();
    const long long item = blockIdx.x / a.groups;
    const long long chunk_raw = (long long)(blockIdx.x % a.groups) * 16 + c;
    const bool active = chunk_raw < a.launched;
    const long long chunk = active ? chunk_raw : a.launched - 1; // (idle columns follow the last chunk and store nothing)
    const long long t0 = chunk * a.L;
    const int len = (int)(a.T - t0 < a.L ? a.T - t0 : a.L); // of this lane's chunk
    const int steps = (int)(a.T < a.L ? a.T : a.L);         // of any (only an item's last chunk is shorter)
    const int row0 = 16 * wave + Comp<R>::row_of(g, 0);     // this lane's rows of the result: row0 + v * dr
    constexpr int dr = sizeof(R) == 4 ? 1 : 4;

    // ---- the matrix: row 16 wave + c, columns 16 kt + 4 g + v; its rows' powers of two for this lane's rows of the result
    R am[KT][4], nv[4];
    {
        const unsigned char *pp = a.prepared + item * a.prepared_stride;
        const bool f64 = sizeof(R) == 8 || a.prepared_f64;
        const int row = 16 * wave + c;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 16 * kt + 4 * g + v;
                const bool ok = row < d && k < d;
                const size_t at = ok ? (size_t)row * a.prepared_cols + k : 0;
                const R x = f64 ? (R) reinterpret_cast<const double *>(pp)[at] : (R) reinterpret_cast<const float *>(pp)[at];
                am[kt][v] = ok ? x : (R)0;
            }
        const double *np = reinterpret_cast<const double *>(pp + (size_t)DP * a.prepared_cols * (f64 ? 8 : 4));
#pragma unroll
        for (int v = 0; v < 4; ++v) nv[v] = row0 + v * dr < d ? (R)np[row0 + v * dr] : (R)0;
    }

    // ---- the incoming vector
    R own[4], ownx = (R)0;
    double E = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) own[v] = (R)0;
    if (a.init) {
        long long idx = item * a.C + chunk;
        if (a.init_group > 0) {
            long long grp = chunk / a.init_group;
            if (grp >= a.init_ngroups) grp = a.init_ngroups - 1;
            idx = (item * a.init_ngroups + grp) * (a.init_group + 1) + (chunk - grp * a.init_group);
        }
        const unsigned char *ip = a.init + idx * a.init_stride;
        const bool f64 = sizeof(R) == 8 || a.fact_f64;
        R some = (R)0;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (row0 + v * dr < d) {
                const size_t at = (size_t)(row0 + v * dr) * a.fact_cols;
                own[v] = f64 ? (R) reinterpret_cast<const double *>(ip)[at] : (R) reinterpret_cast<const float *>(ip)[at];
                some = own[v] != (R)0 ? (R)1 : some;
            }
        E = *reinterpret_cast<const double *>(ip + (size_t)DP * a.fact_cols * (f64 ? 8 : 4));
        // (a zero vector's exponent says nothing: without rows that are not zero the column has none, see combine)
        if (!(Comp<R>::xor16_32_max(some) > (R)0)) ownx = kNegInf;
    }
    auto publish = [&](int buf) {
        if (sizeof(R) == 4) {
            *reinterpret_cast<vec4 *>(&state[buf][c * LDC + row0]) = vec4{own[0], own[1], own[2], own[3]};
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) state[buf][c * LDC + row0 + v * dr] = own[v];
        }
        if (g == 0) expo[buf][c * LDX + wave] = ownx;
    };

    // ---- what a step reads
    struct Rest {
        R2 b[4];
        float shift;
    };
    const R2 *bias0 = reinterpret_cast<const R2 *>(a.bias) + (size_t)(item * a.T + t0) * d;
    const float *shift0 = SHIFT ? a.io_shift + item * a.T + t0 : nullptr;
    unsigned brow[4];
    bool past[4]; // rows beyond the matrix
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        past[v] = !FULL && row0 + v * dr >= d;
        brow[v] = (unsigned)(past[v] ? d - 1 : row0 + v * dr);
    }
    auto load = [&](int t, Rest &r) {
        const size_t tt = (size_t)(t < len ? t : len - 1); // (a chunk may be longer than 2^32 entries)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (FULL && sizeof(R) == 4) { // four entries side by side
                if (v & 1) continue;
                const vec4 w = *reinterpret_cast<const vec4 *>(bias0 + tt * DP + row0 + v);
                r.b[v] = R2{w[0], w[1]};
                r.b[v + 1] = R2{w[2], w[3]};
            } else {
                r.b[v] = bias0[tt * (size_t)d + brow[v]];
            }
        }
        if (SHIFT) r.shift = shift0[tt];
    };

    R *scaled = reinterpret_cast<R *>(a.out_scaled), *logscale = reinterpret_cast<R *>(a.out_logscale);
    R cs = (R)0;
    double ecol = 0.0;
    bool col_zero = false;
    vec4 sv[KT];
    // the state as every wave reads it, brought onto the column's largest exponent
    auto combine = [&](int buf) {
        R x[KT], mx = kNegInf;
        if (KT % 4 == 0) {
#pragma unroll
            for (int k = 0; k < KT; k += 4) {
                const vec4 w = *reinterpret_cast<const vec4 *>(&expo[buf][c * LDX + k]);
#pragma unroll
                for (int v = 0; v < 4; ++v) x[(k + v) % KT] = w[v];
            }
        } else {
#pragma unroll
            for (int k = 0; k < KT; ++k) x[k] = expo[buf][c * LDX + k];
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) sv[kt] = *reinterpret_cast<const vec4 *>(&state[buf][c * LDC + 16 * kt + 4 * g]);
#pragma unroll
        for (int k = 0; k < KT; ++k) mx = raw_max(mx, x[k]);
        col_zero = !(mx > kNegInf);
        cs = col_zero ? (R)0 : mx;
        ecol = col_zero ? 0.0 : E + (double)cs;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const int sh = (int)Comp<R>::clamp_shift(x[kt] - cs);
#pragma unroll
            for (int v = 0; v < 4; ++v) sv[kt][v] = Comp<R>::ldexp_(sv[kt][v], sh);
        }
    };
    // exp(z - c + 2), c the log of the largest magnitude: the mantissa over the largest one, times e^2 (a NaN stays one, and so does the log scale)
    auto store_scaled = [&](int t) {
        R top = (R)0, bad = (R)0;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                top = raw_max(top, Comp<R>::abs_(sv[kt][v]));
                bad = sv[kt][v] != sv[kt][v] ? (R)1 : bad;
            }
        top = Comp<R>::xor16_32_max(top);
        bad = Comp<R>::xor16_32_max(bad);
        const R f = top > (R)0 ? (R)7.38905609893065022723 / top : (R)0;
        const int sh = (int)Comp<R>::clamp_shift(ownx - cs);
        if (active & (t >= 0) & (t < len)) {
            const size_t at = (size_t)(item * a.T + t0 + t);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (!past[v]) scaled[at * d + row0 + v * dr] = Comp<R>::ldexp_(own[v], sh) * f;
            if (logscale && wave == 0 && g == 0)
                logscale[at] = bad > (R)0 ? (R)__builtin_nan("") : top > (R)0 ? (R)(((double)Comp<R>::log2_abs(top) + ecol) * kLn2) : kNegInf;
        }
    };

    Rest ring[PD];
#pragma unroll
    for (int u = 0; u < PD; ++u) load(u, ring[u]);
    publish(0);
    __syncthreads();

    auto step = [&](int t, Rest &r) __attribute__((always_inline)) {
        const int buf = t & 1;
        combine(buf);
        if (scaled) store_scaled(t - 1);
        // (Sums of sixteen terms, and these in pairs, as short as the vector kernel's: one sum over all of them is no faster, and rounds further off.  192
        // rotations of d = 128, relative error of the states 5.1e-7, now 2.5e-7, and 3.1e-7 with one chain a wave.)
        vec4 part[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            part[kt] = vec4{0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) part[kt] = Comp<R>::mfma(am[kt][v], sv[kt][v], part[kt]);
        }
#pragma unroll
        for (int h = KT / 2; h >= 1; h /= 2)
#pragma unroll
            for (int kt = 0; kt < h; ++kt) part[kt] += part[kt + h];
        const vec4 acc = part[0];
        E = ecol;
        // ---- the bias on the same base
        R bm[4], be[4];
        const double cshift = SHIFT ? (double)r.shift * kLog2e : 0.0; // rescaled bias and states, in powers of two
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double x = __builtin_fma((double)r.b[v][0], kLog2e, -(cshift + E));
            const bool none = (x < (double)kNone) | past[v]; // (NaN goes on)
            const double xe = __builtin_rint(x);
            be[v] = none ? (R)kNone : (R)xe;
            if constexpr (sizeof(R) == 4)
                bm[v] = Comp<float>::apply_sign(__builtin_amdgcn_exp2f((float)(x - xe)), (float)r.b[v][1]);
            else
                bm[v] = Comp<double>::apply_sign(Comp<double>::exp2_small(x - xe), (double)r.b[v][1]);
            bm[v] = none ? (R)0 : bm[v];
        }
        load(t + PD, r);
        // A bias below the last place of terms that cancel exactly does not outlive them; beside a large entry of A that meets a zero of the
        // vector it is the result (see goom_vec.hip).  Rare: the terms' magnitudes are summed where it may be so.
        bool alone = false;
#pragma unroll
        for (int v = 0; v < 4; ++v) alone |= (acc[v] == (R)0) & (be[v] < nv[v] - kLast) & (be[v] > (R)kNone);
        if (__builtin_amdgcn_ballot_w64(alone) != 0) {
            vec4 mag = vec4{0, 0, 0, 0};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    R x = am[kt][v];
                    if constexpr (sizeof(R) == 4) asm volatile("" : "+v"(x)); // (worked out here, not once for all steps in registers of its own)
                    mag = Comp<R>::mfma(Comp<R>::abs_(x), Comp<R>::abs_(sv[kt][v]), mag);
                }
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (acc[v] == (R)0 && mag[v] > (R)0 && be[v] < Comp<R>::exponent_of(mag[v]) + nv[v] - kLast) {
                    bm[v] = (R)0;
                    be[v] = (R)kNone;
                }
        }
        // ---- the sums on the larger exponents, the rows' largest
        R m[4], ex[4], mx = kNegInf;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const R pe = acc[v] != (R)0 ? Comp<R>::exponent_of(acc[v]) + nv[v] : (R)kNone;
            ex[v] = raw_max(be[v], pe);
            m[v] = Comp<R>::ldexp_(acc[v], (int)Comp<R>::clamp_shift(nv[v] - ex[v])) + Comp<R>::ldexp_(bm[v], (int)Comp<R>::clamp_shift(be[v] - ex[v]));
            mx = raw_max(m[v] != (R)0 ? ex[v] : kNegInf, mx);
        }
        mx = Comp<R>::xor16_32_max(mx);
        const R ref = mx > kNegInf ? mx : (R)0;
#pragma unroll
        for (int v = 0; v < 4; ++v) own[v] = Comp<R>::ldexp_(m[v], (int)Comp<R>::clamp_shift(ex[v] - ref));
        ownx = mx;
        publish(buf ^ 1);
        if (a.out_goom) {
            R2 z[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) z[v] = R2{log_of(m[v], ex[v], E + cshift), m[v] < (R)0 ? Comp<R>::pi() : (R)0};
            if (active & (t < len)) {
                R2 *o = reinterpret_cast<R2 *>(a.out_goom) + (size_t)(item * a.T + t0 + t) * d + row0;
                if constexpr (FULL && sizeof(R) == 4) {
#pragma unroll
                    for (int v = 0; v < 4; v += 2) *reinterpret_cast<vec4 *>(o + v) = vec4{z[v][0], z[v][1], z[v + 1][0], z[v + 1][1]};
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (!past[v]) o[v * dr] = z[v];
                }
            }
        }
        __syncthreads();
    };
    // whole turns of the ring, then what is left, whose values are there already or are loaded again
    int t = 0;
    for (; t + PD <= steps; t += PD) {
#pragma unroll
        for (int u = 0; u < PD; ++u) step(t + u, ring[u]);
    }
#pragma unroll 1
    for (; t < steps; ++t) {
        load(t, ring[0]);
        step(t, ring[0]);
    }
    combine(steps & 1);
    if (scaled) store_scaled(steps - 1);
    if (a.out_fact && active) { // (full chunks only)
        unsigned char *dst = a.out_fact + (item * a.C + chunk) * a.fact_stride;
        const int sh = (int)Comp<R>::clamp_shift(ownx - cs);
        const bool f64 = sizeof(R) == 8 || a.fact_f64;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const size_t at = (size_t)(row0 + v * dr) * a.fact_cols + a.fact_col;
            const R x = Comp<R>::ldexp_(own[v], sh);
            if (f64)
                reinterpret_cast<double *>(dst)[at] = (double)x;
            else
                reinterpret_cast<float *>(dst)[at] = (float)x;
        }
        if (wave == 0 && g == 0) reinterpret_cast<double *>(dst + (size_t)DP * a.fact_cols * (f64 ? 8 : 4))[a.fact_col] = ecol;
    }
}

template <typename R, int DP, int PD> void launch_walk(hipStream_t st, const OneMatrixArgs &a, unsigned grid)
{
    const bool full = a.d == DP;
    if (a.io_shift && full)
        hipLaunchKernelGGL((one_matrix_walk_kernel<R, DP, true, true, PD>), dim3(grid), dim3(4 * DP), 0, st, a);
    else if (a.io_shift)
        hipLaunchKernelGGL((one_matrix_walk_kernel<R, DP, false, true, PD>), dim3(grid), dim3(4 * DP), 0, st, a);
    else if (full)
        hipLaunchKernelGGL((one_matrix_walk_kernel<R, DP, true, false, PD>), dim3(grid), dim3(4 * DP), 0, st, a);
    else
        hipLaunchKernelGGL((one_matrix_walk_kernel<R, DP, false, false, PD>), dim3(grid), dim3(4 * DP), 0, st, a);
}

} // namespace

// (complex128 above 64: a wave's state and matrix do not fit its registers beside each other; at 16 rows a step of one chain a wave is short
// already: 32 x 1000 x 16 took 83 us a pass this way, 68 that.  The vector kernels take both.)
bool one_matrix_walk_applies(int dp, int dtype) { return dp >= 32 && (dtype == GOOM_C64 || dp <= 64); }

int launch_one_matrix_walk(goom_ctx *ctx, const goom::ChainLaunch &l, int dp)
{
    OneMatrixArgs a;
    a.prepared = static_cast<const unsigned char *>(l.left_prepared);
    a.prepared_stride = l.prepared_stride;
    a.prepared_cols = l.prepared_cols;
    a.prepared_f64 = l.prepared_f64;
    a.bias = static_cast<const unsigned char *>(l.bias);
    a.io_shift = l.io_shift;
    a.T = l.steps;
    a.L = l.chunk_len;
    a.C = (l.steps + l.chunk_len - 1) / l.chunk_len;
    a.launched = l.chunks_launched;
    a.d = l.d;
    a.groups = (int)((l.chunks_launched + 15) / 16);
    a.init = l.init_mode == 1 ? static_cast<const unsigned char *>(l.init) : nullptr;
    a.init_stride = l.init_stride;
    a.init_group = l.init_group;
    a.init_ngroups = l.init_ngroups;
    a.fact_cols = l.fact_cols;
    a.fact_f64 = l.fact_f64;
    a.out_goom = static_cast<unsigned char *>(l.out_goom);
    a.out_scaled = l.out_scaled;
    a.out_logscale = l.out_logscale;
    a.out_fact = static_cast<unsigned char *>(l.out_fact_final);
    a.fact_stride = l.fact_stride;
    a.fact_col = l.bias_col;
    const long long grid = l.batch * a.groups;
    if (grid <= 0) return GOOM_OK;
    if (grid > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many chains for one launch (%lld)", grid);
    const unsigned n = (unsigned)grid;
    hipStream_t st = ctx->stream;
    goom::prof_begin(ctx, l.label);
    if (l.dtype == GOOM_C128) {
        if (dp == 32) launch_walk<double, 32, 4>(st, a, n);
        else launch_walk<double, 64, 4>(st, a, n);
    } else {
        if (dp == 32) launch_walk<float, 32, 4>(st, a, n);
        else if (dp == 64) launch_walk<float, 64, 4>(st, a, n);
        else launch_walk<float, 128, 4>(st, a, n);
    }
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch one_matrix_walk_kernel");
}

} // namespace goom_chain
