// Chains over factored matrices with a matrix state: the carries of a scan (prefixes of its chunk products), the products of
// groups and of spans of chunk products.  Few chains, each a serial sequence of products S <- T_c S of matrices that lie in
// memory as mantissas with one exponent (goom_internal.h: FactLayout): what counts is the latency of one step.
//
// The general chain kernel gives a chain to one workgroup, a wave to 16 state columns, and takes every factor through LDS: 64 x 64,
// float, 3.0 us a step, of which the matrix instructions of a wave (64 of 32 cycles) are 0.85; double 5 us.  Here
//   * a workgroup owns 16 state columns only (they do not depend on the others) and a wave 16 of the rows: a quarter of the matrix
//     instructions a step at 64 x 64, an eighth at 128 x 128; the slabs of a chain are different workgroups;
//   * a wave then needs 16 rows of the factor and nobody else does: they go from memory straight into the operand registers, NPF
//     factors ahead, and are brought onto their rows' powers of two between the matrix instructions of the step before;
//   * the state (DP x 16) passes through LDS, one barrier a step: a wave writes its 16 rows on an exponent of their own per column,
//     every wave brings what it reads onto the column's largest.
// Measured (a launch of 15 to 22 steps, its start of about 10 us included): 64 x 64 float 69 -> 30 us, 50 x 50 57 -> 27, 64 x 64 double 112 -> 51, 8 x 8
// 19.7 -> 11.4.  What is left of a step (0.85 us, float 64 x 64) is issue: some 250 vector instructions a wave around 16 matrix
// instructions of 32 cycles.
// Sums run over the contraction index in the order of the general kernel: float prefixes are the same in every bit.
#include "goom_chain_kernel.h"

namespace goom_chain {

namespace {

template <typename R, int DP, int NPF, bool FULL, bool BIAS> __global__ __launch_bounds__(DP * 4) void carry_kernel(ChainArgs a)
{
    typedef typename Comp<R>::vec4 vec4;
    constexpr int KT = DP / 16;
    constexpr int LDC = DP + Comp<R>::kPad; // a state column in LDS
    constexpr int LDX = KT + (KT > 4 ? 4 : 0);
    __shared__ __align__(16) R state[2][16 * LDC];
    __shared__ __align__(16) R expo[2][16 * LDX];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int n_rows = a.n, d = a.d, m = a.m, lfc = a.left_fact_cols;
    const R kNegInf = Comp<R>::neg_inf();
    const long long nchains = (long long)gridDim.x / a.nslabs;
    const int slab = (int)((long long)blockIdx.x / nchains);
    const long long chain = (long long)blockIdx.x % nchains;
    const long long item = chain / a.chunks_launched, chunk = chain % a.chunks_launched;
    const long long t0 = chunk * a.chunk_len;
    long long len = a.steps - t0;
    if (len > a.chunk_len) len = a.chunk_len;
    if (len < 1) return; // the whole workgroup
    const long long chain_global = item * a.chunks_per_item + chunk;
    const int col = 16 * slab + c;
    const size_t mant_bytes = (size_t)DP * lfc * sizeof(R);
    const size_t fact_mant_bytes = (size_t)DP * a.fact_cols * sizeof(R);

    // ---- factors.  Entry (kt, v) of a lane: row 16 wave + c, column 16 kt + 4 g + v (any order of the contraction index will do
    // as long as the state is read in the same one)
    const unsigned char *left0 = a.left + item * a.left_batch_stride + t0 * a.left_step_stride;
    const unsigned lane_off = (unsigned)(((16 * wave + c) * lfc + 4 * g) * (int)sizeof(R));
    unsigned zero = 0; // keeps the loads below on the vector path: a scalar load's return would be waited for with every LDS read
    asm volatile("" : "+v"(zero));
    struct Raw {
        R x[KT][4];
        double common;
        R b[BIAS ? 4 : 1];
        double be;
    };
    auto load = [&](long long t, Raw &r) {
        const unsigned char *src = left0 + (t < len ? t : len - 1) * a.left_step_stride;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const vec4 w = *reinterpret_cast<const vec4 *>(src + lane_off + (FULL || 16 * kt < lfc ? 16 * kt : 0) * (int)sizeof(R));
#pragma unroll
            for (int v = 0; v < 4; ++v) r.x[kt][v] = w[v];
        }
        r.common = *reinterpret_cast<const double *>(src + mant_bytes + zero);
        if (BIAS) { // column d, the entries of this lane's rows of the result
#pragma unroll
            for (int v = 0; v < 4; ++v) r.b[v] = *reinterpret_cast<const R *>(src + ((16 * wave + Comp<R>::row_of(g, v)) * lfc + d) * (int)sizeof(R));
            r.be = *reinterpret_cast<const double *>(src + mant_bytes + d * sizeof(double) + zero);
        }
    };
    // the row's power of two; the rows' shifts of this lane's part of the result
    auto row_exponent = [&](Raw &r, R (&nv)[4]) {
        R mx = (R)0;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (!FULL && !(16 * wave + c < n_rows && 16 * kt + 4 * g + v < d)) r.x[kt][v] = (R)0;
                mx = sizeof(R) == 4 ? (R)__builtin_fmaxf((float)mx, __builtin_fabsf((float)r.x[kt][v])) : (R)__builtin_fmax((double)mx, __builtin_fabs((double)r.x[kt][v]));
            }
        mx = Comp<R>::xor16_32_max(mx);
        const int e = (mx > (R)0 && mx < -kNegInf) ? Comp<R>::frexp_exp(mx) : 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) nv[v] = (R)__shfl(e, Comp<R>::row_of(g, v), 64);
        return e;
    };

    // ---- initial state: rows 16 wave + row_of(g, v) of column col
    R own[4];        // this lane's part of the state as last written to LDS, on the exponent ownx (of the column, among the wave's rows)
    R ownx = (R)0;
    double E = 0.0;  // the exponent below which the waves' exponents count
    if (a.init_mode == 1) {
        long long iidx = chain_global;
        if (a.init_group > 0) {
            long long grp = chunk / a.init_group;
            if (grp >= a.init_ngroups) grp = a.init_ngroups - 1;
            iidx = (item * a.init_ngroups + grp) * (a.init_group + 1) + (chunk - grp * a.init_group);
        }
        const unsigned char *ip = a.init + iidx * a.init_stride;
#pragma unroll
        for (int v = 0; v < 4; ++v) own[v] = reinterpret_cast<const R *>(ip)[(size_t)(16 * wave + Comp<R>::row_of(g, v)) * a.fact_cols + col];
        E = reinterpret_cast<const double *>(ip + fact_mant_bytes)[col];
    } else if (a.init_mode == 2) { // GOOMs [d, m]
        const R *gp = reinterpret_cast<const R *>(a.init + item * a.init_stride);
        R re[4], im[4], mx = kNegInf;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * wave + Comp<R>::row_of(g, v);
            const bool ok = row < d && col < m;
            re[v] = ok ? gp[((size_t)row * m + col) * 2] : kNegInf;
            im[v] = ok ? gp[((size_t)row * m + col) * 2 + 1] : (R)0;
            mx = re[v] > mx ? re[v] : mx;
        }
        mx = wave_xor_max<R>(mx, 16);
        mx = wave_xor_max<R>(mx, 32);
        ownx = mx > kNegInf ? (R)__builtin_ceil((double)mx * kLog2e) : kNegInf;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const R x = exp2_of<R>(__builtin_fma((double)re[v], kLog2e, mx > kNegInf ? -(double)ownx : 0.0));
            own[v] = Comp<R>::is_negative(im[v]) ? -x : x;
        }
    } else { // identity, zero
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * wave + Comp<R>::row_of(g, v);
            own[v] = (a.init_mode == 0 && row == col && row < d && col < m) ? (R)1 : (R)0;
        }
    }
    auto publish = [&](int buf) {
        if (sizeof(R) == 4) {
            *reinterpret_cast<vec4 *>(&state[buf][c * LDC + 16 * wave + 4 * g]) = vec4{own[0], own[1], own[2], own[3]};
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) state[buf][c * LDC + 16 * wave + Comp<R>::row_of(g, v)] = own[v];
        }
        if (g == 0) expo[buf][c * LDX + wave] = ownx;
    };

    unsigned char *fact_steps = a.out_fact_steps ? a.out_fact_steps + chain_global * (a.chunk_len + 1) * a.fact_stride : nullptr;
    const size_t own_at = (size_t)(16 * wave + Comp<R>::row_of(g, 0)) * a.fact_cols + col;
    const int own_step = Comp<R>::row_of(0, 1) * a.fact_cols;
    auto store_fact = [&](unsigned char *dst, R cs, double e) { // e: the columns' exponents
        const int sh = (int)Comp<R>::clamp_shift(ownx - cs);
        R *mp = reinterpret_cast<R *>(dst) + own_at;
#pragma unroll
        for (int v = 0; v < 4; ++v) mp[(size_t)v * own_step] = Comp<R>::ldexp_(own[v], sh);
        if (wave == 0 && g == 0) reinterpret_cast<double *>(dst + fact_mant_bytes)[col] = e;
    };

    Raw raw[NPF], first;
    R conv[KT][4], nv[4];
    load(0, first);
#pragma unroll
    for (int u = 0; u < NPF; ++u) load(u + 1, raw[u]);
    {
        const int e = row_exponent(first, nv);
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) conv[kt][v] = Comp<R>::ldexp_(first.x[kt][v], -e);
    }
    double common = first.common, be = BIAS ? first.be : 0.0;
    R bias[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) bias[v] = BIAS ? first.b[v] : (R)0;
    publish(0);
    __syncthreads();

    R cs = (R)0;       // the column's largest exponent among the waves
    double ecol = 0.0; // E + cs
    bool col_zero = false;
    auto combine = [&](int buf, R (&x)[KT]) {
        R mx = kNegInf;
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
        for (int k = 0; k < KT; ++k) mx = x[k] > mx ? x[k] : mx;
        col_zero = !(mx > kNegInf);
        cs = col_zero ? (R)0 : mx;
        ecol = E + (double)cs;
    };

    // ring: where factor t + 1 waits
    auto step = [&](long long t, Raw &ring) __attribute__((always_inline)) {
        const int buf = (int)(t & 1);
        R bx[KT];
        combine(buf, bx);
        vec4 sv[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) sv[kt] = *reinterpret_cast<const vec4 *>(&state[buf][c * LDC + 16 * kt + 4 * g]);
        if (fact_steps && t <= len) store_fact(fact_steps + t * a.fact_stride, cs, ecol);
        // (a column of zeros has no say in the exponent that the columns will share)
        if (a.out_fact_final && t == len) store_fact(a.out_fact_final + chain_global * a.fact_stride, cs, a.final_common_exponent && col_zero ? kNegBig : ecol);
        R nn[4];
        const int e = row_exponent(ring, nn);
        vec4 acc = vec4{0, 0, 0, 0};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const int sh = (int)Comp<R>::clamp_shift(bx[kt] - cs);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc = Comp<R>::mfma(conv[kt][v], Comp<R>::ldexp_(sv[kt][v], sh), acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) conv[kt][v] = Comp<R>::ldexp_(ring.x[kt][v], -e);
        }
        // entry (row, col) is acc 2^(nv + E) (+ bias 2^be) now
        E = ecol + common;
        R mx = kNegInf;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const R lg = acc[v] != (R)0 ? Comp<R>::exponent_of(acc[v]) + nv[v] : kNegInf;
            mx = Comp<R>::max_(lg, mx);
        }
        const bool bias_lane = BIAS && col == a.bias_col;
        double bsh = 0.0;
        if (BIAS) {
            bsh = be - E;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (!FULL && 16 * wave + Comp<R>::row_of(g, v) >= n_rows) bias[v] = (R)0;
                const R lb = bias[v] != (R)0 ? Comp<R>::exponent_of(bias[v]) + (R)bsh : kNegInf;
                if (bias_lane) mx = Comp<R>::max_(lb, mx);
            }
        }
        mx = Comp<R>::xor16_32_max(mx);
        if (bias_lane && mx > kNegInf) mx += (R)1; // room for the sum of two terms
        const R ref = mx > kNegInf ? mx : (R)0;
        if (a.out_goom && t == len - 1 && col < m) { // the last prefix, as GOOMs (from the product itself: nothing is rescaled away)
            R *o = reinterpret_cast<R *>(a.out_goom) + ((size_t)chain_global * n_rows * m + col) * 2;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * wave + Comp<R>::row_of(g, v);
                if (FULL || row < n_rows) {
                    o[(size_t)row * m * 2] = Comp<R>::out_re(acc[v], nv[v], E);
                    o[(size_t)row * m * 2 + 1] = acc[v] < (R)0 ? Comp<R>::pi() : (R)0;
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            own[v] = Comp<R>::ldexp_(acc[v], (int)Comp<R>::clamp_shift(nv[v] - ref));
            if (BIAS) {
                double s = bsh - (double)ref;
                s = s > -4000.0 ? (s < 4000.0 ? s : 4000.0) : -4000.0;
                const R xb = Comp<R>::ldexp_(bias[v], (int)s);
                if (bias_lane) own[v] += xb;
            }
        }
        ownx = mx;
        publish(buf ^ 1);
        // the next step's factor, and the place of it in the ring
#pragma unroll
        for (int v = 0; v < 4; ++v) nv[v] = nn[v];
        // (copied in so many instructions: left to itself the compiler loads the next ones into other registers and copies those, waiting)
        common = ring.common;
        asm volatile("" : "+v"(common));
        if (BIAS) {
            be = ring.be;
            asm volatile("" : "+v"(be));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                bias[v] = ring.b[v];
                asm volatile("" : "+v"(bias[v]));
            }
        }
        load(t + 1 + NPF, ring);
        __syncthreads();
    };
    // Whole turns of the ring, the chain's end (step len: the last state is stored) somewhere in the last one, what follows it being
    // dropped: a way out between two steps of a turn makes the compiler copy the ring's registers, and wait for the loads in them.
    for (long long t = 0; t <= len; t += NPF) {
#pragma unroll
        for (int u = 0; u < NPF; ++u) step(t + u, raw[u]);
    }
}

// Columns 0 .. ncommon - 1 of a factored matrix onto their largest exponent (which a left factor's columns share).  A workgroup a matrix:
// the first `launched` of every item's `per_item`.
template <typename R>
__global__ __launch_bounds__(256) void common_exponent_kernel(unsigned char *fact, long long stride, long long launched, long long per_item, int rows, int cols,
                                                              int ncommon)
{
    unsigned char *f = fact + ((long long)blockIdx.x / launched * per_item + (long long)blockIdx.x % launched) * stride;
    R *mp = reinterpret_cast<R *>(f);
    double *ep = reinterpret_cast<double *>(f + (size_t)rows * cols * sizeof(R));
    double emax = kNegBig;
    for (int j = threadIdx.x & 63; j < ncommon; j += 64) emax = ep[j] > emax ? ep[j] : emax;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) emax = fmax(emax, __shfl_xor(emax, s, 64));
    if (emax == kNegBig) emax = 0.0;
    for (int i = threadIdx.x; i < rows * cols; i += 256) {
        const int j = i % cols;
        const double e = j < ncommon ? ep[j] - emax : 0.0;
        mp[i] = Comp<R>::ldexp_(mp[i], (int)(e > -4000.0 ? e : -4000.0));
    }
    __syncthreads(); // every exponent has been read
    for (int j = threadIdx.x; j < cols; j += 256) ep[j] = j < ncommon ? emax : ep[j] == kNegBig ? 0.0 : ep[j];
}

template <typename R, int DP, int NPF> void launch_one_carry(hipStream_t st, const ChainArgs &a, unsigned grid)
{
    const bool full = a.n == DP && a.d == DP;
    if (a.bias_mode)
        hipLaunchKernelGGL((carry_kernel<R, DP, NPF, false, true>), dim3(grid), dim3(4 * DP), 0, st, a);
    else if (full)
        hipLaunchKernelGGL((carry_kernel<R, DP, NPF, true, false>), dim3(grid), dim3(4 * DP), 0, st, a);
    else
        hipLaunchKernelGGL((carry_kernel<R, DP, NPF, false, false>), dim3(grid), dim3(4 * DP), 0, st, a);
}

} // namespace

int launch_carry(goom_ctx *ctx, const ChainArgs &args, int dp, int f64, long long grid, const char *label)
{
    if (args.out_goom && !args.out_goom_last_only) return goom::fail(ctx, GOOM_EUNSUPPORTED, "chains of factored matrices store their last state only");
    if (grid <= 0) return GOOM_OK;
    if (grid * args.nslabs > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many chains for one launch (%lld)", grid);
    const unsigned n = (unsigned)(grid * args.nslabs);
    hipStream_t st = ctx->stream;
    goom::prof_begin(ctx, label);
    if (f64) {
        if (dp == 16) launch_one_carry<double, 16, 4>(st, args, n);
        else if (dp == 32) launch_one_carry<double, 32, 4>(st, args, n);
        else if (dp == 64) launch_one_carry<double, 64, 3>(st, args, n);
        else launch_one_carry<double, 128, 1>(st, args, n);
    } else {
        if (dp == 16) launch_one_carry<float, 16, 4>(st, args, n);
        else if (dp == 32) launch_one_carry<float, 32, 4>(st, args, n);
        else if (dp == 64) launch_one_carry<float, 64, 4>(st, args, n);
        else launch_one_carry<float, 128, 2>(st, args, n);
    }
    if (args.out_fact_final && args.final_common_exponent && args.m > 1) {
        const int ncommon = args.bias_mode ? args.d : args.m;
        unsigned char *f = args.out_fact_final;
        if (f64)
            hipLaunchKernelGGL(common_exponent_kernel<double>, dim3((unsigned)grid), dim3(256), 0, st, f, args.fact_stride, args.chunks_launched,
                               args.chunks_per_item, dp, args.fact_cols, ncommon);
        else
            hipLaunchKernelGGL(common_exponent_kernel<float>, dim3((unsigned)grid), dim3(256), 0, st, f, args.fact_stride, args.chunks_launched,
                               args.chunks_per_item, dp, args.fact_cols, ncommon);
    }
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch carry_kernel");
}

} // namespace goom_chain
