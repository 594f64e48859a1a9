// Backward passes (paper Section 3.1: the redefined finite derivatives of the real absolute value, the real
// logarithm and the complex exponential; Section 4.3: the recurrence h_t = A_t h_{t-1} + b_t over GOOMs).
//
// Codecs.  The log-magnitude of a GOOM is log(abs(x)) with d abs / dx := +-1 (+1 at zero, never 0) and
// d log(u) / du := 1 / (u + eps); the real value of a GOOM is Re exp(x') with d exp(x') / dx' := exp(x') +- eps.
// Both are one multiply per element around the forward value.
//
// Recurrence.  With G_t[i] the gradient of a loss with respect to the log-magnitude of h_t[i], the adjoint of the
// value h_t[i] is lam_t = G_t / h_t + A_{t+1}^T lam_{t+1}: the same kind of recurrence in reverse time over the
// transposed matrices, so it runs through the forward scan itself on operands prepared here (matrices transposed
// and reversed in time, bias G_t / h_t as GOOMs: the adjoints shrink as fast as the states grow, and only their
// products with states and matrix entries return to ordinary magnitudes).  The gradients with respect to
// log-magnitudes are lam_t[i] A_t[i, j] h_{t-1}[j] and lam_t[i] b_t[i].
//
// A float log-magnitude near 1000 is only good to 6e-5, and the adjoints are signed sums with cancellation, so the
// adjoint recurrence is not run on the adjoints themselves but on lamhat_t = lam_t e^(c_t), c_t the whole number
// nearest the largest log-magnitude of h_t: lamhat_t = G_t / (h_t e^(-c_t)) + (e^(c_t - c_{t+1}) A_{t+1}^T) lamhat_{t+1},
// whose operands all have log-magnitudes of ordinary size (h'_t - c_t is exact in the component type; the matrices
// move by the whole number c_t - c_{t+1}).  The shift is undone, in double, where the gradients are formed.
#include "goom_vec.h"

namespace {

constexpr double kInvPi = 0.318309886183790671538;

template <typename R> struct C2;
template <> struct C2<float> { typedef float2 type; };
template <> struct C2<double> { typedef double2 type; };

template <typename R> __device__ inline bool odd_phase(R im)
{
    const int k = (int)__builtin_rint((double)im * kInvPi);
    return (k & 1) != 0;
}
// e^s for a double sum of log-magnitudes, to the accuracy of the result type: float results take the hardware
// exponential on the rounded argument (its error, |s| 2^-24, is far inside a gradient's tolerance)
template <typename R> __device__ inline double exp_for(double s)
{
    if (sizeof(R) == 4) return (double)__builtin_amdgcn_exp2f((float)(s * 1.44269504088896340736));
    return exp(s);
}
// log of a positive real to the accuracy of the result type
template <typename R> __device__ inline double log_for(double g)
{
    if (sizeof(R) == 4) return (double)__builtin_logf((float)g);
    return log(g);
}
template <typename R> __device__ inline R pi_of() { return sizeof(R) == 4 ? (R)3.14159274101257324219f : (R)3.14159265358979311600; }

// ---- codecs -----------------------------------------------------------------------------------------------
template <typename R> __global__ __launch_bounds__(256) void to_goom_backward_kernel(const R *__restrict__ x, const R *__restrict__ g,
                                                                                     R *__restrict__ gx, size_t n, double eps)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double v = (double)x[i];
        const double s = v < 0.0 ? -1.0 : 1.0; // zero counts as non-negative
        gx[i] = (R)((double)g[i] * s / (__builtin_fabs(v) + eps));
    }
}

template <typename R> __global__ __launch_bounds__(256) void from_goom_backward_kernel(const typename C2<R>::type *__restrict__ y,
                                                                                       const R *__restrict__ gx, R *__restrict__ g, size_t n, double eps)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const typename C2<R>::type z = y[i];
        const double mag = exp((double)z.x);
        const double v = odd_phase<R>(z.y) ? -mag : mag;
        g[i] = (R)((double)gx[i] * (v + (v < 0.0 ? -eps : eps)));
    }
}

// scaled exponentiation (Section 4.3): the log-scaling constant takes no gradient, so the gradient with respect to the
// log-magnitude is the scaled value times the gradient with respect to it
template <typename R> __global__ __launch_bounds__(256) void scaled_exp_backward_kernel(const R *__restrict__ scaled, const R *__restrict__ g, R *__restrict__ gre,
                                                                                        size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) gre[i] = scaled[i] * g[i];
}

// ---- recurrence -------------------------------------------------------------------------------------------
// Operands of the adjoint recurrence, indexed by s = T - 1 - t, for the scan kernels that read A transposed and in reverse order
// themselves: gt[b, s, i] = GOOM(G[b, t, i]) - H[b, t, i] (zero where G is zero or the state is
// zero) on the scale e^(c_t), and the shift of step s's log-magnitudes, shift[b, s] = c_t - c_{t+1} (-inf for s = 0: the zero
// matrix).  A group of lanes per (b, s), so that a wave serves two to eight steps of short vectors.
template <typename R> __global__ __launch_bounds__(256) void bwd_shift_kernel(const typename C2<R>::type *__restrict__ H, const R *__restrict__ G,
                                                                             float *__restrict__ shift, typename C2<R>::type *__restrict__ gt,
                                                                             long long T, int d, long long nsteps, int group, int absolute)
{
    // absolute: shift[b, s] = c_t itself (for a scan that rescales its bias and its stored states by it, its factors unchanged)
    // a group of `group` lanes (8, 16, 32 or 64: the power of two that holds d, or the whole wave) per (b, s)
    typedef typename C2<R>::type c2;
    const int lane = threadIdx.x & 63, sub = lane % group;
    const long long step = ((long long)blockIdx.x * 256 + threadIdx.x) / group;
    const bool active = step < nsteps;
    const long long b = active ? step / T : 0, s = active ? step % T : 0;
    const R ninf = sizeof(R) == 4 ? (R)-__builtin_huge_valf() : (R)-__builtin_huge_val();
    const long long t = T - 1 - s;
    // c_t and c_{t+1}: the whole numbers nearest the largest log-magnitudes of h_t and h_{t+1} (0 for a zero state)
    auto scale_of = [&](long long tt) {
        R top = ninf;
        if (active && tt < T)
            for (int i = sub; i < d; i += group) {
                const R v = H[(size_t)(b * T + tt) * d + i].x;
                top = v > top ? v : top;
            }
        for (int sft = group >> 1; sft > 0; sft >>= 1) {
            const R o = __shfl_xor(top, sft, 64);
            top = o > top ? o : top;
        }
        const bool finite = top > ninf && top < -ninf;
        return finite ? (R)__builtin_rint((double)top) : (R)0;
    };
    const R ct = scale_of(t);
    const R cnext = absolute ? (R)0 : scale_of(t + 1); // (uniform: a kernel argument)
    if (!active) return;
    if (sub == 0) shift[b * T + s] = absolute ? (float)ct : s == 0 ? (float)ninf : (float)(ct - cnext);
    for (int i = sub; i < d; i += group) {
        const R gv = G[(size_t)(b * T + t) * d + i];
        const c2 h = H[(size_t)(b * T + t) * d + i];
        c2 o;
        const bool live = gv != (R)0 && h.x > ninf;
        o.x = live ? (R)(log_for<R>(__builtin_fabs((double)gv)) - ((double)h.x - (double)ct)) : ninf;
        o.y = (live && ((gv < (R)0) != odd_phase<R>(h.y))) ? pi_of<R>() : (R)0;
        gt[(size_t)(b * T + s) * d + i] = o;
    }
}

// Gradients from the scaled adjoints mu[b, s] = lam[b, T - 1 - s] e^(c_{T-1-s}) (GOOMs), one wave per (b, t), no
// workgroup barrier:
//   gA[b, t, i, j] = lam_t[i] A_t[i, j] h_{t-1}[j],   gb[b, t, i] = lam_t[i] b_t[i].
// Sums of three log-magnitudes are formed in double (the adjoint and the state are large and opposite); the wave
// keeps the adjoint's and the previous state's log-magnitudes and signs in LDS words of its own.
constexpr int kGradWaves = 4;

template <typename R> __global__ __launch_bounds__(kGradWaves * 64) void bwd_grad_kernel(const typename C2<R>::type *__restrict__ A,
                                                                                         const typename C2<R>::type *__restrict__ bias,
                                                                                         const typename C2<R>::type *__restrict__ h0,
                                                                                         const typename C2<R>::type *__restrict__ H,
                                                                                         const typename C2<R>::type *__restrict__ mu, R *__restrict__ gA,
                                                                                         R *__restrict__ gb, long long T, int d, long long nsteps)
{
    typedef typename C2<R>::type c2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long step = (long long)blockIdx.x * kGradWaves + wave;
    if (step >= nsteps) return; // whole wave
    const long long b = step / T, t = step % T;
    // this wave's words: lre[d], pre[d] (double), signs packed with them as separate int arrays
    double *lre = reinterpret_cast<double *>(smem) + (size_t)wave * 2 * d;
    double *pre = lre + d;
    int *lneg = reinterpret_cast<int *>(reinterpret_cast<double *>(smem) + (size_t)kGradWaves * 2 * d) + (size_t)wave * 2 * d;
    int *pneg = lneg + d;
    const double ninf = -__builtin_huge_val();
    // c_t: the whole number nearest the largest log-magnitude of h_t
    const c2 *ht = H + (size_t)(b * T + t) * d;
    R top = sizeof(R) == 4 ? (R)-__builtin_huge_valf() : (R)-__builtin_huge_val();
    for (int i = lane; i < d; i += 64) {
        const R v = ht[i].x;
        top = v > top ? v : top;
    }
    for (int sft = 32; sft > 0; sft >>= 1) {
        const R o = __shfl_xor(top, sft, 64);
        top = o > top ? o : top;
    }
    const bool finite = (double)top > ninf && (double)top < -ninf;
    const double ct = finite ? __builtin_rint((double)top) : 0.0;
    for (int i = lane; i < d; i += 64) {
        const c2 l = mu[(size_t)(b * T + (T - 1 - t)) * d + i];
        lre[i] = (double)l.x - ct; // -inf stays -inf
        lneg[i] = odd_phase<R>(l.y) ? 1 : 0;
        c2 p = c2{(R)ninf, (R)0};
        if (t > 0) p = H[(size_t)(b * T + t - 1) * d + i];
        else if (h0) p = h0[(size_t)b * d + i];
        pre[i] = (double)p.x;
        pneg[i] = odd_phase<R>(p.y) ? 1 : 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const c2 *ap = A + (size_t)(b * T + t) * d * d;
    R *op = gA + (size_t)(b * T + t) * d * d;
    auto one = [&](int e, c2 a) {
        const int i = e / d, j = e - i * d;
        const double s = lre[i] + (double)a.x + pre[j];
        const bool live = lre[i] > ninf && (double)a.x > ninf && pre[j] > ninf;
        const double v = live ? exp_for<R>(s) : 0.0;
        const bool neg = (lneg[i] ^ pneg[j] ^ (odd_phase<R>(a.y) ? 1 : 0)) != 0;
        return (R)(neg ? -v : v);
    };
    const int nn = d * d;
    if (sizeof(R) == 4 && (nn & 1) == 0) {
        // two adjacent entries per lane and pass: one 16-byte load, one 8-byte store
        const float4 *ap4 = reinterpret_cast<const float4 *>(ap);
        float2 *op2 = reinterpret_cast<float2 *>(op);
        for (int q = lane; q < nn / 2; q += 64) {
            const float4 w = ap4[q];
            float2 o;
            o.x = (float)one(2 * q, c2{(R)w.x, (R)w.y});
            o.y = (float)one(2 * q + 1, c2{(R)w.z, (R)w.w});
            op2[q] = o;
        }
    } else {
        for (int e = lane; e < nn; e += 64) op[e] = one(e, ap[e]);
    }
    if (gb) {
        for (int i = lane; i < d; i += 64) {
            const c2 bb = bias[(size_t)(b * T + t) * d + i];
            const bool live = lre[i] > ninf && (double)bb.x > ninf;
            const double v = live ? exp_for<R>(lre[i] + (double)bb.x) : 0.0;
            const bool neg = (lneg[i] ^ (odd_phase<R>(bb.y) ? 1 : 0)) != 0;
            gb[(size_t)(b * T + t) * d + i] = (R)(neg ? -v : v);
        }
    }
}

// gh0[b, j] = sum_i gA[b, 0, i, j]   (= h_{-1}[j] sum_i lam_0[i] A_0[i, j]), summed in a fixed order
template <typename R> __global__ __launch_bounds__(128) void bwd_h0_kernel(const R *__restrict__ gA, R *__restrict__ gh0, long long T, int d)
{
    const long long b = blockIdx.x;
    for (int j = threadIdx.x; j < d; j += 128) {
        double acc = 0.0;
        for (int i = 0; i < d; ++i) acc += (double)gA[((size_t)b * T * d + i) * d + j];
        gh0[(size_t)b * d + j] = (R)acc;
    }
}

// One matrix for all steps: its gradient is A[i, j] sum_t lam_t[i] h_{t-1}[j].  partial[b, q] = sum over the steps of span q of
// u_t v_t^T, DP x DP doubles (rows and columns beyond d are zero), with u_t[i] = lam_t[i] e^r and v_t[j] = h_{t-1}[j] e^(-r), r the
// largest log-magnitude of h_{t-1} (|v| <= 1; u is of the size of the gradient's terms).  u and v of step 0 are kept for the initial state's
// gradient.
//
// Sixteen steps at a time.  Each of the four waves forms u and v of four of them in LDS (side by side where DP <= 32) and writes those steps'
// bias gradients lam_t[i] b_t[i]; their operands were loaded a turn before.  The sum over the sixteen steps is then a matrix product on the double
// matrix instruction, 16 x 16 x 4: a wave owns a row of tiles and reads five doubles a lane for every four steps of DP = 64.  As a sum in
// registers, sixteen neighbouring entries a thread, each step read sixteen doubles a lane, and the 64 x 1000 steps of d = 64 took 75 us with 64
// steps a workgroup, now 38 with 125 (and the sums over workgroups 14, now 8); bound by the loads of 115 MB and the conversions on them.
constexpr int kOuterSteps = 16;

typedef double outer_d4 __attribute__((ext_vector_type(4)));

// the largest of a group of lanes (16, 32 or 64 of them; none of the values NaN)
template <typename R, int GROUP> __device__ inline R group_max(R x)
{
    x = goom_chain::max16(x);
    if (GROUP == 64) return goom_chain::Comp<R>::xor16_32_max(x);
    if (GROUP == 32) {
        const R o = __shfl_xor(x, 16, 64);
        x = o > x ? o : x;
    }
    return x;
}

template <typename R, int DP> __global__ __launch_bounds__(256) void bwd_outer_kernel(const typename C2<R>::type *__restrict__ bias,
                                                                                     const typename C2<R>::type *__restrict__ h0,
                                                                                     const typename C2<R>::type *__restrict__ H,
                                                                                     const typename C2<R>::type *__restrict__ mu, R *__restrict__ gb,
                                                                                     double *__restrict__ partial, double *__restrict__ uv0, long long T, int d,
                                                                                     int nsplit)
{
    typedef typename C2<R>::type c2;
    constexpr int GROUP = DP < 64 ? DP : 64; // lanes that serve one step
    constexpr int NE = DP / GROUP;           // entries a lane
    constexpr int SPW = 64 / GROUP;          // steps of a wave at once
    constexpr int ROUNDS = kOuterSteps / 4 / SPW;
    constexpr int NT = DP / 16;              // tiles in a row
    constexpr int TPW = NT >= 4 ? NT / 4 : 1; // rows of tiles a wave
    constexpr int LD = DP + 2;
    __shared__ double u[kOuterSteps][LD], v[kOuterSteps][LD];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), sub = lane % GROUP;
    const int g = lane >> 4, c = lane & 15;
    const long long b = blockIdx.x / nsplit;
    const int q = (int)(blockIdx.x - b * nsplit);
    const long long per = (T + nsplit - 1) / nsplit, t0 = q * per, t1 = t0 + per < T ? t0 + per : T;
    const R ninf = sizeof(R) == 4 ? (R)-__builtin_huge_valf() : (R)-__builtin_huge_val();
    const c2 none = {ninf, (R)0};

    struct Operands {
        c2 h[NE], p[NE], l[NE], b[NE];
    };
    Operands ring[ROUNDS];
    auto load = [&](long long tb, int round, Operands &o) {
        const long long t = tb + 4 * wave + round * SPW + lane / GROUP;
        const bool in = t < t1;
        const size_t at = (size_t)(b * T + (in ? t : t0)) * d;
        const c2 *prev = t > 0 ? H + at - d : h0 ? h0 + (size_t)b * d : nullptr;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = sub + GROUP * e;
            const bool live = in && i < d;
            o.h[e] = o.p[e] = o.l[e] = o.b[e] = none;
            if (live) {
                o.h[e] = H[at + i];
                o.l[e] = mu[(size_t)(b * T + (T - 1 - t)) * d + i];
                if (prev) o.p[e] = prev[i];
                if (gb) o.b[e] = bias[at + i];
            }
        }
    };
    auto form = [&](long long tb, int round, const Operands &o) {
        const int kb = 4 * wave + round * SPW + lane / GROUP;
        const long long t = tb + kb;
        // c_t: the whole number nearest the largest log-magnitude of h_t; r: the largest log-magnitude of h_{t-1}
        R top = ninf, big = ninf;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            top = o.h[e].x > top ? o.h[e].x : top;
            big = o.p[e].x > big ? o.p[e].x : big;
        }
        top = group_max<R, GROUP>(top);
        big = group_max<R, GROUP>(big);
        const double ct = (top > ninf && top < -ninf) ? __builtin_rint((double)top) : 0.0;
        const double r = (double)big;
        const bool any = big > ninf && big < -ninf;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = sub + GROUP * e;
            const double lre = (double)o.l[e].x - ct; // log-magnitude of lam_t[i]; -inf stays -inf
            const bool lneg = odd_phase<R>(o.l[e].y);
            double uu = (any && lre > (double)ninf) ? exp_for<R>(lre + r) : 0.0; // (float GOOMs: the hardware exponential of the small double sum)
            double vv = (any && o.p[e].x > ninf) ? exp_for<R>((double)o.p[e].x - r) : 0.0;
            uu = lneg ? -uu : uu;
            vv = odd_phase<R>(o.p[e].y) ? -vv : vv;
            if (gb && t < t1 && i < d) {
                const bool live = lre > (double)ninf && o.b[e].x > ninf;
                const double w = live ? exp_for<R>(lre + (double)o.b[e].x) : 0.0;
                gb[(size_t)(b * T + t) * d + i] = (R)(lneg != odd_phase<R>(o.b[e].y) ? -w : w);
            }
            if (t == 0 && i < d) {
                uv0[((size_t)b * 2) * d + i] = uu;
                uv0[((size_t)b * 2 + 1) * d + i] = vv;
            }
            u[kb][i] = uu;
            v[kb][i] = vv;
        }
    };

    outer_d4 acc[TPW][NT];
#pragma unroll
    for (int w = 0; w < TPW; ++w)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[w][n] = outer_d4{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) load(t0, k, ring[k]);
    for (long long tb = t0; tb < t1; tb += kOuterSteps) {
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            form(tb, k, ring[k]);
            load(tb + kOuterSteps, k, ring[k]);
        }
        __syncthreads();
        if (wave * TPW < NT) {
#pragma unroll
            for (int k = 0; k < kOuterSteps; k += 4) {
                double y[NT];
#pragma unroll
                for (int n = 0; n < NT; ++n) y[n] = v[k + g][16 * n + c];
#pragma unroll
                for (int w = 0; w < TPW; ++w) {
                    const double x = u[k + g][16 * (wave * TPW + w) + c];
#pragma unroll
                    for (int n = 0; n < NT; ++n) acc[w][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y[n], acc[w][n], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    if (wave * TPW >= NT) return;
    double *out = partial + (size_t)blockIdx.x * DP * DP;
#pragma unroll
    for (int w = 0; w < TPW; ++w)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int x = 0; x < 4; ++x) out[(size_t)(16 * (wave * TPW + w) + 4 * x + g) * DP + 16 * n + c] = acc[w][n][x];
}

// gA[b, i, j] = A[b, i, j] sum_q partial[b, q, i, j] (in the order of q);  gh0[b, j] = v_0[j] sum_i u_0[i] A[b, i, j]  (uv0[b] = u_0, v_0)
template <typename R> __global__ __launch_bounds__(256) void bwd_outer_finish_kernel(const typename C2<R>::type *__restrict__ A, const double *__restrict__ partial,
                                                                                     const double *__restrict__ uv0, R *__restrict__ gA,
                                                                                     R *__restrict__ gh0, int d, int dp, int nsplit)
{
    typedef typename C2<R>::type c2;
    // A workgroup an item summed the spans and took an exponential and a logarithm in double for every entry, and for every entry once more for
    // gh0: 104 us for 64 items of d = 64 (16 spans).  Now 256 entries a workgroup, and gh0 in workgroups of its own.
    const long long b = blockIdx.x;
    const double ninf = -__builtin_huge_val();
    const int e = (int)blockIdx.y * 256 + threadIdx.x;
    if (blockIdx.y < (unsigned)((d * d + 255) / 256)) {
        if (e >= d * d) return;
        const int i = e / d, j = e - i * d;
        double acc = 0.0;
        for (int q = 0; q < nsplit; ++q) acc += partial[((size_t)b * nsplit + q) * dp * dp + (size_t)i * dp + j];
        const c2 a = A[(size_t)b * d * d + e];
        // (through the logarithm of the sum: the entry alone may lie outside the range of a double)
        const double mag = (acc != 0.0 && (double)a.x > ninf) ? exp((double)a.x + log(__builtin_fabs(acc))) : 0.0;
        gA[(size_t)b * d * d + e] = (R)((acc < 0.0) != odd_phase<R>(a.y) ? -mag : mag);
        return;
    }
    // the item's workgroups after those, where there are any: gh0, sixteen columns each, sixteen threads a column (four threads a column in one
    // workgroup took sixteen exponentials and logarithms one after the other, and the launch 14 us for d = 64)
    __shared__ double part[16][17];
    const int c = threadIdx.x & 15, p = threadIdx.x >> 4;
    const int j = ((int)blockIdx.y - (d * d + 255) / 256) * 16 + c;
    double acc = 0.0;
    for (int i = p; i < d && j < d; i += 16) {
        const c2 a = A[(size_t)b * d * d + (size_t)i * d + j];
        const double ui = uv0[((size_t)b * 2) * d + i];
        const double mag = (ui != 0.0 && (double)a.x > ninf) ? exp((double)a.x + log(__builtin_fabs(ui))) : 0.0;
        acc += (ui < 0.0) != odd_phase<R>(a.y) ? -mag : mag;
    }
    part[p][c] = acc;
    __syncthreads();
    if (p == 0 && j < d) {
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) sum += part[k][c];
        gh0[(size_t)b * d + j] = (R)(sum * uv0[((size_t)b * 2 + 1) * d + j]);
    }
}

unsigned blocks_for(size_t n)
{
    const size_t b = (n + 255) / 256;
    return (unsigned)(b < 65536 * 16 ? (b ? b : 1) : 65536 * 16);
}

} // namespace

namespace goom {

int launch_to_goom_backward(goom_ctx *ctx, const void *x, const void *g, void *gx, size_t n, int dtype, double eps)
{
    if (n == 0) return GOOM_OK;
    prof_begin(ctx, "to_goom_backward");
    if (dtype == GOOM_C64)
        hipLaunchKernelGGL(to_goom_backward_kernel<float>, dim3(blocks_for(n)), dim3(256), 0, ctx->stream, static_cast<const float *>(x),
                           static_cast<const float *>(g), static_cast<float *>(gx), n, eps);
    else
        hipLaunchKernelGGL(to_goom_backward_kernel<double>, dim3(blocks_for(n)), dim3(256), 0, ctx->stream, static_cast<const double *>(x),
                           static_cast<const double *>(g), static_cast<double *>(gx), n, eps);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch to_goom_backward");
}

int launch_scaled_exp_backward(goom_ctx *ctx, const void *scaled, const void *g, void *gre, size_t n, int dtype)
{
    if (n == 0) return GOOM_OK;
    prof_begin(ctx, "scaled_exp_backward");
    if (dtype == GOOM_C64)
        hipLaunchKernelGGL(scaled_exp_backward_kernel<float>, dim3(blocks_for(n)), dim3(256), 0, ctx->stream, static_cast<const float *>(scaled),
                           static_cast<const float *>(g), static_cast<float *>(gre), n);
    else
        hipLaunchKernelGGL(scaled_exp_backward_kernel<double>, dim3(blocks_for(n)), dim3(256), 0, ctx->stream, static_cast<const double *>(scaled),
                           static_cast<const double *>(g), static_cast<double *>(gre), n);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch scaled_exp_backward");
}

int launch_from_goom_backward(goom_ctx *ctx, const void *y, const void *gx, void *g, size_t n, int dtype, double eps)
{
    if (n == 0) return GOOM_OK;
    prof_begin(ctx, "from_goom_backward");
    if (dtype == GOOM_C64)
        hipLaunchKernelGGL(from_goom_backward_kernel<float>, dim3(blocks_for(n)), dim3(256), 0, ctx->stream, static_cast<const float2 *>(y),
                           static_cast<const float *>(gx), static_cast<float *>(g), n, eps);
    else
        hipLaunchKernelGGL(from_goom_backward_kernel<double>, dim3(blocks_for(n)), dim3(256), 0, ctx->stream, static_cast<const double2 *>(y),
                           static_cast<const double *>(gx), static_cast<double *>(g), n, eps);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch from_goom_backward");
}

// At[b] = A[b]^T, d x d (one matrix per batch item)
template <typename R> __global__ __launch_bounds__(256) void bwd_transpose_kernel(const typename C2<R>::type *__restrict__ A, typename C2<R>::type *__restrict__ At, int d)
{
    const size_t base = (size_t)blockIdx.x * d * d;
    for (int e = threadIdx.x; e < d * d; e += 256) At[base + e] = A[base + (size_t)(e % d) * d + e / d];
}

template <typename R> static int bwd_shift_t(goom_ctx *ctx, const void *H, const void *G, float *shift, void *gt, long long T, int d, long long batch,
                                             const void *A = nullptr, void *At = nullptr)
{
    typedef typename C2<R>::type c2;
    const long long nsteps = batch * T;
    prof_begin(ctx, "affine_backward_prepare_operands");
    const int group = d <= 8 ? 8 : d <= 16 ? 16 : d <= 32 ? 32 : 64;
    const long long per_block = 256 / group;
    hipLaunchKernelGGL(bwd_shift_kernel<R>, dim3((unsigned)((nsteps + per_block - 1) / per_block)), dim3(256), 0, ctx->stream, static_cast<const c2 *>(H),
                       static_cast<const R *>(G), shift, static_cast<c2 *>(gt), T, d, nsteps, group, At ? 1 : 0);
    if (At) hipLaunchKernelGGL(bwd_transpose_kernel<R>, dim3((unsigned)batch), dim3(256), 0, ctx->stream, static_cast<const c2 *>(A), static_cast<c2 *>(At), d);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch bwd_shift_kernel");
}

// (float components, d = 16 and 32: every other size and type is walked by goom_vec_adjoint.hip)
int launch_affine_backward_prepare(goom_ctx *ctx, const void *H, const void *G, float *shift, void *gt, long long T, int d, long long batch)
{
    if (batch * T > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    return bwd_shift_t<float>(ctx, H, G, shift, gt, T, d, batch);
}

int launch_initial_state_gradient(goom_ctx *ctx, const void *gA, void *gh0, long long T, int d, long long batch)
{
    prof_begin(ctx, "affine_backward_initial_state");
    hipLaunchKernelGGL(bwd_h0_kernel<float>, dim3((unsigned)batch), dim3(128), 0, ctx->stream, static_cast<const float *>(gA), static_cast<float *>(gh0), T, d);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch bwd_h0_kernel");
}

// One matrix for all steps, scan over the matrix itself: At [batch, d, d] = A^T, shift[b, s] = c_t, gt as above
int launch_affine_backward_prepare_one_matrix(goom_ctx *ctx, const void *A, const void *H, const void *G, void *At, float *shift, void *gt, long long T, int d,
                                              long long batch, int dtype)
{
    if (batch * T > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    return dtype == GOOM_C64 ? bwd_shift_t<float>(ctx, H, G, shift, gt, T, d, batch, A, At) : bwd_shift_t<double>(ctx, H, G, shift, gt, T, d, batch, A, At);
}

template <typename R> static int bwd_grad_t(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *mu, void *gA,
                                            void *gb, void *gh0, long long T, int d, long long batch)
{
    typedef typename C2<R>::type c2;
    const size_t lds = (size_t)kGradWaves * d * (2 * sizeof(double) + 2 * sizeof(int));
    const long long nsteps = batch * T;
    prof_begin(ctx, "affine_backward_gradients");
    hipLaunchKernelGGL(bwd_grad_kernel<R>, dim3((unsigned)((nsteps + kGradWaves - 1) / kGradWaves)), dim3(kGradWaves * 64), lds, ctx->stream,
                       static_cast<const c2 *>(A), static_cast<const c2 *>(bias), static_cast<const c2 *>(h0), static_cast<const c2 *>(H),
                       static_cast<const c2 *>(mu), static_cast<R *>(gA), static_cast<R *>(gb), T, d, nsteps);
    if (gh0) hipLaunchKernelGGL(bwd_h0_kernel<R>, dim3((unsigned)batch), dim3(128), 0, ctx->stream, static_cast<const R *>(gA), static_cast<R *>(gh0), T, d);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch bwd_grad_kernel");
}

int launch_affine_backward_gradients(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *mu, void *gA,
                                     void *gb, void *gh0, long long T, int d, long long batch)
{
    if (batch * T > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    return bwd_grad_t<float>(ctx, A, bias, h0, H, mu, gA, gb, gh0, T, d, batch);
}

// One matrix for all steps.  partial: [batch, nsplit, dp, dp] doubles (dp: d padded to 16, 32, 64 or 128); uv0: [batch, 2, d] doubles
template <typename R> static int bwd_grad_ti_t(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *mu, void *gA, void *gb,
                                               void *gh0, double *uv0, double *partial, int nsplit, long long T, int d, long long batch)
{
    typedef typename C2<R>::type c2;
    const int dp = d <= 16 ? 16 : d <= 32 ? 32 : d <= 64 ? 64 : 128;
    prof_begin(ctx, "affine_backward_gradients");
    const dim3 grid((unsigned)(batch * nsplit));
    const c2 *bp = static_cast<const c2 *>(bias), *hp = static_cast<const c2 *>(h0), *Hp = static_cast<const c2 *>(H), *mp = static_cast<const c2 *>(mu);
    R *gbp = static_cast<R *>(gb);
    if (dp == 16) hipLaunchKernelGGL((bwd_outer_kernel<R, 16>), grid, dim3(256), 0, ctx->stream, bp, hp, Hp, mp, gbp, partial, uv0, T, d, nsplit);
    else if (dp == 32) hipLaunchKernelGGL((bwd_outer_kernel<R, 32>), grid, dim3(256), 0, ctx->stream, bp, hp, Hp, mp, gbp, partial, uv0, T, d, nsplit);
    else if (dp == 64) hipLaunchKernelGGL((bwd_outer_kernel<R, 64>), grid, dim3(256), 0, ctx->stream, bp, hp, Hp, mp, gbp, partial, uv0, T, d, nsplit);
    else hipLaunchKernelGGL((bwd_outer_kernel<R, 128>), grid, dim3(256), 0, ctx->stream, bp, hp, Hp, mp, gbp, partial, uv0, T, d, nsplit);
    hipLaunchKernelGGL(bwd_outer_finish_kernel<R>, dim3((unsigned)batch, (unsigned)((d * d + 255) / 256 + (gh0 ? (d + 15) / 16 : 0))), dim3(256), 0, ctx->stream, static_cast<const c2 *>(A), partial, uv0, static_cast<R *>(gA),
                       static_cast<R *>(gh0), d, dp, nsplit);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch bwd_outer_kernel");
}

int launch_affine_backward_gradients_one_matrix(goom_ctx *ctx, const void *A, const void *bias, const void *h0, const void *H, const void *mu, void *gA,
                                                void *gb, void *gh0, void *uv0, void *partial, int nsplit, long long T, int d, long long batch, int dtype)
{
    if (batch * T > 0x7fffffffLL || batch * nsplit > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    return dtype == GOOM_C64 ? bwd_grad_ti_t<float>(ctx, A, bias, h0, H, mu, gA, gb, gh0, static_cast<double *>(uv0), static_cast<double *>(partial), nsplit, T, d, batch)
                             : bwd_grad_ti_t<double>(ctx, A, bias, h0, H, mu, gA, gb, gh0, static_cast<double *>(uv0), static_cast<double *>(partial), nsplit, T, d,
                                                     batch);
}

} // namespace goom
