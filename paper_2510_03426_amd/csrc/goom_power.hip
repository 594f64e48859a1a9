// Powers of one matrix, for the recurrence with one matrix for all steps (paper Section 4.3, eq. 25): every full chunk's product is A^L.
//
// The power is a serial chain of products, by squaring and multiplying along L's bits (log2(L) products for the library's own chunk
// lengths, powers of two; a chain of L1 + L2 products before: 115 us at L = 64, d = 64), one workgroup a matrix, so its latency is all that counts.  The
// product of a group of chunks is the same power squared on, in the same launch.  The matrix lies in LDS in double on its rows' powers of two; a wave owns
// sixteen rows, keeps them as left operands in registers (with the rows' powers of two of the step before moved into the columns and
// taken out again as the row's own largest), and reads the right operand straight from LDS.  All in double for both component types:
// the power is applied to a carried vector, where an error relative to its norm has no bound relative to the result.
#include "goom_vec.h"

namespace goom_chain {

namespace {

template <typename V> __device__ inline double entry_of(V re, V im, double n) { return scaled_entry((double)re, (double)im, n); }

// A [batch][d][d] GOOMs of component IO; power: mantissas of component F on their rows' powers of two, row i's at exponent i (a factored matrix
// that every step of a chain shares; on one exponent a matrix in units of its own, D A D^-1, would lose its small columns); prepared: NULL, or the
// matrix itself in the same form; group: NULL, or that power squared `squarings` times more
template <typename IO, typename F, int DP>
__global__ __launch_bounds__((DP / 16) * 64) void power_kernel(const IO *A, int d, long long exponent, unsigned char *power, unsigned char *prepared,
                                                               long long stride, int squarings, unsigned char *group, long long group_stride, int fact_cols)
{
    typedef IO IO2 __attribute__((ext_vector_type(2)));
    constexpr int KS = DP / 4;  // steps of four inner indices
    constexpr int NT = DP / 16; // column tiles, and waves
    constexpr int LD = DP + 2;
    extern __shared__ __align__(16) double lds[];
    double *P = lds;             // [DP][LD], rows on their own powers of two
    double *D = lds + DP * LD;   // [DP] those powers of two
    double *R = D + DP;          // [DP] the rows' scales within a product
    double *DA = R + DP;         // [DP] the matrix's own rows' powers of two

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    const IO2 *src = reinterpret_cast<const IO2 *>(A) + (size_t)blockIdx.x * d * d;

    // the matrix: row by row, sixteen lanes a row
    for (int r0 = 0; r0 < 16; r0 += 4) {
        const int row = 16 * wave + r0 + g;
        IO2 z[NT];
        double u = -__builtin_huge_val();
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            const bool ok = row < d && c + 16 * k < d;
            z[k] = src[ok ? (size_t)row * d + c + 16 * k : 0];
            if (!ok) z[k][0] = -__builtin_huge_val();
            u = raw_max(u, (double)z[k][0]);
        }
        u = max16(u);
        const double n = u > -1.0e300 ? __builtin_ceil(u * kLog2e) : 0.0;
        unsigned char *prep = prepared ? prepared + blockIdx.x * stride : nullptr;
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            const double v = entry_of(z[k][0], z[k][1], n);
            P[row * LD + c + 16 * k] = v;
            if (prep && row < d && c + 16 * k < d) reinterpret_cast<F *>(prep)[(size_t)row * fact_cols + c + 16 * k] = (F)v;
        }
        if (c == 0) {
            D[row] = DA[row] = n;
            if (prep && row < d) reinterpret_cast<double *>(prep + (size_t)DP * fact_cols * sizeof(F))[row] = u > -1.0e300 ? n : (double)kNone;
        }
    }
    __syncthreads();
    int bit = 62;
    while (bit > 0 && !((exponent >> bit) & 1)) --bit;
    unsigned char *dst = power + blockIdx.x * stride;
    for (;;) {
        bool by_matrix = false; // this product: the matrix times the power so far, or its square
        while (bit > 0) {
            // left operand: row 16 wave + c, inner index 4 k + g
            const int arow = 16 * wave + c;
            double a[KS];
            double top = kNegBig;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                if (by_matrix) {
                    const bool ok = arow < d && 4 * k + g < d;
                    const IO2 z = src[ok ? (size_t)arow * d + 4 * k + g : 0];
                    a[k] = ok ? entry_of(z[0], z[1], DA[arow]) : 0.0;
                } else {
                    a[k] = P[arow * LD + 4 * k + g];
                }
                const double e = a[k] != 0.0 ? Comp<double>::exponent_of(a[k]) + D[4 * k + g] : kNegBig;
                top = raw_max(top, e);
            }
            top = Comp<double>::xor16_32_max(top);
            const double row_scale = top > 0.5 * kNegBig ? top : 0.0;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const double sh = D[4 * k + g] - row_scale;
                a[k] = __builtin_ldexp(a[k], (int)Comp<double>::clamp_shift(sh));
            }
            if (g == 0) R[arow] = row_scale + (by_matrix ? DA[arow] : D[arow]); // (read by this wave alone)
            d4 acc[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[nt] = d4{0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[nt] = Comp<double>::mfma(a[k], P[(4 * k + g) * LD + 16 * nt + c], acc[nt]);
            __syncthreads(); // every wave is done with P and D
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * wave + 4 * v + g;
                double m = 0.0;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) m = raw_max(m, __builtin_fabs(acc[nt][v]));
                m = max16(m);
                const double e = m > 0.0 ? Comp<double>::exponent_of(m) : 0.0;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) P[row * LD + 16 * nt + c] = __builtin_ldexp(acc[nt][v], -(int)e);
                if (c == 0) D[row] = m > 0.0 ? R[row] + e : 0.0;
            }
            __syncthreads();
            // (squared: times the matrix where the next bit down is set, and on to that bit)
            if (!by_matrix && ((exponent >> (bit - 1)) & 1)) {
                by_matrix = true;
            } else {
                by_matrix = false;
                --bit;
            }
        }
        // (a zero row has no power of two)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * wave + 4 * v + g;
            double some = 0.0;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) some = P[row * LD + 16 * nt + c] != 0.0 ? 1.0 : some;
            some = max16(some);
            if (c == 0 && row < d) reinterpret_cast<double *>(dst + (size_t)DP * fact_cols * sizeof(F))[row] = some > 0.0 ? D[row] : kNegBig;
        }
        for (int e = threadIdx.x; e < d * d; e += (int)blockDim.x) {
            const int i = e / d, j = e - i * d;
            reinterpret_cast<F *>(dst)[(size_t)i * fact_cols + j] = (F)P[i * LD + j];
        }
        if (!group) return;
        dst = group + blockIdx.x * group_stride;
        group = nullptr;
        bit = squarings; // (that many bits, all zero)
        exponent = 0;
        __syncthreads(); // every wave is done with P and D
    }
}

template <typename IO, typename F, int DP>
int launch(goom_ctx *ctx, const void *A, int d, long long batch, long long exponent, void *power, void *prepared, long long stride,
           int squarings, void *group, long long group_stride, int fact_cols)
{
    const size_t lds = ((size_t)DP * (DP + 2) + 3 * DP) * sizeof(double);
    auto kern = power_kernel<IO, F, DP>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return goom::check_hip(ctx, e, "hipFuncSetAttribute(power_kernel)");
    }
    if (batch > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many matrices for one launch");
    goom::prof_begin(ctx, "affine_phase1_matrix_power");
    hipLaunchKernelGGL(kern, dim3((unsigned)batch), dim3((DP / 16) * 64), lds, ctx->stream, static_cast<const IO *>(A), d, exponent,
                       static_cast<unsigned char *>(power), static_cast<unsigned char *>(prepared), stride, squarings, static_cast<unsigned char *>(group), group_stride,
                       fact_cols);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch power_kernel");
}

template <typename IO, typename F>
int by_size(goom_ctx *ctx, int dp, const void *A, int d, long long batch, long long exponent, void *power, void *prepared, long long stride, int squarings,
            void *group, long long group_stride, int fact_cols)
{
    switch (dp) {
    case 16: return launch<IO, F, 16>(ctx, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols);
    case 32: return launch<IO, F, 32>(ctx, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols);
    case 64: return launch<IO, F, 64>(ctx, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols);
    default: return launch<IO, F, 128>(ctx, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols);
    }
}

} // namespace

int launch_matrix_power(goom_ctx *ctx, const void *A, int d, long long batch, int dtype, int fact_f64, int dp, long long exponent, void *power, void *prepared,
                        long long stride, int squarings, void *group, long long group_stride, int fact_cols)
{
    if (dtype == GOOM_C128) return by_size<double, double>(ctx, dp, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols);
    return fact_f64 ? by_size<float, double>(ctx, dp, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols)
                    : by_size<float, float>(ctx, dp, A, d, batch, exponent, power, prepared, stride, squarings, group, group_stride, fact_cols);
}

} // namespace goom_chain
