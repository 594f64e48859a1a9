// The adjoints of the prefix scan once more (goom_scan_adjoint.hip), for batch items whose magnitudes lie too far apart for mantissas
// with one power of two a column: rows of a state e^60 apart, a column of a chunk product that its common exponent leaves no room for,
// log-magnitudes beyond 3e8 in double.  Here every entry has a whole-number exponent of its own, held in double (exact up to 2^53), so
// that only a term which is 2^-1000 of its own sum's largest is lost.
//
// The walk sets an item's flag where something may not have fitted; only then does a workgroup here do anything, and it overwrites that item's
// gradients.  Same chunks, three kernels: chunk products and vectors (A_c^T column by column beside the vectors: columns of one adjoint
// recurrence, the former without gradients), carries, gradients.  K and Lam lie in the workspace, where the walk had its own chunk products.
// Vector instructions only, bound by their number: a sum's exponent first, then its terms on it, nine instructions in double a term and the
// loads; with an exponent carried along instead, 17 and 8.4 ms where now 16 and 5.3 (64 x 128 steps of complex64 64 x 64; 16 x 128 of complex128).
// A column is as good as another, so a workgroup has sixteen of them (gradients: all), a thread four of one row, which share the
// conversion of the matrix's entries.  Four times the waves a workgroup, with spills: 21 to 25 ms.
#include "goom_chain_kernel.h"

namespace {

using namespace goom_chain;

template <typename R> struct C2;
template <> struct C2<float> { typedef float2 type; };
template <> struct C2<double> { typedef double2 type; };

constexpr double kZeroExp = -1.0e300; // exponent of a zero
constexpr int kCols = 16, kPer = 4;   // columns of a group, of a thread
constexpr int kThreads = 256;
constexpr int kItems = GOOM_MAX_DIM / 64; // rows that a thread has, four columns each

struct Entry { // m 2^e
    double m, e;
};

template <typename R> struct WideArgs {
    typedef typename C2<R>::type c2;
    const c2 *M, *P, *S0;
    const R *G;
    R *gM, *gS0;
    const int *wide;
    unsigned char *slots; // [batch][C]: exponents, then mantissas, [columns][d]; the first ncols - m columns are A_c^T
    long long slot_stride, T, L, C;
    int d, m, ncols;
};

__device__ inline int shift_of(double x) { return (int)__builtin_fmax(x, -4000.0); }
__device__ inline Entry zero_entry() { return Entry{0.0, kZeroExp}; }
__device__ inline void add_term(Entry &s, double m, double e)
{
    const double top = __builtin_fmax(s.e, e);
    s.m = __builtin_ldexp(s.m, shift_of(s.e - top)) + __builtin_ldexp(m, shift_of(e - top));
    s.e = top;
}
__device__ inline Entry normal(Entry s)
{
    if (s.m == 0.0) return zero_entry();
    return Entry{__builtin_amdgcn_frexp_mant(s.m), s.e + (double)__builtin_amdgcn_frexp_exp(s.m)};
}
// a GOOM's magnitude and sign, negated: its reciprocal's
template <typename R> __device__ inline Entry entry_of(typename C2<R>::type x, bool inverse = false)
{
    const double re = inverse ? -(double)x.x : (double)x.x;
    if (!__builtin_isfinite(x.x)) return zero_entry();
    const double n = __builtin_rint(re * kLog2e);
    double f = __builtin_fma(re, kLog2e, -n);
    f = __builtin_fma(re, 2.0355273740931033e-17, f); // log2(e) - kLog2e
    const double y = Comp<double>::exp2_small(f); // (|f| is 1/2 and what the product with log2(e) was rounded by)
    return Entry{Comp<R>::is_negative(x.y) ? -y : y, n};
}
// sum over i < n of x(i) l(u, i) for four u: the exponent first, then the terms on it
template <class X, class L> __device__ inline void sums(int n, X &&x, L &&l, Entry (&out)[kPer])
{
    double top[kPer], m[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        top[u] = -1.0e290; // (above what a zero's can be)
        m[u] = 0.0;
    }
#pragma unroll 4
    for (int i = 0; i < n; ++i) {
        const double e = x(i).e;
#pragma unroll
        for (int u = 0; u < kPer; ++u) top[u] = __builtin_fmax(top[u], e + l(u, i).e);
    }
#pragma unroll 2
    for (int i = 0; i < n; ++i) {
        const Entry a = x(i);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const Entry b = l(u, i);
            // 2^t for a whole t from -1000 to 0: t + 1023 in the last bits of a double between 2^52 and 2^53, moved to an exponent's place
            const double t = __builtin_fmax(a.e + (b.e - top[u]), -1000.0) + 4503599627371519.0;
            const double scale = __builtin_bit_cast(double, (unsigned long long)((unsigned)__builtin_bit_cast(unsigned long long, t) << 20) << 32);
            m[u] = __builtin_fma(a.m * b.m, scale, m[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) out[u] = Entry{m[u], top[u]};
}
template <typename R> __device__ inline R value_of(Entry s)
{
    const double x = s.e + 1200.0; // (far out: zero or infinity either way)
    return (R)__builtin_ldexp(s.m, (int)__builtin_fmin(__builtin_fmax(x, -4000.0), 8000.0) - 1200);
}

// whether a workgroup of the walk has said of this item that it may have lost something
template <typename R> __device__ bool item_is_wide(const WideArgs<R> &a, long long b)
{
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    int mine = 0;
    for (long long at = threadIdx.x; at < 2 * a.C; at += kThreads) mine |= a.wide[b * 2 * a.C + at];
    if (mine) any = 1;
    __syncthreads();
    return any != 0;
}

template <typename R> struct Slot {
    double *e;
    R *m;
    __device__ Slot(const WideArgs<R> &a, long long at)
    {
        unsigned char *p = a.slots + at * a.slot_stride;
        e = reinterpret_cast<double *>(p);
        m = reinterpret_cast<R *>(p + (size_t)a.ncols * a.d * sizeof(double));
    }
    __device__ Entry get(int at) const { return Entry{(double)m[at], e[at]}; }
    __device__ void put(int at, Entry s) const
    {
        m[at] = (R)s.m;
        e[at] = s.e;
    }
};

// item q of a thread: row j and columns k .. k + 3 of a group of sixteen that begins at k0 and ends before k1
#define GOOM_WIDE_ITEM(q, k0, k1)                                                                                                                            \
    const int j = 64 * (q) + (int)threadIdx.x % 64, k = (k0) + kPer * ((int)threadIdx.x / 64);                                                                  \
    const bool mine = j < a.d && k < (k1);

// columns k0 .. of the slot, Lam, become K = M^T Lam (all threads of the workgroup come here)
template <typename R> __device__ void propagate(const WideArgs<R> &a, const Slot<R> &s, const typename C2<R>::type *Mt, int k0, int k1)
{
    const int d = a.d;
    Entry out[kItems][kPer];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        GOOM_WIDE_ITEM(q, k0, k1)
#pragma unroll
        for (int u = 0; u < kPer; ++u) out[q][u] = zero_entry();
        if (!mine) continue;
        sums(d, [&](int i) { return entry_of<R>(Mt[i * d + j]); }, [&](int u, int i) { return s.get((k + u < k1 ? k + u : k) * d + i); }, out[q]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        GOOM_WIDE_ITEM(q, k0, k1)
        if (!mine) continue;
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (k + u < k1) s.put((k + u) * d + j, normal(out[q][u]));
    }
    __syncthreads();
}

// columns of K in the slot (state columns k0 .. k1 - 1, `first` before them) become Lam = K + G / P
template <typename R> __device__ void join(const WideArgs<R> &a, const Slot<R> &s, size_t step, int first, int k0, int k1)
{
    const int d = a.d, m = a.m, w = k1 - k0;
    for (int at = threadIdx.x; at < d * w; at += kThreads) {
        const int j = at / w, k = k0 + at % w;
        const double g = (double)a.G[step * d * m + (size_t)j * m + k];
        const auto p = a.P[step * d * m + (size_t)j * m + k];
        if (g == 0.0 || !__builtin_isfinite(p.x)) continue;
        const Entry x = entry_of<R>(p, true);
        Entry l = s.get((first + k) * d + j);
        add_term(l, __builtin_amdgcn_frexp_mant(g) * x.m, x.e + (double)__builtin_amdgcn_frexp_exp(g));
        s.put((first + k) * d + j, normal(l));
    }
    __syncthreads();
}

// a chunk (not the first), sixteen columns: from the identity without gradients, or from zero with them
template <typename R> __global__ __launch_bounds__(kThreads) void wide_vectors_kernel(WideArgs<R> a)
{
    const int groups_d = (a.d + kCols - 1) / kCols;
    const long long chunk = blockIdx.x % (a.C - 1) + 1, b = blockIdx.x / (a.C - 1);
    if (!item_is_wide(a, b)) return;
    const bool product = (int)blockIdx.y < groups_d;
    const int k0 = kCols * (product ? (int)blockIdx.y : (int)blockIdx.y - groups_d), kend = product ? a.d : a.m;
    const int k1 = k0 + kCols < kend ? k0 + kCols : kend, first = product ? 0 : a.d;
    const Slot<R> s(a, b * a.C + chunk);
    for (int at = threadIdx.x; at < (k1 - k0) * a.d; at += kThreads) {
        const int k = k0 + at / a.d, j = at % a.d;
        s.put((first + k) * a.d + j, product && j == k ? Entry{1.0, 0.0} : zero_entry());
    }
    __syncthreads();
    const long long lo = chunk * a.L, hi = lo + a.L < a.T ? lo + a.L : a.T;
    for (long long t = hi - 1; t >= lo; --t) {
        const size_t step = (size_t)(b * a.T + t);
        if (!product) join(a, s, step, first, k0, k1);
        propagate(a, s, a.M + step * a.d * a.d, first + k0, first + k1);
    }
}

// K at every chunk's end, sixteen columns, in the places of the chunk vectors
template <typename R> __global__ __launch_bounds__(kThreads) void wide_carries_kernel(WideArgs<R> a)
{
    const long long b = blockIdx.x;
    if (!item_is_wide(a, b)) return;
    const int d = a.d, k0 = kCols * (int)blockIdx.y, k1 = k0 + kCols < a.m ? k0 + kCols : a.m;
    Entry K[kItems][kPer];
#pragma unroll
    for (int q = 0; q < kItems; ++q)
#pragma unroll
        for (int u = 0; u < kPer; ++u) K[q][u] = zero_entry();
    for (long long c = a.C - 1; c >= 0; --c) {
        const Slot<R> s(a, b * a.C + c);
        Entry V[kItems][kPer];
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            GOOM_WIDE_ITEM(q, k0, k1)
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                V[q][u] = zero_entry();
                if (!mine || k + u >= k1) continue;
                if (c > 0) V[q][u] = s.get((d + k + u) * d + j);
                s.put((d + k + u) * d + j, K[q][u]); // (each thread in the places it read)
            }
        }
        if (c == 0) break;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            GOOM_WIDE_ITEM(q, k0, k1)
            if (!mine) continue;
            Entry sum[kPer]; // of A_c[i, j] K[i, k]
            sums(d, [&](int i) { return s.get(i * d + j); }, [&](int u, int i) { return s.get((d + (k + u < k1 ? k + u : k)) * d + i); }, sum);
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                add_term(V[q][u], sum[u].m, sum[u].e);
                K[q][u] = normal(V[q][u]);
            }
        }
    }
}

// a chunk with its gradients
template <typename R> __global__ __launch_bounds__(kThreads) void wide_gradients_kernel(WideArgs<R> a)
{
    typedef typename C2<R>::type c2;
    const long long chunk = blockIdx.x % a.C, b = blockIdx.x / a.C;
    if (!item_is_wide(a, b)) return;
    const int d = a.d, m = a.m, first = a.ncols - m;
    const Slot<R> s(a, b * a.C + chunk);
    if (a.C == 1) {
        for (int at = threadIdx.x; at < m * d; at += kThreads) s.put(first * d + at, zero_entry());
        __syncthreads();
    }
    const c2 *S0 = a.S0 ? a.S0 + (size_t)b * d * m : nullptr;
    const long long lo = chunk * a.L, hi = lo + a.L < a.T ? lo + a.L : a.T;
    for (long long t = hi - 1; t >= lo; --t) {
        const size_t step = (size_t)(b * a.T + t);
        join(a, s, step, first, 0, m);
        const c2 *Mt = a.M + step * d * d, *prev = t > 0 ? a.P + (step - 1) * d * m : S0;
        const int rows4 = (d + kPer - 1) / kPer;
        for (int at = threadIdx.x; at < rows4 * d; at += kThreads) {
            const int j = at % d, i = kPer * (at / d);
            Entry sum[kPer];
            sums(m, [&](int k) { return prev ? entry_of<R>(prev[j * m + k]) : j == k ? Entry{1.0, 0.0} : zero_entry(); },
                 [&](int u, int k) { return s.get((first + k) * d + (i + u < d ? i + u : i)); }, sum);
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                if (i + u >= d) continue;
                const Entry x = entry_of<R>(Mt[(i + u) * d + j]);
                a.gM[step * d * d + (size_t)(i + u) * d + j] = value_of<R>(Entry{sum[u].m * x.m, sum[u].e + x.e});
            }
        }
        __syncthreads(); // (Lam has been read)
        if (t > lo || (chunk == 0 && a.gS0))
            for (int k0 = 0; k0 < m; k0 += kCols) propagate(a, s, Mt, first + k0, first + (k0 + kCols < m ? k0 + kCols : m));
    }
    if (chunk == 0 && a.gS0)
        for (int at = threadIdx.x; at < d * m; at += kThreads) {
            const int j = at / m, k = at % m;
            const Entry x = entry_of<R>(S0[j * m + k]), l = s.get((first + k) * d + j);
            a.gS0[(size_t)b * d * m + at] = value_of<R>(Entry{l.m * x.m, l.e + x.e});
        }
}
#undef GOOM_WIDE_ITEM

template <typename R> int launch_wide_t(goom_ctx *ctx, const goom::ScanAdjointLaunch &l)
{
    typedef typename C2<R>::type c2;
    WideArgs<R> a;
    a.M = static_cast<const c2 *>(l.M);
    a.P = static_cast<const c2 *>(l.P);
    a.S0 = static_cast<const c2 *>(l.S0);
    a.G = static_cast<const R *>(l.G);
    a.gM = static_cast<R *>(l.gM);
    a.gS0 = static_cast<R *>(l.gS0);
    a.wide = l.wide;
    a.slots = static_cast<unsigned char *>(l.slots);
    a.slot_stride = (long long)l.slot_stride;
    a.T = l.T;
    a.L = l.L;
    a.C = l.C;
    a.d = l.d;
    a.m = l.m;
    a.ncols = l.C > 1 ? l.d + l.m : l.m;
    goom::prof_begin(ctx, "scan_adjoint_wide");
    if (l.C > 1) {
        const unsigned gd = (unsigned)((l.d + kCols - 1) / kCols), gm = (unsigned)((l.m + kCols - 1) / kCols);
        hipLaunchKernelGGL(wide_vectors_kernel<R>, dim3((unsigned)(l.batch * (l.C - 1)), gd + gm), dim3(kThreads), 0, ctx->stream, a);
        hipLaunchKernelGGL(wide_carries_kernel<R>, dim3((unsigned)l.batch, gm), dim3(kThreads), 0, ctx->stream, a);
    }
    hipLaunchKernelGGL(wide_gradients_kernel<R>, dim3((unsigned)(l.batch * l.C)), dim3(kThreads), 0, ctx->stream, a);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch wide_gradients_kernel");
}

} // namespace

namespace goom {

size_t scan_adjoint_slot_bytes(long long C, int d, int m, int dtype)
{
    const size_t entries = (size_t)((C > 1 ? d : 0) + m) * d, entry = sizeof(double) + (dtype == GOOM_C64 ? sizeof(float) : sizeof(double));
    return (entries * entry + 15) / 16 * 16;
}

int launch_scan_adjoint_wide(goom_ctx *ctx, const ScanAdjointLaunch &l)
{
    return l.dtype == GOOM_C64 ? launch_wide_t<float>(ctx, l) : launch_wide_t<double>(ctx, l);
}

} // namespace goom
