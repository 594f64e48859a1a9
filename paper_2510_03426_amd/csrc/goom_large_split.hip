// Products of large float matrices on the bf16 matrix instruction: a float is the sum of three bf16 (8 bits each, rounded to nearest: 24
// bits, so the sum is exact), and a product of two floats is six products of such parts; the three left out reach 2^-24 of it (2^-27.5 in
// the root mean square, of either sign).  The parts' products are exact in float and are summed in float, as the float instruction sums its own.  The float matrix
// instruction does 157 TFLOP/s, the bf16 one 2500: six of them are 2.6 times as fast.
// Measured: 32 products of 1024^3 913 -> 650 us (the kernel alone 447: 154 TFLOP/s, its matrix cores busy for 55 % of the cycles), scan of 192 x 512 x 512 2790 ->
// 1170.  Error against 64 bits, floats -> parts: the scan 1.05e-5 -> 6.0e-6, products of N(0, 1) 300 x 200 x 150 1.24e-6 -> 5.9e-7 (products of
// the leading parts and all others in sums of their own; logarithms of mantissas, not of lifted numbers; the lift applied to exponentials, not to
// their arguments: without the last two the error is 1.4 to 2.4 times the floats').
//
// Magnitudes: bf16 has float's exponents, but the last part of a number lies 2^-16 below the first, so a number below 2^-110
// would lose it.  Both operands are therefore held with their largest entries at 2^kLift instead of 1: products reach 2^80 times the inner size
// and everything down to 2^-150 of the largest entries keeps its 24 bits, where float operands scaled to 1 end at 2^-126.
//
// Matrix products of GOOMs above 128 (LMME) and scans of large matrices (Section 4.1) run through one kernel,
//     C[i][n] = sum_k X[i][k] Y[n][k],
// with X, the left factor, as three planes of bf16 with K contiguous, and Y either the same (LMME) or the running state of a
// chain as the last product left it: plain floats Ct[n][k].  A state is never rescaled by a pass of its own: the kernel that
// writes it finds every column's largest exponent (an integer maximum by atomics), and the kernel that reads it applies the factor's row shifts
// and that exponent, and splits into parts, on the way into LDS.  Row shifts are taken relative to the factor's largest there (whole numbers of
// any size themselves, the differences that matter are small and exact); the largest joins the columns' exponents, in double.
#include <climits>
#include <cmath>

#include "goom_large_scan.h"

namespace {

using goom_chain::Comp;
using goom_chain::f4;
using goom_large::pad_to;
typedef Comp<float> CF;
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

constexpr float kLift = 40.0f;
constexpr float kLog2eF = 1.44269504088896340736f;

// natural log of |x| 2^s, x not zero: the hardware logarithm of a mantissa in [1/2, 1), whose last place is that of a number below 1 (taken of x
// itself, which lies near 2^80 here, it would be that of 80)
__device__ inline float log_of(float x, double s)
{
#pragma clang fp contract(off)
    const float kLn2Hi = 0.693147182464599609375f;
    const float kLn2Lo = -1.90465429995776806e-9f;
    const float e = CF::exponent_of(x);
    const float l2 = __builtin_amdgcn_logf(__builtin_fabsf(__builtin_ldexpf(x, -(int)e)));
    const float w = (float)(s + (double)e);
    return __builtin_fmaf(w, kLn2Hi, __builtin_fmaf(w, kLn2Lo, l2 * kLn2Hi));
}

// +-2^(re log2(e) - shift), shift being a row's (column's) whole number less kLift: Comp<float>::exp2_shifted with the lift applied to the result.  (In
// the exponent it would cost the bits below the last place of 40; far down, where there are none of these, it is taken there first.)
__device__ inline float lifted(float2 z, float shift)
{
#pragma clang fp contract(off)
    const float kHi = 1.44269502162933349609375f, kLo = 1.925963033500011e-8f, kLn2 = 0.693147182464599609375f;
    const float p_hi = z.x * kHi;
    float p_lo = __builtin_fmaf(z.x, kHi, -p_hi);
    p_lo = __builtin_fmaf(z.x, kLo, p_lo);
    const float t_hi = p_hi - (shift + kLift);
    const bool far = t_hi < -60.0f;
    const float y = __builtin_amdgcn_exp2f(far ? t_hi + kLift : t_hi);
    const float yc = CF::ldexp_(__builtin_fmaf(y, p_lo * kLn2, y), far ? 0 : (int)kLift);
    return CF::apply_sign(t_hi > -190.0f ? yc : 0.0f, z.y); // false for -inf and NaN as well: they become zero
}

// two floats into their three parts, packed (first in the low half)
__device__ inline void split2(float a, float b, unsigned &hi, unsigned &mid, unsigned &lo)
{
    auto pack = [](float x, float y) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{x, y}, bf2)); };
    auto low = [](unsigned p) { return __builtin_bit_cast(float, p << 16); };
    auto high = [](unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); };
    hi = pack(a, b);
    a -= low(hi);
    b -= high(hi);
    mid = pack(a, b);
    lo = pack(a - low(mid), b - high(mid));
}
__device__ inline void split8(const float (&x)[8], u4 (&p)[3])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        unsigned h, m, l;
        split2(x[2 * q], x[2 * q + 1], h, m, l);
        p[0][q] = h;
        p[1][q] = m;
        p[2][q] = l;
    }
}

// an array with one piece per chunk of every item
template <typename T> struct Pieces {
    T *p;
    long long item, chunk; // strides
    __device__ __host__ T *at(long long i, long long c) const { return p + i * item + c * chunk; }
};

__device__ inline int exponent_key(float e) { return (int)e; }

// A row this far below its factor's largest (in powers of two) counts as no farther: such shifts, two of them and a float's exponent add up
// exactly in float.  (No sum in float reaches so far down; a column that has entries in such rows alone is kept, on a wrong exponent.)
constexpr double kFarRow = -4.0e6;

struct SplitGemm {
    int chunks;                            // products: blockIdx.z = item * chunks + chunk
    int M, N, K;                           // padded: M, N to the tile, K to 16
    Pieces<const __bf16> X;                // planes [3][K / 16][M][16]
    Pieces<const float> row_shift;         // [M]: the factor's row i stands for itself times 2^row_shift
    // Y as planes [3][K / 16][N][16], columns times 2^col_shift[n] (LMME) ...
    Pieces<const __bf16> Yp;
    Pieces<const float> col_shift;
    // ... or as the raw product Yr [K / 16][N][16] of the step before: entry k times 2^fold[k] (no more than 1), column n's largest exponent with
    // these key[n], exponent of the column outside of these e_in[n] + extra
    Pieces<const float> Yr, fold;
    Pieces<const int> key;
    Pieces<const double> e_in;
    Pieces<const double> extra;
    Pieces<double> e_out;                  // of the product's columns
    // outputs
    Pieces<float> Ct, C;                   // p NULL or the product as [M / 16][N][16] / [M][N]
    Pieces<const float> fold1, fold2;      // p NULL: no shifts
    Pieces<int> key1, key2;                // p NULL or the columns' largest exponents, entry i times 2^fold[i]
    Pieces<int> clear;                     // p NULL or keys to be set back
    // GOOMs out: [item][slots][n][m], slot = chunk * L + step (stored if below slots and step < L), or `last` of a single slot
    float2 *P;
    long long slots, L, step;
    int n, m;
};

// What becomes of a product: v[i][j] holds four consecutive rows from row[i] on of column col0 + 32 j.  once: this wave stands for its columns.
template <int NI, int NJ, bool RAW>
__device__ inline void finish(const SplitGemm &a, long long item, long long chunk, const f4 (&v)[NI][NJ], const int (&row)[NI], int col0, bool once, int h)
{
    double eo[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = col0 + 32 * j;
        if constexpr (RAW) {
            const int key = a.key.at(item, chunk)[col];
            eo[j] = a.e_in.at(item, chunk)[col] + *a.extra.at(item, chunk) + ((key > INT_MIN ? (double)key : 0.0) - (double)kLift);
            if (once && h == 0 && a.e_out.p) a.e_out.at(item, chunk)[col] = eo[j];
        } else {
            eo[j] = (double)a.col_shift.at(item, chunk)[col];
        }
        if (once && h == 0 && a.clear.p) a.clear.at(item, chunk)[col] = INT_MIN;
    }
    if (a.Ct.p) {
        float *o = a.Ct.at(item, chunk);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) *reinterpret_cast<f4 *>(o + ((size_t)(row[i] >> 4) * a.N + col0 + 32 * j) * 16 + (row[i] & 15)) = v[i][j];
    }
    if (a.C.p) {
        float *o = a.C.at(item, chunk);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[(size_t)(row[i] + r) * a.N + col0 + 32 * j] = v[i][j][r];
    }
    auto largest = [&](const Pieces<const float> &fold_next, const Pieces<int> &keys) {
        const float *f = fold_next.p ? fold_next.at(item, chunk) : nullptr;
        float mx[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) mx[j] = CF::neg_inf();
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const f4 w = f ? *reinterpret_cast<const f4 *>(f + row[i]) : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = v[i][j][r];
                    mx[j] = CF::max_(x != 0.f ? CF::exponent_of(x) + w[r] : CF::neg_inf(), mx[j]);
                }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const float m = CF::xor32_max(mx[j]);
            if (h == 0 && m > CF::neg_inf()) atomicMax(&keys.at(item, chunk)[col0 + 32 * j], exponent_key(m));
        }
    };
    if (a.key1.p) largest(a.fold1, a.key1);
    if (a.key2.p) largest(a.fold2, a.key2);
    const long long slot = chunk * a.L + a.step;
    if (a.P && a.step < a.L && slot < a.slots) {
        const float *ns = a.row_shift.at(item, chunk);
        float2 *o = a.P + ((size_t)item * a.slots + slot) * a.n * a.m;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const f4 w = *reinterpret_cast<const f4 *>(ns + row[i]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const float x = v[i][j][r];
                    const float zero = RAW && w[r] == -CF::neg_inf() ? w[r] : CF::neg_inf(); // (a chain's row that is not finite)
                    if (row[i] + r < a.n && col0 + 32 * j < a.m)
                        o[(size_t)(row[i] + r) * a.m + col0 + 32 * j] =
                            float2{x != 0.0f ? log_of(x, eo[j] + (double)w[r]) : zero, x < 0.0f ? CF::pi() : 0.0f};
                }
        }
    }
}

// the six products of parts, the smallest first: into `rest`, and the leading parts' own
template <int NI, int NJ> __device__ inline void multiply(const bf8 (&av)[3][NI], const bf8 (&bv)[3][NJ], f16v (&acc)[NI][NJ], f16v (&rest)[NI][NJ])
{
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                f16v &sum = q < 5 ? rest[i][j] : acc[i][j];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[pa[q]][i], bv[pb[q]][j], sum, 0, 0, 0);
            }
}

// A plane lies in memory sixteen values of K at a time, [K / 16][rows][16]: what a step of K needs of a tile is one piece.
// 128 x 128 tiles: grid (N / 128, M / 128, products), 256 threads = 2 x 2 waves of 64 x 64.  Steps of sixteen K through two LDS buffers, one barrier a
// step; the values of the two steps after that are on their way in registers.  In LDS a row is 32 bytes; the halves of
// every other eight rows change places, so that sixteen lanes' reads and writes of 16 bytes meet sixteen different groups of four banks.
template <bool RAW> __global__ __launch_bounds__(256, 2) void gemm_split_kernel(SplitGemm a)
{
    constexpr int TM = 128, PL = TM * 16;
    __shared__ __align__(16) __bf16 xs[2][3][PL];
    __shared__ __align__(16) __bf16 ys[2][3][PL];
    __shared__ __align__(16) float fold[RAW ? GOOM_MAX_DIM_LMME : 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, c = lane & 31;
    const int wm = wave >> 1, wn = wave & 1;
    // workgroups go to the eight XCDs in turn: renumber them so that one XCD works on a contiguous range of tiles and
    // shares their operands in its L2
    const unsigned tx = gridDim.x, ty = gridDim.y;
    const unsigned long long nwg = (unsigned long long)tx * ty * gridDim.z;
    unsigned long long lin = ((unsigned long long)blockIdx.z * ty + blockIdx.y) * tx + blockIdx.x;
    if (nwg % 8 == 0) lin = (lin % 8) * (nwg / 8) + lin / 8;
    const unsigned bx = (unsigned)(lin % tx), by = (unsigned)((lin / tx) % ty);
    const long long z = (long long)(lin / ((unsigned long long)tx * ty)), item = z / a.chunks, chunk = z % a.chunks;
    const int K = a.K, nk = K / 16;
    const size_t xplane = (size_t)a.M * K, yplane = (size_t)a.N * K;

    const int r0 = tid >> 1, k8 = (tid & 1) * 8; // this thread's piece: row r0 of the tile, values k8 .. k8 + 7 of the step
    const __bf16 *Xb = a.X.at(item, chunk) + ((size_t)by * TM + r0) * 16 + k8;
    const __bf16 *Ypb = RAW ? nullptr : a.Yp.at(item, chunk) + ((size_t)bx * TM + r0) * 16 + k8;
    const float *Yrb = RAW ? a.Yr.at(item, chunk) + (size_t)(bx * TM + r0) * 16 + k8 : nullptr;
    float lift = 0.f; // kLift less the exponent of this thread's column
    if constexpr (RAW) {
        const int key = a.key.at(item, chunk)[bx * TM + r0];
        lift = kLift - (key > INT_MIN ? (float)key : 0.0f);
        for (int k = tid; k < K; k += 256) fold[k] = a.fold.p ? a.fold.at(item, chunk)[k] : 0.0f;
        __syncthreads();
    }
    struct Piece {
        u4 x[3], y[RAW ? 2 : 3]; // (y: floats if RAW)
    };
    auto load_tiles = [&](int k, Piece &t) {
        const size_t k0 = 16 * (size_t)(k < nk ? k : 0);
#pragma unroll
        for (int p = 0; p < 3; ++p) t.x[p] = *reinterpret_cast<const u4 *>(Xb + p * xplane + k0 * a.M);
        if constexpr (RAW) {
#pragma unroll
            for (int e = 0; e < 2; ++e) t.y[e] = *reinterpret_cast<const u4 *>(Yrb + k0 * a.N + 4 * e);
        } else {
#pragma unroll
            for (int p = 0; p < 3; ++p) t.y[p] = *reinterpret_cast<const u4 *>(Ypb + p * yplane + k0 * a.N);
        }
    };
    const int at = r0 * 16 + (k8 ^ ((r0 & 8) ? 8 : 0));
    auto store_tiles = [&](int k, const Piece &t, int buf) {
        u4 y[3];
        if constexpr (RAW) {
            float v[8];
            const int kk = 16 * (k < nk ? k : 0) + k8;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const f4 f = *reinterpret_cast<const f4 *>(&fold[kk + 4 * e]), x = __builtin_bit_cast(f4, t.y[e]);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[4 * e + q] = CF::ldexp_(x[q], (int)CF::clamp_shift(f[q] + lift));
            }
            split8(v, y);
        } else {
#pragma unroll
            for (int p = 0; p < 3; ++p) y[p] = t.y[p];
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            *reinterpret_cast<u4 *>(&xs[buf][p][at]) = k < nk ? t.x[p] : u4{0, 0, 0, 0};
            *reinterpret_cast<u4 *>(&ys[buf][p][at]) = y[p];
        }
    };
    f16v acc[2][2], rest[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = rest[i][j][e] = 0.f;
    Piece ahead[2];
    load_tiles(0, ahead[0]);
    load_tiles(1, ahead[1]);
    store_tiles(0, ahead[0], 0);
    load_tiles(2, ahead[0]);
    __syncthreads();
    const int half = (8 * h) ^ ((c & 8) ? 8 : 0); // lane l: row (column) l % 32, K = 8 (l / 32) + 0 .. 7
    for (int k0 = 0; k0 < nk; k0 += 2) { // (a last odd step is followed by one of zeros)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            bf8 av[3][2], bv[3][2];
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    av[p][i] = *reinterpret_cast<const bf8 *>(&xs[u][p][(wm * 64 + 32 * i + c) * 16 + half]);
                    bv[p][i] = *reinterpret_cast<const bf8 *>(&ys[u][p][(wn * 64 + 32 * i + c) * 16 + half]);
                }
            store_tiles(k0 + u + 1, ahead[1 - u], 1 - u);
            load_tiles(k0 + u + 3, ahead[1 - u]);
            multiply<2, 2>(av, bv, acc, rest);
            __syncthreads();
        }
    }
    // register r of a 32 x 32 block: row 8 (r / 4) + 4 h + r % 4 of column c
    f4 v[8][2];
    int row[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        row[i] = by * TM + wm * 64 + 32 * (i >> 2) + 8 * (i & 3) + 4 * h;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[i][j][r] = acc[i >> 2][j][4 * (i & 3) + r] + rest[i >> 2][j][4 * (i & 3) + r];
    }
    finish<8, 2, RAW>(a, item, chunk, v, row, bx * TM + wn * 64 + c, by == 0 && wm == 0, h);
}

// Products too few to fill the chip with such tiles (the carries of a scan, one after the other): 32 x 32 tiles, a workgroup's four waves share K
// and add their sums in LDS.  A wave's operands come straight from memory, DEPTH steps of sixteen K at a time in flight.
template <bool RAW> __global__ __launch_bounds__(256, 2) void gemm_split_few_kernel(SplitGemm a)
{
    constexpr int DEPTH = 4;
    __shared__ __align__(16) float part[4][4][64 * 4]; // [rows' quarter][wave][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, c = lane & 31;
    const int bx = blockIdx.x, by = blockIdx.y;
    const long long item = blockIdx.z / a.chunks, chunk = blockIdx.z % a.chunks;
    const int K = a.K, steps = K / 16;
    const size_t xplane = (size_t)a.M * K, yplane = (size_t)a.N * K;
    const __bf16 *Xb = a.X.at(item, chunk) + ((size_t)by * 32 + c) * 16 + 8 * h;
    const __bf16 *Ypb = RAW ? nullptr : a.Yp.at(item, chunk) + ((size_t)bx * 32 + c) * 16 + 8 * h;
    const float *Yrb = RAW ? a.Yr.at(item, chunk) + (size_t)(bx * 32 + c) * 16 + 8 * h : nullptr;
    const float *fold = RAW && a.fold.p ? a.fold.at(item, chunk) + 8 * h : nullptr;
    float lift = 0.f;
    if (RAW) {
        const int key = a.key.at(item, chunk)[bx * 32 + c];
        lift = kLift - (key > INT_MIN ? (float)key : 0.0f);
    }
    f16v acc[1][1], rest[1][1];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][0][e] = rest[0][0][e] = 0.f;
    // wave w takes steps w, w + 4, ...; beyond the last one a zero stands in for the left operand
    for (int s0 = wave; s0 < steps; s0 += 4 * DEPTH) {
        u4 xr[DEPTH][3], yp[DEPTH][3];
        f4 yr[DEPTH][2], fr[DEPTH][2];
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int k0 = 16 * (s0 + 4 * u < steps ? s0 + 4 * u : s0);
#pragma unroll
            for (int p = 0; p < 3; ++p) xr[u][p] = *reinterpret_cast<const u4 *>(Xb + p * xplane + (size_t)k0 * a.M);
            if constexpr (RAW) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    yr[u][e] = *reinterpret_cast<const f4 *>(Yrb + (size_t)k0 * a.N + 4 * e);
                    fr[u][e] = fold ? *reinterpret_cast<const f4 *>(fold + k0 + 4 * e) : f4{0.f, 0.f, 0.f, 0.f};
                }
            } else {
#pragma unroll
                for (int p = 0; p < 3; ++p) yp[u][p] = *reinterpret_cast<const u4 *>(Ypb + p * yplane + (size_t)k0 * a.N);
            }
        }
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            bf8 av[3][1], bv[3][1];
            if constexpr (RAW) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = CF::ldexp_(yr[u][e >> 2][e & 3], (int)CF::clamp_shift(fr[u][e >> 2][e & 3] + lift));
                split8(v, yp[u]);
            }
            const bool there = s0 + 4 * u < steps;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                av[p][0] = __builtin_bit_cast(bf8, there ? xr[u][p] : u4{0, 0, 0, 0});
                bv[p][0] = __builtin_bit_cast(bf8, yp[u][p]);
            }
            multiply<1, 1>(av, bv, acc, rest);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f4 x;
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = acc[0][0][4 * q + r] + rest[0][0][4 * q + r];
        *reinterpret_cast<f4 *>(&part[q][wave][4 * lane]) = x;
    }
    __syncthreads();
    f4 v[1][1];
    v[0][0] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) v[0][0] += *reinterpret_cast<const f4 *>(&part[wave][w][4 * lane]);
    const int row[1] = {by * 32 + 8 * wave + 4 * h};
    finish<1, 1, RAW>(a, item, chunk, v, row, bx * 32 + c, by == 0 && wave == 0, h);
}

// Do products of n x m (any sizes) fill the chip in 128 x 128 tiles, and the tiles?  Before, the large kernel's sharing of operands does not count for its
// latency, and tiles that are more than two thirds padding cost more than it saves.  In us, an LMME in these tiles / in the other kernel's of 32 x 32 (which
// have `few` entries in all, padding included): 64 tiles, 4 x 512^3 52 / 37, 64 x 128 x 1024 x 128 101 / 97; 80 and more, 32 x 200^3 44 / 46, 64 x 200^3
// 51 / 74, 128 x 128 x 1024 x 128 174 / 204, 64 x 160 x 1000 x 160 149 / 163; mostly padding, 256 x 64 x 1000 x 64 282 / 171, 1024 of them 1114 /
// 673, 1000 x 130 x 300 x 20 448 / 248.
bool split_in_tiles(int n, int m, long long products)
{
    const double few = (double)pad_to(n, 32) * pad_to(m, 32) * (double)products, tiles = (double)pad_to(n, 128) * pad_to(m, 128) * (double)products;
    return few >= 80.0 * 128 * 128 && tiles <= 3.0 * few;
}

// products: of M x N x K (padded: K to 16, M and N to 128, or to 32 if they are too few)
template <bool RAW> void launch_gemm_split(hipStream_t st, const SplitGemm &a, unsigned products, bool in_tiles)
{
    if (in_tiles)
        hipLaunchKernelGGL(gemm_split_kernel<RAW>, dim3(a.N / 128, a.M / 128, products), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(gemm_split_few_kernel<RAW>, dim3(a.N / 32, a.M / 32, products), dim3(256), 0, st, a);
}

// ---- rows of GOOM matrices into planes.  Row r of matrix b: 2^(log2|x| - shift), shift = the row's whole power of two less kLift.  One wave a
// row (up to 1024 entries, sixteen a lane, in pairs), four rows a workgroup: grid (rows_padded / 4, matrices), 256 threads.  A row without entries
// has the shift -inf; of a chain's matrices a row with an infinite entry (or, if nan_shows, a NaN; it counts as zero otherwise) has inf, and no
// entries: the product's row is infinite then, and so are all states after it.
// A chain of matrices (L > 0): matrix b is step s = s0 + b % per_chain of chain b / per_chain = item * C + chunk, and goes to place
// chain * places + s % places; beyond the chunk or T it is the identity.
struct RowsArgs {
    const float2 *A;
    __bf16 *X;
    float *shifts;
    int n, d, rows_padded, k_padded;
    long long T, L, C, per_chain, s0, places;
    bool nan_shows;
};
__global__ __launch_bounds__(256) void split_rows_kernel(RowsArgs a)
{
    __shared__ __align__(16) __bf16 parts[3][4][GOOM_MAX_DIM_LMME + 8];
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long b = blockIdx.y;
    const size_t plane = (size_t)a.rows_padded * a.k_padded;
    bool active = true;
    long long mat = b, place = b;
    if (a.L > 0) {
        const long long chain = b / a.per_chain, s = a.s0 + b % a.per_chain, t = (chain % a.C) * a.L + s;
        active = s < a.L && t < a.T;
        mat = chain / a.C * a.T + t;
        place = chain * a.places + s % a.places;
    }
    float *shift = a.shifts + (size_t)place * a.rows_padded + row;
    const int wave = threadIdx.x >> 6;
    auto put = [&](int j, float x0, float x1) {
        unsigned p[3];
        split2(x0, x1, p[0], p[1], p[2]);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<unsigned *>(&parts[q][wave][j]) = p[q];
    };
    // the four rows' pieces of sixteen lie side by side: whole lines of 128 bytes
    auto write_out = [&]() {
        __syncthreads();
        const int count = a.k_padded / 2; // pieces of 16 bytes of a plane's four rows
        __bf16 *out = a.X + (size_t)place * 3 * plane + (size_t)blockIdx.x * 64;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            for (int i = threadIdx.x; i < count; i += 256)
                *reinterpret_cast<u4 *>(out + q * plane + (size_t)(i >> 3) * a.rows_padded * 16 + (i & 7) * 8) =
                    *reinterpret_cast<const u4 *>(&parts[q][(i >> 1) & 3][(i >> 3) * 16 + (i & 1) * 8]);
    };
    if (!active || row >= a.n) {
        const float one = !active && row < a.n ? 1.0f : 0.0f; // (a power of two: 2^kLift with the shift -kLift)
        for (int j = 2 * lane; j < a.k_padded; j += 128)
            put(j, j == row ? one * 1099511627776.0f : 0.f, j + 1 == row ? one * 1099511627776.0f : 0.f);
        if (lane == 0) *shift = !active && row < a.n ? -kLift : CF::neg_inf();
        write_out();
        return;
    }
    const float2 *arow = a.A + ((size_t)mat * a.n + row) * a.d;
    const bool pairs = (a.d & 1) == 0;
    float2 e[8][2];
    float mx = CF::neg_inf();
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int j = 2 * lane + 128 * r;
        e[r][0] = e[r][1] = float2{CF::neg_inf(), 0.f};
        if (j < a.d) {
            if (pairs) {
                const f4 w = *reinterpret_cast<const f4 *>(arow + j);
                e[r][0] = float2{w[0], w[1]};
                e[r][1] = float2{w[2], w[3]};
            } else {
                e[r][0] = arow[j];
                if (j + 1 < a.d) e[r][1] = arow[j + 1];
            }
        }
        mx = fmaxf(mx, fmaxf(e[r][0].x, e[r][1].x));
        bad = bad || e[r][0].x != e[r][0].x || e[r][1].x != e[r][1].x;
    }
    if (a.nan_shows && bad) mx = -CF::neg_inf();
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s, 64));
    const float sh = ceilf(mx * kLog2eF) - kLift;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int j = 2 * lane + 128 * r;
        if (j < a.k_padded)
            put(j, lifted(e[r][0], sh), lifted(e[r][1], sh));
    }
    if (lane == 0) *shift = sh;
    write_out();
}

// The row shifts of the matrices that split_rows_kernel has converted, relative to each one's largest, and these (infinite: a row is).
// grid (matrices), 256 threads; places as there.
struct RelativeArgs {
    const float *shifts;
    float *rel;
    double *top;
    int dp;
    long long per_chain, s0, places;
};
__global__ __launch_bounds__(256) void relative_shifts_kernel(RelativeArgs a)
{
    __shared__ float red[4];
    const long long b = blockIdx.x, place = b / a.per_chain * a.places + (a.s0 + b % a.per_chain) % a.places;
    const float *sh = a.shifts + (size_t)place * a.dp;
    float x[GOOM_MAX_DIM_LMME / 256], mx = CF::neg_inf();
#pragma unroll
    for (int r = 0; r < GOOM_MAX_DIM_LMME / 256; ++r) {
        const int k = threadIdx.x + 256 * r;
        x[r] = k < a.dp ? sh[k] : CF::neg_inf();
        mx = fmaxf(mx, x[r]);
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    const double top = mx > CF::neg_inf() ? (double)mx : 0.0;
#pragma unroll
    for (int r = 0; r < GOOM_MAX_DIM_LMME / 256; ++r) {
        const int k = threadIdx.x + 256 * r;
        const double rel = (double)x[r] - top; // (NaN: such a row)
        if (k < a.dp) a.rel[(size_t)place * a.dp + k] = (float)(rel > kFarRow ? rel : kFarRow);
    }
    if (threadIdx.x == 0) a.top[place] = top;
}

// ---- columns of a GOOM matrix [d][m]: their shifts (less kLift); grid (cols_padded / 64 rounded up, matrices), block 64 x 4
__global__ __launch_bounds__(256) void split_column_shift_kernel(const float2 *__restrict__ B, float *__restrict__ shifts, int d, int m, int cols_padded)
{
    __shared__ float red[4][64];
    const int cx = threadIdx.x & 63, ry = threadIdx.x >> 6;
    const int col = blockIdx.x * 64 + cx;
    const long long b = blockIdx.y;
    float mx = CF::neg_inf();
    if (col < m) {
        // eight independent loads in flight per thread: the loop is bound by memory latency otherwise
        float part[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) part[u] = CF::neg_inf();
        const float2 *base = B + (size_t)b * d * m + col;
        int j = ry;
        for (; j + 28 < d; j += 32) {
#pragma unroll
            for (int u = 0; u < 8; ++u) part[u] = fmaxf(part[u], base[(size_t)(j + 4 * u) * m].x);
        }
        for (; j < d; j += 4) part[0] = fmaxf(part[0], base[(size_t)j * m].x);
#pragma unroll
        for (int u = 0; u < 8; ++u) mx = fmaxf(mx, part[u]);
    }
    red[ry][cx] = mx;
    __syncthreads();
    if (ry == 0 && col < cols_padded) {
        mx = fmaxf(fmaxf(red[0][cx], red[1][cx]), fmaxf(red[2][cx], red[3][cx]));
        shifts[(size_t)b * cols_padded + col] = (mx > CF::neg_inf() ? ceilf(mx * kLog2eF) : 0.0f) - kLift;
    }
}

// transposed, as planes Y[3][k_padded / 16][cols_padded][16] (FLOATS: as floats, one of them), a matrix every `stride` values.  grid (cols_padded /
// 32, k_padded / 32 rounded up, matrices), 256 threads.
template <bool FLOATS>
__global__ __launch_bounds__(256) void split_columns_kernel(const float2 *__restrict__ B, const float *__restrict__ shifts, void *__restrict__ Yv, long long stride,
                                                            int d, int m, int cols_padded, int k_padded)
{
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int c0 = blockIdx.x * 32, j0 = blockIdx.y * 32;
    const long long b = blockIdx.z;
    const int col = c0 + tx;
    const float sh = shifts[(size_t)b * cols_padded + col];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = j0 + ty + 8 * r;
        float v = 0.0f;
        if (j < d && col < m) {
            v = lifted(B[((size_t)b * d + j) * m + col], sh);
        }
        tile[ty + 8 * r][tx] = v; // [j][col]
    }
    __syncthreads();
    if constexpr (FLOATS) {
        float *Y = static_cast<float *>(Yv) + b * stride;
#pragma unroll
        for (int r = 0; r < 4; ++r) Y[((size_t)((j0 + tx) >> 4) * cols_padded + c0 + ty + 8 * r) * 16 + (tx & 15)] = tile[tx][ty + 8 * r];
    } else {
        const size_t plane = (size_t)cols_padded * k_padded;
        __bf16 *Y = static_cast<__bf16 *>(Yv) + b * stride;
        const int jj = 2 * (threadIdx.x & 15), cc = threadIdx.x >> 4;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            unsigned p[3];
            split2(tile[jj][cc + 16 * r], tile[jj + 1][cc + 16 * r], p[0], p[1], p[2]);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (j0 + jj < k_padded)
                    *reinterpret_cast<unsigned *>(Y + q * plane + ((size_t)((j0 + jj) >> 4) * cols_padded + c0 + cc + 16 * r) * 16 + (jj & 15)) = p[q];
        }
    }
}

// ---- the chunks' first matrices as the states after their first step: Ct[chain][i / 16][n][i % 16] = row i, column n of A scaled as in split_rows_kernel (whose
// shifts these are), and the columns' keys under those shifts, relative to their largest.
// grid (dp / 32, dp / 32, chains), 256 threads.
struct FirstArgs {
    const float2 *A;
    Pieces<const float> shifts, rel;
    Pieces<float> Ct;
    Pieces<int> key;
    int d, dp, chunks;
    long long T, L;
};
__global__ __launch_bounds__(256) void first_state_kernel(FirstArgs a)
{
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int n0 = blockIdx.x * 32, i0 = blockIdx.y * 32;
    const long long item = blockIdx.z / a.chunks, chunk = blockIdx.z % a.chunks;
    const float2 *A = a.A + ((size_t)item * a.T + chunk * a.L) * a.d * a.d;
    const float *sh = a.shifts.at(item, chunk), *rel = a.rel.at(item, chunk);
    float mx = CF::neg_inf();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + ty + 8 * r, n = n0 + tx;
        const float ri = rel[i];
        float v = 0.0f;
        if (i < a.d && n < a.d) {
            v = lifted(A[(size_t)i * a.d + n], sh[i]);
            if (v != 0.f) mx = fmaxf(mx, CF::exponent_of(v) + ri);
        }
        tile[ty + 8 * r][tx] = v; // [i][n]
    }
    if (mx > CF::neg_inf()) atomicMax(&a.key.at(item, chunk)[n0 + tx], exponent_key(mx));
    __syncthreads();
    float *o = a.Ct.at(item, chunk);
#pragma unroll
    for (int r = 0; r < 4; ++r) o[((size_t)((i0 + tx) >> 4) * a.dp + n0 + ty + 8 * r) * 16 + (tx & 15)] = tile[tx][ty + 8 * r]; // [i / 16][n][i % 16]
}

// ---- chunk products C[chunk][i][j] (columns' keys without shifts, exponents e) as left factors: planes with column j on 2^kLift, what that
// takes out of the column (g) relative to the largest of them (gmax) joining the row shifts of the factor before it: fold[k].
// grid (dp / 4, chunks, items), 256 threads; one wave a row.
struct TotalsArgs {
    const float *C;      // [item][chunk][dp][dp]
    const int *key;      // [item][chunk][dp]
    const double *e;     // [item][chunk][dp]
    __bf16 *X;           // [item][chunk], planes
    int dp;
    long long chunks;    // per item, of the arrays
};
__global__ __launch_bounds__(256) void totals_planes_kernel(TotalsArgs a)
{
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long at = (long long)blockIdx.z * a.chunks + blockIdx.y;
    const size_t plane = (size_t)a.dp * a.dp;
    const float *src = a.C + (size_t)at * plane + (size_t)row * a.dp;
    const int *key = a.key + at * a.dp;
    __bf16 *out = a.X + (size_t)at * 3 * plane + (size_t)row * 16;
    for (int j = 2 * lane; j < a.dp; j += 128) {
        const int k0 = key[j], k1 = key[j + 1];
        unsigned hi, mid, lo;
        split2(CF::ldexp_(src[j], (int)CF::clamp_shift(kLift - (k0 > INT_MIN ? (float)k0 : 0.f))),
               CF::ldexp_(src[j + 1], (int)CF::clamp_shift(kLift - (k1 > INT_MIN ? (float)k1 : 0.f))), hi, mid, lo);
        __bf16 *o = out + (size_t)(j >> 4) * a.dp * 16 + (j & 15);
        *reinterpret_cast<unsigned *>(o) = hi;
        *reinterpret_cast<unsigned *>(o + plane) = mid;
        *reinterpret_cast<unsigned *>(o + 2 * plane) = lo;
    }
}
// What the carries' entries have to be multiplied by.  The carry into chunk c still lacks the row shifts of total c - 1 (fold2, and their largest,
// top2; none for c = 0); as the operand of the next product it takes the exponents of total c's columns too, g(c)[k] relative to the largest of
// them, which joins gmax (fold1).  grid (chunks, items), 256 threads.
struct FoldArgs {
    const int *key;             // as above; NULL: the totals are the matrices themselves, g = 0
    const double *e;
    Pieces<const float> rel;    // rows of total c
    Pieces<const double> top;
    float *fold1, *fold2;       // [item][chunk][dp]
    double *gmax, *top2;        // [item][chunk]
    int dp, d;
    long long chunks, totals;
};
__global__ __launch_bounds__(256) void totals_fold_kernel(FoldArgs a)
{
    __shared__ double red[4];
    const long long chunk = blockIdx.x, item = blockIdx.y, at = item * a.chunks + chunk;
    const float *before = chunk > 0 ? a.rel.at(item, chunk - 1) : nullptr;
    const double top2 = chunk > 0 ? *a.top.at(item, chunk - 1) : 0.0;
    if (threadIdx.x == 0) a.top2[at] = top2;
    double g[4], mx = -1.0e300;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int k = threadIdx.x + 256 * r;
        g[r] = -1.0e300; // an empty column, which meets nothing of the state
        if (k < a.dp) {
            a.fold2[at * a.dp + k] = before ? before[k] : 0.0f;
            if (chunk < a.totals) {
                if (!a.key) g[r] = k < a.d ? 0.0 : g[r];
                else if (a.key[at * a.dp + k] > INT_MIN) g[r] = a.e[at * a.dp + k] + (double)a.key[at * a.dp + k] - (double)kLift;
                mx = fmax(mx, g[r]);
            }
        }
    }
    if (chunk >= a.totals) return; // the whole workgroup
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) mx = fmax(mx, __shfl_xor(mx, s, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    if (!(mx > -1.0e300)) mx = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int k = threadIdx.x + 256 * r;
        if (k < a.dp) {
            const double rel = g[r] - mx;
            a.fold1[at * a.dp + k] = (float)(rel > kFarRow ? rel : kFarRow) + (before ? before[k] : 0.0f);
        }
    }
    if (threadIdx.x == 0) a.gmax[at] = mx + top2;
}

// the initial state (identity, or a converted one that lies there already): its entries, its keys under the first total's fold and without.
// One wave a column n; grid (mp / 4, items), 256 threads.
struct StartArgs {
    Pieces<float> Ct;    // [dp / 16][mp][16]
    Pieces<int> key1, key2; // key1.p NULL: there is no total
    Pieces<double> e;
    Pieces<const float> fold;
    const float *shifts; // NULL: identity; else [item][mp], the converted columns' shifts
    int d, dp, mp;
};
__global__ __launch_bounds__(256) void start_state_kernel(StartArgs a)
{
    const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long item = blockIdx.y;
    float *col = a.Ct.at(item, 0) + (size_t)n * 16;
    const float *fold = a.key1.p ? a.fold.at(item, 0) : nullptr;
    float m1 = CF::neg_inf(), m2 = CF::neg_inf();
    for (int i = lane; i < a.dp; i += 64) {
        float &at = col[(size_t)(i >> 4) * a.mp * 16 + (i & 15)];
        if (!a.shifts) at = i == n && n < a.d ? 1.0f : 0.0f;
        const float x = at;
        if (x != 0.f) {
            m2 = fmaxf(m2, CF::exponent_of(x));
            if (fold) m1 = fmaxf(m1, CF::exponent_of(x) + fold[i]);
        }
    }
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        m1 = fmaxf(m1, __shfl_xor(m1, s, 64));
        m2 = fmaxf(m2, __shfl_xor(m2, s, 64));
    }
    if (lane == 0) {
        if (a.key1.p) a.key1.at(item, 0)[n] = m1 > CF::neg_inf() ? exponent_key(m1) : INT_MIN;
        a.key2.at(item, 0)[n] = m2 > CF::neg_inf() ? exponent_key(m2) : INT_MIN;
        a.e.at(item, 0)[n] = a.shifts ? (double)a.shifts[(size_t)item * a.mp + n] : 0.0;
    }
}

// n keys; nz zeros (no more than keys)
__global__ __launch_bounds__(256) void fill_keys_kernel(int *p, size_t n, double *z, size_t nz)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        p[i] = INT_MIN;
        if (i < nz) z[i] = 0.0;
    }
}

struct LmmeSplitPlan {
    int Np, Mp, Kp;
    size_t off_rs, off_y, off_cs, total;
};
LmmeSplitPlan plan_lmme_split(long long batch, int n, int d, int m)
{
    LmmeSplitPlan p;
    const int tile = split_in_tiles(n, m, batch) ? 128 : 32;
    p.Kp = pad_to(d, 16);
    p.Np = pad_to(n, tile);
    p.Mp = pad_to(m, tile);
    size_t off = goom::align_up((size_t)batch * 3 * p.Np * p.Kp * 2, 256);
    p.off_rs = off;
    off += goom::align_up((size_t)batch * p.Np * 4, 256);
    p.off_y = off;
    off += goom::align_up((size_t)batch * 3 * p.Mp * p.Kp * 2, 256);
    p.off_cs = off;
    off += goom::align_up((size_t)batch * p.Mp * 4, 256);
    p.total = off;
    return p;
}

} // namespace

namespace goom {

size_t lmme_split_workspace_bytes(long long batch, int n, int d, int m) { return plan_lmme_split(batch, n, d, m).total; }

int launch_lmme_split(goom_ctx *ctx, const void *A, const void *B, void *C, long long batch, int n, int d, int m, void *ws)
{
    const LmmeSplitPlan p = plan_lmme_split(batch, n, d, m);
    if (batch > 65535) return fail(ctx, GOOM_EUNSUPPORTED, "at most 65535 pairs per call for shapes above 128 (batch=%lld)", batch);
    unsigned char *w = static_cast<unsigned char *>(ws);
    __bf16 *X = reinterpret_cast<__bf16 *>(w), *Y = reinterpret_cast<__bf16 *>(w + p.off_y);
    float *rs = reinterpret_cast<float *>(w + p.off_rs), *cs = reinterpret_cast<float *>(w + p.off_cs);
    hipStream_t st = ctx->stream;
    const unsigned nb = (unsigned)batch;
    prof_begin(ctx, "lmme_large_scale_operands");
    RowsArgs r{static_cast<const float2 *>(A), X, rs, n, d, p.Np, p.Kp, 0, 0, 0, 0, 0, 0, false};
    hipLaunchKernelGGL(split_rows_kernel, dim3(p.Np / 4, nb), dim3(256), 0, st, r);
    hipLaunchKernelGGL(split_column_shift_kernel, dim3((p.Mp + 63) / 64, nb), dim3(256), 0, st, static_cast<const float2 *>(B), cs, d, m, p.Mp);
    hipLaunchKernelGGL(split_columns_kernel<false>, dim3(p.Mp / 32, (p.Kp + 31) / 32, nb), dim3(256), 0, st, static_cast<const float2 *>(B), cs, Y,
                       3LL * p.Mp * p.Kp, d, m, p.Mp, p.Kp);
    prof_end(ctx);
    if (int s = check_hip(ctx, hipGetLastError(), "launch LMME operand kernels")) return s;
    prof_begin(ctx, "lmme_large_gemm");
    SplitGemm a{};
    a.chunks = 1;
    a.M = p.Np;
    a.N = p.Mp;
    a.K = p.Kp;
    a.X = {X, 3LL * p.Np * p.Kp, 0};
    a.row_shift = {rs, p.Np, 0};
    a.Yp = {Y, 3LL * p.Mp * p.Kp, 0};
    a.col_shift = {cs, p.Mp, 0};
    a.P = static_cast<float2 *>(C);
    a.slots = 1;
    a.L = 1;
    a.step = 0;
    a.n = n;
    a.m = m;
    launch_gemm_split<false>(st, a, nb, split_in_tiles(n, m, batch));
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch gemm_split_kernel");
}

} // namespace goom

// ------------------------------------------------------------------------------------------------
// Scans and reductions: the three phases of the chunked scan, every phase advancing all of its chains by one step per launch.
// ------------------------------------------------------------------------------------------------
namespace {

struct SplitPlan {
    long long L, C, C1;  // chunk length, chunks per item, chunks whose products phase 1 forms
    long long places;    // of converted matrices a chain: all of them, converted once, or two, converted step by step in both phases
    int dp, mp;
    size_t x, shifts, rel, top, xt, raw, tot, fold1, fold2, gmax, top2, car, start_shifts, keys, keys_count, e, total;
    size_t key_round, key_tot, key_car1, key_car2, e_round, e_tot, e_car; // offsets in elements within keys, e
};

// least: two converted matrices a chain whatever the room (the same chunks, and the same results in every bit)
SplitPlan plan_split(long long T, int d, int m, long long batch, long long requested, bool final_only, bool least)
{
    SplitPlan p;
    p.dp = pad_to(d, 128);
    p.mp = pad_to(m, 128);
    const long long tiles = (long long)(p.dp / 128) * (p.dp / 128);
    const size_t mat = (size_t)p.dp * p.dp;
    long long c;
    if (requested > 0) {
        c = (T + requested - 1) / requested;
    } else {
        // The number of chunks by what the launches cost.  Measured with an inner size of 512, in us: a round of all chains 37 while every compute
        // unit has one tile, 58 with two, about 27 for each further one; a carry 10 (16 tiles of 128 x 128 in its own tiling), a third of it the launch.
        // 192 x 512 x 512: 6 steps a chunk 1233, 10 (as many chunks as 2 sqrt(T / 2)) 1480, 12 1266, 24 2015.
        long long most = (long long)(((size_t)8 << 30) / ((mat * 22 + (size_t)p.mp * p.dp * 8) * (size_t)batch));
        if (most > T / 2) most = T / 2;
        if (most > 65535 / batch) most = 65535 / batch;
        const double inner = p.dp / 512.0, carry = 3.0 + 7.0 * inner * std::fmax(1.0, (double)(batch * (p.dp / 128) * (p.mp / 128)) / 16.0 * 0.4);
        auto round = [&](long long n) {
            const double full = (double)((n + 255) / 256);
            return inner * (full <= 1.0 ? 37.0 : 58.0 + 27.0 * (full - 2.0));
        };
        double best = 1e300;
        c = 1;
        for (long long k = 1; k <= most && k <= 1024; ++k) {
            const long long len = (T + k - 1) / k, used = (T + len - 1) / len;
            if (used != k) continue;
            const double rounds = (used > 1 ? (double)(len - 1) * round(batch * used * tiles) : 0.0) +
                                  (final_only && used > 1 ? 0.0 : (double)len * round(batch * used * (p.dp / 128) * (p.mp / 128)));
            const double cost = rounds + (double)(used - 1) * carry;
            if (cost < best) {
                best = cost;
                c = k;
            }
        }
    }
    if (c < 1) c = 1;
    p.L = (T + c - 1) / c;
    p.C = (T + p.L - 1) / p.L;
    p.C1 = p.C <= 1 ? 0 : (final_only ? p.C : p.C - 1);
    const size_t chains = (size_t)batch * p.C;
    p.places = (!least && chains * p.L * mat * 6 <= ((size_t)4 << 30)) || p.L < 2 ? p.L : 2;
    const size_t slots = chains * p.places;
    const int rows = p.mp > p.dp ? p.mp : p.dp;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += goom::align_up(bytes, 256); return o; };
    p.x = take(slots * mat * 6);
    p.shifts = take(slots * p.dp * 4);
    p.rel = take(slots * p.dp * 4);
    p.top = take(slots * 8);
    const bool products = p.C1 > 0 && p.L > 1;
    p.xt = take(products ? chains * mat * 6 : 0);
    p.tot = take(products ? chains * mat * 4 : 0);
    p.raw = take(2 * chains * (size_t)rows * p.dp * 4);
    p.fold1 = take(chains * p.dp * 4);
    p.fold2 = take(chains * p.dp * 4);
    p.gmax = take(chains * 8);
    p.top2 = take(chains * 8);
    p.car = take((size_t)batch * (p.C + 1) * p.mp * p.dp * 4);
    p.start_shifts = take((size_t)batch * p.mp * 4);
    size_t k = 0;
    p.key_round = k; k += 3 * chains * rows;
    p.key_tot = k; k += chains * p.dp;
    p.key_car1 = k; k += (size_t)batch * (p.C + 1) * p.mp;
    p.key_car2 = k; k += (size_t)batch * (p.C + 1) * p.mp;
    p.keys_count = k;
    p.keys = take(k * 4);
    k = 0;
    p.e_round = k; k += 2 * chains * rows;
    p.e_tot = k; k += chains * p.dp;
    p.e_car = k; k += (size_t)batch * (p.C + 1) * p.mp;
    p.e = take(k * 8);
    p.total = off;
    return p;
}

} // namespace

namespace goom {

// Long chains of 128 < d <= 256 with states as wide keep their states in registers (goom_chain256.hip), which takes a chip full of chains of some length.
// Measured, 256 x 256, states in registers against this: T = 64 675 / 284 us, 512 1929 / 986, 4096 5982 / 4476, 16 384 15.6 / 19.2 ms.
bool scan_split_applies(long long T, int d, int m, long long batch) { return !(d > 128 && d <= 256 && m <= 256 && T * batch > 8192); }

size_t scan_split_workspace_bytes(long long T, int d, int m, long long batch, long long requested_chunk, bool final_only, bool least)
{
    return plan_split(T, d, m, batch, requested_chunk, final_only, least).total;
}

int run_scan_split(goom_ctx *ctx, const void *M, const void *init, void *P, long long T, int d, int m, long long batch, long long requested_chunk, void *ws,
                   size_t ws_bytes, bool final_only)
{
    SplitPlan p = plan_split(T, d, m, batch, requested_chunk, final_only, false);
    if (p.total > ws_bytes) p = plan_split(T, d, m, batch, requested_chunk, final_only, true);
    const long long C = p.C, L = p.L, chains = batch * C;
    if (chains > 65535) return fail(ctx, GOOM_EUNSUPPORTED, "too many chains (%lld) for matrices above %d", chains, GOOM_MAX_DIM);
    unsigned char *w = static_cast<unsigned char *>(ws);
    const int dp = p.dp, mp = p.mp;
    const long long mat = (long long)dp * dp, state = (long long)mp * dp;
    const int rows = mp > dp ? mp : dp;
    const float2 *Mg = static_cast<const float2 *>(M);
    __bf16 *X = reinterpret_cast<__bf16 *>(w + p.x);
    float *shifts = reinterpret_cast<float *>(w + p.shifts), *rel = reinterpret_cast<float *>(w + p.rel);
    double *top = reinterpret_cast<double *>(w + p.top), *top2 = reinterpret_cast<double *>(w + p.top2);
    float *raw[2] = {reinterpret_cast<float *>(w + p.raw), reinterpret_cast<float *>(w + p.raw) + chains * rows * dp};
    float *car = reinterpret_cast<float *>(w + p.car);
    float *fold1 = reinterpret_cast<float *>(w + p.fold1), *fold2 = reinterpret_cast<float *>(w + p.fold2);
    double *gmax = reinterpret_cast<double *>(w + p.gmax);
    int *keys = reinterpret_cast<int *>(w + p.keys);
    double *es = reinterpret_cast<double *>(w + p.e);
    int *key_round[3] = {keys + p.key_round, keys + p.key_round + chains * rows, keys + p.key_round + 2 * chains * rows};
    int *key_tot = keys + p.key_tot, *key_car1 = keys + p.key_car1, *key_car2 = keys + p.key_car2;
    double *e_round[2] = {es + p.e_round, es + p.e_round + chains * rows};
    double *e_tot = es + p.e_tot, *e_car = es + p.e_car;
    hipStream_t st = ctx->stream;
    auto ok = [&](const char *what) { return check_hip(ctx, hipGetLastError(), what); };
    const long long car_item = (C + 1) * state, carm = (C + 1) * mp; // strides of the carries' arrays

    const bool all = p.places == L;
    // steps s0 .. of all chains: their matrices' planes and row shifts
    auto convert = [&](long long s0, long long per_chain) {
        // (a NaN shows where states as wide run in registers, and in long chains of these sizes still do; in larger products it counts as zero)
        RowsArgs r{Mg, X, shifts, d, d, dp, dp, T, L, C, per_chain, s0, p.places, d <= 256 && m <= 256};
        hipLaunchKernelGGL(split_rows_kernel, dim3(dp / 4, (unsigned)(chains * per_chain)), dim3(256), 0, st, r);
        RelativeArgs q{shifts, rel, top, dp, per_chain, s0, p.places};
        hipLaunchKernelGGL(relative_shifts_kernel, dim3((unsigned)(chains * per_chain)), dim3(256), 0, st, q);
    };
    auto planes = [&](long long s) { return Pieces<const __bf16>{X + s % p.places * 3 * mat, C * p.places * 3 * mat, p.places * 3 * mat}; };
    auto row_shifts = [&](long long s) { return Pieces<const float>{shifts + s % p.places * dp, C * p.places * dp, p.places * dp}; };
    auto relative = [&](long long s) { return Pieces<const float>{rel + s % p.places * dp, C * p.places * dp, p.places * dp}; };
    auto tops = [&](long long s) { return Pieces<const double>{top + s % p.places, C * p.places, p.places}; };
    auto fill_keys = [&](int *k, size_t n, double *z, size_t nz) {
        const unsigned g = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
        hipLaunchKernelGGL(fill_keys_kernel, dim3(g), dim3(256), 0, st, k, n, z, nz);
    };

    prof_begin(ctx, "scan_large_convert");
    fill_keys(keys, p.keys_count, e_round[0], (size_t)chains * rows); // (the exponents outside of the chunks' first matrices)
    const long long together = chains * L <= 65535 ? L : 1; // (a grid's second dimension; chunks of two steps reach further)
    for (long long s = 0; all && s < L; s += together) convert(s, together);
    prof_end(ctx);

    // ---- phase 1: chunk products, stored by rows in the last step
    const bool products = p.C1 > 0 && L > 1;
    if (products) {
        prof_begin(ctx, "scan_large_phase1_chunk_products");
        const unsigned nchains = (unsigned)(batch * p.C1);
        if (!all) convert(0, 1);
        FirstArgs f{Mg, row_shifts(0), relative(0), {raw[0], C * rows * dp, (long long)rows * dp}, {key_round[0], C * rows, rows}, d, dp, (int)p.C1, T, L};
        hipLaunchKernelGGL(first_state_kernel, dim3(dp / 32, dp / 32, nchains), dim3(256), 0, st, f);
        for (long long s = 1; s < L; ++s) {
            if (!all) convert(s, 1);
            SplitGemm a{};
            a.chunks = (int)p.C1;
            a.M = a.N = a.K = dp;
            a.X = planes(s);
            a.row_shift = row_shifts(s);
            a.Yr = {raw[(s - 1) & 1], C * rows * dp, (long long)rows * dp};
            a.fold = relative(s - 1);
            a.extra = tops(s - 1);
            a.key = {key_round[(s - 1) % 3], C * rows, rows};
            a.e_in = {e_round[(s - 1) & 1], C * rows, rows};
            if (s + 1 < L) {
                a.Ct = {raw[s & 1], C * rows * dp, (long long)rows * dp};
                a.fold1 = relative(s);
                a.key1 = {key_round[s % 3], C * rows, rows};
                a.clear = {key_round[(s + 1) % 3], C * rows, rows};
                a.e_out = {e_round[s & 1], C * rows, rows};
            } else {
                a.C = {reinterpret_cast<float *>(w + p.tot), C * mat, mat};
                a.key1 = {key_tot, C * dp, dp};
                a.e_out = {e_tot, C * dp, dp};
            }
            launch_gemm_split<true>(st, a, nchains, split_in_tiles(dp, dp, nchains));
        }
        prof_end(ctx);
        if (int e = ok("scan_large phase 1")) return e;
    }

    // ---- phase 2: prefixes at the chunk boundaries (and, for a reduction, the final product)
    prof_begin(ctx, "scan_large_phase2_carries");
    Pieces<const __bf16> xt = planes(0); // (chunks of one step are their own products)
    const Pieces<const float> tot_shifts = row_shifts(L - 1), tot_rel = relative(L - 1);
    const Pieces<const double> tot_top = tops(L - 1);
    if (products) {
        __bf16 *xtp = reinterpret_cast<__bf16 *>(w + p.xt);
        TotalsArgs t{reinterpret_cast<const float *>(w + p.tot), key_tot, e_tot, xtp, dp, C};
        hipLaunchKernelGGL(totals_planes_kernel, dim3(dp / 4, (unsigned)p.C1, (unsigned)batch), dim3(256), 0, st, t);
        xt = {xtp, C * 3 * mat, 3 * mat};
    }
    FoldArgs f{products ? key_tot : nullptr, e_tot, tot_rel, tot_top, fold1, fold2, gmax, top2, dp, d, C, p.C1};
    hipLaunchKernelGGL(totals_fold_kernel, dim3((unsigned)C, (unsigned)batch), dim3(256), 0, st, f);
    float *start_shifts = reinterpret_cast<float *>(w + p.start_shifts);
    if (init) {
        hipLaunchKernelGGL(split_column_shift_kernel, dim3(mp / 64, (unsigned)batch), dim3(256), 0, st, static_cast<const float2 *>(init), start_shifts, d, m, mp);
        // (into the first carry's place, which lies a whole item of carries from the next item's)
        hipLaunchKernelGGL(split_columns_kernel<true>, dim3(mp / 32, dp / 32, (unsigned)batch), dim3(256), 0, st, static_cast<const float2 *>(init), start_shifts,
                           static_cast<void *>(car), car_item, d, m, mp, dp);
    }
    StartArgs s0{{car, car_item, state}, {p.C1 > 0 ? key_car1 : nullptr, carm, mp}, {key_car2, carm, mp}, {e_car, carm, mp}, {fold1, C * dp, dp},
                 init ? start_shifts : nullptr, d, dp, mp};
    hipLaunchKernelGGL(start_state_kernel, dim3(mp / 4, (unsigned)batch), dim3(256), 0, st, s0);
    for (long long c = 0; c < p.C1; ++c) {
        const bool last = c + 1 == p.C1;
        SplitGemm a{};
        a.chunks = 1;
        a.M = a.K = dp;
        a.N = mp;
        a.X = {xt.p + c * xt.chunk, xt.item, 0};
        a.row_shift = {tot_shifts.p + c * tot_shifts.chunk, tot_shifts.item, 0};
        a.Yr = {car + c * state, car_item, 0};
        a.fold = {fold1 + c * dp, C * dp, 0};
        a.key = {key_car1 + c * mp, carm, 0};
        a.e_in = {e_car + c * mp, carm, 0};
        a.extra = {gmax + c, C, 0};
        a.e_out = {e_car + (c + 1) * mp, carm, 0};
        if (!(final_only && last)) a.Ct = {car + (c + 1) * state, car_item, 0};
        if (!last) {
            a.fold1 = {fold1 + (c + 1) * dp, C * dp, 0};
            a.key1 = {key_car1 + (c + 1) * mp, carm, 0};
        }
        if (!final_only) { // as chunk c + 1 reads it
            a.fold2 = {tot_rel.p + c * tot_rel.chunk, tot_rel.item, 0};
            a.key2 = {key_car2 + (c + 1) * mp, carm, 0};
        } else if (last) {
            a.P = static_cast<float2 *>(P);
            a.slots = a.L = 1;
            a.n = d;
            a.m = m;
        }
        launch_gemm_split<true>(st, a, (unsigned)batch, split_in_tiles(dp, mp, batch));
    }
    prof_end(ctx);
    if (int e = ok("scan_large phase 2")) return e;
    if (final_only && p.C1 > 0) return GOOM_OK;

    // ---- phase 3: every chunk from its incoming prefix, all prefixes stored (a reduction of a single chunk stores the last)
    prof_begin(ctx, final_only ? "scan_large_single_chunk" : "scan_large_phase3_outputs");
    fill_keys(keys + p.key_round, 3 * chains * rows, nullptr, 0);
    for (long long s = 0; s < L; ++s) {
        if (!all) convert(s, 1);
        SplitGemm a{};
        a.chunks = (int)C;
        a.M = a.K = dp;
        a.N = mp;
        a.X = planes(s);
        a.row_shift = row_shifts(s);
        if (s == 0) {
            a.Yr = {car, car_item, state};
            a.fold = {fold2, C * dp, dp};
            a.extra = {top2, C, 1};
            a.key = {key_car2, carm, mp};
            a.e_in = {e_car, carm, mp};
        } else {
            a.Yr = {raw[(s - 1) & 1], C * rows * dp, (long long)rows * dp};
            a.fold = relative(s - 1);
            a.extra = tops(s - 1);
            a.key = {key_round[(s - 1) % 3], C * rows, rows};
            a.e_in = {e_round[(s - 1) & 1], C * rows, rows};
        }
        if (s + 1 < L) {
            a.Ct = {raw[s & 1], C * rows * dp, (long long)rows * dp};
            a.fold1 = relative(s);
            a.key1 = {key_round[s % 3], C * rows, rows};
            a.clear = {key_round[(s + 1) % 3], C * rows, rows};
            a.e_out = {e_round[s & 1], C * rows, rows};
        }
        if (!final_only || s + 1 == L) {
            a.P = static_cast<float2 *>(P);
            a.n = d;
            a.m = m;
            a.slots = final_only ? 1 : T;
            a.L = final_only ? 1 : L;
            a.step = final_only ? 0 : s;
        }
        launch_gemm_split<true>(st, a, (unsigned)chains, split_in_tiles(dp, mp, chains));
    }
    prof_end(ctx);
    return ok("scan_large phase 3");
}

} // namespace goom
