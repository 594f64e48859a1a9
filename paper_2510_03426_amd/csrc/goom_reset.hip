// Carry phase of the selectively reset scan (paper Section 5; Section 4.2.1 item (a)).
//
// The reset scan cuts the chain into chunks like the plain scan.  Phase 1 (chain kernel)
// multiplies every chunk down to one factored matrix T_c.  This kernel is phase 2: one
// workgroup per batch item walks the chunks in order, keeping the true prefix state
//     Z = T_c Y_c            (the state at step (c + 1) L),
// examines it with the selection function S (always / near-colinear columns / never), and
// when selected replaces it by R(Z): columns scaled to unit norm, then the orthonormal
// factor Q of a QR factorisation with positive diagonal.  The prefix that enters chunk
// c + 1, Y_{c+1}, is written for phase 3 (chain kernel), which re-walks every chunk and
// stores all states.  Because S and R are applied only to true prefix states, left to
// right, the result does not depend on a scan tree: it is the sequential recurrence with
// its states examined every L steps.
//
// Per column k a reset removes log R_kk + log(norm of column k) of log-growth from the
// state; these accumulate (in double) into growth[k], plus the same quantities for the
// final state, so growth / (dt T) is the Lyapunov spectrum (paper Section 4.2.1, eq. 20, with the
// triangular factors taken at the resets: triangular factors multiply, so their diagonals
// accumulate exactly as in the step-by-step method).
//
// The chain of chunks is inherently serial (each reset depends on the previous one), so this
// phase is latency bound: what counts is the length of the dependent instruction chain per
// chunk.  One wave per batch item holds the whole state in registers (policies that look at a
// state first), or one wave per panel of it, the panels' waves a chunk apart (policy "always").
#include <cmath>
#include <cstring>
#include <type_traits>

#include "goom_internal.h"

namespace {

constexpr double kLn2 = 0.693147180559945309417;
constexpr double kLog2e = 1.44269504088896340736;
constexpr int kThreads = 256;

struct ResetArgs {
    const unsigned char *totals; // [batch][C] factored chunk products (common exponent), DP x tot_cols
    long long tot_stride;
    int tot_cols;
    unsigned char *carries;      // [batch][C + 1] factored prefixes entering each chunk (and the final state), DP x car_cols
    long long car_stride;
    int car_cols;
    const void *s0;              // NULL or GOOM initial state [batch][d][d] (complex64 or complex128)
    unsigned char *chunk_flags;  // [batch][C]: 1 where the state at the end of chunk c was reset
    double *growth;              // NULL or [batch][d]
    double growth_scale;         // 1, or 1 / (dt T) to return exponents
    long long T, L, C;
    int d;
    int policy;
    float cos_threshold;
    const int *only_if;          // staged kernel: NULL, or [batch]: items for which it has work
    // spectra in segments (see reset_carry_staged_kernel): room for their results, [batch][segments] of SegmentRoom doubles
    double *segments_room;
    const double *frames;        // NULL, or as much: the chain's states at the segments' ends, as a first pass has put them together
    int segments;
    long long per_segment;
};

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

__device__ inline f4 mfma4(float x, float y, f4 acc) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0); }

__device__ inline float read_lane(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// LDS operations of one wave complete in program order; this only keeps the compiler from
// moving them across the point where lanes hand data to each other.
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef double d4 __attribute__((ext_vector_type(4)));

// One wave per batch item.  All DP x DP matrices live in registers in the layout the
// 16 x 16 x 4 matrix instruction leaves its result in: lane (g = lane / 16, c = lane % 16),
// register [nt][mt][v] holds entry (row 16 mt + 4 g + v, column 16 nt + c).  That layout is
// also the instruction's B operand, and, read as "column block first", the A operand of the
// transpose, so both Z = T Y and the Gram matrix G = Z^T Z run on the matrix unit without
// moving the state; only the chunk product T goes through LDS (it arrives row by row).
//
// QR by the Gram matrix: Cholesky elimination G = R^T R, one column per step, with the same
// column operations applied to Z, which turns Z into Q = Z R^-1 in place; row k of G and
// column k of Z reach the other lanes through a few words of LDS.  The pivots are the
// squares of R's diagonal.  G is formed and eliminated in double (the double-precision
// matrix instruction; its result has row 16 mt + 4 v + g in register v), so the pivots stay
// accurate up to cond(Z)^2 of about 1e12; the columns of Z are updated in float, which
// costs orthogonality in proportion to sqrt(largest ratio of a column's squared norm to its
// pivot).  When that ratio is large the factorisation is repeated on Q, which restores
// orthogonality to rounding level, and the two diagonals multiply.
template <int DP> struct Wave {
    static constexpr int KT = DP / 16;
    static constexpr int LDT = DP + 4;
    float tile[DP * LDT]; // chunk product, row-major, rows padded against bank conflicts
    double rrow[2][DP];   // row k of G at step k, entry j at position j (two sets, used alternately)
    double rperm[2][DP];  // the same with entry 16 mt + 4 v + g at position 16 mt + 4 g + v
    float qcol[2][DP];    // column k of Z at step k
    double diag[DP];      // diagonal of the Gram matrix
    float qpanel[DP / 16][DP * 20]; // finished panels of Q, [row][column within the panel], rows padded to 20
};

// The factorisation runs panel by panel (16 columns at a time), in square-root-free form: a step
// subtracts (G_kj / p_k) times row / column k from every later one of the panel, p_k = G_kk being the
// pivot, and the columns are scaled by 1 / sqrt(p) at the end of the panel.  The row and the column of
// step k go to LDS as they are, so their round trip overlaps with the reciprocal of the pivot, the
// other half of the dependent chain.  A panel is first made orthogonal to the finished panels on the matrix unit (R_qp = Q_q^T Z_p, then
// Z_p -= Q_q R_qp: the first product reads both operands in place, the second takes Q_q from LDS as
// its left operand and R_qp, as the matrix instruction left it, as its right operand), then its own
// 16 x 16 Gram matrix is eliminated as above.  A step then touches 16 columns instead of all of
// them, and only one 16 x 16 tile of G is alive at a time.

// elimination of one panel: G is its 16 x 16 Gram matrix (register v = row 4 v + g, column c),
// Zp its columns; pivots to piv for the lanes that own the column
template <int DP> __device__ void eliminate_panel(d4 &G, f4 (&Zp)[DP / 16], double &piv, Wave<DP> &s, int g, int c)
{
    constexpr int KT = DP / 16;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int gk = k % 4, vk = k / 4; // row k of G: lanes with g == gk, register vk
        const int buf = k & 1;
        double *rrow = s.rrow[buf];
        double *rperm = s.rperm[buf];
        float *qcol = s.qcol[buf];
        if (g == gk) {
            const double r = c > k ? G[vk] : 0.0; // zero left of the diagonal: finished columns stay put
            rrow[c] = r;
            rperm[((c & 3) << 2) | (c >> 2)] = r;
        }
        if (c == k) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) *reinterpret_cast<f4 *>(&qcol[16 * mt + 4 * g]) = Zp[mt];
        }
        const double pv = G[vk];
        const int lo = __builtin_amdgcn_readlane((int)(__builtin_bit_cast(unsigned long long, pv) & 0xffffffffull), 16 * gk + k);
        const int hi = __builtin_amdgcn_readlane((int)(__builtin_bit_cast(unsigned long long, pv) >> 32), 16 * gk + k);
        const double pivot = __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
        if (c == k) piv = pivot;
        const bool live = pivot > 1.0e-30;
        const double r0 = (double)__builtin_amdgcn_rcpf((float)pivot);
        const double inv = live ? r0 * (2.0 - pivot * r0) : 0.0;
        wave_sync();
        const double tj = rrow[c] * inv;
        const d4 ri = *reinterpret_cast<const d4 *>(&rperm[4 * g]); // rows 4 v + g, v = 0..3
        G -= ri * tj;
        const float tjf = (float)tj;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) {
            const f4 zk = *reinterpret_cast<const f4 *>(&qcol[16 * mt + 4 * g]);
            Zp[mt] -= zk * tjf;
        }
    }
    wave_sync();
}

// QR of Z in place (Z <- Q), panel by panel; piv[nt] = squared diagonal of R for column 16 nt + c.
// Returns the largest ratio (squared column norm) / pivot, a measure of cond(Z)^2.
template <int DP> __device__ float qr_panels(f4 (&Z)[DP / 16][DP / 16], double (&piv)[DP / 16], Wave<DP> &s, int g, int c)
{
    constexpr int KT = DP / 16;
    float norm2[KT];
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        float a = 0.0f;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) a = __builtin_fmaf(Z[nt][mt][v], Z[nt][mt][v], a);
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        norm2[nt] = a;
    }
#pragma unroll
    for (int p = 0; p < KT; ++p) {
        // orthogonal to the finished panels; twice, because one float projection leaves about
        // 2^-24 of the panel's norm behind, which the panel's own (much smaller) remainder would magnify
#pragma unroll
        for (int rep = 0; rep < (p > 0 ? 2 : 0); ++rep)
#pragma unroll
        for (int q = 0; q < p; ++q) {
            f4 R = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) R = mfma4(Z[q][kt][v], Z[p][kt][v], R);
            R = -R;
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const f4 av = *reinterpret_cast<const f4 *>(&s.qpanel[q][(16 * mt + c) * 20 + 4 * g]);
#pragma unroll
                for (int v = 0; v < 4; ++v) Z[p][mt] = mfma4(av[v], R[v], Z[p][mt]);
            }
        }
        // the panel's own Gram matrix, in double
        d4 G = {0., 0., 0., 0.};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) G = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Z[p][kt][v], (double)Z[p][kt][v], G, 0, 0, 0);
        piv[p] = 1.0;
        eliminate_panel<DP>(G, Z[p], piv[p], s, g, c);
        const bool live = piv[p] > 1.0e-30;
        const float sc = live ? __builtin_amdgcn_rsqf((float)piv[p]) : 0.0f;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) Z[p][mt] *= sc;
        if (p + 1 < KT) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) s.qpanel[p][(16 * mt + 4 * g + v) * 20 + c] = Z[p][mt][v];
            wave_sync();
        }
    }
    float worst = 1.0f;
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        const float ratio = piv[nt] > 1.0e-30 ? norm2[nt] * __builtin_amdgcn_rcpf((float)piv[nt]) : 1.0f;
        worst = fmaxf(worst, ratio);
    }
#pragma unroll
    for (int sft = 1; sft < 16; sft <<= 1) worst = fmaxf(worst, __shfl_xor(worst, sft, 64));
    return read_lane(worst, 0); // the same in every lane; this tells the compiler so
}

// ---------------------------------------------------------------------------------------------------
// The carry kernel keeps everything in double: the chunk products arrive in double, Z = T Y and every step
// of the factorisation run on the double-precision matrix instruction and the double vector ALU.  The
// 16 x 16 x 4 double instruction leaves rows 4 v + g of column c in register v of lane (g, c), takes
// A[row c][k = g] and B[k = g][column c] from lane (g, c); so a matrix held as [nt][mt] tiles in that result
// layout is, register for register, a B operand whose contraction index runs 4 v + g, and an A operand of
// its transpose.  Whatever is read from LDS as a four-vector therefore stores index 4 v + g at position
// 4 g + v (perm16 below).
__device__ inline int perm16(int j) { return (j & ~15) | ((j & 3) << 2) | ((j >> 2) & 3); }

template <int DP> struct WaveD {
    static constexpr int LDT = DP + 2;  // row stride of the chunk product (doubles)
    static constexpr int LDQ = 18;      // row stride of a finished panel
    double tile[DP * LDT]; // chunk product, rows in order, columns in perm16 order
    double gram[16 * 18]; // a panel's Gram matrix on its way into the lanes
    double diag[DP];      // diagonal of the Gram matrix (selection by cosines)
    double qpanel[DP / 16 > 1 ? DP / 16 - 1 : 1][DP * LDQ]; // finished panels of Q: [row][column within the panel, perm16 order]
};

__device__ inline d4 mfma8(double x, double y, d4 acc) { return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc, 0, 0, 0); }

__device__ inline double read_lane_d(double v, int lane)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffffull), lane);
    const int hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// 1 / x and 1 / sqrt(x) to double precision from the float hardware approximations (x within float range)
__device__ inline double rcp_d(double x)
{
    double r = (double)__builtin_amdgcn_rcpf((float)x);
    r = r * (2.0 - x * r);
    return r * (2.0 - x * r);
}
__device__ inline double rsqrt_d(double x)
{
    double r = (double)__builtin_amdgcn_rsqf((float)x);
    r = r * (1.5 - 0.5 * x * r * r);
    return r * (1.5 - 0.5 * x * r * r);
}

// lane K of every row of sixteen lanes, to all lanes of that row
template <int K> __device__ inline double row_bcast(double x)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffull), 0x150 + K, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), 0x150 + K, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// x[i] += (src of lane i of the row of sixteen) * mul, for i = FROM .. TO - 1: one instruction each, the broadcast being part of
// the multiply-add.  (A register that a vector instruction has just written may be read across lanes two issue slots later:
// every block opens with that wait, since the compiler does not look into it.)
#define GOOM_FMAC_BCAST(ACC, LANE) "v_fmac_f64_dpp " ACC ", %[s], %[m] row_newbcast:" LANE " row_mask:0xf bank_mask:0xf\n\t"
template <int FROM, int TO = 16> __device__ inline void fmac_bcast(double (&x)[16], double src, double mul)
{
    if constexpr (FROM + 8 <= TO) {
        asm("s_nop 1\n\t" GOOM_FMAC_BCAST("%0", "%[k0]") GOOM_FMAC_BCAST("%1", "%[k1]") GOOM_FMAC_BCAST("%2", "%[k2]") GOOM_FMAC_BCAST("%3", "%[k3]")
                GOOM_FMAC_BCAST("%4", "%[k4]") GOOM_FMAC_BCAST("%5", "%[k5]") GOOM_FMAC_BCAST("%6", "%[k6]") GOOM_FMAC_BCAST("%7", "%[k7]")
            : "+v"(x[FROM]), "+v"(x[FROM + 1]), "+v"(x[FROM + 2]), "+v"(x[FROM + 3]), "+v"(x[FROM + 4]), "+v"(x[FROM + 5]), "+v"(x[FROM + 6]), "+v"(x[FROM + 7])
            : [s] "v"(src), [m] "v"(mul), [k0] "n"(FROM), [k1] "n"(FROM + 1), [k2] "n"(FROM + 2), [k3] "n"(FROM + 3), [k4] "n"(FROM + 4), [k5] "n"(FROM + 5),
              [k6] "n"(FROM + 6), [k7] "n"(FROM + 7));
        fmac_bcast<FROM + 8, TO>(x, src, mul);
    } else if constexpr (FROM + 4 <= TO) {
        asm("s_nop 1\n\t" GOOM_FMAC_BCAST("%0", "%[k0]") GOOM_FMAC_BCAST("%1", "%[k1]") GOOM_FMAC_BCAST("%2", "%[k2]") GOOM_FMAC_BCAST("%3", "%[k3]")
            : "+v"(x[FROM]), "+v"(x[FROM + 1]), "+v"(x[FROM + 2]), "+v"(x[FROM + 3])
            : [s] "v"(src), [m] "v"(mul), [k0] "n"(FROM), [k1] "n"(FROM + 1), [k2] "n"(FROM + 2), [k3] "n"(FROM + 3));
        fmac_bcast<FROM + 4, TO>(x, src, mul);
    } else if constexpr (FROM + 2 <= TO) {
        asm("s_nop 1\n\t" GOOM_FMAC_BCAST("%0", "%[k0]") GOOM_FMAC_BCAST("%1", "%[k1]")
            : "+v"(x[FROM]), "+v"(x[FROM + 1])
            : [s] "v"(src), [m] "v"(mul), [k0] "n"(FROM), [k1] "n"(FROM + 1));
        fmac_bcast<FROM + 2, TO>(x, src, mul);
    } else if constexpr (FROM + 1 <= TO) {
        asm("s_nop 1\n\t" GOOM_FMAC_BCAST("%0", "%[k0]") : "+v"(x[FROM]) : [s] "v"(src), [m] "v"(mul), [k0] "n"(FROM));
    }
}

// over the four lanes that hold a column (lane, lane ^ 16, lane ^ 32, lane ^ 48): the largest / the sum
__device__ inline unsigned column_max(unsigned x)
{
    auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = max((unsigned)a[0], (unsigned)a[1]);
    a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return max((unsigned)a[0], (unsigned)a[1]);
}
__device__ inline double column_sum(double x)
{
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
        const auto l = half == 0 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false) : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = half == 0 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false) : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        x = __builtin_bit_cast(double, ((unsigned long long)h[0] << 32) | l[0]) + __builtin_bit_cast(double, ((unsigned long long)h[1] << 32) | l[1]);
    }
    return x;
}
// binary exponent of the largest entry of a column (rows in Z and in the three other lanes that hold it): entries times 2^-it lie
// below 1.  (An empty column: -1022, which changes nothing of it.)
template <int KT> __device__ inline int column_exponent(const d4 (&Z)[KT])
{
    unsigned key = 0;
#pragma unroll
    for (int mt = 0; mt < KT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double x = Z[mt][v]; // (a vector's element inside the cast would be read as element 0)
            key = max(key, (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32) & 0x7fffffffu);
        }
    return (int)(column_max(key) >> 20) - 1022;
}

constexpr int kPanelLd = 18; // row stride of a 16-column panel (or of its Gram matrix) in LDS, in doubles

// One pivot of the elimination below (by recursion, so that every index is a constant).  neg: minus the multipliers of step K.
// The order is the source's: the next pivot's row is updated first, and its reciprocal (rcp_d, step by step), a chain of dependent
// instructions, is formed between the updates that nothing waits for.
// KEEP: the multipliers stay in u: row K of the panel's unit triangular factor, lane c its column.
template <int K, int NR, bool KEEP>
__device__ inline void eliminate_from(double (&G)[16], double (&z)[NR][16], double neg, double &piv, int c, double (&u)[KEEP ? 16 : 1])
{
    if constexpr (KEEP) u[K] = -neg;
    if constexpr (K < 15) {
        // (with two rows a lane the second row's updates are filler enough, and fewer pieces leave the registers alone)
        constexpr int Z1 = NR > 1 ? 16 : K + 1 + (17 - K) / 3, Z2 = Z1 + (17 - Z1) / 2, G1 = NR > 1 ? 16 : K + 2 + (15 - K) / 2;
        asm("s_nop 1\n\t" GOOM_FMAC_BCAST("%0", "%[k]") : "+v"(G[K + 1]) : [s] "v"(G[K]), [m] "v"(neg), [k] "n"(K + 1));
        __builtin_amdgcn_sched_barrier(0);
        fmac_bcast<K + 1, Z1>(z[0], neg, z[0][K]);
        __builtin_amdgcn_sched_barrier(0);
        const double pivot = row_bcast<K + 1>(G[K + 1]);
        const float coarse = (float)pivot;
        __builtin_amdgcn_sched_barrier(0);
        fmac_bcast<K + 2, G1>(G, G[K], neg);
        __builtin_amdgcn_sched_barrier(0);
        const float estimate = __builtin_amdgcn_rcpf(coarse);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NR > 1) {
            fmac_bcast<K + 1>(z[1], neg, z[1][K]);
            __builtin_amdgcn_sched_barrier(0);
        }
        fmac_bcast<Z1, Z2>(z[0], neg, z[0][K]);
        __builtin_amdgcn_sched_barrier(0);
        const double r = (double)estimate;
        const double t = 2.0 - pivot * r;
        __builtin_amdgcn_sched_barrier(0);
        fmac_bcast<G1>(G, G[K], neg);
        __builtin_amdgcn_sched_barrier(0);
        const double r1 = r * t;
        __builtin_amdgcn_sched_barrier(0);
        fmac_bcast<Z2>(z[0], neg, z[0][K]);
        __builtin_amdgcn_sched_barrier(0);
        piv = c == K + 1 ? G[K + 1] : piv;
        const double inv = r1 * (2.0 - pivot * r1);
        eliminate_from<K + 1, NR, KEEP>(G, z, -(G[K + 1] * (pivot > 1.0e-280 ? inv : 0.0)), piv, c, u);
    }
}

// Orthonormal factor of one panel (DP rows, 16 columns, Zp in the matrix instruction's layout) by its Gram matrix G, in
// square-root-free form: step k subtracts (G_kj / p_k) times row / column k from every later one, p_k = G_kk being the pivot; at
// the end the columns are scaled by 1 / sqrt(p).  The panel leaves as rows: lane r holds row r (and r + 64) in z, and `panel`
// ([DP][18], columns in perm16 order) receives them.  piv: the pivot of column c.
//
// A chain of sixteen pivots is all latency, so nothing in it leaves the registers: every row of sixteen lanes holds the whole
// Gram matrix, lane c its column c, every lane one row of the panel; what a step needs of other lanes is one lane's value for
// sixteen others, which the multiply-add itself can fetch (at half its rate: 9 cycles; a broadcast into a register and two
// multiply-adds that share it cost the same, and the compiler then puts the updates after the chain instead of into it).  (560 cycles a
// pivot when rows and columns of the step went through LDS, now about 200.)
//
// A pivot that comes out negative is a column that is nothing but rounding beside its norm: in a first pass it stays as it is,
// its residual, with a pivot of 1, and the caller (told so) factors once more, where the residual stands for itself; in the
// `last` one it is dropped, like a column that is zero.
//
// tri: (KEEP) receives the triangular factor, [16][18].
template <int DP, bool KEEP = false> __device__ inline bool factor_panel_rows(const d4 (&Zp)[DP / 16], double &piv, double *panel, double *gram,
                                                                              double (&z)[DP > 64 ? 2 : 1][16], int lane, bool last, double *tri = nullptr)
{
    constexpr int KT = DP / 16, NR = DP > 64 ? 2 : 1;
    const int g = lane >> 4, c = lane & 15;
    const int pc = ((c & 3) << 2) | (c >> 2);
    wave_sync();
#pragma unroll
    for (int mt = 0; mt < KT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) panel[(16 * mt + 4 * v + g) * kPanelLd + pc] = Zp[mt][v];
    wave_sync();
    const int row = lane & (DP < 64 ? DP - 1 : 63);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int q = 0; q < 16; q += 2) { // positions q, q + 1 hold columns 4 (q % 4) + q / 4 and the same plus 4
            const d2 x = *reinterpret_cast<const d2 *>(&panel[(row + 64 * r) * kPanelLd + q]);
            z[r][4 * (q & 3) + (q >> 2)] = x[0];
            z[r][4 * ((q + 1) & 3) + (q >> 2)] = x[1];
        }
    d4 Gt = {0., 0., 0., 0.};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int v = 0; v < 4; ++v) Gt = mfma8(Zp[kt][v], Zp[kt][v], Gt);
#pragma unroll
    for (int v = 0; v < 4; ++v) gram[(4 * v + g) * kPanelLd + c] = Gt[v];
    wave_sync();
    double G[16];
#pragma unroll
    for (int j = 0; j < 16; j += 2) { // (symmetric to the last bit: row c is column c)
        const d2 x = *reinterpret_cast<const d2 *>(&gram[c * kPanelLd + j]);
        G[j] = x[0];
        G[j + 1] = x[1];
    }
    const double first = row_bcast<0>(G[0]);
    piv = G[0];
    double u[KEEP ? 16 : 1];
    eliminate_from<0, NR, KEEP>(G, z, -(G[0] * (first > 1.0e-280 ? rcp_d(first) : 0.0)), piv, c, u);
    const bool live = piv > 1.0e-280, open = !live && !last && piv != 0.0;
    const double sc = live ? rsqrt_d(piv) : open ? 1.0 : 0.0;
    if constexpr (KEEP) {
        gram[c] = live ? piv * sc : sc; // (the Gram matrix has been read) the factor's diagonal
        wave_sync();
        if (g == 0) {
#pragma unroll
            for (int k = 0; k < 16; ++k) tri[k * kPanelLd + c] = c < k ? 0.0 : c == k ? gram[k] : gram[k] * u[k];
        }
    }
    piv = open ? 1.0 : piv;
    const double cols[16] = {row_bcast<0>(sc),  row_bcast<1>(sc),  row_bcast<2>(sc),  row_bcast<3>(sc), row_bcast<4>(sc),  row_bcast<5>(sc),
                             row_bcast<6>(sc),  row_bcast<7>(sc),  row_bcast<8>(sc),  row_bcast<9>(sc), row_bcast<10>(sc), row_bcast<11>(sc),
                             row_bcast<12>(sc), row_bcast<13>(sc), row_bcast<14>(sc), row_bcast<15>(sc)};
#pragma unroll
    for (int r = 0; r < NR; ++r) {
#pragma unroll
        for (int j = 0; j < 16; ++j) z[r][j] *= cols[j];
#pragma unroll
        for (int q = 0; q < 16; q += 2) {
            const d2 x = {z[r][4 * (q & 3) + (q >> 2)], z[r][4 * ((q + 1) & 3) + (q >> 2)]};
            *reinterpret_cast<d2 *>(&panel[(row + 64 * r) * kPanelLd + q]) = x;
        }
    }
    wave_sync();
    return __builtin_amdgcn_ballot_w64(open) != 0;
}

// a panel from LDS, in the matrix instruction's layout (rows 16 mt + 4 v + g of column c)
template <int DP> __device__ inline void panel_tiles(d4 (&Zp)[DP / 16], const double *panel, int g, int c)
{
    const int pc = ((c & 3) << 2) | (c >> 2);
#pragma unroll
    for (int mt = 0; mt < DP / 16; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) Zp[mt][v] = panel[(16 * mt + 4 * v + g) * kPanelLd + pc];
}

// QR of Z in place (Z <- Q), panel by panel; piv[nt] = squared diagonal of R for column 16 nt + c.  Returns the
// largest ratio (squared column norm) / pivot, a measure of cond(Z)^2.  Before the factorisation every column
// is scaled by a power of two to a largest entry near 1 (cexp receives the exponents).
template <int DP> __device__ double qr_panels_d(d4 (&Z)[DP / 16][DP / 16], double (&piv)[DP / 16], double (&cexp)[DP / 16], WaveD<DP> &s, int g, int c, bool last)
{
    bool open = false;
    constexpr int KT = DP / 16;
    constexpr int LDQ = WaveD<DP>::LDQ;
    double norm2[KT];
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        double mx = 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) mx = fmax(mx, fabs(Z[nt][mt][v]));
        mx = fmax(mx, __shfl_xor(mx, 16, 64));
        mx = fmax(mx, __shfl_xor(mx, 32, 64));
        int ex = 0;
        if (mx > 0.0) (void)frexp(mx, &ex);
        cexp[nt] = (double)ex;
        double a = 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Z[nt][mt][v] = ldexp(Z[nt][mt][v], -ex);
                a = fma(Z[nt][mt][v], Z[nt][mt][v], a);
            }
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        norm2[nt] = a;
    }
#pragma unroll
    for (int p = 0; p < KT; ++p) {
        // orthogonal to the finished panels (twice: one projection leaves rounding-level remainders of the
        // panel's norm behind, which the panel's own, much smaller, remainder would magnify)
#pragma unroll
        for (int rep = 0; rep < (p > 0 ? 2 : 0); ++rep)
#pragma unroll
            for (int q = 0; q < p; ++q) {
                d4 R = {0., 0., 0., 0.};
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) R = mfma8(Z[q][kt][v], Z[p][kt][v], R);
                R = -R;
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) {
                    const d4 av = *reinterpret_cast<const d4 *>(&s.qpanel[q][(16 * mt + c) * LDQ + 4 * g]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) Z[p][mt] = mfma8(av[v], R[v], Z[p][mt]);
                }
            }
        double rows[1][16];
        double *panel = p + 1 < KT ? s.qpanel[p] : s.tile; // (the chunk product's tile is free by now)
        open |= factor_panel_rows<DP>(Z[p], piv[p], panel, s.gram, rows, (g << 4) | c, last);
        panel_tiles<DP>(Z[p], panel, g, c);
    }
    wave_sync();
    double worst = 1.0;
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        const double ratio = piv[nt] > 1.0e-280 ? norm2[nt] * rcp_d(piv[nt]) : 1.0;
        worst = fmax(worst, ratio);
    }
#pragma unroll
    for (int sft = 1; sft < 16; sft <<= 1) worst = fmax(worst, __shfl_xor(worst, sft, 64));
    return open ? 1.0e300 : read_lane_d(worst, 0);
}

// IO: component type of the GOOM initial state (float for complex64, double for complex128)
template <int DP, typename IO> __global__ __launch_bounds__(64) void reset_carry_kernel(ResetArgs a)
{
    constexpr int KT = DP / 16;
    constexpr int LDT = WaveD<DP>::LDT;
    constexpr int TQ = DP * DP / 4 / 64; // 32-byte pieces (four doubles) of the chunk product per lane
    constexpr bool PREFETCH = DP <= 32;  // the next chunk product waits in registers during the factorisation
    __shared__ __align__(32) WaveD<DP> s;
    const int lane = threadIdx.x;
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const long long b = blockIdx.x;
    const size_t tot_mant = (size_t)DP * a.tot_cols * sizeof(double);
    const size_t car_mant = (size_t)DP * a.car_cols * sizeof(double);

    d4 Y[KT][KT];    // state: Y[nt][mt][v] = entry (row 16 mt + 4 v + g, column 16 nt + c), columns scaled by 2^yexp
    double yexp[KT];
    double pprod[KT], pexp[KT]; // product of all pivots so far = pprod 2^pexp (column exponents counted twice: pivots are squares)
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        yexp[nt] = 0.0;
        pprod[nt] = 1.0;
        pexp[nt] = 0.0;
    }
    // ---- initial state: identity or the given GOOM matrix; rows and columns past d carry an identity block,
    // which stays orthogonal to everything and never reaches the outputs
#pragma unroll
    for (int nt = 0; nt < KT; ++nt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) Y[nt][mt][v] = (16 * mt + 4 * v + g == 16 * nt + c) ? 1.0 : 0.0;
    if (a.s0) {
        const IO *gp = reinterpret_cast<const IO *>(a.s0) + (size_t)b * d * d * 2;
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            const int col = 16 * nt + c;
            if (col < d) {
                double cmax = -__builtin_huge_val();
                for (int i = 0; i < d; ++i) cmax = fmax(cmax, (double)gp[((size_t)i * d + col) * 2]);
                yexp[nt] = cmax > -__builtin_huge_val() ? ceil(cmax * kLog2e) : 0.0;
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * mt + 4 * v + g;
                        double val = 0.0;
                        if (row < d) {
                            const IO *e = gp + ((size_t)row * d + col) * 2;
                            const double t = (double)e[0] * kLog2e - yexp[nt];
                            val = t > -1000.0 ? exp2(t) : 0.0;
                            if ((int)rint((double)e[1] * 0.318309886183790671538) & 1) val = -val;
                        }
                        Y[nt][mt][v] = val;
                    }
            }
        }
    }

    auto store_carry = [&](long long cc) {
        unsigned char *dst = a.carries + (b * (a.C + 1) + cc) * a.car_stride;
        double *mp = reinterpret_cast<double *>(dst);
        double *ep = reinterpret_cast<double *>(dst + car_mant);
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            const int col = 16 * nt + c;
            if (col < a.car_cols) {
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * mt + 4 * v + g;
                        mp[(size_t)row * a.car_cols + col] = (row < d && col < d) ? Y[nt][mt][v] : 0.0;
                    }
                if (g == 0) ep[col] = col < d ? yexp[nt] : 0.0;
            }
        }
    };

    // chunk product cc: mantissas as pieces of four doubles (row = piece / (DP / 4)), and its common exponent
    auto total_ptr = [&](long long cc) { return a.totals + (b * a.C + cc) * a.tot_stride; };
    auto load_piece = [&](const unsigned char *tp, int q) {
        const int piece = lane + 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
        return *reinterpret_cast<const d4 *>(reinterpret_cast<const double *>(tp) + (size_t)row * a.tot_cols + c4);
    };
    auto tile_piece = [&](double *tile, int q, d4 val) {
        const int piece = lane + 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
        const int p4 = (c4 & ~15) | ((c4 >> 2) & 3);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double x = val[e];
            if (row >= d || c4 + e >= d) x = (c4 + e == row) ? 1.0 : 0.0; // identity block past d
            tile[row * LDT + p4 + 4 * e] = x;
        }
    };

    // QR of Z in place (Z <- Q).  The growth it removes, ln R_kk + ln 2 * (exponent of column k), is kept as a
    // running product of pivots (mantissa and binary exponent apart) plus a sum of exponents, so that no logarithm
    // is taken inside the chain of chunks.
    auto qr_in_place = [&](d4 (&Z)[KT][KT], const double (&colexp)[KT]) {
        double piv[KT], piv2[KT], ce[KT], ce2[KT];
        const double amp = qr_panels_d<DP>(Z, piv, ce, s, g, c, false);
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            piv2[nt] = 1.0;
            ce2[nt] = 0.0;
        }
        // The factor Q comes out with errors of about amp 2^-53 relative to its columns' norms (amp: the squared
        // condition number).  For complex64 states, which are rounded to float, that is repaired by a second
        // factorisation from amp = 1e10 on; complex128 states take the second factorisation from 1e3 on.
        if (amp > (sizeof(IO) == 4 ? 1.0e10 : 1.0e3)) (void)qr_panels_d<DP>(Z, piv2, ce2, s, g, c, true);
#pragma unroll
        for (int nt = 0; nt < KT; ++nt)
            if (piv[nt] > 1.0e-280 && piv2[nt] > 1.0e-280) {
                int e;
                pprod[nt] = frexp(pprod[nt] * piv[nt] * piv2[nt], &e);
                pexp[nt] += 2.0 * (colexp[nt] + ce[nt] + ce2[nt]) + (double)e;
            }
    };

    d4 tq[PREFETCH ? TQ : 1];
    double tex_next = 0.0;
    if (PREFETCH && a.C > 0) {
        const unsigned char *tp = total_ptr(0);
        tex_next = *reinterpret_cast<const double *>(tp + tot_mant);
#pragma unroll
        for (int q = 0; q < TQ; ++q) tq[q] = load_piece(tp, q);
    }

    for (long long cc = 0; cc < a.C; ++cc) {
        store_carry(cc);
        double tex = tex_next;
        double *tile = s.tile;
        if (PREFETCH) {
#pragma unroll
            for (int q = 0; q < TQ; ++q) tile_piece(tile, q, tq[q]);
        } else { // (64-wide: the registers are taken by the state; the chunk product goes straight to LDS)
            const unsigned char *tp = total_ptr(cc);
            tex = *reinterpret_cast<const double *>(tp + tot_mant);
#pragma unroll 4
            for (int q = 0; q < TQ; ++q) tile_piece(tile, q, load_piece(tp, q));
        }
        wave_sync();
        if (PREFETCH && cc + 1 < a.C) {
            const unsigned char *tp = total_ptr(cc + 1);
            tex_next = *reinterpret_cast<const double *>(tp + tot_mant);
#pragma unroll
            for (int q = 0; q < TQ; ++q) tq[q] = load_piece(tp, q);
        }
        // ---- Z = T_c Y
        d4 Z[KT][KT];
#pragma unroll
        for (int nt = 0; nt < KT; ++nt)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) Z[nt][mt] = d4{0., 0., 0., 0.};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const d4 av = *reinterpret_cast<const d4 *>(&tile[(16 * mt + c) * LDT + 16 * kt + 4 * g]);
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int nt = 0; nt < KT; ++nt) Z[nt][mt] = mfma8(av[v], Y[nt][kt][v], Z[nt][mt]);
            }
        wave_sync(); // the tile is free again
        double zexp[KT];
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) zexp[nt] = yexp[nt] + tex;

        const long long t_end = (cc + 1) * a.L; // 1-based step this chunk ends at (if it is a full chunk)
        const bool boundary = t_end <= a.T && a.policy >= 0;
        bool did_reset = false;
        if (boundary) {
            did_reset = a.policy == 1;
            if (!did_reset) {
                // squared cosines between columns, tile by tile of the Gram matrix: any pair above the threshold?
#pragma unroll
                for (int nt = 0; nt < KT; ++nt) {
                    d4 Gd = {0., 0., 0., 0.};
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int v = 0; v < 4; ++v) Gd = mfma8(Z[nt][kt][v], Z[nt][kt][v], Gd);
                    // G[j][j] for column j = 16 nt + c sits in lane (c % 4, c), register c / 4
                    double dsel = Gd[0];
                    dsel = (c >> 2) == 1 ? Gd[1] : dsel;
                    dsel = (c >> 2) == 2 ? Gd[2] : dsel;
                    dsel = (c >> 2) == 3 ? Gd[3] : dsel;
                    if (g == (c & 3)) s.diag[16 * nt + c] = dsel;
                }
                wave_sync();
                bool hit = false;
                const double thr2 = (double)a.cos_threshold * (double)a.cos_threshold;
#pragma unroll
                for (int nt = 0; nt < KT; ++nt) {
                    const double dc = s.diag[16 * nt + c];
#pragma unroll
                    for (int mt = 0; mt <= nt; ++mt) {
                        d4 Gt = {0., 0., 0., 0.}; // rows: columns 16 mt + .. of Z, columns: 16 nt + c
#pragma unroll
                        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                            for (int v = 0; v < 4; ++v) Gt = mfma8(Z[mt][kt][v], Z[nt][kt][v], Gt);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int row = 16 * mt + 4 * v + g, col = 16 * nt + c;
                            const double dr = s.diag[row];
                            const double x = Gt[v];
                            if (row < col && col < d && x * x > thr2 * dr * dc) hit = true;
                        }
                    }
                }
                wave_sync();
                did_reset = __builtin_amdgcn_ballot_w64(hit) != 0;
            }
        }
        if (did_reset) {
            qr_in_place(Z, zexp);
#pragma unroll
            for (int nt = 0; nt < KT; ++nt) {
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) Y[nt][mt] = Z[nt][mt];
                yexp[nt] = 0.0;
            }
        } else {
            // Y <- Z with every column renormalised by a power of two
#pragma unroll
            for (int nt = 0; nt < KT; ++nt) {
                double mx = 0.0;
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) mx = fmax(mx, fabs(Z[nt][mt][v]));
                mx = fmax(mx, __shfl_xor(mx, 16, 64));
                mx = fmax(mx, __shfl_xor(mx, 32, 64));
                int ex = 0;
                if (mx > 0.0) (void)frexp(mx, &ex);
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) Y[nt][mt][v] = ldexp(Z[nt][mt][v], -ex);
                yexp[nt] = zexp[nt] + (double)ex;
            }
        }
        if (lane == 0) a.chunk_flags[b * a.C + cc] = did_reset ? 1 : 0;
    }

    store_carry(a.C); // the final state

    // ---- growth of the final state (factorised, not replaced)
    if (a.growth) {
        d4 Z[KT][KT];
#pragma unroll
        for (int nt = 0; nt < KT; ++nt)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) Z[nt][mt] = Y[nt][mt];
        qr_in_place(Z, yexp);
        if (g == 0) {
#pragma unroll
            for (int nt = 0; nt < KT; ++nt)
                if (16 * nt + c < d) a.growth[b * d + 16 * nt + c] = 0.5 * (log(pprod[nt]) + pexp[nt] * kLn2) * a.growth_scale;
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// The carry kernel where every boundary is reset (policy "always") and d <= 64.  Panel p of a state depends on the panels
// before it at the same boundary and on itself at the boundary before: Z_p = T_c Q_p, then Z_p made orthogonal to
// Q_0 .. Q_{p-1}, then its own factorisation.  So a workgroup gives a wave to every panel and runs them as
// stages of a pipeline, wave p at chunk s - p in stage s; the chain's pace is the last wave's stage and not the whole
// factorisation.  Finished panels pass through LDS: panel q of a chunk is read up to KT - 1 - q stages after it was written, so a
// ring of KT of them serves (one for the last panel, which only its own wave reads).
//
// The arithmetic is reset_carry_kernel's, operation for operation: a late column of 128 steps can be 10^-8 of its norm off the
// others, and what rounding leaves of it then moves the spectrum's tenth digit (both are 9e-10 off sequential QR
// there), so results stay the same only if every bit does.  That includes when a state is factored a second time, which its worst column
// decides and which replaces all panels: known only when the last wave is done with the chunk, KT - 1 stages after
// the first.  The pipeline goes on as if there were none; when there is one, what was begun since is dropped, the chunk
// goes through the waves a second time (each has its panel of the first in the ring) and those after it follow.  Growth is
// booked once the decision is there.
//
// Rows and columns past d are zero throughout: a zero pivot leaves a zero column, and nothing of it reaches the others.
//
// Bound by the last wave's chain of dependent instructions and double matrix instructions (64 cycles each): product, two projections,
// Gram matrix and rows, sixteen pivots, scaling.
// Carries of 512 chunks of 32 x 32: 4.34 -> 2.55 ms (0.2 of it second factorisations), one wave with a whole state having
// taken 20 400 cycles a chunk.  Whole spectra: 14 000 steps of 64 x 64 12.1 -> 1.89 ms, complex128 50 x 50 12.1 -> 2.03, complex128
// 65 536 of 32 x 32, where nearly every chunk is factored twice (three stages a chunk instead of one), 7.5 -> 5.9.
//
// SEG: the spectrum of a long chain.  Its stages are a serial chain, but the growth is the diagonal of one triangular factor: that of
// the whole chain's product times the initial state, and this can be put together from pieces.  Each segment of the chunks is walked by a workgroup of its
// own, and what it keeps is its product as Q_e R Q_s^T: the states at its ends and the product of its triangular factors, R = diag(2^E) N, on exponents of
// its rows (R's entries lie e^+-1000 apart).  segment_join_kernel makes one of two.  R is put together by a wave beside the panels' waves, a
// stage behind the decision about a chunk, from the projections' coefficients and the panels' triangles that they leave in LDS.
// Twice: joined from segments that begin at the identity, the growth has lost what the joins magnify (weakly separated directions, I + 0.15 N(0, 1) /
// sqrt(32), 128 chunks of 8 steps: 3e-13 of growth, 4e-14 in order), and the more the longer it takes the states to come close to the chain's.  But the
// chain's states at the segments' ends come out good to 1e-7 and better, and from these the second pass's joins magnify nothing: 4e-14.
// Error against extended precision, in order -> so, the worst of three chains: 8 x 8 3.7e-14 -> 6.4e-14, 16 x 16 6.6e-14 -> 5.6e-14, 32 x 32 4.8e-14 -> 4.4e-14,
// Lorenz-96 of d = 32, 96 chunks of 64 8.6e-11 -> 5.9e-11.
// 512 chunks of 32 x 32: 2532 -> 550 us (two walks of 64 segments 63 each, twelve joins of 34); whole spectra, T = 65 536: 2.80 -> 0.83 ms; 128 chunks 626 ->
// 417 us, 96 of them 478 -> 415, complex128 (nearly every chunk factored twice) 1138 -> 610, 64 of these 768 -> 528; but complex64 64 chunks 362 -> 387.
// Chains that do not join (directions that grow alike and turn) are found out in the first joins and walked in order: 128 chunks 615 -> 812 us, 512 of
// them 2390 -> 2590.
constexpr int kTriSlots = 5; // four chunks, and a second factorisation
constexpr long long kSegmentChunks = 8;
template <int DP, bool SEG = false> constexpr size_t staged_lds()
{
    constexpr int KT = DP / 16;
    return (((size_t)((KT - 1) * KT + 1) * DP + DP) * kPanelLd + KT * DP * 2 + 4 + (SEG ? kTriSlots * (3 * 16 * kPanelLd + DP) + DP : 0)) * sizeof(double);
}
// a segment's results: Q_s, N, Q_e (DP x DP), E, its growth (of the first one, from its true start), whether it is of no use
template <int DP> constexpr int segment_room() { return 3 * DP * DP + 2 * DP + 2; }
template <int DP> constexpr int kSegmentLost = 3 * DP * DP + 2 * DP;

template <int DP, typename IO, bool SEG = false> __global__ __launch_bounds__(DP * 4 + (SEG ? 64 : 0)) void reset_carry_staged_kernel(ResetArgs a)
{
    static_assert(!SEG || DP <= 32, "two panels at most");
    constexpr int KT = DP / 16, PANEL = DP * kPanelLd;
    extern __shared__ __align__(32) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int p = __builtin_amdgcn_readfirstlane(tid >> 6); // this wave's panel
    const int g = lane >> 4, c = lane & 15;
    const int pc = ((c & 3) << 2) | (c >> 2);
    const int d = a.d, col = 16 * p + c;
    const long long b = SEG ? blockIdx.x / a.segments : blockIdx.x;
    if (a.only_if && !a.only_if[b]) return; // the whole workgroup
    const int segment = SEG ? (int)(blockIdx.x % a.segments) : 0;
    const bool last_segment = !SEG || segment + 1 == a.segments;
    const long long begin = SEG ? segment * a.per_segment : 0;
    const size_t tot_mant = (size_t)DP * a.tot_cols * sizeof(double);
    const size_t car_mant = (size_t)DP * a.car_cols * sizeof(double);
    auto slot = [&](int q, long long i) { return reinterpret_cast<double *>(smem) + (size_t)(q * KT + (q + 1 < KT ? (int)(i & (KT - 1)) : 0)) * PANEL; };
    double *gram = reinterpret_cast<double *>(smem) + (size_t)((KT - 1) * KT + 1) * PANEL + p * 16 * kPanelLd;
    // of the chunks that are not decided yet: a column's pivot and the exponents taken out of it
    d2 *undecided = reinterpret_cast<d2 *>(reinterpret_cast<double *>(smem) + (size_t)((KT - 1) * KT + 1) * PANEL + DP * kPanelLd);
    int *worst = reinterpret_cast<int *>(undecided + KT * DP); // [2][KT]: does a chunk's state have to be factored again, so far as waves 0 .. p know
    // SEG: per slot the triangular factor's blocks (0, 0), (1, 1), (0, 1) and its columns' exponents; E
    [[maybe_unused]] double *tri = reinterpret_cast<double *>(worst) + 4;
    auto tri_block = [&](int sl, int q) { return tri + (size_t)(sl * 3 + q) * 16 * kPanelLd; };
    [[maybe_unused]] double *tri_exp = tri + (size_t)kTriSlots * 3 * 16 * kPanelLd; // [slot][DP]
    [[maybe_unused]] double *row_exp = tri_exp + kTriSlots * DP;
    [[maybe_unused]] double *room = SEG ? a.segments_room + (size_t)blockIdx.x * segment_room<DP>() : nullptr;
    [[maybe_unused]] const double *frame = SEG && a.frames && segment > 0 ? a.frames + ((size_t)blockIdx.x - 1) * segment_room<DP>() : nullptr;
    if constexpr (SEG) {
        if (frame && frame[kSegmentLost<DP>] != 0.0) { // the whole workgroup
            if (tid == 0) room[kSegmentLost<DP>] = 1.0;
            return;
        }
    }

    d4 Y[KT]; // Y[mt][v] = entry (row 16 mt + 4 v + g, column 16 p + c), columns scaled by 2^yexp
    double yexp = 0.0, pprod = 1.0, pexp = 0.0; // product of all pivots so far = pprod 2^pexp (column exponents counted twice)
#pragma unroll
    for (int mt = 0; mt < KT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) Y[mt][v] = (16 * mt + 4 * v + g == col && col < d) ? 1.0 : 0.0;
    if constexpr (SEG) {
        if (frame && p < KT) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) Y[mt][v] = frame[2 * DP * DP + (16 * mt + 4 * v + g) * DP + col];
        }
    }
    if (a.s0 && col < d && segment == 0) {
        const IO *gp = reinterpret_cast<const IO *>(a.s0) + (size_t)b * d * d * 2;
        double cmax = -__builtin_huge_val();
        for (int i = 0; i < d; ++i) cmax = fmax(cmax, (double)gp[((size_t)i * d + col) * 2]);
        yexp = cmax > -__builtin_huge_val() ? ceil(cmax * kLog2e) : 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                double val = 0.0;
                if (row < d) {
                    const IO *e = gp + ((size_t)row * d + col) * 2;
                    const double t = (double)e[0] * kLog2e - yexp;
                    val = t > -1000.0 ? exp2(t) : 0.0;
                    if ((int)rint((double)e[1] * 0.318309886183790671538) & 1) val = -val;
                }
                Y[mt][v] = val;
            }
    }
    auto carry = [&](long long i) { return a.carries + (b * (a.C + 1) + i) * a.car_stride; };
    if (a.carries) { // the state that enters the first chunk
        double *mp = reinterpret_cast<double *>(carry(0));
        if (col < a.car_cols) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) mp[(size_t)(16 * mt + 4 * v + g) * a.car_cols + col] = Y[mt][v];
            if (g == 0) reinterpret_cast<double *>(carry(0) + car_mant)[col] = yexp;
        }
    }
    // later ones from rows: lane r holds row r of the panel
    auto store_carry = [&](long long i, const double (&rows)[1][16]) {
        if (16 * p < a.car_cols) {
            double *mp = reinterpret_cast<double *>(carry(i)) + (size_t)lane * a.car_cols + 16 * p;
            if (lane < DP) {
#pragma unroll
                for (int j = 0; j < 16; j += 2) *reinterpret_cast<d2 *>(mp + j) = d2{rows[0][j], rows[0][j + 1]};
            }
            if (g == 0) reinterpret_cast<double *>(carry(i) + car_mant)[col] = yexp;
        }
    };

    // The next chunk product.  d <= 32: as operands, row 16 mt + c, columns 16 kt + 4 v + g.  d <= 64: a row's 128 bytes by eight
    // lanes (as operands each load touches sixteen lines, and four waves' loads kept the memory pipe busy for half a stage).
    constexpr bool SLICES = DP > 32;
    double tq[KT][KT][4];
    double tex;
    const unsigned lane_at = (unsigned)((SLICES ? (lane >> 3) * a.tot_cols + 2 * (lane & 7) : c * a.tot_cols + g) * sizeof(double));
    auto load_total = [&](long long i) {
        const unsigned char *tp = a.totals + (b * a.C + i) * a.tot_stride;
        tex = *reinterpret_cast<const double *>(tp + tot_mant);
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const int at = 16 * kt < a.tot_cols ? 16 * kt : 0;
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
                if constexpr (SLICES) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) { // (one base for the wave, one offset for the lane)
                        const d2 x = *reinterpret_cast<const d2 *>(tp + (size_t)((16 * mt + 8 * h) * a.tot_cols + at) * sizeof(double) + lane_at);
                        tq[mt][kt][2 * h] = x[0];
                        tq[mt][kt][2 * h + 1] = x[1];
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        tq[mt][kt][v] = *reinterpret_cast<const double *>(tp + (size_t)(16 * mt * a.tot_cols + at + 4 * v) * sizeof(double) + lane_at);
                }
        }
    };
    auto clear_past_d = [&]() {
        if (d != DP) {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = SLICES ? 16 * mt + 8 * (v >> 1) + (lane >> 3) : 16 * mt + c, k = 16 * kt + (SLICES ? 2 * (lane & 7) + (v & 1) : 4 * v + g);
                        if (row >= d || k >= d) tq[mt][kt][v] = 0.0;
                    }
        }
    };

    // a finished panel: rows 16 mt + 4 v + g of column c, and, negated, row 16 mt + c, columns 4 v + g
    d4 qt[KT];
    d2 qa[KT][2];
    auto load_panel = [&](int q, long long i) {
        const double *pq = slot(q, i);
        panel_tiles<DP>(qt, pq, g, c);
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int h = 0; h < 2; ++h) qa[mt][h] = -*reinterpret_cast<const d2 *>(&pq[(16 * mt + c) * kPanelLd + 4 * g + 2 * h]);
    };
    // Q of Z (in the matrix instruction's layout) to `out` and, as rows, to `rows`; the columns' pivots and exponents.  Returns whether
    // one of the columns asks for a second factorisation (see qr_panels_d and its callers).
    auto factor = [&](d4 (&Z)[KT], long long i, double *out, double (&rows)[1][16], double &piv, double &expo, bool second) {
        [[maybe_unused]] d4 coefficients = {0., 0., 0., 0.};
        auto project = [&]() {
            d4 R = {0., 0., 0., 0.};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) R = mfma8(qt[kt][v], Z[kt][v], R);
            if constexpr (SEG) coefficients += R;
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) Z[mt] = mfma8(qa[mt][v >> 1][v & 1], R[v], Z[mt]);
        };
        const int ex = column_exponent(Z);
        expo = (double)ex;
        double norm2 = 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Z[mt][v] = ldexp(Z[mt][v], -ex);
                norm2 = fma(Z[mt][v], Z[mt][v], norm2);
            }
        norm2 = column_sum(norm2);
        // orthogonal to the finished panels, twice (see qr_panels_d)
#pragma unroll 1
        for (int rep = 0; rep < 2; ++rep)
#pragma unroll 1
            for (int q = 0; q < p; ++q) {
                if (KT > 2) load_panel(q, i);
                project();
            }
        const int sl = second ? kTriSlots - 1 : (int)(i & 3);
        if constexpr (SEG) {
            if (p > 0) {
                double *t = tri_block(sl, 2);
#pragma unroll
                for (int v = 0; v < 4; ++v) t[(4 * v + g) * kPanelLd + c] = coefficients[v];
            }
        }
        const bool open = factor_panel_rows<DP, SEG>(Z, piv, out, gram, rows, lane, second, SEG ? tri_block(sl, p) : nullptr);
        return open || __builtin_amdgcn_ballot_w64(piv > 1.0e-280 && norm2 > (sizeof(IO) == 4 ? 1.0e10 : 1.0e3) * piv) != 0;
    };
    // growth as in reset_carry_kernel (a column that is zero has none)
    auto grow = [&](double first, double second, double expo) {
        if (first > 1.0e-280 && second > 1.0e-280) {
            int e;
            pprod = frexp(pprod * first * second, &e);
            pexp += 2.0 * expo + (double)e;
        }
    };

    load_total(begin);
    // (the last one: growth of the final state, factorised, not replaced)
    const long long items = last_segment ? a.C + (a.growth ? 1 : 0) : (segment + 1) * a.per_segment;
    // SEG: N in the matrix instruction's layout, E in LDS
    [[maybe_unused]] d4 N[KT][KT];
    [[maybe_unused]] bool lost = false;
    if constexpr (SEG) {
        if (p == KT) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int nt = 0; nt < KT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) N[kt][nt][v] = kt == nt && 4 * v + g == c ? 1.0 : 0.0;
            if (lane < DP) row_exp[lane] = 0.0;
            wave_sync();
        }
    }
    // N <- R N, rows on exponents of their own
    auto accumulate = [&](int sl) {
        double rv[KT][KT][4], ek[KT][4], top[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) ek[kt][v] = row_exp[16 * kt + 4 * v + g] + tri_exp[sl * DP + 16 * kt + 4 * v + g];
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) {
            top[mt] = -1.0e300;
#pragma unroll
            for (int kt = mt; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    rv[mt][kt][v] = tri_block(sl, mt == kt ? mt : 2)[c * kPanelLd + 4 * v + g];
                    if (rv[mt][kt][v] != 0.0) {
                        int e;
                        (void)frexp(rv[mt][kt][v], &e);
                        top[mt] = fmax(top[mt], (double)e + ek[kt][v]);
                    }
                }
            top[mt] = fmax(top[mt], __shfl_xor(top[mt], 16, 64));
            top[mt] = fmax(top[mt], __shfl_xor(top[mt], 32, 64));
            const bool empty = !(top[mt] > -1.0e299);
            lost = lost || (empty && 16 * mt + c < d);
            if (empty) top[mt] = 0.0;
        }
        wave_sync();
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) {
            if (g == 0) row_exp[16 * mt + c] = top[mt];
#pragma unroll
            for (int kt = mt; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) rv[mt][kt][v] = ldexp(rv[mt][kt][v], (int)fmax(ek[kt][v] - top[mt], -4000.0));
        }
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) // (upper triangular: the rows below a row's block are the old ones still)
#pragma unroll
            for (int nt = mt; nt < KT; ++nt) {
                d4 sum = {0., 0., 0., 0.};
#pragma unroll
                for (int kt = mt; kt <= nt; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum = mfma8(rv[mt][kt][v], N[kt][nt][v], sum);
                N[mt][nt] = sum;
            }
        wave_sync();
    };
    // wave p is at chunk from + n - p in stage n since the last (re)start, which begins with the second factorisation of chunk `from` if `redo`
    long long from = begin, n = 0;
    bool redo = false;
    int pending = -1; // SEG: the slot of a factor that has been decided
    double redo_piv = 1.0, redo_expo = 0.0; // pivots and exponents of that chunk's first factorisation
    d2 own; // what this wave has left in `undecided` last
    bool hit = false;
    for (int stage = 0;; stage ^= 1, ++n) {
        const long long i = from + n - p;
        const bool second = redo && i == from;
        if constexpr (SEG) {
            if (p == KT && pending >= 0) accumulate(pending);
            pending = -1;
            if (p < KT && n >= p && i == begin && !second && segment > 0) {
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) room[(16 * mt + 4 * v + g) * DP + col] = Y[mt][v];
            }
        }
        if ((!SEG || p < KT) && n >= p && i < items) { // (the same for the whole wave)
            double *out = slot(p, i);
            double rows[1][16], piv, expo, zexp = yexp;
            d4 Z[KT];
            hit = false;
            const bool boundary = i == a.C || (i + 1) * a.L <= a.T; // (a last, shorter chunk ends at no boundary)
            if (KT == 2 && p > 0) load_panel(0, i); // (it is there since the stage before)
            if (second) {
                panel_tiles<DP>(Z, out, g, c);
            } else if (i < a.C) {
                zexp = yexp + tex;
                clear_past_d();
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) Z[mt] = d4{0., 0., 0., 0.};
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    double ta[KT][4];
                    if constexpr (SLICES) { // (sixteen columns at a time through this panel's own place, column j at position perm16(j))
                        const int j = 2 * (lane & 7), pj = ((j & 3) << 2) | (j >> 2); // (column j + 1: four places on)
                        wave_sync();
#pragma unroll
                        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                            for (int v = 0; v < 4; ++v) out[(16 * mt + 8 * (v >> 1) + (lane >> 3)) * kPanelLd + pj + 4 * (v & 1)] = tq[mt][kt][v];
                        wave_sync();
                    }
#pragma unroll
                    for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const d2 x = SLICES ? *reinterpret_cast<const d2 *>(&out[(16 * mt + c) * kPanelLd + 4 * g + 2 * h]) : d2{tq[mt][kt][2 * h], tq[mt][kt][2 * h + 1]};
                            ta[mt][2 * h] = x[0];
                            ta[mt][2 * h + 1] = x[1];
                        }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int mt = 0; mt < KT; ++mt) Z[mt] = mfma8(ta[mt][v], Y[kt][v], Z[mt]);
                }
            } else {
                panel_tiles<DP>(Z, slot(p, i - 1), g, c);
            }
            load_total(i + 1 < a.C ? i + 1 : a.C - 1); // (in one place: loads in several would be copied together, and waited for, where they meet)
            if (boundary) {
                hit = factor(Z, i, out, rows, piv, expo, second);
                if constexpr (SEG) {
                    if (g == 0) tri_exp[(second ? kTriSlots - 1 : (int)(i & 3)) * DP + col] = second ? expo : zexp + expo;
                }
                if (second) {
                    grow(redo_piv, piv, redo_expo + expo);
                } else {
                    own = d2{piv, zexp + expo};
                    if (KT > 1 && g == 0) undecided[(i & (KT - 1)) * DP + col] = own;
                }
                if (i < a.C) yexp = 0.0;
            } else { // columns renormalised by a power of two
                const int ex = column_exponent(Z);
                yexp = col < d ? zexp + (double)ex : 0.0;
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) out[(16 * mt + 4 * v + g) * kPanelLd + pc] = ldexp(Z[mt][v], -ex);
                wave_sync();
#pragma unroll
                for (int j = 0; j < 16; ++j) rows[0][j] = out[(lane & (DP - 1)) * kPanelLd + (((j & 3) << 2) | (j >> 2))];
            }
            if (i < a.C) {
                panel_tiles<DP>(Y, out, g, c);
                if (a.carries) store_carry(i + 1, rows);
                if (tid == 0) a.chunk_flags[b * a.C + i] = boundary ? 1 : 0;
            }
            if ((KT > 1 || SEG) && lane == 0) worst[stage * KT + p] = (hit && !second) || (p > 0 && !second && worst[(stage ^ 1) * KT + p - 1]);
        }
        // (LDS only: the loads of the next chunk product and the stores of carries stay in flight)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        // the chunk that the last wave has finished (all waves come to the same answer)
        if (n < KT - 1) continue;
        const long long done = from + n - (KT - 1);
        if (SEG && redo && done == from && segment > 0) pending = kTriSlots - 1;
        if (!(redo && done == from) && (done == a.C || (done + 1) * a.L <= a.T)) {
            if (SEG && segment > 0) pending = (int)(done & 3);
            const d2 first = KT > 1 ? (!SEG || p < KT ? undecided[(done & (KT - 1)) * DP + col] : d2{1.0, 0.0}) : own;
            if (KT > 1 || SEG ? __builtin_amdgcn_readfirstlane(worst[stage * KT + KT - 1]) != 0 : hit) {
                from = done;
                n = -1;
                redo = true;
                redo_piv = first[0];
                redo_expo = first[1];
                yexp = 0.0;
                continue;
            }
            grow(first[0], 1.0, first[1]);
        }
        if (done + 1 == items) break;
    }
    if constexpr (SEG) {
        if (p == KT) {
            if (pending >= 0) accumulate(pending);
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int nt = 0; nt < KT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) room[DP * DP + (16 * mt + 4 * v + g) * DP + 16 * nt + c] = N[mt][nt][v];
            if (lane < DP) room[3 * DP * DP + lane] = row_exp[lane];
            const bool any = __builtin_amdgcn_ballot_w64(lost) != 0;
            if (lane == 0) room[kSegmentLost<DP>] = any ? 1.0 : 0.0;
        } else {
#pragma unroll
            for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) room[2 * DP * DP + (16 * mt + 4 * v + g) * DP + col] = Y[mt][v];
            if (g == 0) room[3 * DP * DP + DP + col] = col < d ? 0.5 * (log(pprod) + pexp * kLn2) : 0.0;
        }
    } else if (a.growth && g == 0 && col < d) {
        a.growth[b * d + col] = 0.5 * (log(pprod) + pexp * kLn2) * a.growth_scale;
    }
}

// sum over the eight lanes that share a row (column) below
__device__ inline double eight_sum(double x)
{
    auto moved = [](double v, auto ctrl) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffull), decltype(ctrl)::value, 0xf, 0xf, true);
        const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
    };
    x += moved(x, std::integral_constant<int, 0xB1>{});  // quad_perm [1,0,3,2]
    x += moved(x, std::integral_constant<int, 0x4E>{});  // quad_perm [2,3,0,1]
    x += moved(x, std::integral_constant<int, 0x141>{}); // row_half_mirror
    return x;
}
__device__ inline double eight_max(double x)
{
#pragma unroll
    for (int s = 1; s < 8; s <<= 1) x = fmax(x, __shfl_xor(x, s, 64));
    return x;
}

// Two neighbouring segments of reset_carry_staged_kernel<., ., true> become one (a tree of launches makes one of all).  With Q_s, E, N, Q_e of the first (1) and
// of the second (2),
//     Q_e2 diag(2^E2) N2 W diag(2^E1) N1 Q_s1^-1,  Q_s2 W = Q_e1,
// and what is needed is the triangular factorisation of diag(2^E2) N2 W, whose rows lie e^+-1000 apart: from the columns as they are, everything
// below the largest rows would be rounding.  N2 W = L U without exchanges first; then
//     diag(2^E2) L U = (diag(2^E2) L diag(2^-E2)) diag(2^E2) U,
// where the bracket is 1 on the diagonal, small below it where the exponents are in order (they are, but for directions of nearly equal
// growth), and is factored by columns, Q' R'.  An error of U's is magnified as L's entries are large: in the first pass, from the identity, up to
// 1e9 times, which leaves the states at the ends good to some digits (out: every segment joined with the one `stride` before it, so that the
// tree gives them at all ends).  In the second, where Q_s2 is such a state, L is the identity to 1e-7 and better, and is refused beyond `limit`; as
// it is where a segment has lost a row (singular chunks): the chain is walked in order after all.  For what begins with the chain's first segment
// only the growth counts: the diagonals' logarithms.  One workgroup a pair, eight threads a row.  Bound by the 2 d dependent steps of the two
// factorisations.
template <int DP> __global__ __launch_bounds__(DP * 8) void segment_join_kernel(ResetArgs a, double *out, int stride, double limit, int *again)
{
    constexpr int LD = DP + 1, W = DP / 8, KT = DP / 16;
    __shared__ double X[DP * LD], Y[DP * LD], Z[DP * LD], low[DP * LD], rest[DP * LD];
    __shared__ double E1[DP], E2[DP];
    __shared__ int bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = tid >> 3, s = tid & 7, d = a.d;
    const int g = lane >> 4, c = lane & 15;
    const int pairs = out ? a.segments : (a.segments - stride + 2 * stride - 1) / (2 * stride);
    const long long b = blockIdx.x / pairs;
    const int first = out ? (int)(blockIdx.x % pairs) - stride : (int)(blockIdx.x % pairs) * 2 * stride;
    const bool from_start = out ? first < stride : first == 0; // what the first segment stands for begins where the chain does
    double *room1 = a.segments_room + ((ptrdiff_t)b * a.segments + first) * segment_room<DP>();
    const double *room2 = room1 + (ptrdiff_t)stride * segment_room<DP>();
    double *to = out ? out + (size_t)blockIdx.x * segment_room<DP>() : room1;
    if (first < 0) { // (the chain's state at this end is there)
        for (int m = 0; m < W; ++m) to[2 * DP * DP + r * DP + s + 8 * m] = room2[2 * DP * DP + r * DP + s + 8 * m];
        if (tid == 0) to[kSegmentLost<DP>] = room2[kSegmentLost<DP>];
        return;
    }
    const bool last_pair = !out && first == 0 && 2 * stride >= a.segments;
    auto fetch = [&](double *to, const double *from) {
        for (int m = 0; m < W; ++m) to[r * LD + s + 8 * m] = from[r * DP + s + 8 * m];
    };
    // C <- base + sign * A B (or A^T B); a wave a tile
    auto multiply = [&](double *C, const double *base, double sign, const double *A, bool transposed, const double *B) {
        if (wave < KT * KT) {
            const int mt = wave / KT, nt = wave % KT;
            d4 sum = {0., 0., 0., 0.};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int k = 16 * kt + 4 * v + g, i = 16 * mt + c;
                    sum = mfma8(transposed ? A[k * LD + i] : A[i * LD + k], B[k * LD + 16 * nt + c], sum);
                }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = (16 * mt + 4 * v + g) * LD + 16 * nt + c;
                C[at] = base ? base[at] + sign * sum[v] : sum[v];
            }
        }
        __syncthreads();
    };
    fetch(Y, room2);                   // Q_s2
    fetch(Z, room1 + 2 * DP * DP);     // Q_e1
    fetch(low, room2 + DP * DP);       // N2
    if (tid < DP) {
        E2[tid] = room2[3 * DP * DP + tid];
        E1[tid] = room1[3 * DP * DP + tid];
    }
    if (tid == 0) bad = room1[kSegmentLost<DP>] != 0.0 || room2[kSegmentLost<DP>] != 0.0;
    __syncthreads();
    if (bad) { // the whole workgroup
        if (tid == 0) {
            to[kSegmentLost<DP>] = 1.0;
            if (last_pair) again[b] = 1;
        }
        return;
    }
    // W: Q_s2^T Q_e1, and corrected twice (states of complex64 chains are orthonormal to 1e-6 only, where a chunk was not factored twice)
    multiply(X, nullptr, 1.0, Y, true, Z);
    for (int turn = 0; turn < 2; ++turn) {
        multiply(rest, Z, -1.0, Y, false, X);
        multiply(X, X, 1.0, Y, true, rest);
    }
    multiply(Z, nullptr, 1.0, low, false, X); // N2 W
    for (int m = 0; m < W; ++m) low[r * LD + s + 8 * m] = 0.0;
    __syncthreads();
    // Z = L U, U in place; the bracket in `low`
    bool wrong = false;
    for (int k = 0; k < d; ++k) {
        const double pivot = Z[k * LD + k];
        if (r > k && r < d) {
            const double l = Z[r * LD + k] / pivot;
#pragma unroll
            for (int m = 0; m < W; ++m)
                if (s + 8 * m > k) Z[r * LD + s + 8 * m] = fma(-l, Z[k * LD + s + 8 * m], Z[r * LD + s + 8 * m]);
            wrong = wrong || !(fabs(l) <= limit); // (also a pivot of zero)
            if (s == 0) {
                const double x = ldexp(l, (int)fmin(fmax(E2[r] - E2[k], -4000.0), 1000.0));
                wrong = wrong || !(fabs(x) <= fmax(limit, 1.0e6));
                low[r * LD + k] = x;
            }
        }
        __syncthreads();
    }
    if (s == 0) low[r * LD + r] = r < d ? 1.0 : 0.0;
    for (int m = 0; m < W; ++m) {
        const int j = s + 8 * m;
        if (j < r || r >= d) Z[r * LD + j] = 0.0;
        rest[r * LD + j] = 0.0;
    }
    if (tid < d) wrong = wrong || !(fabs(Z[tid * LD + tid]) > 0.0);
    __syncthreads();
    // the bracket's columns one after the other: Q' to X, R' to rest.  r is a column here
    for (int k = 0; k < d; ++k) {
        double n2 = 0.0, dot = 0.0, ck[W], cr[W];
#pragma unroll
        for (int m = 0; m < W; ++m) {
            ck[m] = low[(s + 8 * m) * LD + k];
            cr[m] = low[(s + 8 * m) * LD + r];
            n2 = fma(ck[m], ck[m], n2);
            dot = fma(ck[m], cr[m], dot);
        }
        n2 = eight_sum(n2);
        dot = eight_sum(dot);
        if (r >= k && r < d) {
            const double norm = sqrt(n2), f = dot / n2;
            if (s == 0) rest[k * LD + r] = f * norm;
            if (r > k) {
#pragma unroll
                for (int m = 0; m < W; ++m) low[(s + 8 * m) * LD + r] = fma(-f, ck[m], cr[m]);
            } else {
                const double inv = 1.0 / norm;
#pragma unroll
                for (int m = 0; m < W; ++m) X[(s + 8 * m) * LD + k] = ck[m] * inv;
            }
        }
        __syncthreads();
    }
    for (int m = 0; m < W; ++m)
        if (r >= d || s + 8 * m >= d) X[r * LD + s + 8 * m] = 0.0;
    if (from_start) {
        if (!out && tid < d) {
            double &growth = room1[3 * DP * DP + DP + tid];
            growth += log(fabs(Z[tid * LD + tid])) + log(rest[tid * LD + tid]) + E2[tid] * kLn2;
            if (last_pair) {
                const double x = growth * a.growth_scale;
                if (!(fabs(x) < 1.0e300)) bad = 1;
                a.growth[b * d + tid] = x;
            }
        }
    } else {
        // N1 <- R' diag(2^E2) U diag(2^E1) N1, rows on exponents of their own
        fetch(Y, room1 + DP * DP);
        for (int turn = 0; turn < 2; ++turn) {
            double *A = turn ? rest : Z;
            __syncthreads();
            double top = -1.0e300;
            for (int m = 0; m < W; ++m) {
                const int j = s + 8 * m;
                const double x = A[r * LD + j];
                if (x != 0.0) {
                    int e;
                    (void)frexp(x, &e);
                    top = fmax(top, (double)e + E1[j]);
                }
            }
            top = eight_max(top);
            const bool empty = !(top > -1.0e299);
            wrong = wrong || (empty && r < d);
            if (empty) top = 0.0;
            for (int m = 0; m < W; ++m) {
                const int j = s + 8 * m;
                A[r * LD + j] = ldexp(A[r * LD + j], (int)fmax(E1[j] - top, -4000.0));
            }
            __syncthreads();
            if (s == 0) E1[r] = top + (turn == 0 ? E2[r] : 0.0);
            multiply(turn ? Y : low, nullptr, 1.0, A, false, turn ? low : Y);
        }
        for (int m = 0; m < W; ++m) {
            to[DP * DP + r * DP + s + 8 * m] = Y[r * LD + s + 8 * m];
            if (out) to[r * DP + s + 8 * m] = room1[r * DP + s + 8 * m]; // Q_s1
        }
        if (tid < DP) to[3 * DP * DP + tid] = E1[tid];
    }
    if (wrong) bad = 1;
    __syncthreads();
    // Q_e1 <- Q_e2 Q'
    fetch(Z, room2 + 2 * DP * DP);
    __syncthreads();
    multiply(Y, nullptr, 1.0, Z, false, X);
    for (int m = 0; m < W; ++m) to[2 * DP * DP + r * DP + s + 8 * m] = Y[r * LD + s + 8 * m];
    if (tid == 0) {
        to[kSegmentLost<DP>] = bad ? 1.0 : 0.0;
        if (last_pair) again[b] = bad;
    }
}

// ---------------------------------------------------------------------------------------------------
// The carry kernel for 64 < d <= 128.  A state of 128 x 128 doubles is more than one wave's registers hold, so a
// workgroup of four waves owns a batch item, wave w the columns 32 w .. 32 w + 31 of the state (two panels of
// sixteen).  Z = T_c Y is formed slab by slab from one LDS tile of the chunk product; the factorisation then
// walks the eight panels in order: the wave that owns a panel makes it orthogonal to the finished ones (which
// lie in LDS, in the tile's place), factorises it as above and lays it down for the others.  Arithmetic, layouts
// and bookkeeping are those of the one-wave kernel.
struct WideScratch {
    double gram[16 * 18];
    double diag[128];
    double red[4];
    int hit;
};

// One factorisation of a 128 x 128 matrix held by four waves (wave w: columns 32 w .. 32 w + 31 as two panels) in
// place, Z <- Q: see qr_panels_d.  piv, cexp: pivots and column exponents of this wave's two panels.  Returns the
// largest (squared column norm) / pivot over the whole matrix, the same in every wave.  Finished panels lie in
// LDS at `panels` ([8][128][18] doubles); all four waves must call this together.
__device__ double wide_qr_pass(d4 (&Z)[2][8], double (&piv)[2], double (&cexp)[2], double *panels, WideScratch &s, int wave, int lane, bool last)
{
    constexpr int DP = 128, KT = 8, NL = 2, LDQ = 18;
    const int g = lane >> 4, c = lane & 15;
    const int pc = ((c & 3) << 2) | (c >> 2);
    auto panel = [&](int q) { return panels + (size_t)q * DP * LDQ; };
    bool open = false;
    double norm2[NL];
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        double mx = 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) mx = fmax(mx, fabs(Z[nl][mt][v]));
        mx = fmax(mx, __shfl_xor(mx, 16, 64));
        mx = fmax(mx, __shfl_xor(mx, 32, 64));
        int ex = 0;
        if (mx > 0.0) (void)frexp(mx, &ex);
        cexp[nl] = (double)ex;
        double sum = 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Z[nl][mt][v] = ldexp(Z[nl][mt][v], -ex);
                sum = fma(Z[nl][mt][v], Z[nl][mt][v], sum);
            }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        norm2[nl] = sum;
        piv[nl] = 1.0;
    }
    __syncthreads(); // (whoever still read the LDS panels or the tile is done)
    // Panel by panel: its owner factorises panel P (by then orthogonal to all finished ones) and lays it down; then
    // every wave makes those of its own panels that come later orthogonal to it, twice in a row (one projection
    // leaves rounding-level remainders of the panel's norm behind), all four waves at work at once.
    auto factor_panel = [&](int P, d4 (&Zp)[KT], double &pv) {
        double rows[2][16];
        open |= factor_panel_rows<DP>(Zp, pv, panel(P), s.gram, rows, lane, last);
        panel_tiles<DP>(Zp, panel(P), g, c);
    };
    auto project_out = [&](int P, d4 (&Zp)[KT]) {
        const double *pq = panel(P);
#pragma unroll 1
        for (int rep = 0; rep < 2; ++rep) {
            d4 R = {0., 0., 0., 0.};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) R = mfma8(pq[(16 * kt + 4 * v + g) * LDQ + pc], Zp[kt][v], R);
            R = -R;
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const d4 av = *reinterpret_cast<const d4 *>(&pq[(16 * mt + c) * LDQ + 4 * g]);
#pragma unroll
                for (int v = 0; v < 4; ++v) Zp[mt] = mfma8(av[v], R[v], Zp[mt]);
            }
        }
    };
#pragma unroll 1
    for (int P = 0; P < KT; ++P) {
        if (wave == P / NL) {
            if (P % NL == 0)
                factor_panel(P, Z[0], piv[0]);
            else
                factor_panel(P, Z[1], piv[1]);
        }
        __syncthreads();
        if (NL * wave > P) project_out(P, Z[0]);
        if (NL * wave + 1 > P) project_out(P, Z[1]);
        // (no barrier: the next panel is written elsewhere, and its owner reads nothing but its own registers before)
    }
    __syncthreads();
    double worst = 1.0;
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        const double ratio = piv[nl] > 1.0e-280 ? norm2[nl] * rcp_d(piv[nl]) : 1.0;
        worst = fmax(worst, ratio);
    }
#pragma unroll
    for (int sft = 1; sft < 16; sft <<= 1) worst = fmax(worst, __shfl_xor(worst, sft, 64));
    if (lane == 0) s.red[wave] = open ? 1.0e300 : worst;
    __syncthreads();
    worst = fmax(fmax(s.red[0], s.red[1]), fmax(s.red[2], s.red[3]));
    __syncthreads();
    return worst;
}

// Is there a pair of columns of the 128 x 128 matrix Z (held by four waves as in wide_qr_pass) whose squared cosine
// exceeds thr2?  Z goes to LDS panel by panel; every wave takes the pairs whose second column is its own.  The same
// answer in every wave; all four waves must call this together.
__device__ bool wide_colinear(const d4 (&Z)[2][8], double *panels, WideScratch &s, int wave, int lane, int d, double thr2)
{
    constexpr int DP = 128, KT = 8, NL = 2, LDQ = 18;
    const int g = lane >> 4, c = lane & 15;
    const int pc = ((c & 3) << 2) | (c >> 2);
    auto panel = [&](int q) { return panels + (size_t)q * DP * LDQ; };
    __syncthreads(); // the tile, or the panels of a factorisation, are free
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        double *pp = panel(NL * wave + nl);
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) pp[(16 * mt + 4 * v + g) * LDQ + pc] = Z[nl][mt][v];
        d4 Gd = {0., 0., 0., 0.};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int v = 0; v < 4; ++v) Gd = mfma8(Z[nl][kt][v], Z[nl][kt][v], Gd);
        // G[j][j] for column j = 16 P + c sits in lane (c % 4, c), register c / 4
        double dsel = Gd[0];
        dsel = (c >> 2) == 1 ? Gd[1] : dsel;
        dsel = (c >> 2) == 2 ? Gd[2] : dsel;
        dsel = (c >> 2) == 3 ? Gd[3] : dsel;
        if (g == (c & 3)) s.diag[32 * wave + 16 * nl + c] = dsel;
    }
    if (threadIdx.x == 0) s.hit = 0;
    __syncthreads();
    bool hit = false;
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        const int P = NL * wave + nl;
        const double dc = s.diag[16 * P + c];
        for (int q = 0; q <= P; ++q) {
            const double *pq = panel(q);
            d4 Gt = {0., 0., 0., 0.}; // rows: columns 16 q + .. of Z, columns: 16 P + c
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) Gt = mfma8(pq[(16 * kt + 4 * v + g) * LDQ + pc], Z[nl][kt][v], Gt);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * q + 4 * v + g, col = 16 * P + c;
                const double dr = s.diag[row];
                const double x = Gt[v];
                if (row < col && col < d && x * x > thr2 * dr * dc) hit = true;
            }
        }
    }
    if (__builtin_amdgcn_ballot_w64(hit) != 0 && lane == 0) s.hit = 1;
    __syncthreads();
    return s.hit != 0;
}

template <typename IO> __global__ __launch_bounds__(256) void reset_carry_wide_kernel(ResetArgs a)
{
    constexpr int DP = 128, KT = DP / 16, NL = 2, NW = 4, LDT = DP + 2, LDQ = 18;
    constexpr int TQ = DP * DP / 4 / (NW * 64); // 32-byte pieces of the chunk product per thread
    extern __shared__ __align__(32) unsigned char smem[];
    double *tile = reinterpret_cast<double *>(smem); // [128][130]: chunk product, columns in perm16 order
    auto panel = [&](int q) { return reinterpret_cast<double *>(smem) + (size_t)q * DP * LDQ; }; // [8][128][18], after the product
    WideScratch &s = *reinterpret_cast<WideScratch *>(smem + (size_t)KT * DP * LDQ * sizeof(double));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const long long b = blockIdx.x;
    const size_t tot_mant = (size_t)DP * a.tot_cols * sizeof(double);
    const size_t car_mant = (size_t)DP * a.car_cols * sizeof(double);

    d4 Y[NL][KT]; // Y[nl][mt][v] = entry (row 16 mt + 4 v + g, column 32 wave + 16 nl + c), columns scaled by 2^yexp
    double yexp[NL], pprod[NL], pexp[NL];
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        yexp[nl] = 0.0;
        pprod[nl] = 1.0;
        pexp[nl] = 0.0;
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) Y[nl][mt][v] = (16 * mt + 4 * v + g == 32 * wave + 16 * nl + c) ? 1.0 : 0.0;
    }
    if (a.s0) {
        const IO *gp = reinterpret_cast<const IO *>(a.s0) + (size_t)b * d * d * 2;
#pragma unroll
        for (int nl = 0; nl < NL; ++nl) {
            const int col = 32 * wave + 16 * nl + c;
            if (col < d) {
                double cmax = -__builtin_huge_val();
                for (int i = 0; i < d; ++i) cmax = fmax(cmax, (double)gp[((size_t)i * d + col) * 2]);
                yexp[nl] = cmax > -__builtin_huge_val() ? ceil(cmax * kLog2e) : 0.0;
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * mt + 4 * v + g;
                        double val = 0.0;
                        if (row < d) {
                            const IO *e = gp + ((size_t)row * d + col) * 2;
                            const double t = (double)e[0] * kLog2e - yexp[nl];
                            val = t > -1000.0 ? exp2(t) : 0.0;
                            if ((int)rint((double)e[1] * 0.318309886183790671538) & 1) val = -val;
                        }
                        Y[nl][mt][v] = val;
                    }
            }
        }
    }

    auto store_carry = [&](long long cc) {
        unsigned char *dst = a.carries + (b * (a.C + 1) + cc) * a.car_stride;
        double *mp = reinterpret_cast<double *>(dst);
        double *ep = reinterpret_cast<double *>(dst + car_mant);
#pragma unroll
        for (int nl = 0; nl < NL; ++nl) {
            const int col = 32 * wave + 16 * nl + c;
            if (col < a.car_cols) {
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int row = 16 * mt + 4 * v + g;
                        mp[(size_t)row * a.car_cols + col] = (row < d && col < d) ? Y[nl][mt][v] : 0.0;
                    }
                if (g == 0) ep[col] = col < d ? yexp[nl] : 0.0;
            }
        }
    };

    auto qr_pass = [&](d4 (&Z)[NL][KT], double (&piv)[NL], double (&cexp)[NL], bool last) { return wide_qr_pass(Z, piv, cexp, panel(0), s, wave, lane, last); };
    auto qr_in_place = [&](d4 (&Z)[NL][KT], const double (&colexp)[NL]) {
        double piv[NL], piv2[NL], ce[NL], ce2[NL];
        const double amp = qr_pass(Z, piv, ce, false);
#pragma unroll
        for (int nl = 0; nl < NL; ++nl) {
            piv2[nl] = 1.0;
            ce2[nl] = 0.0;
        }
        if (amp > (sizeof(IO) == 4 ? 1.0e10 : 1.0e3)) (void)qr_pass(Z, piv2, ce2, true); // (the same in every wave)
#pragma unroll
        for (int nl = 0; nl < NL; ++nl)
            if (piv[nl] > 1.0e-280 && piv2[nl] > 1.0e-280) {
                int e;
                pprod[nl] = frexp(pprod[nl] * piv[nl] * piv2[nl], &e);
                pexp[nl] += 2.0 * (colexp[nl] + ce[nl] + ce2[nl]) + (double)e;
            }
    };

    for (long long cc = 0; cc < a.C; ++cc) {
        store_carry(cc);
        const unsigned char *tp = a.totals + (b * a.C + cc) * a.tot_stride;
        const double tex = *reinterpret_cast<const double *>(tp + tot_mant);
        __syncthreads(); // (the panels of the chunk before are done with)
#pragma unroll 4
        for (int q = 0; q < TQ; ++q) {
            const int piece = tid + NW * 64 * q;
            const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
            const int p4 = (c4 & ~15) | ((c4 >> 2) & 3);
            d4 val = {0., 0., 0., 0.};
            if (c4 < a.tot_cols) val = *reinterpret_cast<const d4 *>(reinterpret_cast<const double *>(tp) + (size_t)row * a.tot_cols + c4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double x = val[e];
                if (row >= d || c4 + e >= d) x = (c4 + e == row) ? 1.0 : 0.0; // identity block past d
                tile[row * LDT + p4 + 4 * e] = x;
            }
        }
        __syncthreads();
        // ---- Z = T_c Y
        d4 Z[NL][KT];
#pragma unroll
        for (int nl = 0; nl < NL; ++nl)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) Z[nl][mt] = d4{0., 0., 0., 0.};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) {
                const d4 av = *reinterpret_cast<const d4 *>(&tile[(16 * mt + c) * LDT + 16 * kt + 4 * g]);
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int nl = 0; nl < NL; ++nl) Z[nl][mt] = mfma8(av[v], Y[nl][kt][v], Z[nl][mt]);
            }
        double zexp[NL];
#pragma unroll
        for (int nl = 0; nl < NL; ++nl) zexp[nl] = yexp[nl] + tex;

        const long long t_end = (cc + 1) * a.L;
        const bool boundary = t_end <= a.T && a.policy >= 0;
        bool did_reset = false;
        if (boundary) {
            did_reset = a.policy == 1;
            if (!did_reset) {
                did_reset = wide_colinear(Z, panel(0), s, wave, lane, d, (double)a.cos_threshold * (double)a.cos_threshold);
            }
        }
        if (did_reset) {
            qr_in_place(Z, zexp);
#pragma unroll
            for (int nl = 0; nl < NL; ++nl) {
#pragma unroll
                for (int mt = 0; mt < KT; ++mt) Y[nl][mt] = Z[nl][mt];
                yexp[nl] = 0.0;
            }
        } else {
#pragma unroll
            for (int nl = 0; nl < NL; ++nl) {
                double mx = 0.0;
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) mx = fmax(mx, fabs(Z[nl][mt][v]));
                mx = fmax(mx, __shfl_xor(mx, 16, 64));
                mx = fmax(mx, __shfl_xor(mx, 32, 64));
                int ex = 0;
                if (mx > 0.0) (void)frexp(mx, &ex);
#pragma unroll
                for (int mt = 0; mt < KT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) Y[nl][mt][v] = ldexp(Z[nl][mt][v], -ex);
                yexp[nl] = zexp[nl] + (double)ex;
            }
        }
        if (tid == 0) a.chunk_flags[b * a.C + cc] = did_reset ? 1 : 0;
    }

    store_carry(a.C); // the final state

    if (a.growth) { // growth of the final state (factorised, not replaced)
        d4 Z[NL][KT];
#pragma unroll
        for (int nl = 0; nl < NL; ++nl)
#pragma unroll
            for (int mt = 0; mt < KT; ++mt) Z[nl][mt] = Y[nl][mt];
        qr_in_place(Z, yexp);
        if (g == 0) {
#pragma unroll
            for (int nl = 0; nl < NL; ++nl) {
                const int col = 32 * wave + 16 * nl + c;
                if (col < d) a.growth[b * d + col] = 0.5 * (log(pprod[nl]) + pexp[nl] * kLn2) * a.growth_scale;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// The selective-resetting scan in the order of the paper's own parallel prefix scan (Section 5, eq. 28;
// Appendix C).  Elements (X_0, A_1, ..., A_T) are GOOM matrices; parallel step k works on blocks of 2^k
// elements, updating every element of a block's upper half from the last element of its lower half.  With all
// bias slots zero at the start every tuple (A*, B*) has one non-zero slot, so an element is one matrix M and a
// flag "has been reset" (the bias slot is the occupied one): a flagged element ignores what precedes it
// (A* = 0), an unflagged one becomes LMME(M_curr, M_prev) and inherits the flag of prev.  Before each parallel
// step every unflagged element that S selects is replaced by R(M) and flagged (tree_reset_kernel); the
// products of a step are batched LMMEs of the chain kernel, scattered back by tree_scatter_kernel.
struct TreeResetArgs {
    void *M;             // [n][d][d] GOOMs of one batch item, n = T + 1 elements
    unsigned char *flag; // [n]
    long long n;
    int d;
    int policy;
    float cos_threshold;
};

template <int DP, typename IO> __global__ __launch_bounds__(64) void tree_reset_kernel(TreeResetArgs a)
{
    constexpr int KT = DP / 16;
    __shared__ __align__(32) WaveD<DP> s;
    const int lane = threadIdx.x;
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const long long i = blockIdx.x;
    if (a.flag[i] || a.policy < 0) return; // whole wave
    IO *mp = static_cast<IO *>(a.M) + (size_t)i * d * d * 2;
    // columns scaled to a largest entry of 1 (identity block past d)
    d4 Z[KT][KT];
    bool any = false;
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        const int col = 16 * nt + c;
        double re[KT][4], im[KT][4];
        double cmax = -__builtin_huge_val();
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                double r = row == col ? 0.0 : -__builtin_huge_val(), im_ = 0.0;
                if (row < d && col < d) {
                    r = (double)mp[((size_t)row * d + col) * 2];
                    im_ = (double)mp[((size_t)row * d + col) * 2 + 1];
                    any = any || r > -__builtin_huge_val();
                }
                re[mt][v] = r;
                im[mt][v] = im_;
                cmax = fmax(cmax, r);
            }
        cmax = fmax(cmax, __shfl_xor(cmax, 16, 64));
        cmax = fmax(cmax, __shfl_xor(cmax, 32, 64));
        const bool zero_col = !(cmax > -__builtin_huge_val());
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double x = zero_col ? 0.0 : exp(re[mt][v] - cmax);
                if ((int)rint(im[mt][v] * 0.318309886183790671538) & 1) x = -x;
                Z[nt][mt][v] = x;
            }
    }
    if (__builtin_amdgcn_ballot_w64(any) == 0) return; // a zero matrix is never selected
    bool sel = a.policy == 1;
    if (!sel) {
        // squared cosines between columns, tile by tile of the Gram matrix
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            d4 Gd = {0., 0., 0., 0.};
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int v = 0; v < 4; ++v) Gd = mfma8(Z[nt][kt][v], Z[nt][kt][v], Gd);
            double dsel = Gd[0];
            dsel = (c >> 2) == 1 ? Gd[1] : dsel;
            dsel = (c >> 2) == 2 ? Gd[2] : dsel;
            dsel = (c >> 2) == 3 ? Gd[3] : dsel;
            if (g == (c & 3)) s.diag[16 * nt + c] = dsel;
        }
        wave_sync();
        bool hit = false;
        const double thr2 = (double)a.cos_threshold * (double)a.cos_threshold;
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            const double dc = s.diag[16 * nt + c];
#pragma unroll
            for (int mt = 0; mt <= nt; ++mt) {
                d4 Gt = {0., 0., 0., 0.};
#pragma unroll
                for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) Gt = mfma8(Z[mt][kt][v], Z[nt][kt][v], Gt);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * mt + 4 * v + g, col = 16 * nt + c;
                    const double dr = s.diag[row];
                    if (row < col && col < d && Gt[v] * Gt[v] > thr2 * dr * dc) hit = true;
                }
            }
        }
        wave_sync();
        sel = __builtin_amdgcn_ballot_w64(hit) != 0;
    }
    if (!sel) return;
    double piv[KT], ce[KT];
    const double amp = qr_panels_d<DP>(Z, piv, ce, s, g, c, false);
    if (amp > (sizeof(IO) == 4 ? 1.0e10 : 1.0e3)) (void)qr_panels_d<DP>(Z, piv, ce, s, g, c, true);
    const IO pi = sizeof(IO) == 4 ? (IO)3.14159274101257324219f : (IO)3.14159265358979311600;
#pragma unroll
    for (int nt = 0; nt < KT; ++nt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g, col = 16 * nt + c;
                if (row < d && col < d) {
                    const double q = Z[nt][mt][v];
                    mp[((size_t)row * d + col) * 2] = (IO)(q != 0.0 ? log(fabs(q)) : -__builtin_huge_val());
                    mp[((size_t)row * d + col) * 2 + 1] = q < 0.0 ? pi : (IO)0;
                }
            }
    if (lane == 0) a.flag[i] = 1;
}

// The same for 64 < d <= 128: four waves per element, the factorisation and the cosine test of the wide carry kernel.
template <typename IO> __global__ __launch_bounds__(256) void tree_reset_wide_kernel(TreeResetArgs a)
{
    constexpr int DP = 128, KT = 8, NL = 2, LDQ = 18;
    extern __shared__ __align__(32) unsigned char smem[];
    double *panels = reinterpret_cast<double *>(smem);
    WideScratch &s = *reinterpret_cast<WideScratch *>(smem + (size_t)KT * DP * LDQ * sizeof(double));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const long long i = blockIdx.x;
    if (a.flag[i] || a.policy < 0) return; // whole workgroup
    IO *mp = static_cast<IO *>(a.M) + (size_t)i * d * d * 2;
    d4 Z[NL][KT];
    bool any = false;
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        const int col = 32 * wave + 16 * nl + c;
        double cmax = -__builtin_huge_val();
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                double r = row == col ? 0.0 : -__builtin_huge_val();
                if (row < d && col < d) {
                    r = (double)mp[((size_t)row * d + col) * 2];
                    any = any || r > -__builtin_huge_val();
                }
                Z[nl][mt][v] = r;
                cmax = fmax(cmax, r);
            }
        cmax = fmax(cmax, __shfl_xor(cmax, 16, 64));
        cmax = fmax(cmax, __shfl_xor(cmax, 32, 64));
        const bool zero_col = !(cmax > -__builtin_huge_val());
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                double x = zero_col ? 0.0 : exp(Z[nl][mt][v] - cmax);
                if (row < d && col < d && ((int)rint((double)mp[((size_t)row * d + col) * 2 + 1] * 0.318309886183790671538) & 1)) x = -x;
                Z[nl][mt][v] = x;
            }
    }
    if (tid == 0) s.hit = 0;
    __syncthreads();
    if (__builtin_amdgcn_ballot_w64(any) != 0 && lane == 0) s.hit = 1;
    __syncthreads();
    if (s.hit == 0) return; // a zero matrix is never selected (the same in every wave)
    bool sel = a.policy == 1;
    if (!sel) sel = wide_colinear(Z, panels, s, wave, lane, d, (double)a.cos_threshold * (double)a.cos_threshold);
    if (!sel) return;
    double piv[NL], ce[NL];
    const double amp = wide_qr_pass(Z, piv, ce, panels, s, wave, lane, false);
    if (amp > (sizeof(IO) == 4 ? 1.0e10 : 1.0e3)) (void)wide_qr_pass(Z, piv, ce, panels, s, wave, lane, true);
    const IO pi = sizeof(IO) == 4 ? (IO)3.14159274101257324219f : (IO)3.14159265358979311600;
#pragma unroll
    for (int nl = 0; nl < NL; ++nl)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g, col = 32 * wave + 16 * nl + c;
                if (row < d && col < d) {
                    const double q = Z[nl][mt][v];
                    mp[((size_t)row * d + col) * 2] = (IO)(q != 0.0 ? log(fabs(q)) : -__builtin_huge_val());
                    mp[((size_t)row * d + col) * 2 + 1] = q < 0.0 ? pi : (IO)0;
                }
            }
    if (tid == 0) a.flag[i] = 1;
}

// After the products of a parallel step: element i = block * 2 half + half + u takes tmp[block][u] unless it is
// flagged, and inherits the flag of j = block * 2 half + half - 1.  One workgroup per element.
template <typename IO> __global__ __launch_bounds__(256) void tree_scatter_kernel(IO *M, const IO *tmp, unsigned char *flag, long long n, int d,
                                                                                  long long half)
{
    const long long e = blockIdx.x; // index among the updated elements, block by block
    const long long block = e / half, u = e % half;
    const long long i = block * 2 * half + half + u, j = block * 2 * half + half - 1;
    if (i >= n) return;
    const unsigned char fi = flag[i], fj = flag[j];
    __syncthreads();
    if (!fi) {
        const size_t nn = (size_t)d * d * 2;
        for (size_t q = threadIdx.x; q < nn; q += 256) M[(size_t)i * nn + q] = tmp[(size_t)e * nn + q];
        if (threadIdx.x == 0) flag[i] = fj;
    }
}

// elements of one batch item: X_0 (given, or the identity) and the T matrices; flags cleared
template <typename IO> __global__ __launch_bounds__(256) void tree_init_kernel(const IO *J, const IO *S0, IO *M, unsigned char *flag, long long n, int d)
{
    const long long i = blockIdx.x;
    const size_t nn = (size_t)d * d * 2;
    const IO ninf = sizeof(IO) == 4 ? (IO)-__builtin_huge_valf() : (IO)-__builtin_huge_val();
    for (size_t q = threadIdx.x; q < nn; q += 256) {
        IO v;
        if (i > 0) v = J[(size_t)(i - 1) * nn + q];
        else if (S0) v = S0[q];
        else v = (q & 1) ? (IO)0 : (((q / 2) / d == (q / 2) % d) ? (IO)0 : ninf);
        M[(size_t)i * nn + q] = v;
    }
    if (threadIdx.x == 0) flag[i] = 0;
}

template <typename IO> __global__ __launch_bounds__(256) void tree_finish_kernel(const IO *M, const unsigned char *flag, IO *states, unsigned char *out_flags,
                                                                                 long long n, int d)
{
    const long long t = blockIdx.x; // state after step t + 1 = element t + 1
    const size_t nn = (size_t)d * d * 2;
    for (size_t q = threadIdx.x; q < nn; q += 256) states[(size_t)t * nn + q] = M[(size_t)(t + 1) * nn + q];
    if (out_flags && threadIdx.x == 0) out_flags[t] = flag[t + 1];
}

// Spectrum from the input states (paper Section 4.2.1, groups (b)-(d)): one wave per step t.
// The input state S_{t-1} is log-scaled column by column and exponentiated, its QR gives the
// orthonormal basis Q_{t-1}; J_t (scaled by one power of two for the whole matrix) is applied to
// it on the matrix unit, and the QR of the result gives R_t; log R_kk goes to steplog[b][t][k].
// Every step is independent of the others.
struct StepArgs {
    const float *J;      // [batch][T][d][d] GOOMs
    const float *S0;     // NULL (identity) or [batch][d][d] GOOMs
    const float *states; // [batch][T][d][d] GOOMs: entry t holds the state after step t + 1
    double *steplog;     // [batch][T][d]
    long long T;
    int d;
};

template <int DP> __global__ __launch_bounds__(64) void lyap_step_kernel(StepArgs a)
{
    constexpr int KT = DP / 16;
    constexpr int LDT = DP + 4;
    constexpr int TQ = DP * DP / 4 / 64;
    __shared__ __align__(16) Wave<DP> s;
    const int lane = threadIdx.x;
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const long long b = blockIdx.x / a.T, t = blockIdx.x % a.T;
    const float kLog2eF = 1.44269504088896340736f;

    // ---- input state, columns scaled to largest entry 1 (identity block past d)
    const float *src = t == 0 ? (a.S0 ? a.S0 + (size_t)b * d * d * 2 : nullptr) : a.states + (size_t)(b * a.T + t - 1) * d * d * 2;
    f4 Q[KT][KT];
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        const int col = 16 * nt + c;
        float re[KT][4], im[KT][4];
        float cmax = -__builtin_huge_valf();
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * g + v;
                float r = row == col ? 0.0f : -__builtin_huge_valf(), i = 0.0f;
                if (src && row < d && col < d) {
                    const float2 e = *reinterpret_cast<const float2 *>(src + ((size_t)row * d + col) * 2);
                    r = e.x;
                    i = e.y;
                }
                re[mt][v] = r;
                im[mt][v] = i;
                cmax = fmaxf(cmax, r);
            }
        cmax = fmaxf(cmax, __shfl_xor(cmax, 16, 64));
        cmax = fmaxf(cmax, __shfl_xor(cmax, 32, 64));
        const bool zero_col = !(cmax > -__builtin_huge_valf());
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float x = zero_col ? 0.0f : __builtin_amdgcn_exp2f((re[mt][v] - cmax) * kLog2eF);
                if ((int)rintf(im[mt][v] * 0.318309886183790671538f) & 1) x = -x;
                Q[nt][mt][v] = x;
            }
    }
    {
        double piv[KT];
        const float amp = qr_panels<DP>(Q, piv, s, g, c);
        if (amp > 65536.0f) (void)qr_panels<DP>(Q, piv, s, g, c);
    }

    // ---- J_t as reals scaled by 2^-sh, sh from the largest entry; identity block past d
    const float *jp = a.J + (size_t)(b * a.T + t) * d * d * 2;
    float jre[TQ][4], jim[TQ][4];
    float jmax = -__builtin_huge_valf();
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        const int piece = lane + 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float r = -__builtin_huge_valf(), i = 0.0f;
            if (row < d && c4 + e < d) {
                const float2 v = *reinterpret_cast<const float2 *>(jp + ((size_t)row * d + c4 + e) * 2);
                r = v.x;
                i = v.y;
            }
            jre[q][e] = r;
            jim[q][e] = i;
            jmax = fmaxf(jmax, r);
        }
    }
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) jmax = fmaxf(jmax, __shfl_xor(jmax, sft, 64));
    const float sh = jmax > -__builtin_huge_valf() ? ceilf(jmax * kLog2eF) : 0.0f;
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
        const int piece = lane + 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
        f4 val;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x = __builtin_amdgcn_exp2f(__builtin_fmaf(jre[q][e], kLog2eF, -sh));
            if ((int)rintf(jim[q][e] * 0.318309886183790671538f) & 1) x = -x;
            if (row >= d || c4 + e >= d) x = (c4 + e == row) ? 1.0f : 0.0f;
            val[e] = x;
        }
        *reinterpret_cast<f4 *>(&s.tile[row * LDT + c4]) = val;
    }
    wave_sync();
    f4 Z[KT][KT];
#pragma unroll
    for (int nt = 0; nt < KT; ++nt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) Z[nt][mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) {
            const f4 av = *reinterpret_cast<const f4 *>(&s.tile[(16 * mt + c) * LDT + 16 * kt + 4 * g]);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int nt = 0; nt < KT; ++nt) Z[nt][mt] = mfma4(av[v], Q[nt][kt][v], Z[nt][mt]);
        }
    wave_sync();
    double piv[KT], piv2[KT];
    const float amp = qr_panels<DP>(Z, piv, s, g, c);
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) piv2[nt] = 1.0;
    if (amp > 65536.0f) (void)qr_panels<DP>(Z, piv2, s, g, c);
    if (g == 0) {
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            const int col = 16 * nt + c;
            if (col < d) {
                const double p = piv[nt] * piv2[nt];
                a.steplog[(size_t)(b * a.T + t) * d + col] = p > 1.0e-60 ? 0.5 * log(p) + (double)sh * kLn2 : -__builtin_huge_val();
            }
        }
    }
}

// The same for complex128 GOOMs, in double throughout: the factorisations and the product run on the double matrix
// instruction in the layout of the carry kernel above (register v of lane (g, c) holds row 4 v + g; whatever is read
// from LDS as a four-vector stores index 4 v + g at position 4 g + v).
struct StepArgsD {
    const double *J, *S0, *states;
    double *steplog;
    long long T;
    int d;
};

template <int DP> __global__ __launch_bounds__(64) void lyap_step_kernel_d(StepArgsD a)
{
    constexpr int KT = DP / 16;
    constexpr int LDT = WaveD<DP>::LDT;
    constexpr int TQ = DP * DP / 4 / 64;
    __shared__ __align__(32) WaveD<DP> s;
    const int lane = threadIdx.x;
    const int g = lane >> 4, c = lane & 15;
    const int d = a.d;
    const long long b = blockIdx.x / a.T, t = blockIdx.x % a.T;
    auto is_odd = [](double im) { return ((int)rint(im * 0.318309886183790671538) & 1) != 0; };

    // ---- input state, columns scaled to largest entry 1 (identity block past d)
    const double *src = t == 0 ? (a.S0 ? a.S0 + (size_t)b * d * d * 2 : nullptr) : a.states + (size_t)(b * a.T + t - 1) * d * d * 2;
    d4 Q[KT][KT];
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        const int col = 16 * nt + c;
        double cmax = -__builtin_huge_val();
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                double r = row == col ? 0.0 : -__builtin_huge_val();
                if (src && row < d && col < d) r = src[((size_t)row * d + col) * 2];
                Q[nt][mt][v] = r;
                cmax = fmax(cmax, r);
            }
        cmax = fmax(cmax, __shfl_xor(cmax, 16, 64));
        cmax = fmax(cmax, __shfl_xor(cmax, 32, 64));
        const bool zero_col = !(cmax > -__builtin_huge_val());
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                const double tt = (Q[nt][mt][v] - cmax) * kLog2e;
                double x = (zero_col || !(tt > -1000.0)) ? 0.0 : exp2(tt);
                if (src && row < d && col < d && is_odd(src[((size_t)row * d + col) * 2 + 1])) x = -x;
                Q[nt][mt][v] = x;
            }
    }
    {
        double piv[KT], ce[KT];
        const double amp = qr_panels_d<DP>(Q, piv, ce, s, g, c, false);
        if (amp > 1.0e3) (void)qr_panels_d<DP>(Q, piv, ce, s, g, c, true);
    }

    // ---- J_t as reals scaled by 2^-sh, sh from the largest entry; identity block past d
    const double *jp = a.J + (size_t)(b * a.T + t) * d * d * 2;
    double jmax = -__builtin_huge_val();
    for (int q = 0; q < TQ; ++q) {
        const int piece = lane + 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (row < d && c4 + e < d) jmax = fmax(jmax, jp[((size_t)row * d + c4 + e) * 2]);
    }
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) jmax = fmax(jmax, __shfl_xor(jmax, sft, 64));
    const double sh = jmax > -__builtin_huge_val() ? ceil(jmax * kLog2e) : 0.0;
    for (int q = 0; q < TQ; ++q) {
        const int piece = lane + 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
        const int p4 = (c4 & ~15) | ((c4 >> 2) & 3);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double x = (c4 + e == row) ? 1.0 : 0.0;
            if (row < d && c4 + e < d) {
                const double *v = jp + ((size_t)row * d + c4 + e) * 2;
                const double tt = __builtin_fma(v[0], kLog2e, -sh);
                x = tt > -1000.0 ? exp2(tt) : 0.0;
                if (is_odd(v[1])) x = -x;
            }
            s.tile[row * LDT + p4 + 4 * e] = x;
        }
    }
    wave_sync();
    d4 Z[KT][KT];
#pragma unroll
    for (int nt = 0; nt < KT; ++nt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) Z[nt][mt] = d4{0., 0., 0., 0.};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) {
            const d4 av = *reinterpret_cast<const d4 *>(&s.tile[(16 * mt + c) * LDT + 16 * kt + 4 * g]);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int nt = 0; nt < KT; ++nt) Z[nt][mt] = mfma8(av[v], Q[nt][kt][v], Z[nt][mt]);
        }
    wave_sync();
    double piv[KT], piv2[KT], ce[KT], ce2[KT];
    const double amp = qr_panels_d<DP>(Z, piv, ce, s, g, c, false);
#pragma unroll
    for (int nt = 0; nt < KT; ++nt) {
        piv2[nt] = 1.0;
        ce2[nt] = 0.0;
    }
    if (amp > 1.0e3) (void)qr_panels_d<DP>(Z, piv2, ce2, s, g, c, true);
    if (g == 0) {
#pragma unroll
        for (int nt = 0; nt < KT; ++nt) {
            const int col = 16 * nt + c;
            if (col < d) {
                const bool ok = piv[nt] > 1.0e-280 && piv2[nt] > 1.0e-280;
                a.steplog[(size_t)(b * a.T + t) * d + col] =
                    ok ? 0.5 * (log(piv[nt]) + log(piv2[nt])) + (ce[nt] + ce2[nt] + sh) * kLn2 : -__builtin_huge_val();
            }
        }
    }
}

// The per-step estimator for 64 < d <= 128: a workgroup of four waves per step, the state's columns divided among
// them as in reset_carry_wide_kernel, everything in double for both formats.
template <typename IO> __global__ __launch_bounds__(256) void lyap_step_wide_kernel(const IO *J, const IO *S0, const IO *states, double *steplog,
                                                                                    long long T, int d)
{
    constexpr int DP = 128, KT = 8, NL = 2, NW = 4, LDT = DP + 2, LDQ = 18;
    constexpr int TQ = DP * DP / 4 / (NW * 64);
    extern __shared__ __align__(32) unsigned char smem[];
    double *tile = reinterpret_cast<double *>(smem);
    double *panels = reinterpret_cast<double *>(smem);
    WideScratch &s = *reinterpret_cast<WideScratch *>(smem + (size_t)KT * DP * LDQ * sizeof(double));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    const long long b = blockIdx.x / T, t = blockIdx.x % T;
    auto is_odd = [](double im) { return ((int)rint(im * 0.318309886183790671538) & 1) != 0; };

    // ---- input state, columns scaled to largest entry 1 (identity block past d), then its orthonormal factor
    const IO *src = t == 0 ? (S0 ? S0 + (size_t)b * d * d * 2 : nullptr) : states + (size_t)(b * T + t - 1) * d * d * 2;
    d4 Q[NL][KT];
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        const int col = 32 * wave + 16 * nl + c;
        double cmax = -__builtin_huge_val();
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                double r = row == col ? 0.0 : -__builtin_huge_val();
                if (src && row < d && col < d) r = (double)src[((size_t)row * d + col) * 2];
                Q[nl][mt][v] = r;
                cmax = fmax(cmax, r);
            }
        cmax = fmax(cmax, __shfl_xor(cmax, 16, 64));
        cmax = fmax(cmax, __shfl_xor(cmax, 32, 64));
        const bool zero_col = !(cmax > -__builtin_huge_val());
#pragma unroll
        for (int mt = 0; mt < KT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * mt + 4 * v + g;
                const double tt = (Q[nl][mt][v] - cmax) * kLog2e;
                double x = (zero_col || !(tt > -1000.0)) ? 0.0 : exp2(tt);
                if (src && row < d && col < d && is_odd((double)src[((size_t)row * d + col) * 2 + 1])) x = -x;
                Q[nl][mt][v] = x;
            }
    }
    {
        double piv[NL], ce[NL];
        const double amp = wide_qr_pass(Q, piv, ce, panels, s, wave, lane, false);
        if (amp > 1.0e3) (void)wide_qr_pass(Q, piv, ce, panels, s, wave, lane, true);
    }

    // ---- J_t as reals scaled by 2^-sh, sh from the largest entry; identity block past d
    const IO *jp = J + (size_t)(b * T + t) * d * d * 2;
    double jmax = -__builtin_huge_val();
    for (int e = tid; e < d * d; e += NW * 64) jmax = fmax(jmax, (double)jp[(size_t)e * 2]);
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) jmax = fmax(jmax, __shfl_xor(jmax, sft, 64));
    __syncthreads(); // (the panels of the factorisation above are done with; s.red is free)
    if (lane == 0) s.red[wave] = jmax;
    __syncthreads();
    jmax = fmax(fmax(s.red[0], s.red[1]), fmax(s.red[2], s.red[3]));
    const double sh = jmax > -__builtin_huge_val() ? ceil(jmax * kLog2e) : 0.0;
    for (int q = 0; q < TQ; ++q) {
        const int piece = tid + NW * 64 * q;
        const int row = piece / (DP / 4), c4 = 4 * (piece % (DP / 4));
        const int p4 = (c4 & ~15) | ((c4 >> 2) & 3);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double x = (c4 + e == row) ? 1.0 : 0.0;
            if (row < d && c4 + e < d) {
                const IO *v = jp + ((size_t)row * d + c4 + e) * 2;
                const double tt = __builtin_fma((double)v[0], kLog2e, -sh);
                x = tt > -1000.0 ? exp2(tt) : 0.0;
                if (is_odd((double)v[1])) x = -x;
            }
            tile[row * LDT + p4 + 4 * e] = x;
        }
    }
    __syncthreads();
    d4 Z[NL][KT];
#pragma unroll
    for (int nl = 0; nl < NL; ++nl)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) Z[nl][mt] = d4{0., 0., 0., 0.};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int mt = 0; mt < KT; ++mt) {
            const d4 av = *reinterpret_cast<const d4 *>(&tile[(16 * mt + c) * LDT + 16 * kt + 4 * g]);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int nl = 0; nl < NL; ++nl) Z[nl][mt] = mfma8(av[v], Q[nl][kt][v], Z[nl][mt]);
        }
    double piv[NL], piv2[NL], ce[NL], ce2[NL];
    const double amp = wide_qr_pass(Z, piv, ce, panels, s, wave, lane, false); // (its first barrier comes after the reads of the tile)
#pragma unroll
    for (int nl = 0; nl < NL; ++nl) {
        piv2[nl] = 1.0;
        ce2[nl] = 0.0;
    }
    if (amp > 1.0e3) (void)wide_qr_pass(Z, piv2, ce2, panels, s, wave, lane, true);
    if (g == 0) {
#pragma unroll
        for (int nl = 0; nl < NL; ++nl) {
            const int col = 32 * wave + 16 * nl + c;
            if (col < d) {
                const bool ok = piv[nl] > 1.0e-280 && piv2[nl] > 1.0e-280;
                steplog[(size_t)(b * T + t) * d + col] = ok ? 0.5 * (log(piv[nl]) + log(piv2[nl])) + (ce[nl] + ce2[nl] + sh) * kLn2 : -__builtin_huge_val();
            }
        }
    }
}

// lambda[b][k] = scale * sum_t steplog[b][t][k], summed in a fixed order: kSlices slices of the
// steps per batch item, partial sums in the workspace, then one block adds the slices.
constexpr int kSlices = 64;

__global__ __launch_bounds__(256) void steplog_partial_kernel(const double *steplog, double *partial, long long T, int d)
{
    __shared__ double red[256];
    const long long b = blockIdx.x / kSlices;
    const int slice = blockIdx.x % kSlices;
    const int r = threadIdx.x >> 6; // 4 groups of 64 threads; thread k < d of a group owns exponent k (and k + 64 above 64)
    const long long per = (T + kSlices - 1) / kSlices;
    const long long lo = slice * per, hi = lo + per < T ? lo + per : T;
    for (int k0 = 0; k0 < d; k0 += 64) { // (the same trips for every thread: there are barriers inside)
        const int kk = threadIdx.x & 63, k = k0 + kk;
        double acc = 0.0;
        if (k < d)
            for (long long t = lo + r; t < hi; t += 4) acc += steplog[(size_t)(b * T + t) * d + k];
        __syncthreads();
        red[threadIdx.x] = acc;
        __syncthreads();
        if (r == 0 && k < d) partial[(size_t)(b * kSlices + slice) * d + k] = ((red[kk] + red[64 + kk]) + red[128 + kk]) + red[192 + kk];
    }
}

__global__ void steplog_final_kernel(const double *partial, double *lambda, int d, double scale)
{
    const long long b = blockIdx.x;
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        double acc = 0.0;
        for (int sl = 0; sl < kSlices; ++sl) acc += partial[(size_t)(b * kSlices + sl) * d + k];
        lambda[b * d + k] = acc * scale;
    }
}

// Largest exponent from the final vector v = J_T ... J_1 u_0 (paper Section 4.2.2):
// LSE(2 Re v') / (2 dt T); one thread per batch item.
template <typename R> __global__ void lle_epilogue_kernel(const R *v, double *lle, long long batch, int d, double scale)
{
    const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= batch) return;
    const R *p = v + (size_t)b * d * 2;
    double m = -__builtin_huge_val();
    for (int i = 0; i < d; ++i) m = fmax(m, 2.0 * (double)p[2 * i]);
    if (!(m > -__builtin_huge_val())) {
        lle[b] = -__builtin_huge_val();
        return;
    }
    double acc = 0.0;
    for (int i = 0; i < d; ++i) acc += exp(2.0 * (double)p[2 * i] - m);
    lle[b] = (m + log(acc)) * scale;
}

// u_0 = (1, ..., 1) / sqrt(d) as GOOMs
template <typename R> __global__ void uniform_u0_kernel(R *u, long long n, int d)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    u[2 * i] = (R)(-0.5 * log((double)d));
    u[2 * i + 1] = (R)0;
}

// After phase 3 has stored the states of every chunk: the state at a reset step is the
// reset one, which is the prefix entering the next chunk; also fills the per-step flags.
struct ResetPostArgs {
    const unsigned char *carries; // factored prefixes with double mantissas
    long long car_stride;
    int car_cols;
    int dp;
    const unsigned char *chunk_flags;
    void *states;         // NULL or [batch][T][d][d] GOOMs
    unsigned char *flags; // NULL or [batch][T]
    long long T, L, C;
    int d;
};

template <typename IO> __global__ __launch_bounds__(kThreads) void reset_post_kernel(ResetPostArgs a)
{
    const long long b = blockIdx.x / a.C, c = blockIdx.x % a.C;
    const int tid = threadIdx.x, d = a.d;
    const long long t_first = c * a.L;
    long long len = a.T - t_first;
    if (len > a.L) len = a.L;
    const bool was_reset = a.chunk_flags[b * a.C + c] != 0;
    if (a.flags)
        for (long long t = tid; t < len; t += kThreads) a.flags[b * a.T + t_first + t] = (was_reset && t == len - 1) ? 1 : 0;
    if (!was_reset || !a.states) return;
    const unsigned char *src = a.carries + (b * (a.C + 1) + c + 1) * a.car_stride;
    const double *mp = reinterpret_cast<const double *>(src);
    const double *ep = reinterpret_cast<const double *>(src + (size_t)a.dp * a.car_cols * sizeof(double));
    IO *op = static_cast<IO *>(a.states) + ((size_t)(b * a.T + t_first + len - 1) * d * d) * 2;
    const IO pi = sizeof(IO) == 4 ? (IO)3.14159274101257324219f : (IO)3.14159265358979311600;
    for (int e = tid; e < d * d; e += kThreads) {
        const int i = e / d, k = e % d;
        const double v = mp[(size_t)i * a.car_cols + k];
        const double re = v != 0.0 ? log(fabs(v)) + ep[k] * kLn2 : -__builtin_huge_val();
        op[(size_t)e * 2] = (IO)re;
        op[(size_t)e * 2 + 1] = v < 0.0 ? pi : (IO)0;
    }
}

} // namespace

namespace goom {

int launch_reset_post(goom_ctx *ctx, const ResetLaunch &l)
{
    ResetPostArgs a;
    a.carries = static_cast<const unsigned char *>(l.carries);
    a.car_stride = l.car_stride;
    a.car_cols = l.car_cols;
    a.dp = padded_dim(l.d);
    a.chunk_flags = l.chunk_flags;
    a.states = l.post_states;
    a.flags = l.flags;
    a.T = l.T;
    a.L = l.L;
    a.C = l.C;
    a.d = l.d;
    const long long grid = l.batch * l.C;
    if (grid > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many chunks for one launch");
    prof_begin(ctx, "reset_post_states_flags");
    if (l.dtype == GOOM_C64)
        hipLaunchKernelGGL(reset_post_kernel<float>, dim3((unsigned)grid), dim3(kThreads), 0, ctx->stream, a);
    else
        hipLaunchKernelGGL(reset_post_kernel<double>, dim3((unsigned)grid), dim3(kThreads), 0, ctx->stream, a);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch reset_post_kernel");
}


int launch_lyap_steps(goom_ctx *ctx, const void *J, const void *S0, const void *states, double *steplog, double *partial,
                      double *lambda, long long T, int d, long long batch, int dtype, double scale)
{
    const long long grid = batch * T;
    if (grid > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    const int dp = padded_dim(d);
    if (d > 128) return fail(ctx, GOOM_EUNSUPPORTED, "the per-step estimator supports d <= 128 (d=%d)", d);
    prof_begin(ctx, "lyapunov_per_step_qr");
    if (dp == 128) { // four waves per step
        const size_t lds = (size_t)8 * 128 * 18 * sizeof(double) + sizeof(WideScratch);
        const void *kern = dtype == GOOM_C64 ? reinterpret_cast<const void *>(lyap_step_wide_kernel<float>) : reinterpret_cast<const void *>(lyap_step_wide_kernel<double>);
        if (int st = check_hip(ctx, hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds), "hipFuncSetAttribute(lyap_step_wide_kernel)")) return st;
        if (dtype == GOOM_C64)
            hipLaunchKernelGGL(lyap_step_wide_kernel<float>, dim3((unsigned)grid), dim3(256), lds, ctx->stream, static_cast<const float *>(J),
                               static_cast<const float *>(S0), static_cast<const float *>(states), steplog, T, d);
        else
            hipLaunchKernelGGL(lyap_step_wide_kernel<double>, dim3((unsigned)grid), dim3(256), lds, ctx->stream, static_cast<const double *>(J),
                               static_cast<const double *>(S0), static_cast<const double *>(states), steplog, T, d);
    } else
    if (dtype == GOOM_C64) {
        StepArgs a;
        a.J = static_cast<const float *>(J);
        a.S0 = static_cast<const float *>(S0);
        a.states = static_cast<const float *>(states);
        a.steplog = steplog;
        a.T = T;
        a.d = d;
        if (dp == 16)
            hipLaunchKernelGGL(lyap_step_kernel<16>, dim3((unsigned)grid), dim3(64), 0, ctx->stream, a);
        else if (dp == 32)
            hipLaunchKernelGGL(lyap_step_kernel<32>, dim3((unsigned)grid), dim3(64), 0, ctx->stream, a);
        else
            hipLaunchKernelGGL(lyap_step_kernel<64>, dim3((unsigned)grid), dim3(64), 0, ctx->stream, a);
    } else {
        StepArgsD a;
        a.J = static_cast<const double *>(J);
        a.S0 = static_cast<const double *>(S0);
        a.states = static_cast<const double *>(states);
        a.steplog = steplog;
        a.T = T;
        a.d = d;
        if (dp == 16)
            hipLaunchKernelGGL(lyap_step_kernel_d<16>, dim3((unsigned)grid), dim3(64), 0, ctx->stream, a);
        else if (dp == 32)
            hipLaunchKernelGGL(lyap_step_kernel_d<32>, dim3((unsigned)grid), dim3(64), 0, ctx->stream, a);
        else
            hipLaunchKernelGGL(lyap_step_kernel_d<64>, dim3((unsigned)grid), dim3(64), 0, ctx->stream, a);
    }
    prof_end(ctx);
    if (int st = check_hip(ctx, hipGetLastError(), "launch lyap_step_kernel")) return st;
    prof_begin(ctx, "lyapunov_mean_of_logs");
    hipLaunchKernelGGL(steplog_partial_kernel, dim3((unsigned)(batch * kSlices)), dim3(256), 0, ctx->stream, steplog, partial, T, d);
    hipLaunchKernelGGL(steplog_final_kernel, dim3((unsigned)batch), dim3(64), 0, ctx->stream, partial, lambda, d, scale);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch steplog kernels");
}

size_t lyap_steps_partial_bytes(long long batch, int d) { return align_up((size_t)batch * kSlices * d * sizeof(double), 256); }

int launch_lle_epilogue(goom_ctx *ctx, const void *v, double *lle, long long batch, int d, int dtype, double scale)
{
    const unsigned blocks = (unsigned)((batch + 63) / 64);
    prof_begin(ctx, "lle_log_norm");
    if (dtype == GOOM_C64)
        hipLaunchKernelGGL(lle_epilogue_kernel<float>, dim3(blocks), dim3(64), 0, ctx->stream, static_cast<const float *>(v), lle, batch, d, scale);
    else
        hipLaunchKernelGGL(lle_epilogue_kernel<double>, dim3(blocks), dim3(64), 0, ctx->stream, static_cast<const double *>(v), lle, batch, d, scale);
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch lle_epilogue_kernel");
}

int launch_uniform_u0(goom_ctx *ctx, void *u, long long batch, int d, int dtype)
{
    const long long n = batch * d;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (dtype == GOOM_C64)
        hipLaunchKernelGGL(uniform_u0_kernel<float>, dim3(blocks), dim3(256), 0, ctx->stream, static_cast<float *>(u), n, d);
    else
        hipLaunchKernelGGL(uniform_u0_kernel<double>, dim3(blocks), dim3(256), 0, ctx->stream, static_cast<double *>(u), n, d);
    return check_hip(ctx, hipGetLastError(), "launch uniform_u0_kernel");
}

size_t reset_tree_workspace_bytes(long long T, int d, long long batch, int dtype)
{
    const size_t mat = (size_t)d * d * 2 * (dtype == GOOM_C64 ? 4 : 8);
    return align_up((size_t)batch * (T + 1) * mat, 256) + align_up((size_t)(T + 1) * mat, 256) + align_up((size_t)batch * (T + 1), 256);
}

template <typename IO> static int run_reset_tree_t(goom_ctx *ctx, const void *J, const void *S0, void *states, unsigned char *out_flags, long long T, int d,
                                                   long long batch, int dtype, int policy, float cos_threshold, void *ws)
{
    const long long n = T + 1;
    const size_t mat = (size_t)d * d * 2 * sizeof(IO);
    unsigned char *w = static_cast<unsigned char *>(ws);
    unsigned char *Mall = w;
    unsigned char *tmp = w + align_up((size_t)batch * n * mat, 256);
    unsigned char *flags = tmp + align_up((size_t)n * mat, 256);
    const int dp = padded_dim(d);
    if (n > 0x7fffffffLL) return fail(ctx, GOOM_EUNSUPPORTED, "too many steps for one launch");
    const size_t wide_lds = (size_t)8 * 128 * 18 * sizeof(double) + sizeof(WideScratch);
    if (dp == 128)
        if (int st = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(tree_reset_wide_kernel<IO>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)wide_lds),
                               "hipFuncSetAttribute(tree_reset_wide_kernel)"))
            return st;
    for (long long b = 0; b < batch; ++b) {
        IO *M = reinterpret_cast<IO *>(Mall + (size_t)b * n * mat);
        unsigned char *flag = flags + (size_t)b * n;
        hipLaunchKernelGGL(tree_init_kernel<IO>, dim3((unsigned)n), dim3(256), 0, ctx->stream, static_cast<const IO *>(J) + (size_t)b * T * d * d * 2,
                           S0 ? static_cast<const IO *>(S0) + (size_t)b * d * d * 2 : nullptr, M, flag, n, d);
        for (long long half = 1; half < n; half *= 2) {
            TreeResetArgs a;
            a.M = M;
            a.flag = flag;
            a.n = n;
            a.d = d;
            a.policy = policy;
            a.cos_threshold = cos_threshold;
            prof_begin(ctx, "reset_tree_select_and_reset");
            if (dp == 16) hipLaunchKernelGGL((tree_reset_kernel<16, IO>), dim3((unsigned)n), dim3(64), 0, ctx->stream, a);
            else if (dp == 32) hipLaunchKernelGGL((tree_reset_kernel<32, IO>), dim3((unsigned)n), dim3(64), 0, ctx->stream, a);
            else if (dp == 64) hipLaunchKernelGGL((tree_reset_kernel<64, IO>), dim3((unsigned)n), dim3(64), 0, ctx->stream, a);
            else hipLaunchKernelGGL(tree_reset_wide_kernel<IO>, dim3((unsigned)n), dim3(256), wide_lds, ctx->stream, a);
            prof_end(ctx);
            if (int st = check_hip(ctx, hipGetLastError(), "launch tree_reset_kernel")) return st;
            // products of this parallel step: whole blocks, then the ragged last one
            const long long full = n / (2 * half), rest = n % (2 * half) > half ? n % (2 * half) - half : 0;
            for (int part = 0; part < 2; ++part) {
                const long long items = part == 0 ? full : (rest ? 1 : 0), steps = part == 0 ? half : rest;
                if (items == 0) continue;
                const long long first = part == 0 ? 0 : full * 2 * half; // first element of the first block of this part
                ChainLaunch l;
                std::memset(&l, 0, sizeof l);
                l.dtype = dtype;
                l.n = l.d = l.m = d;
                l.left = reinterpret_cast<unsigned char *>(M) + (size_t)(first + half) * mat;
                l.left_batch_stride = (long long)(2 * half * mat);
                l.left_step_stride = (long long)mat;
                l.steps = steps;
                l.chunk_len = 1;
                l.chunks_launched = steps;
                l.batch = items;
                l.init_mode = 2;
                l.init = reinterpret_cast<unsigned char *>(M) + (size_t)(first + half - 1) * mat;
                l.init_stride = (long long)(2 * half * mat);
                l.out_goom = tmp + (size_t)(part == 0 ? 0 : full * half) * mat;
                l.label = "reset_tree_products";
                if (int st = launch_chain(ctx, l)) return st;
            }
            const long long updated = full * half + rest;
            if (updated > 0)
                hipLaunchKernelGGL(tree_scatter_kernel<IO>, dim3((unsigned)updated), dim3(256), 0, ctx->stream, M, reinterpret_cast<const IO *>(tmp), flag, n, d, half);
            if (int st = check_hip(ctx, hipGetLastError(), "launch tree_scatter_kernel")) return st;
        }
        hipLaunchKernelGGL(tree_finish_kernel<IO>, dim3((unsigned)T), dim3(256), 0, ctx->stream, M, flag, static_cast<IO *>(states) + (size_t)b * T * d * d * 2,
                           out_flags ? out_flags + (size_t)b * T : nullptr, n, d);
        if (int st = check_hip(ctx, hipGetLastError(), "launch tree_finish_kernel")) return st;
    }
    return GOOM_OK;
}

int run_reset_tree(goom_ctx *ctx, const void *J, const void *S0, void *states, unsigned char *out_flags, long long T, int d, long long batch,
                   int dtype, int policy, float cos_threshold, void *ws)
{
    return dtype == GOOM_C64 ? run_reset_tree_t<float>(ctx, J, S0, states, out_flags, T, d, batch, dtype, policy, cos_threshold, ws)
                             : run_reset_tree_t<double>(ctx, J, S0, states, out_flags, T, d, batch, dtype, policy, cos_threshold, ws);
}

int launch_reset_carry(goom_ctx *ctx, const ResetLaunch &l)
{
    ResetArgs a;
    a.totals = static_cast<const unsigned char *>(l.totals);
    a.tot_stride = l.tot_stride;
    a.tot_cols = l.tot_cols;
    a.carries = static_cast<unsigned char *>(l.carries);
    a.car_stride = l.car_stride;
    a.car_cols = l.car_cols;
    a.s0 = l.s0;
    a.chunk_flags = l.chunk_flags;
    a.growth = l.growth;
    a.growth_scale = l.growth_scale;
    a.T = l.T;
    a.L = l.L;
    a.C = l.C;
    a.d = l.d;
    a.policy = l.policy;
    a.cos_threshold = l.cos_threshold;
    a.only_if = nullptr;
    a.segments_room = nullptr;
    a.frames = nullptr;
    a.segments = 0;
    a.per_segment = 0;
    const int dp = padded_dim(l.d);
    unsigned char *const carries = static_cast<unsigned char *>(l.carries);
    if (l.policy == GOOM_RESET_ALWAYS && dp <= 64 && !l.post_states) a.carries = nullptr; // (without states nobody reads them)
    if (l.d > 128) return fail(ctx, GOOM_EUNSUPPORTED, "the reset scan supports d <= 128 (d=%d)", l.d);
    if (dp == 128) { // four waves per batch item, the state's columns divided among them
        const size_t lds = (size_t)8 * 128 * 18 * sizeof(double) + sizeof(WideScratch);
        const void *kern = l.dtype == GOOM_C64 ? reinterpret_cast<const void *>(reset_carry_wide_kernel<float>) : reinterpret_cast<const void *>(reset_carry_wide_kernel<double>);
        if (int st = check_hip(ctx, hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds), "hipFuncSetAttribute(reset_carry_wide_kernel)")) return st;
        prof_begin(ctx, "reset_phase2_carries_qr");
        if (l.dtype == GOOM_C64)
            hipLaunchKernelGGL(reset_carry_wide_kernel<float>, dim3((unsigned)l.batch), dim3(256), lds, ctx->stream, a);
        else
            hipLaunchKernelGGL(reset_carry_wide_kernel<double>, dim3((unsigned)l.batch), dim3(256), lds, ctx->stream, a);
        prof_end(ctx);
        return check_hip(ctx, hipGetLastError(), "launch reset_carry_wide_kernel");
    }
    // The spectrum alone of a long chain: in segments of eight chunks and more, whose results lie where the carries would (twice: for a chunk two times
    // 3 / 8 of a matrix, and the carries are a matrix each).
    long long segments = l.C / kSegmentChunks;
    if (segments > 256 / l.batch) segments = 256 / l.batch; // a compute unit each
    if (!a.carries && l.policy == GOOM_RESET_ALWAYS && dp <= 32 && l.growth && l.C >= (l.dtype == GOOM_C64 ? 80 : 64) && segments >= 4) {
        a.per_segment = (l.C + segments - 1) / segments;
        a.segments = (int)((l.C + a.per_segment - 1) / a.per_segment);
        const size_t all = (size_t)l.batch * a.segments * (dp == 16 ? segment_room<16>() : segment_room<32>());
        double *rooms[2] = {reinterpret_cast<double *>(carries), reinterpret_cast<double *>(carries) + all};
        int *again = reinterpret_cast<int *>(rooms[1] + all);
        a.segments_room = rooms[0];
        prof_begin(ctx, "reset_phase2_segments_qr");
        const dim3 grid((unsigned)(l.batch * a.segments));
        auto join = [&](double *out, int stride, double limit) {
            const unsigned pairs = out ? (unsigned)a.segments : (unsigned)((a.segments - stride + 2 * stride - 1) / (2 * stride));
            if (dp == 16) hipLaunchKernelGGL(segment_join_kernel<16>, dim3(pairs * (unsigned)l.batch), dim3(128), 0, ctx->stream, a, out, stride, limit, again);
            else hipLaunchKernelGGL(segment_join_kernel<32>, dim3(pairs * (unsigned)l.batch), dim3(256), 0, ctx->stream, a, out, stride, limit, again);
        };
#define GOOM_SEGMENT_CASE(DPV, IO)                                                                                                                        \
    {                                                                                                                                                      \
        if (int st = check_hip(ctx,                                                                                                                        \
                               hipFuncSetAttribute(reinterpret_cast<const void *>(reset_carry_staged_kernel<DPV, IO, true>),                               \
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)staged_lds<DPV, true>()),                              \
                               "hipFuncSetAttribute(reset_carry_staged_kernel)"))                                                                          \
            return st;                                                                                                                                     \
        hipLaunchKernelGGL((reset_carry_staged_kernel<DPV, IO, true>), grid, dim3(4 * DPV + 64), (staged_lds<DPV, true>()), ctx->stream, a);               \
    }
        for (int pass = 0; pass < 2; ++pass) {
            if (dp == 16) {
                if (l.dtype == GOOM_C64) GOOM_SEGMENT_CASE(16, float) else GOOM_SEGMENT_CASE(16, double)
            } else {
                if (l.dtype == GOOM_C64) GOOM_SEGMENT_CASE(32, float) else GOOM_SEGMENT_CASE(32, double)
            }
            if (pass == 0) {
                for (int stride = 1; stride < a.segments; stride *= 2) {
                    double *to = a.segments_room == rooms[0] ? rooms[1] : rooms[0];
                    join(to, stride, 1.0e12);
                    a.segments_room = to;
                }
                a.frames = a.segments_room;
                a.segments_room = a.segments_room == rooms[0] ? rooms[1] : rooms[0];
            } else {
                for (int stride = 1; stride < a.segments; stride *= 2) join(nullptr, stride, 1.0e-2);
            }
        }
#undef GOOM_SEGMENT_CASE
        prof_end(ctx);
        if (int st = check_hip(ctx, hipGetLastError(), "launch reset_carry_staged_kernel in segments")) return st;
        a.only_if = again; // and in order those that did not come out
    }
    prof_begin(ctx, "reset_phase2_carries_qr");
#define GOOM_STAGED_CASE(DPV)                                                                                                  \
    if (l.policy == GOOM_RESET_ALWAYS && dp == DPV) {                                                                          \
        const void *kern = l.dtype == GOOM_C64 ? reinterpret_cast<const void *>(reset_carry_staged_kernel<DPV, float>)         \
                                               : reinterpret_cast<const void *>(reset_carry_staged_kernel<DPV, double>);       \
        if (int st = check_hip(ctx, hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)staged_lds<DPV>()), \
                               "hipFuncSetAttribute(reset_carry_staged_kernel)"))                                              \
            return st;                                                                                                         \
        if (l.dtype == GOOM_C64)                                                                                               \
            hipLaunchKernelGGL((reset_carry_staged_kernel<DPV, float>), dim3((unsigned)l.batch), dim3(4 * DPV), staged_lds<DPV>(), ctx->stream, a); \
        else                                                                                                                   \
            hipLaunchKernelGGL((reset_carry_staged_kernel<DPV, double>), dim3((unsigned)l.batch), dim3(4 * DPV), staged_lds<DPV>(), ctx->stream, a); \
        prof_end(ctx);                                                                                                         \
        return check_hip(ctx, hipGetLastError(), "launch reset_carry_staged_kernel");                                          \
    }
    GOOM_STAGED_CASE(16)
    GOOM_STAGED_CASE(32)
    GOOM_STAGED_CASE(64)
#undef GOOM_STAGED_CASE
#define GOOM_RESET_CASE(DPV)                                                                                                   \
    if (dp == DPV) {                                                                                                           \
        if (l.dtype == GOOM_C64)                                                                                               \
            hipLaunchKernelGGL((reset_carry_kernel<DPV, float>), dim3((unsigned)l.batch), dim3(64), 0, ctx->stream, a);       \
        else                                                                                                                   \
            hipLaunchKernelGGL((reset_carry_kernel<DPV, double>), dim3((unsigned)l.batch), dim3(64), 0, ctx->stream, a);      \
    }
    GOOM_RESET_CASE(16)
    GOOM_RESET_CASE(32)
    GOOM_RESET_CASE(64)
#undef GOOM_RESET_CASE
    prof_end(ctx);
    return check_hip(ctx, hipGetLastError(), "launch reset_carry_kernel");
}

} // namespace goom
