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
//   * one factor for all steps (SAME) is converted once and stays in registers;
//   * the loop has no branch around a load (the bias's kind is a template parameter, steps past the end are computed and dropped):
//     behind one the compiler cannot count the loads in flight and waits for all of them (1.5 us a carry step of d = 64 then).
// Carries (factored matrices) are multiplied and added in double for float components too.
// Measured against the general chain kernel with one column: 63 carries of 16 sequences of d = 64 (float) 1018 -> 64 us; states of
// 8 x 2000 matrices of d = 100 3680 -> 307 us (0.35 -> 4.2 TB/s), of complex128 matrices of d = 48 1053 -> 196 us; a step of one
// chain takes 0.7 (d = 8), 1.4 (d = 64) and 2.9 us (d = 128).
#include "goom_vec.h"

namespace goom_chain {

namespace {

// no bias, GOOM vectors, GOOM vectors with io_shift, column d of the factored left factor
constexpr int kBiasNone = 0, kBiasGoom = 1, kBiasShifted = 2, kBiasFact = 3;

// natural log of |x| 2^s, s a whole number: the hardware logarithm of a mantissa in [1/2, 1), where its error is a unit in the last place
// of 1 (of a number scaled by 2^32, as the tile kernels take it, the logarithm is near 32 and so is its last place: 1.5e-6 against
// 2e-7 on states of one step)
__device__ inline float log_of(float x, double s)
{
#pragma clang fp contract(off)
    const float kLn2Hi = 0.693147182464599609375f;
    const float kLn2Lo = -1.90465429995776806e-9f;
    const float e = Comp<float>::exponent_of(x); // (zero: -126, and the logarithm is -inf)
    const float l2 = __builtin_amdgcn_logf(__builtin_fabsf(__builtin_ldexpf(x, -(int)e)));
    const float w = (float)(s + (double)e);
    return __builtin_fmaf(w, kLn2Hi, __builtin_fmaf(w, kLn2Lo, l2 * kLn2Hi));
}

template <typename R, typename IO, int DP, int NW, bool FACT, bool FULL, bool SAME, int BIAS, int PD>
__global__ __launch_bounds__(NW * 64) void vec_walk_kernel(ChainArgs a)
{
    typedef typename std::conditional<FACT || sizeof(R) == 8, double, float>::type V; // the vector and the sums
    typedef IO IO2 __attribute__((ext_vector_type(2)));
    constexpr int K = DP / 16;  // entries of a row per lane
    constexpr int RW = DP / NW; // rows of a wave
    constexpr int Q = RW / 4;   // passes of four rows
    constexpr int RD = PD % 2 == 0 ? 2 : 1; // depth of the ring of biases
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
    [[maybe_unused]] const unsigned char *same0 = a.left + item * a.left_batch_stride; // (a shared factored matrix lies in the item's first slot)
    const int lfc = a.left_fact_cols;
    const int row0 = wave * RW + g;           // row of pass q: row0 + 4 q
    const int orow = row0 + 4 * (c < Q ? c : 0); // the row this lane finishes (lanes c >= Q repeat one and store nothing)
    const bool owner = c < Q;
    const bool row_ok = orow < n_rows;
    const size_t bias_row = (size_t)(row_ok ? orow : 0);
    constexpr bool bias_goom = BIAS == kBiasGoom || BIAS == kBiasShifted, bias_fact = BIAS == kBiasFact, shifted = BIAS == kBiasShifted;

    // Entry (q, k) of this lane: row row0 + 4 q, column c + 16 k.  Beyond the matrix the last row (whose result is dropped) and
    // the row's last entry (which meets a zero of the vector, and repeats a value that the row's shift knows already) stand in: no
    // load or entry is masked.
    // Wave-uniform bases plus 32-bit byte offsets.
    const unsigned row_bytes = FACT ? (unsigned)lfc * (unsigned)sizeof(R) : (unsigned)(FULL ? DP : d) * (unsigned)sizeof(IO2);
    constexpr unsigned kEntry = FACT ? sizeof(R) : sizeof(IO2);
    unsigned row_at[FULL ? 1 : Q], col_at[FULL ? 1 : K];
    if constexpr (FULL) {
        row_at[0] = (unsigned)row0 * row_bytes;
        col_at[0] = (unsigned)c * kEntry;
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) row_at[q] = (unsigned)(row0 + 4 * q < n_rows ? row0 + 4 * q : n_rows - 1) * row_bytes;
#pragma unroll
        for (int k = 0; k < K; ++k) col_at[k] = (unsigned)(c + 16 * k < d ? c + 16 * k : d - 1) * kEntry;
    }
    auto offset_of = [&](int q, int k) {
        if constexpr (FULL)
            return row_at[0] + col_at[0] + (unsigned)(4 * q) * (unsigned)(DP * kEntry) + (unsigned)(16 * k) * kEntry;
        else
            return row_at[q] + col_at[k];
    };

    struct Matrix { // a factor as it comes from memory
        IO2 z[FACT || SAME ? 1 : Q][FACT || SAME ? 1 : K];
        R w[FACT && !SAME ? Q : 1][FACT && !SAME ? K : 1];
    };
    struct Rest { // what else a step reads
        IO2 bias;      // GOOM bias of the lane's row
        R bias_m;      // factored bias: mantissa ...
        double bias_e; // ... and exponent
        double common; // the factored matrix's exponent
        float shift;   // io_shift
    };
    auto load_goom = [&](long long t, int q, int k) {
        return *reinterpret_cast<const IO2 *>(left0 + t * a.left_step_stride + offset_of(q, k));
    };
    auto load_fact = [&](long long t, int q, int k) {
        return *reinterpret_cast<const R *>(left0 + t * a.left_step_stride + offset_of(q, k));
    };
    // (a step past the end loads the last one's again)
    auto load = [&](long long t, Matrix &m) {
        t = t < len ? t : len - 1;
        if constexpr (!SAME) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if constexpr (FACT)
                        m.w[q][k] = load_fact(t, q, k);
                    else
                        m.z[q][k] = load_goom(t, q, k);
                }
        }
    };
    auto load_rest = [&](long long t, Rest &r) {
        t = t < len ? t : len - 1;
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
            if (shifted) r.shift = a.io_shift[item * a.steps + t0 + t];
        }
    };

    // ---- one factor's entries, scaled by their rows' powers of two
    // EARLY: the next factor is converted while this step's rows are on their way through LDS
    constexpr bool EARLY = !FACT && !SAME && DP <= 32; // (larger factors' registers are better spent on a deeper ring)
    V same_s[SAME || EARLY ? Q : 1][SAME || EARLY ? K : 1], same_n[SAME || EARLY ? Q : 1];
    double same_common = 0.0;
    auto row_shift_of = [&](const IO2 (&z)[K]) { // a whole number near the row's largest log2|A_ij|
        V u = -__builtin_huge_val();
#pragma unroll
        for (int k = 0; k < K; ++k) u = raw_max(u, (V)z[k][0]);
        u = max16(u);
        return u > (V)kNone ? Comp<V>::ceil_(u * (V)kLog2e) : (V)kNone; // (+inf stays: its row comes out as NaN; a zero row has none)
    };
    if constexpr (SAME) {
        [[maybe_unused]] const double *same_e = reinterpret_cast<const double *>(same0 + (size_t)DP * lfc * sizeof(R));
        if constexpr (FACT) { // rows on their own powers of two (goom_power.hip), these relative to the largest
            double top = kNegBig;
            for (int i = lane; i < n_rows; i += 64) top = raw_max(top, same_e[i]);
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) top = raw_max(top, __shfl_xor(top, s, 64));
            same_common = top > 0.5 * kNegBig ? top : 0.0;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if constexpr (FACT) {
                const double e = same_e[row0 + 4 * q < n_rows ? row0 + 4 * q : n_rows - 1];
#pragma unroll
                for (int k = 0; k < K; ++k) same_s[q][k] = (V) * reinterpret_cast<const R *>(same0 + offset_of(q, k));
                same_n[q] = e > 0.5 * kNegBig ? (V)(e - same_common) : (V)0;
            } else if (a.left_prepared) { // converted once for all chunks (goom_power.hip)
                const unsigned char *pp = a.left_prepared + item * a.prepared_stride;
                const bool f64 = sizeof(R) == 8 || a.prepared_f64;
                const int i = row0 + 4 * q < n_rows ? row0 + 4 * q : n_rows - 1;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const size_t at = (size_t)i * a.prepared_cols + (c + 16 * k < d ? c + 16 * k : d - 1);
                    same_s[q][k] = f64 ? (V) reinterpret_cast<const double *>(pp)[at] : (V) reinterpret_cast<const float *>(pp)[at];
                }
                same_n[q] = (V) reinterpret_cast<const double *>(pp + (size_t)DP * a.prepared_cols * (f64 ? 8 : 4))[i];
            } else {
                IO2 z[K];
#pragma unroll
                for (int k = 0; k < K; ++k) z[k] = load_goom(0, q, k);
                same_n[q] = row_shift_of(z);
                // the one conversion's rounding is the same at every step and adds up along the chain: made in double, rounded once
#pragma unroll
                for (int k = 0; k < K; ++k) same_s[q][k] = (V)scaled_entry((double)z[k][0], (double)z[k][1], (double)same_n[q]);
            }
        }
    }

    auto convert = [&](const Matrix &r) {
        if constexpr (EARLY) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                same_n[q] = row_shift_of(r.z[q]);
#pragma unroll
                for (int k = 0; k < K; ++k) same_s[q][k] = scaled_entry((V)r.z[q][k][0], (V)r.z[q][k][1], same_n[q]);
            }
        }
    };

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

    // mat: the step's matrix, or (EARLY) the one after it, to be converted; either makes room for the one PD steps on
    auto step = [&](long long t, Matrix &mat, Rest &r) {
        const bool live = t < len; // (the whole workgroup; a step past the end is computed on the last factor and dropped)
        // ---- the lane's row of A_t h, as part 2^(n + base)
        V part = (V)0, n = (V)0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            V p = (V)0, nq = (V)0;
            if constexpr (SAME || EARLY) {
#pragma unroll
                for (int k = 0; k < K; ++k) p = p + same_s[q][k] * hm[k];
                nq = same_n[q];
            } else if constexpr (FACT) {
#pragma unroll
                for (int k = 0; k < K; ++k) p = p + (V)mat.w[q][k] * hm[k];
            } else {
                nq = row_shift_of(mat.z[q]);
#pragma unroll
                for (int k = 0; k < K; ++k) p = p + scaled_entry((V)mat.z[q][k][0], (V)mat.z[q][k][1], nq) * hm[k];
            }
            p = sum16(p);
            part = c == q ? p : part;
            n = c == q ? nq : n;
            if (K >= 8) __builtin_amdgcn_sched_barrier(0); // one pass's temporaries at a time: the registers hold two factors
        }
        if constexpr (FACT && sizeof(R) == 8) {
            // A factored matrix has one power of two for all its rows: a row may be 2^-500 of it, and meet an entry of the vector as small.
            // Where a sum comes out so low, the row is taken on a power of two of its own.  (SAME: it is, and its entries may be as far apart.)
            const bool low = owner && Comp<V>::abs_(part) < (V)0x1p-900;
            if (__builtin_amdgcn_ballot_w64(low) != 0) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    auto entry = [&](int k) -> V {
                        if constexpr (SAME)
                            return same_s[q][k];
                        else
                            return (V)mat.w[q][k];
                    };
                    V top = (V)0, p = (V)0;
#pragma unroll
                    for (int k = 0; k < K; ++k) top = raw_max(top, Comp<V>::abs_(entry(k)));
                    top = max16(top);
                    int e = top > (V)0 ? Comp<V>::frexp_exp(top) : 0;
                    asm volatile("" : "+v"(e)); // (worked out here, not once for all steps in registers of its own)
#pragma unroll
                    for (int k = 0; k < K; ++k) p = p + Comp<V>::ldexp_(entry(k), -e) * hm[k];
                    p = sum16(p);
                    part = c == q ? p : part;
                    n = c == q ? (V)e + (SAME ? same_n[SAME ? q : 0] : (V)0) : n;
                    if (K >= 8) __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // ---- the bias on the same base; the sum on the larger exponent
        const double base = eh + (FACT ? (SAME ? same_common : r.common) : 0.0);
        V bm = (V)0, be = (V)kNone;
        double cs = 0.0; // rescaled bias and states, in powers of two
        if (bias_goom) {
            if (shifted) cs = (double)r.shift * kLog2e;
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
        // A bias below the last place of anything that the row's terms could leave does not outlive their exact cancellation (the
        // entry is zero then, and passes no gradient, as where sum and bias share an exponent).  What counts is the terms that there are: a large
        // entry of A that meets a zero of the vector cancels nothing, and the bias is the result.  (Looked for in the rare steps that have
        // such a row: a row with terms keeps a sum, a row without any has seldom so small a bias beside so large an entry.)
        if constexpr (bias_goom) {
            constexpr V kLast = (V)(sizeof(V) == 4 ? 149 : 1074);
            const bool alone = owner && part == (V)0 && be < n - kLast && be > (V)kNone;
            if (__builtin_amdgcn_ballot_w64(alone) != 0) {
                V largest = (V)kNone; // exponent of the row's largest A_ij h_j, on the same base
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    V e = (V)kNone;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        V x; // that of the entry
                        if constexpr (SAME || EARLY) {
                            V v = same_s[q][k];
                            asm volatile("" : "+v"(v)); // (worked out here, not once for all steps in registers of its own)
                            x = v != (V)0 ? Comp<V>::exponent_of(v) + same_n[q] : (V)kNone;
                        } else {
                            x = (V)mat.z[q][k][0] * (V)kLog2e;
                        }
                        if (hm[k] != (V)0) e = raw_max(e, x + Comp<V>::exponent_of(hm[k]));
                    }
                    e = max16(e);
                    largest = c == q ? e : largest;
                }
                if (alone && be < largest - kLast) {
                    bm = (V)0;
                    be = (V)kNone;
                }
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
        if (a.out_goom && live && owner && row_ok && (!last_only || t == len - 1)) {
            const size_t at = (size_t)(last_only ? chain : item * a.steps + t0 + t) * n_rows + orow;
            IO re;
            if constexpr (sizeof(V) == 4 && sizeof(IO) == 4)
                re = log_of(m, (double)ex + base + cs);
            else
                re = (IO)Comp<double>::out_re((double)m, (double)ex, base + cs);
            reinterpret_cast<IO2 *>(a.out_goom)[at] = IO2{re, m < (V)0 ? Comp<IO>::pi() : (IO)0};
        }
        load_rest(t + RD, r);
        convert(mat);
        if (Q * K >= 16) __builtin_amdgcn_sched_barrier(0); // (the new factor takes the old one's registers, not more)
        load(t + PD + (EARLY ? 1 : 0), mat);
        if (Q * K >= 16) __builtin_amdgcn_sched_barrier(0);
        // ---- everyone reads the vector and brings it onto its largest exponent
        if (NW > 1) {
            __syncthreads();
        } else { // a wave's LDS operations complete in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        V xm = (V)kNone;
#pragma unroll
        for (int k = 0; k < K; ++k) xm = raw_max(xm, vx[buf][c + 16 * k]);
        xm = max16(xm);
        const bool none = !(xm > (V)(0.5f * kNone));
        if (none) xm = (V)0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const V h = Comp<V>::ldexp_(vm[buf][c + 16 * k], (int)Comp<V>::clamp_shift(vx[buf][c + 16 * k] - xm));
            hm[k] = live ? h : hm[k];
        }
        const double en = none ? 0.0 : base + (double)xm;
        eh = live ? en : eh;
        if (fact_steps && live) store_fact(fact_steps + (t + 1) * a.fact_stride, 0, sizeof(R) == 8);
        if (scaled && live) {
            // exp(z - c + 2), c the log of the largest magnitude: the mantissa over the largest one, times e^2.  (The maximum passes a NaN
            // by; the entry stays one, and the log scale says so: a zero state is something else.)
            V am = (V)0;
            bool nan = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                am = raw_max(am, Comp<V>::abs_(hm[k]));
                nan = nan || hm[k] != hm[k];
            }
            am = max16(am);
            nan = __builtin_amdgcn_ballot_w64(nan) != 0;
            if (wave == (NW - 1) && g == 3) { // (not the wave that has carries to store)
                const size_t at = (size_t)(item * a.steps + t0 + t);
                const V f = am > (V)0 ? (V)7.38905609893065022723 / am : (V)0;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (c + 16 * k < d) scaled[at * d + c + 16 * k] = (IO)(hm[k] * f);
                if (logscale && c == 0)
                    logscale[at] = nan ? (IO)__builtin_nan("") : am > (V)0 ? (IO)(((double)Comp<V>::log2_abs(am) + eh) * kLn2) : (IO)-__builtin_huge_val();
            }
        }
    };

    Matrix ring[PD];
    Rest rest[RD];
    if constexpr (EARLY) {
        load(0, ring[0]);
        convert(ring[0]);
    }
#pragma unroll
    for (int i = 0; i < PD; ++i) load(i + (EARLY ? 1 : 0), ring[i]);
#pragma unroll
    for (int i = 0; i < RD; ++i) load_rest(i, rest[i]);
    for (long long t = 0; t < len; t += PD) { // (PD steps written out: the rings' slots are known at compile time)
#pragma unroll
        for (int i = 0; i < PD; ++i) step(t + i, ring[i], rest[i % RD]);
    }
    if (a.out_fact_final) store_fact(a.out_fact_final + chain * a.fact_stride, a.bias_mode ? a.bias_col : 0, sizeof(R) == 8 || a.fact_f64);
}

template <typename R, int DP, int NW, bool FACT, bool FULL, bool SAME, int BIAS, int PD>
int launch_vec(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    if (grid <= 0) return GOOM_OK;
    if (grid > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many chains for one launch (%lld)", grid);
    goom::prof_begin(ctx, label);
    hipLaunchKernelGGL((vec_walk_kernel<R, R, DP, NW, FACT, FULL, SAME, BIAS, PD>), dim3((unsigned)grid), dim3(NW * 64), 0, ctx->stream, args);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch vec_walk_kernel");
}

template <typename R, int DP, int NW, int PD> int goom_factors(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    const bool bias = args.bias_mode == 1;
    if (args.left_step_stride == 0 && args.steps > 1) {
        if (bias && args.io_shift) return launch_vec<R, DP, NW, false, false, true, kBiasShifted, 2>(ctx, args, grid, label);
        return bias ? launch_vec<R, DP, NW, false, false, true, kBiasGoom, 2>(ctx, args, grid, label)
                    : launch_vec<R, DP, NW, false, false, true, kBiasNone, 2>(ctx, args, grid, label);
    }
    if (bias && args.io_shift) return launch_vec<R, DP, NW, false, false, false, kBiasShifted, PD>(ctx, args, grid, label);
    if (args.n == DP && args.d == DP)
        return bias ? launch_vec<R, DP, NW, false, true, false, kBiasGoom, PD>(ctx, args, grid, label)
                    : launch_vec<R, DP, NW, false, true, false, kBiasNone, PD>(ctx, args, grid, label);
    return bias ? launch_vec<R, DP, NW, false, false, false, kBiasGoom, PD>(ctx, args, grid, label)
                : launch_vec<R, DP, NW, false, false, false, kBiasNone, PD>(ctx, args, grid, label);
}

template <typename R, int DP, int NW, int PD> int factored(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    if (args.left_same) return launch_vec<R, DP, NW, true, false, true, kBiasFact, 2>(ctx, args, grid, label);
    return args.bias_mode == 2 ? launch_vec<R, DP, NW, true, false, false, kBiasFact, PD>(ctx, args, grid, label)
                               : launch_vec<R, DP, NW, true, false, false, kBiasNone, PD>(ctx, args, grid, label);
}

} // namespace

int dispatch_vec(goom_ctx *ctx, const ChainArgs &args, int dp, int f64, int left_fact, long long grid, const char *label)
{
    if (left_fact) {
        switch (dp) {
        case 16: return f64 ? factored<double, 16, 1, 4>(ctx, args, grid, label) : factored<float, 16, 1, 4>(ctx, args, grid, label);
        case 32: return f64 ? factored<double, 32, 2, 4>(ctx, args, grid, label) : factored<float, 32, 1, 4>(ctx, args, grid, label);
        case 64: return f64 ? factored<double, 64, 8, 4>(ctx, args, grid, label) : factored<float, 64, 4, 4>(ctx, args, grid, label);
        default: return f64 ? factored<double, 128, 8, 1>(ctx, args, grid, label) : factored<float, 128, 8, 1>(ctx, args, grid, label);
        }
    }
    switch (dp) {
    case 16: return f64 ? goom_factors<double, 16, 1, 2>(ctx, args, grid, label) : goom_factors<float, 16, 1, 4>(ctx, args, grid, label);
    case 32: return f64 ? goom_factors<double, 32, 4, 2>(ctx, args, grid, label) : goom_factors<float, 32, 2, 4>(ctx, args, grid, label);
    case 64: return f64 ? goom_factors<double, 64, 8, 2>(ctx, args, grid, label) : goom_factors<float, 64, 4, 4>(ctx, args, grid, label);
    default: return f64 ? goom_factors<double, 128, 8, 1>(ctx, args, grid, label) : goom_factors<float, 128, 8, 1>(ctx, args, grid, label);
    }
}

} // namespace goom_chain
