// Hot chain kernel for square matrices of the sizes between those it is built for (16 < d <= 128) and for states
// of another width than the matrices: the tile is padded to the next of 32, 64, 128 with zero rows and columns,
// and only the ceil(d / 16) blocks of sixteen rows and columns that hold entries are multiplied (paper Section 4.1
// runs chains of d x d matrices; its sizes are powers of two, which the unpadded instantiations serve).
#include "goom_chain_fast.h"

namespace goom_chain {

bool ragged_applies(const ChainArgs &args, int dp, int nw)
{
    const int d = args.d, m = args.m;
    return args.n == d && d > 16 && d <= dp && (d < dp || m != d) && m <= dp && (dp == 32 || dp == 64 || dp == 128) && nw <= dp / 16 &&
           (args.init_mode != 0 || m == d) && args.bias_mode == 0 && args.out_fact_steps == nullptr && !args.left_real && !args.out_scaled;
}

template <int DP, int NW, int KD, int RAG> static int launch_ragged(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    constexpr int LDA = DP + 4;
    const size_t lds = 2 * ((size_t)DP * LDA * sizeof(float) + (size_t)DP * sizeof(float)) + 128;
    void (*kern)(ChainArgs) = chain_kernel_fast_ragged<DP, NW, KD, RAG>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return goom::check_hip(ctx, e, "hipFuncSetAttribute(chain_kernel_fast_ragged)");
    }
    if (grid <= 0) return GOOM_OK;
    if (grid > 0x7fffffffLL) return goom::fail(ctx, GOOM_EUNSUPPORTED, "too many chains for one launch (%lld)", grid);
    goom::prof_begin(ctx, label);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), lds, ctx->stream, args);
    goom::prof_end(ctx);
    return goom::check_hip(ctx, hipGetLastError(), "launch chain_kernel_fast_ragged");
}

// d a multiple of four with a state of d columns spares the lanes the unaligned loads, the moves at the matrix's edge and the
// comparisons of the stores' rows: 20 000 steps of 52 x 52 take 648 us so and of 50 x 50 664 us the other way.  The rest before,
// through the general kernel, and now, whole scans: 40 000 steps of d = 35 1156 -> 614 us, 20 000 of d = 50 932 -> 664, 10 000 of d = 77
// 1847 -> 1071, 6000 of d = 127 1617 -> 1318, a state of 20 columns at d = 64 634 -> 579, one of 3 at d = 100 1230 -> 572; products
// of 50 x 50 with 50 x 33 (2000 pairs) 48.8 -> 32.7 us.  (A third to a half of the shorter ones are the carries.)
template <int DP, int NW, int KD> static int pick_ragged(goom_ctx *ctx, const ChainArgs &args, long long grid, const char *label)
{
    if (args.d % 4 == 0 && args.m == args.d) return launch_ragged<DP, NW, KD, 1>(ctx, args, grid, label);
    return launch_ragged<DP, NW, KD, 2>(ctx, args, grid, label);
}

int dispatch_ragged(goom_ctx *ctx, const ChainArgs &args, int dp, long long grid, const char *label)
{
    const int kd = (args.d + 15) / 16;
    if (dp == 32) return pick_ragged<32, 2, 2>(ctx, args, grid, label);
    if (dp == 64) return kd <= 3 ? pick_ragged<64, 4, 3>(ctx, args, grid, label) : pick_ragged<64, 4, 4>(ctx, args, grid, label);
    switch (kd) {
    case 8: return pick_ragged<128, 8, 8>(ctx, args, grid, label);
    case 7: return pick_ragged<128, 8, 7>(ctx, args, grid, label);
    case 6: return pick_ragged<128, 8, 6>(ctx, args, grid, label);
    default: return pick_ragged<128, 8, 5>(ctx, args, grid, label);
    }
}

} // namespace goom_chain
