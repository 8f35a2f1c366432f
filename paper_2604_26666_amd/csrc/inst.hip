// One tile configuration's kernels (both B layouts).  Built once per row of configs.def with
// -DFACT_ID=.. -DFACT_BM=.. -DFACT_BN=.. -DFACT_WM=.. -DFACT_WN=.. -DFACT_BK=.. -DFACT_STAGES=.., and for 4-wave
// configurations (but 192-wide ones) once more with -DFACT_ODD_ROWS: the kernels for plain outputs with rows at half a word.
#include "launch.h"
#include "lds_limit.h"

namespace fact {

#define FACT_CAT2(a, b) a##b
#define FACT_CAT(a, b) FACT_CAT2(a, b)

#ifdef FACT_ODD_ROWS
constexpr bool ODD = true;
#else
constexpr bool ODD = false;
#endif
hipError_t FACT_CAT(fact_launch_odd_cfg, FACT_ID)(const GemmArgs &args, bool trans_b, int grid_z, hipStream_t stream);

template <bool TRANS_B>
static hipError_t launch_one(const GemmArgs &args, int grid_z, hipStream_t stream)
{
    if constexpr (!TRANS_B && !plain_b_supported(FACT_BN)) {
        (void)args; (void)grid_z; (void)stream;
        return hipErrorInvalidConfiguration;          // (the host side never selects such a tile for this layout)
    } else {
    constexpr bool CAN_PERSIST = FACT_WM * FACT_WN <= 4;      // the persistent form exists for 4-wave configurations
    auto kern = gemm_kernel<FACT_BM, FACT_BN, FACT_WM, FACT_WN, TRANS_B, FACT_BK, FACT_STAGES, false, false, ODD>;
    auto kern_p = gemm_kernel<FACT_BM, FACT_BN, FACT_WM, FACT_WN, TRANS_B, FACT_BK, FACT_STAGES, CAN_PERSIST && !ODD, false, ODD>;
    auto kern_h = gemm_kernel<FACT_BM, FACT_BN, FACT_WM, FACT_WN, TRANS_B, FACT_BK, FACT_STAGES, false, true, ODD>;      // binary16 operands (ordinary launches only)
    if constexpr (CAN_PERSIST && odd_rows_apart(FACT_BN) && !ODD)
        if (args.act != ACT_SILU_GATE && args.splits <= 1 && !args.out_f32 && !args.c_f32 && args.persist_items <= 0 &&
            ((args.ldc & 1) || ((uintptr_t)args.C & 2) || (grid_z > 1 && (args.stride_c & 1))))
            return FACT_CAT(fact_launch_odd_cfg, FACT_ID)(args, TRANS_B, grid_z, stream);
    // 192-wide tiles: a kernel for either store policy
    constexpr bool TWO = FACT_BN == 192;
    auto kern_s = gemm_kernel<FACT_BM, FACT_BN, FACT_WM, FACT_WN, TRANS_B, FACT_BK, FACT_STAGES, false, false, ODD, TWO>;
    auto kern_ps = gemm_kernel<FACT_BM, FACT_BN, FACT_WM, FACT_WN, TRANS_B, FACT_BK, FACT_STAGES, CAN_PERSIST && !ODD, false, ODD, TWO>;
    auto kern_hs = gemm_kernel<FACT_BM, FACT_BN, FACT_WM, FACT_WN, TRANS_B, FACT_BK, FACT_STAGES, false, true, ODD, TWO>;
    const bool persist = CAN_PERSIST && args.persist_items > 0;
    if (args.persist_items > 0 && (!CAN_PERSIST || args.f16)) return hipErrorInvalidConfiguration;     // (the host side never asks for it)
    constexpr int lds = lds_total(FACT_BM, FACT_BN, FACT_WM, FACT_WN, FACT_BK, FACT_STAGES);
    static LdsLimit limit;
    const hipError_t e = raise_lds_limit(limit, lds, {(const void *)kern, (const void *)kern_p, (const void *)kern_h,
                                                      (const void *)kern_s, (const void *)kern_ps, (const void *)kern_hs});     // (kern_p is kern where no persistent form exists)
    if (e != hipSuccess) return e;
    const int tiles = args.tiles_m * args.tiles_n;
    const int grid_x = args.tail_g > 1 ? args.tail_first + (tiles - args.tail_first) * args.tail_g : tiles;
    dim3 grid((unsigned)grid_x, 1, (unsigned)grid_z);
    if (args.persist_items > 0) grid = dim3((unsigned)args.persist_grid, 1, 1);
    dim3 block(FACT_WM * FACT_WN * 64, 1, 1);
    if (args.store_stream) {                                  // (the same kernels where the policy is chosen inside)
        kern = kern_s;
        kern_p = kern_ps;
        kern_h = kern_hs;
    }
    if (args.f16) hipLaunchKernelGGL(kern_h, grid, block, lds, stream, args);
    else if (persist) hipLaunchKernelGGL(kern_p, grid, block, lds, stream, args);
    else hipLaunchKernelGGL(kern, grid, block, lds, stream, args);
    return hipGetLastError();
    }
}

#ifdef FACT_ODD_ROWS
#define FACT_LAUNCH fact_launch_odd_cfg
#else
#define FACT_LAUNCH fact_launch_cfg
#endif
hipError_t FACT_CAT(FACT_LAUNCH, FACT_ID)(const GemmArgs &args, bool trans_b, int grid_z, hipStream_t stream)
{
    return trans_b ? launch_one<true>(args, grid_z, stream) : launch_one<false>(args, grid_z, stream);
}

}  // namespace fact
