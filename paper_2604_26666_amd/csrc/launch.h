// Host-side interface between the C ABI and the per-configuration translation units.
#pragma once
#include <hip/hip_runtime.h>
#include "gemm_kernel.h"

namespace fact {

// Launches configuration `id`'s kernel.  Defined once per configuration (inst.hip).
typedef hipError_t (*launch_fn)(const GemmArgs &args, bool trans_b, int grid_z, hipStream_t stream);

#define FACT_CFG(id, bm, bn, wm, wn, bk, st) hipError_t fact_launch_cfg##id(const GemmArgs &, bool, int, hipStream_t);
#include "configs.def"
#undef FACT_CFG

struct ConfigDesc {
    int id, bm, bn, wm, wn, bk, stages;
    launch_fn launch;
    // operand ring, or the epilogue's per-wave fp32 staging regions if those are larger
    int lds_bytes() const { return fact::lds_total(bm, bn, wm, wn, bk, stages); }
    int threads() const { return wm * wn * 64; }
    bool has_prefetch() const { return fact::has_prefetch(bm, bn, wm, wn, bk, stages); }      // and with it the sink a tail split's collector needs
    bool gate_capable() const { return true; }      // every wave tile has an even number of MFMA tiles along N
    bool serves(int trans_b) const { return trans_b || plain_b_supported(bn); }      // 192-wide tiles: B as [N][K] only
};

// Split-K reduction + epilogue, and the guarded fallback GEMM (aux_kernels.hip).
hipError_t launch_splitk_reduce(const GemmArgs &args, hipStream_t stream);
hipError_t launch_fallback_gemm(const GemmArgs &args, bool trans_b, int grid_z, hipStream_t stream);

// GEMM of few rows against B as [N][K], and small GEMMs of either layout (skinny.hip): the calls of few rows it can take and
// their estimated microseconds (whole_lines: every row of B begins on a 128-byte line); the estimate for a small GEMM with the
// tile that gives it (-1: none serves it); the form that runs for that tile (-1: few rows), a number of FACT_ROUTE_SKINNY; the launch.
bool skinny_takes(const GemmArgs &args, bool trans_b);
double skinny_us(const GemmArgs &args, int64_t batch, bool whole_lines);
double small_us(const GemmArgs &args, bool trans_b, int64_t batch, int most, int *tile);
int skinny_form(const GemmArgs &args, bool trans_b, int64_t batch, int tile);
hipError_t launch_skinny_gemm(const GemmArgs &args, bool trans_b, int form, int grid_z, hipStream_t stream);

// The same kernel's form for operands of any alignment: its estimate with the tile that gives it (-1: none), the launch.
double small_any_us(const GemmArgs &args, bool trans_b, int64_t batch, int *tile);
hipError_t launch_small_any(const GemmArgs &args, bool trans_b, int tile, int grid_z, hipStream_t stream);

// GEMM with operands of any alignment and size on the matrix cores (ragged.hip): the form that runs, a number of
// FACT_ROUTE_RAGGED, and the launch.
bool ragged_serves(const GemmArgs &args, bool trans_b, int64_t batch);
int ragged_form(const GemmArgs &args, bool trans_b, int64_t batch);
hipError_t launch_ragged_gemm(const GemmArgs &args, bool trans_b, int form, int grid_z, hipStream_t stream);

// Workspace of fact_gemm_splitk (any layout and epilogue) and of fact_block_mlp: the least that a call takes, and what the query reports.
struct Workspace { size_t least, full; };
Workspace splitk_workspace(int64_t M, int64_t N, int64_t K);
Workspace mlp_workspace(int64_t T, int64_t d_model, int64_t d_ff, int act);

}  // namespace fact
