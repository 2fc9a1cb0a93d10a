// Launchers of the fp32-operand matrix products.  Each unit's kernels are compiled in a source file of its own
// (gemm_fp32.hip: the fp32 matrix instruction, gemm_split.hip: three-term bf16 splits), so that they build side by side;
// the planner in ulsnn.hip chooses among the tile shapes numbered here.
#pragma once
#include <hip/hip_runtime.h>

#include "gemm.hpp"

namespace ulsnn {

// Tile shapes of the fp32 instruction (order of ULSNN_TILE_*) and of the split.
enum CfgId { CFG_256x128 = 0, CFG_128W8, CFG_128, CFG_128x64, CFG_64x128, CFG_64, CFG_64K64, CFG_160x128, CFG_64K32, CFG_COUNT };

enum SplitId { SP_256x256 = 0, SP_256x128, SP_128W8, SP_128, SP_128x64, SP_64x128, SP_64, SP_64K64, SP_32K128, SP_COUNT };

// The split's tiles address their operands with 32-bit byte offsets (256 rows apart at most), which bounds the leading
// dimension.
constexpr int SPLIT_MAX_LD = (1 << 21) - 64;

// One product: grid (tiles, k splits); a.tiles_m, a.tiles_n and a.kchunk are set.  Which layouts exist for an epilogue:
// EPI_AXPBY and EPI_PARTIAL all four, EPI_BIAS_TANH and EPI_BIAS NN, EPI_TANHGRAD NT.  `mixed` (gemm_split.hpp): EPI_PARTIAL NT
// and EPI_TANHGRAD, which has no other form.
#define ULSNN_HIDDEN __attribute__((visibility("hidden")))
ULSNN_HIDDEN hipError_t launch_fp32(int cfg, int splits, bool a_kc, bool b_kc, int epi, const GemmArgs &a, hipStream_t s);
ULSNN_HIDDEN hipError_t launch_split(int cfg, int splits, bool a_kc, bool b_kc, int epi, bool mixed, const GemmArgs &a, hipStream_t s);

}  // namespace ulsnn
