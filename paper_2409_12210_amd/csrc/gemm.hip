// Ragged grouped GEMMs of the MoDSE layer on gfx950: one problem per expert, M = tokens routed to the
// expert (known only on the device), N or K = the expert's own hidden width d_ff[e] (Sec. 3.1 of
// arXiv 2409.12210).  A block of the launch before turns the device-side counts into a problem table and a tile prefix
// (gemm_plan.h); the workgroups, persistent ones or one per tile, find their tiles in it without any host round trip.
//
// Operand layouts (GemmLayout): every tensor of the layer is used as it lies in memory.  The forward
// GEMMs have both operands K-contiguous; the data-gradient GEMMs read the weights as [K, N]; the
// weight-gradient GEMMs contract over tokens and read both activations as [K, M] and [K, N].
#include <algorithm>

#include "common.h"
#include "gemm_bf16.h"
#include "gemm_block.h"
#include "gemm_choice.h"
#include "gemm_tiles.h"

namespace {
using namespace modse_gemm;

// (of the device that is current at the first launch; only a grid of workgroups that walk the tile list, of any length,
// goes by it)
int num_cus() {
  static const int n = [] {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return GEMM_CUS;
    return prop.multiProcessorCount > 0 ? prop.multiProcessorCount : GEMM_CUS;
  }();
  return n;
}

template <int BM, int BN, int NB, int WAVES_M, int WAVES_N, int EPI, int LAYOUT>
hipError_t run_bf16(const GemmPlan* plan, int n_prob, int accumulate, int option, int64_t max_tiles, hipStream_t s) {
  constexpr int NT = WAVES_M * WAVES_N * 64;
  int64_t grid = num_cus();  // the LDS panels fill a CU: one persistent workgroup per CU
  if (max_tiles < grid) grid = max_tiles;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL((gg_bf16_kernel<BM, BN, NB, WAVES_M, WAVES_N, EPI, LAYOUT>), dim3((unsigned)grid), dim3(NT), 0, s,
                     plan, n_prob, accumulate, option);
  return hipGetLastError();
}

// Workgroups of a launch with one per tile (max_tiles: an upper bound of the tile list's length)
int64_t block_grid(int64_t max_tiles) { return (int64_t)align_up((size_t)std::max<int64_t>(max_tiles, 1), NUM_XCD * TILE_RUN); }

template <typename T, int BM, int BN, int EPI, int LAYOUT, int WAVES_M = 2, int WAVES_N = 2>
hipError_t run_block(const GemmPlan* plan, int n_prob, int accumulate, int option, int64_t max_tiles, hipStream_t s) {
  constexpr int NB = EPI == EPI_SWIGLU ? 2 : 1;
  const int64_t grid = block_grid(max_tiles);
  if constexpr (std::is_same_v<T, float> && BM == 32)
    hipLaunchKernelGGL((gg_f32_small_kernel<NB, EPI, LAYOUT>), dim3((unsigned)grid), dim3(256), 0, s, plan, n_prob, accumulate, option);
  else if constexpr (std::is_same_v<T, float>)
    hipLaunchKernelGGL((gg_f32_kernel<BM, BN, NB, EPI, LAYOUT>), dim3((unsigned)grid), dim3(256), 0, s, plan, n_prob, accumulate,
                       option);
  else if constexpr (BM < 128)
    hipLaunchKernelGGL((gg_bf16_skinny_kernel<BM, BN, NB, WAVES_M, WAVES_N, EPI, LAYOUT>), dim3((unsigned)grid),
                       dim3(WAVES_M * WAVES_N * 64), 0, s, plan, n_prob, accumulate, option);
  else
    hipLaunchKernelGGL((gg_bf16_block_kernel<BM, BN, NB, WAVES_M, WAVES_N, EPI, LAYOUT>), dim3((unsigned)grid),
                       dim3(WAVES_M * WAVES_N * 64), 0, s, plan, n_prob, accumulate, option);
  return hipGetLastError();
}

// EPI_SWIGLU: `bn` columns of each of the two matrices
template <typename T, int EPI, int LAYOUT>
hipError_t run_block_tile(TileShape t, const GemmPlan* plan, int n_prob, int accumulate, int option, int64_t max_tiles, hipStream_t s) {
  if (t.bm == 128) return run_block<T, 128, EPI == EPI_SWIGLU ? 64 : 128, EPI, LAYOUT>(plan, n_prob, accumulate, option, max_tiles, s);
  if constexpr (std::is_same_v<T, float> && EPI != EPI_STORE_F32)
    if (t.bm == 32) return run_block<T, 32, 32, EPI, LAYOUT>(plan, n_prob, accumulate, option, max_tiles, s);
  constexpr int BN = std::is_same_v<T, float> || EPI == EPI_SWIGLU ? 64 : 128;
  if constexpr (!std::is_same_v<T, float> && LAYOUT == LAYOUT_TN && EPI != EPI_SWIGLU)
    if (t.bm == 32) return run_block<T, 32, BN, EPI, LAYOUT, 1, 4>(plan, n_prob, accumulate, option, max_tiles, s);
  if constexpr (!std::is_same_v<T, float> && LAYOUT == LAYOUT_AB_K) return hipErrorInvalidValue;  // (128 rows or 256)
  else return run_block<T, 64, BN, EPI, LAYOUT>(plan, n_prob, accumulate, option, max_tiles, s);
}

// The epilogue fixes the operand layout: forward GEMMs are K-contiguous on both sides, data gradients read
// the weights as [K, N], weight gradients read both activations token-major; split-K partial sums of a forward GEMM
// (EPI_STORE_F32 with LAYOUT_TN) are the one exception.
template <typename T>
hipError_t launch_block(int epilogue, int layout, TileShape t, const GemmPlan* plan, int n_prob, int accumulate, int option,
                        int64_t max_tiles, hipStream_t s) {
  switch (epilogue) {
    case EPI_STORE: return run_block_tile<T, EPI_STORE, LAYOUT_TN>(t, plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_SWIGLU: return run_block_tile<T, EPI_SWIGLU, LAYOUT_TN>(t, plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_SWIGLU_BWD: return run_block_tile<T, EPI_SWIGLU_BWD, LAYOUT_B_KN>(t, plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_STORE_DUALK:
      if constexpr (std::is_same_v<T, float>) return run_block_tile<T, EPI_STORE_DUALK, LAYOUT_B_KN>(t, plan, n_prob, accumulate, option, max_tiles, s);
      else return hipErrorInvalidValue;  // (launch_dx)
    case EPI_STORE_F32:
      if (layout == LAYOUT_B_KN) {
        if constexpr (std::is_same_v<T, float>) return run_block_tile<T, EPI_STORE_F32, LAYOUT_B_KN>(t, plan, n_prob, accumulate, option, max_tiles, s);
        else return hipErrorInvalidValue;
      }
      if (layout == LAYOUT_TN) return run_block_tile<T, EPI_STORE_F32, LAYOUT_TN>(t, plan, n_prob, accumulate, option, max_tiles, s);
      return run_block_tile<T, EPI_STORE_F32, LAYOUT_AB_K>(t, plan, n_prob, accumulate, option, max_tiles, s);  // (bf16: where dX has 256-row tiles)
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_grouped_gemm(modse_dtype dt, int epilogue, TileShape t, const GemmPlan* plan, int n_prob, int accumulate,
                               int option, int64_t max_tiles, hipStream_t s, int layout) {
  if (dt == MODSE_F32) return launch_block<float>(epilogue, layout, t, plan, n_prob, accumulate, option, max_tiles, s);
  if (t.bm <= 128 && t.bn <= 128) return launch_block<bf16_t>(epilogue, layout, t, plan, n_prob, accumulate, option, max_tiles, s);
  switch (epilogue) {
    case EPI_STORE:
      return run_bf16<256, 256, 1, 4, 2, EPI_STORE, LAYOUT_TN>(plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_SWIGLU:
      return run_bf16<256, 128, 2, 4, 2, EPI_SWIGLU, LAYOUT_TN>(plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_SWIGLU_BWD:
      return run_bf16<256, 256, 1, 4, 2, EPI_SWIGLU_BWD, LAYOUT_B_KN>(plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_STORE_DUALK:
      return run_bf16<256, 256, 1, 4, 2, EPI_STORE_DUALK, LAYOUT_B_KN>(plan, n_prob, accumulate, option, max_tiles, s);
    case EPI_STORE_F32:
      return run_bf16<256, 256, 1, 4, 2, EPI_STORE_F32, LAYOUT_AB_K>(plan, n_prob, accumulate, option, max_tiles, s);
  }
  return hipErrorInvalidValue;
}

// Wherever the tiles allow it: in none of 58 layers drawn over the sizes that have such tiles was one launch slower by more than
// the runs differ (figures at the kernels, gemm_block.h).
bool dwg_beside_dx(modse_dtype dt, TileShape dx_tile, TileShape wg_tile) {
  return dt == MODSE_F32 ? dx_tile.bm <= 64 && wg_tile.bm == 64 : dx_tile.bm <= 128;
}
bool wgrad_beside_dx(modse_dtype dt, TileShape dx_tile, TileShape wg_tile) {
  return dwg_beside_dx(dt, dx_tile, wg_tile) && wg_tile.bm <= 128;
}
hipError_t launch_dx(modse_dtype dt, TileShape dx_tile, bool dx_split, const GemmPlan* dx, int n_dx, int64_t dx_tiles, int dx_option,
                     const GemmPlan* wg, int n_wg, int64_t wg_tiles, int accumulate, int wg_option, const DwgArgs* dwg, hipStream_t s) {
  const int64_t dx_blocks = block_grid(dx_tiles), wg_blocks = wg ? block_grid(wg_tiles) : 0;
  const DwgArgs w = dwg ? *dwg : DwgArgs{};
  const int n_dwg = dwg ? dwg_blocks(w) : 0;
  const dim3 grid((unsigned)(n_dwg + dx_blocks + wg_blocks)), block(256);
#define MODSE_LAUNCH_F32(TILE, EPI)                                                                                               \
  hipLaunchKernelGGL((gg_f32_dx_wgrad_kernel<TILE, EPI>), grid, block, 0, s, w, n_dwg, dx, n_dx, (int)dx_blocks, wg, n_wg, accumulate, \
                     wg_option)
#define MODSE_LAUNCH_BF16(TILE, EPI)                                                                                             \
  hipLaunchKernelGGL((gg_bf16_dx_kernel<TILE, EPI>), grid, block, 0, s, dx, n_dx, dx_option, (int)dx_blocks, w, n_dwg, wg, n_wg, \
                     accumulate, wg_option)
  if (dt == MODSE_F32) {
    if (dx_tile.bm == 32) MODSE_LAUNCH_F32(32, EPI_STORE_DUALK);  // (never split)
    else if (dx_split) MODSE_LAUNCH_F32(64, EPI_STORE_F32);
    else MODSE_LAUNCH_F32(64, EPI_STORE_DUALK);
  } else {
    if (dx_tile.bm == 128 && dx_split) MODSE_LAUNCH_BF16(128, EPI_STORE_F32);
    else if (dx_tile.bm == 128) MODSE_LAUNCH_BF16(128, EPI_STORE_DUALK);
    else if (dx_split) MODSE_LAUNCH_BF16(64, EPI_STORE_F32);
    else MODSE_LAUNCH_BF16(64, EPI_STORE_DUALK);
  }
#undef MODSE_LAUNCH_F32
#undef MODSE_LAUNCH_BF16
  return hipGetLastError();
}
