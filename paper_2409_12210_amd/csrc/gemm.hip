// Ragged grouped GEMMs of the MoDSE layer on gfx950: one problem per expert, M = tokens routed to the
// expert (known only on the device), N or K = the expert's own hidden width d_ff[e] (Sec. 3.1 of
// arXiv 2409.12210).  A tiny plan kernel turns the device-side counts into a problem table and a tile
// prefix; persistent GEMM workgroups walk the tile list without any host round trip.
//
// Operand layouts (GemmLayout): every tensor of the layer is used as it lies in memory.  The forward
// GEMMs have both operands K-contiguous; the data-gradient GEMMs read the weights as [K, N]; the
// weight-gradient GEMMs contract over tokens and read both activations as [K, M] and [K, N].
#include <algorithm>

#include "common.h"
#include "gemm_bf16.h"
#include "gemm_bf16_skinny.h"
#include "gemm_block.h"
#include "gemm_plan.h"
#include "gemm_tiles.h"

namespace {
using namespace modse_gemm;

// ------------------------------------------------------------------------------------------------
// plan kernel of the backward GEMMs (single block): device-side counts -> problem tables.  (The forward plans
// are made by the routing stage's scan launch, see gemm_plan.h.)
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void plan_bwd_kernel(LayerDims L, int esize, const int32_t* __restrict__ counts,
                                                      const int32_t* __restrict__ offsets, BwdPlanArgs a) {
  __shared__ int s_tiles[MODSE_MAX_PROBLEMS];
  const int i = threadIdx.x;
  const bool on = i < L.N;
  const int e = on ? L.order[i] : 0;
  size_t hoff = 0;
  for (int q = 0; q < e; ++q) hoff += (size_t)counts[q] * L.f[q];
  const int n_e = counts[e], f = L.f[e], d = L.d;
  const size_t es = esize;
  const size_t woff = (size_t)L.foff[e] * d;   // element offset of expert e in W1/W3/W2 and their gradients
  const size_t roff = (size_t)offsets[e] * d;  // element offset of expert e's rows in [T*k, d] tensors
  if (on) {  // dh = dO W2 (W2_e is [d, f]: a [K, N] operand), fused SwiGLU backward -> dA, dB
    GemmProblem P = {};
    P.A = cadd(a.dO, roff * es);
    P.B = cadd(a.W2, woff * es);
    P.C = vadd(a.dA, hoff * es);
    P.C2 = vadd(a.dB, hoff * es);
    P.E1 = cadd(a.dHdA, hoff * es);
    P.E2 = cadd(a.dHdB, hoff * es);
    P.M = n_e; P.N = f; P.K = d;
    P.lda = d; P.ldb = f; P.ldc = f;
    s_tiles[i] = set_tiles(P, a.dh_tile.bm, a.dh_tile.bn);
    a.dh->prob[i] = P;
  }
  finish_plan(a.dh, i, L.N, s_tiles);
  if (on) {  // dXp = dA W1 + dB W3 (W1_e, W3_e are [f, d]: [K, N] operands)
    GemmProblem P = {};
    P.A = cadd(a.dA, hoff * es);
    P.B = cadd(a.W1, woff * es);
    P.A2 = cadd(a.dB, hoff * es);
    P.B2 = cadd(a.W3, woff * es);
    P.C = vadd(a.dXp, roff * es);
    P.M = n_e; P.N = d; P.K = f;
    P.lda = f; P.ldb = d; P.ldc = d;
    s_tiles[i] = set_tiles(P, a.dx_tile.bm, a.dx_tile.bn);
    a.dx->prob[i] = P;
  }
  finish_plan(a.dx, i, L.N, s_tiles);
  // Weight gradients contract over the expert's tokens, so a tile costs n_e K-steps whatever its expert's
  // width: the three GEMMs of one expert are listed together, experts by falling token count.
  if (on) {
    int rank = 0;
    for (int q = 0; q < L.N; ++q) rank += (counts[q] > n_e || (counts[q] == n_e && q < e)) ? 1 : 0;
    for (int which = 0; which < 2; ++which) {  // dW1 = dA^T Xp, dW3 = dB^T Xp
      GemmProblem P = {};
      P.A = cadd(which ? a.dB : a.dA, hoff * es);  // [K = n_e, M = f]
      P.B = cadd(a.Xp, roff * es);                  // [K = n_e, N = d]
      P.C = (which ? a.dW3 : a.dW1) + woff;
      P.M = f; P.N = d; P.K = n_e;
      P.lda = f; P.ldb = d; P.ldc = d;
      s_tiles[3 * rank + which] = set_tiles(P, a.wg_tile.bm, a.wg_tile.bn);
      a.wg->prob[3 * rank + which] = P;
    }
    GemmProblem P = {};  // dW2 = dO^T H
    P.A = cadd(a.dO, roff * es);  // [K = n_e, M = d]
    P.B = cadd(a.H, hoff * es);   // [K = n_e, N = f]
    P.C = a.dW2 + woff;
    P.M = d; P.N = f; P.K = n_e;
    P.lda = d; P.ldb = f; P.ldc = f;
    s_tiles[3 * rank + 2] = set_tiles(P, a.wg_tile.bm, a.wg_tile.bn);
    a.wg->prob[3 * rank + 2] = P;
  }
  finish_plan(a.wg, i, 3 * L.N, s_tiles);
}

int num_cus() {
  static int n = 0;
  if (n == 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      n = prop.multiProcessorCount;
    if (n <= 0) n = 256;
  }
  return n;
}

template <int BM, int BN, int NB, int WAVES_M, int WAVES_N, int EPI, int LAYOUT>
hipError_t run_bf16(const GemmPlan* plan, int accumulate, int save_pre, int64_t max_tiles, hipStream_t s) {
  constexpr int NT = WAVES_M * WAVES_N * 64;
  int64_t grid = num_cus();  // the LDS panels fill a CU: one persistent workgroup per CU
  if (max_tiles < grid) grid = max_tiles;
  if (grid < 1) grid = 1;
  if constexpr (BM == 64) {  // decode-sized batches
    hipLaunchKernelGGL((gg_bf16_skinny_kernel<BM, BN, NB, WAVES_M, WAVES_N, EPI, LAYOUT>), dim3((unsigned)grid), dim3(NT), 0,
                       s, plan, accumulate, save_pre);
  } else {
    hipLaunchKernelGGL((gg_bf16_kernel<BM, BN, NB, WAVES_M, WAVES_N, EPI, LAYOUT>), dim3((unsigned)grid), dim3(NT), 0, s,
                       plan, accumulate, save_pre);
  }
  return hipGetLastError();
}

// max_tiles: an upper bound of the tile list's length; one workgroup per tile
template <typename T, int BM, int BN, int EPI, int LAYOUT>
hipError_t run_block(const GemmPlan* plan, int accumulate, int save_pre, int64_t max_tiles, hipStream_t s) {
  constexpr int NB = EPI == EPI_SWIGLU ? 2 : 1;
  const int64_t grid = (int64_t)align_up((size_t)std::max<int64_t>(max_tiles, 1), NUM_XCD * TILE_RUN);
  if constexpr (std::is_same_v<T, float>)
    hipLaunchKernelGGL((gg_f32_kernel<BM, BN, NB, EPI, LAYOUT>), dim3((unsigned)grid), dim3(256), 0, s, plan, accumulate,
                       save_pre);
  else
    hipLaunchKernelGGL((gg_bf16_block_kernel<BM, BN, NB, EPI, LAYOUT>), dim3((unsigned)grid), dim3(256), 0, s, plan,
                       accumulate, save_pre);
  return hipGetLastError();
}

// EPI_SWIGLU: `bn` columns of each of the two matrices
template <typename T, int EPI, int LAYOUT>
hipError_t run_block_tile(TileShape t, const GemmPlan* plan, int accumulate, int save_pre, int64_t max_tiles, hipStream_t s) {
  if (t.bm == 128) return run_block<T, 128, EPI == EPI_SWIGLU ? 64 : 128, EPI, LAYOUT>(plan, accumulate, save_pre, max_tiles, s);
  return run_block<T, 64, 64, EPI, LAYOUT>(plan, accumulate, save_pre, max_tiles, s);
}

}  // namespace

namespace {
// tiles of an average batch: every expert has T * k / N rows (of C, or of the contraction for weight gradients)
int64_t expected_tiles(const LayerDims& L, int epilogue, int bm, int bn) {
  const int64_t rows = ((int64_t)L.T * L.k + L.N - 1) / L.N, mt = (rows + bm - 1) / bm, nt_d = (L.d + bn - 1) / bn;
  int64_t n = 0;
  for (int e = 0; e < L.N; ++e) {
    const int64_t nt_f = (L.f[e] + bn - 1) / bn;
    switch (epilogue) {
      case EPI_SWIGLU:
      case EPI_SWIGLU_BWD: n += mt * nt_f; break;
      case EPI_STORE_F32: n += 2 * ((L.f[e] + bm - 1) / bm) * nt_d + ((L.d + bm - 1) / bm) * nt_f; break;
      default: n += mt * nt_d;
    }
  }
  return n;
}
}  // namespace

// Forward GEMMs of a decode-sized batch (no expert can have more than MODSE_SKINNY_TOKENS rows) use tiles
// 64 rows high and 8 waves wide: 8/9 of what a stage loads is weights instead of half.
// float32: 128 x 128 tiles (a wave then needs four LDS reads per sixteen matrix instructions) unless they are too few to
// give every CU two, where 64 x 64 tiles spread the work.
TileShape gemm_tile_shape(const LayerDims& L, modse_dtype dt, int epilogue) {
  if (dt == MODSE_F32) {
    const TileShape t = epilogue == EPI_SWIGLU ? TileShape{128, 64} : TileShape{128, 128};
    return expected_tiles(L, epilogue, t.bm, t.bn) >= 2 * num_cus() ? t : TileShape{64, 64};
  }
  const bool skinny = L.T <= MODSE_SKINNY_TOKENS && (epilogue == EPI_SWIGLU || epilogue == EPI_STORE);
  if (epilogue == EPI_SWIGLU) return skinny ? TileShape{64, 256} : TileShape{256, 128};
  return skinny ? TileShape{64, 512} : TileShape{256, 256};
}

// The epilogue fixes the operand layout: forward GEMMs are K-contiguous on both sides, data gradients read
// the weights as [K, N], weight gradients read both activations token-major; split-K partial sums of a forward GEMM
// (EPI_STORE_F32 with LAYOUT_TN) are the one exception.
hipError_t launch_grouped_gemm(modse_dtype dt, int epilogue, TileShape t, const GemmPlan* plan, int accumulate,
                               int save_pre, int64_t max_tiles, hipStream_t s, int layout) {
  const bool split_k = epilogue == EPI_STORE_F32 && layout == LAYOUT_TN;
  if (dt == MODSE_F32) {
    if (split_k) return run_block_tile<float, EPI_STORE_F32, LAYOUT_TN>(t, plan, accumulate, save_pre, max_tiles, s);
    switch (epilogue) {
      case EPI_STORE: return run_block_tile<float, EPI_STORE, LAYOUT_TN>(t, plan, accumulate, save_pre, max_tiles, s);
      case EPI_SWIGLU: return run_block_tile<float, EPI_SWIGLU, LAYOUT_TN>(t, plan, accumulate, save_pre, max_tiles, s);
      case EPI_SWIGLU_BWD: return run_block_tile<float, EPI_SWIGLU_BWD, LAYOUT_B_KN>(t, plan, accumulate, save_pre, max_tiles, s);
      case EPI_STORE_DUALK: return run_block_tile<float, EPI_STORE_DUALK, LAYOUT_B_KN>(t, plan, accumulate, save_pre, max_tiles, s);
      case EPI_STORE_F32: return run_block_tile<float, EPI_STORE_F32, LAYOUT_AB_K>(t, plan, accumulate, save_pre, max_tiles, s);
    }
    return hipErrorInvalidValue;
  }
  const bool skinny = t.bm == 64;
  if (split_k) {
    if (skinny) return run_bf16<64, 512, 1, 1, 8, EPI_STORE_F32, LAYOUT_TN>(plan, accumulate, save_pre, max_tiles, s);
    return run_bf16<256, 256, 1, 4, 2, EPI_STORE_F32, LAYOUT_TN>(plan, accumulate, save_pre, max_tiles, s);
  }
  switch (epilogue) {
    case EPI_STORE:
      if (skinny) return run_bf16<64, 512, 1, 1, 8, EPI_STORE, LAYOUT_TN>(plan, accumulate, save_pre, max_tiles, s);
      return run_bf16<256, 256, 1, 4, 2, EPI_STORE, LAYOUT_TN>(plan, accumulate, save_pre, max_tiles, s);
    case EPI_SWIGLU:
      if (skinny) return run_bf16<64, 256, 2, 1, 8, EPI_SWIGLU, LAYOUT_TN>(plan, accumulate, save_pre, max_tiles, s);
      return run_bf16<256, 128, 2, 4, 2, EPI_SWIGLU, LAYOUT_TN>(plan, accumulate, save_pre, max_tiles, s);
    case EPI_SWIGLU_BWD:
      return run_bf16<256, 256, 1, 4, 2, EPI_SWIGLU_BWD, LAYOUT_B_KN>(plan, accumulate, save_pre, max_tiles, s);
    case EPI_STORE_DUALK:
      return run_bf16<256, 256, 1, 4, 2, EPI_STORE_DUALK, LAYOUT_B_KN>(plan, accumulate, save_pre, max_tiles, s);
    case EPI_STORE_F32:
      return run_bf16<256, 256, 1, 4, 2, EPI_STORE_F32, LAYOUT_AB_K>(plan, accumulate, save_pre, max_tiles, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_plan_bwd(const LayerDims& L, modse_dtype dt, const int32_t* counts, const int32_t* offsets,
                           const BwdPlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(plan_bwd_kernel, dim3(1), dim3(64), 0, s, L, dt == MODSE_F32 ? 4 : 2, counts, offsets, a);
  return hipGetLastError();
}
