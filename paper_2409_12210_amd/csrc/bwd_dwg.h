// Weight gradient of the router, dW_gate = x^T dl (and dW_noise = x^T du): the shares of the chunks of tokens.  A header because
// layers of small tiles take it in the launch of dX (gemm_block.h).
#pragma once
#include <algorithm>

#include "common.h"

// eight consecutive elements as loaded, and element i of them as float
template <typename T>
struct Raw8;
template <>
struct Raw8<bf16_t> {
  u32x4 v;
  __device__ void load(const bf16_t* p) { v = *reinterpret_cast<const u32x4*>(p); }
  __device__ float get(int i) const {
    const uint32_t w = v[i >> 1];
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
template <>
struct Raw8<float> {
  f32x4 a, b;
  __device__ void load(const float* p) {
    a = *reinterpret_cast<const f32x4*>(p);
    b = *reinterpret_cast<const f32x4*>(p + 4);
  }
  __device__ float get(int i) const { return i < 4 ? a[i] : b[i - 4]; }
};

constexpr int BR_SLAB = 512, BR_TOK = 32;  // columns of d that a wave (eight per lane) owns; tokens per block and step

struct DwgArgs {
  const float *dl, *du;  // [T, N]
  const void* x;         // [T, d]
  float* partial;
  int ntok, d, N, nmat, tok;    // nmat: 2 with the noise term; tok: tokens per chunk
  int nchunk, slabs;
};
inline DwgArgs dwg_args(const LayerDims& L, const void* x, const BwdRouterBufs& B, int nmat) {
  // about 512 blocks: fewer, longer chunks mean fewer partial gradients (two matrices: room for half as many)
  const int slabs = (L.d + BR_SLAB - 1) / BR_SLAB, nb = (L.T + BR_TOK - 1) / BR_TOK, groups = (L.N + 7) / 8 * nmat;
  const int tok = std::max(nmat, std::min(16, nb * slabs * groups / 512)) * BR_TOK;
  return DwgArgs{B.dl, B.du, x, B.dW_partial, L.T, L.d, L.N, nmat, tok, (L.T + tok - 1) / tok, slabs};
}
inline int dwg_blocks(const DwgArgs& a) { return a.nchunk * a.slabs * ((a.N + 7) / 8) * a.nmat; }

typedef float DwgSums[2][64][64];

// partial[chunk][m][c][e] = sum over the chunk's tokens of x[t][c] dl[t][e] (m = 1: du), reduced over the chunks by
// dwg_reduce_kernel.  A block owns a slab, eight columns e and `tok` tokens, a quarter of them per wave.  A lane keeps its 8
// x 8 slice of the sum in registers; one load brings dl of eight tokens, which go to scalar registers; dl and the rows of the
// next batch of tokens are on their way during the arithmetic of one, without any barrier; at the end the waves' sums
// meet in LDS in a fixed order.
// TB: tokens per batch.
template <typename T, int TB>
__device__ __forceinline__ void bwd_dwg_block(const DwgArgs& a, int block, DwgSums& s_sum) {
  const int chunk = block % a.nchunk, slab = block / a.nchunk % a.slabs, group = block / a.nchunk / a.slabs;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = a.d, N = a.N, c = slab * BR_SLAB + lane * 8, cl = min(c, d - 8);
  const int groups = (N + 7) / 8, m = group / groups, e0 = group % groups * 8, ne = min(8, N - e0);
  const float* const dl = (m ? a.du : a.dl) + e0;
  float acc[8][8];
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[q][e] = 0.f;
  const int per = a.tok / 4, t0 = chunk * a.tok + wave * per, t1 = min(t0 + per, a.ntok);
  Raw8<T> cur[TB], nxt[TB];
  auto fetch = [&](Raw8<T> (&r)[TB], int t) {  // (tokens beyond the last repeat it; their dl is zero)
#pragma unroll
    for (int u = 0; u < TB; ++u) r[u].load(static_cast<const T*>(a.x) + (size_t)min(t + u, a.ntok - 1) * d + cl);
  };
  auto fetch_dl = [&](int t) -> float {  // lane 8 u + e: token t + u, column e0 + e
    const int u = lane >> 3, e = lane & 7;
    const float v = dl[(size_t)min(t + u, a.ntok - 1) * N + min(e, ne - 1)];
    return e < ne && t + u < t1 ? v : 0.f;
  };
  float dcur = 0.f;
  if (t0 < t1) {
    fetch(cur, t0);
    dcur = fetch_dl(t0);
  }
#pragma unroll 1
  for (int t = t0; t < t1; t += TB) {
    fetch(nxt, t + TB);
    const float dnxt = fetch_dl(t + TB);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < TB; ++u) {
      float dv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) dv[e] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(dcur), u * 8 + e));
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float xv = cur[u].get(q);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[q][e] = fmaf(xv, dv[e], acc[q][e]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < TB; ++u) cur[u] = nxt[u];
    dcur = dnxt;
  }
  // waves 2 and 3 hand their sums to waves 0 and 1, then wave 1 its own to wave 0
#pragma unroll
  for (int half = 2; half >= 1; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) s_sum[wave - half][q * 8 + e][lane] = acc[q][e];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[q][e] += s_sum[wave][q * 8 + e][lane];
    }
    __syncthreads();
  }
  if (wave != 0 || c >= d) return;
  float* const out = a.partial + (((size_t)chunk * a.nmat + m) * d + c) * N + e0;
  if (N == 8) {  // the lane's 8 x 8 block is 256 consecutive bytes
#pragma unroll
    for (int q = 0; q < 8; ++q) store8(out + q * 8, acc[q]);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e < ne) out[(size_t)q * N + e] = acc[q][e];
  }
}
