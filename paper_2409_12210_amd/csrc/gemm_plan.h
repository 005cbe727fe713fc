// Device-side tile plans of the grouped GEMMs: the counts that the router leaves on the device become a
// problem table and a tile prefix, without a host round trip, in a block of the launch that precedes the GEMMs.
#pragma once
#include "common.h"
#include "gemm_tiles.h"

namespace modse_gemm {

// Tile counts and decode constants of a problem (from the fields in registers, before the problem is stored);
// returns its number of tiles.
__device__ inline int set_tiles(GemmProblem& P, int bm, int bn) {
  P.mtiles = (P.M + bm - 1) / bm;
  P.ntiles = (P.N + bn - 1) / bn;
  const int tiles = P.mtiles * P.ntiles;
  P.magic_group = tile_magic((uint32_t)(GROUP_M * P.ntiles), (uint64_t)tiles);
  P.magic_tail = tile_magic((uint32_t)(P.mtiles % GROUP_M), (uint64_t)GROUP_M * P.ntiles);
  return tiles;
}

// Exclusive sum over the lanes of a wave; total: the sum of all.
template <typename V>
__device__ inline V wave_exclusive(V v, int lane, V& total) {
  V incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const V up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  total = __shfl(incl, 63, 64);
  return incl - v;
}

// One wave fills in the tile prefix of a plan whose n problems have the tile counts in s_tiles.
__device__ inline void finish_plan(GemmPlan* plan, int lane, int n, const int* s_tiles) {
  constexpr int PER = MODSE_MAX_PROBLEMS / 64;
  int v[PER], sum = 0, total;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    v[i] = lane * PER + i < n ? s_tiles[lane * PER + i] : 0;
    sum += v[i];
  }
  int run = wave_exclusive(sum, lane, total);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (lane * PER + i < n) plan->tile_start[lane * PER + i] = run;
    run += v[i];
  }
  if (lane == 0) plan->tile_start[n] = total;
}

// What the planning block keeps in LDS.  It is the tail of a launch whose other blocks are long done (or the body of an
// extra block beside them), a chain of latencies and nothing else: every sum over experts or problems is a wave scan, and
// the problems of all GEMMs are made side by side by different waves.
struct PlanLds {
  long long hoff[MODSE_MAX_EXPERTS];   // elements of the ragged hidden tensors before expert e
  int first[MODSE_MAX_EXPERTS + 1];    // problems of a split product before the i-th listed expert
  int tiles[3][MODSE_MAX_PROBLEMS];
};
// hoff and first (passes * ceil(f / kchunk) problems per expert in listed order; one when kchunk is 0): waves 0 and 1
__device__ inline void plan_offsets(const LayerDims& L, const int* counts, int kchunk, int passes, PlanLds& S) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave == 0) {
    const int e = min(lane, L.N - 1);
    long long total;
    const long long h = wave_exclusive<long long>(lane < L.N ? (long long)counts[e] * L.f[e] : 0, lane, total);
    if (lane < L.N) S.hoff[lane] = h;
  } else if (wave == 1) {
    const int f = L.f[L.order[min(lane, L.N - 1)]];
    int total;
    const int n = lane >= L.N ? 0 : kchunk > 0 ? passes * ((f + kchunk - 1) / kchunk) : 1;
    const int p = wave_exclusive(n, lane, total);
    if (lane < L.N) S.first[lane] = p;
    if (lane == 0) S.first[L.N] = total;
  }
}
// the listed expert that problem p belongs to
__device__ inline int plan_expert(const PlanLds& S, int N, int p) {
  int lo = 0, hi = N;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (S.first[mid] <= p) lo = mid;
    else hi = mid;
  }
  return lo;
}

__device__ inline const char* cadd(const void* p, size_t bytes) { return static_cast<const char*>(p) + bytes; }
__device__ inline char* vadd(void* p, size_t bytes) { return p ? static_cast<char*>(p) + bytes : nullptr; }

// Length (whole K steps) of the nchunk chunks that K = f is cut into: about equal ones.  (The last may be short or even
// empty; an empty one writes a slab of zeros.)
__device__ inline int balanced_chunk(int f, int nchunk) { return ((f + nchunk - 1) / nchunk + 63) / 64 * 64; }

// Problem tables of the two forward GEMMs, by a block of at least 128 threads (counts, offsets: in LDS or memory).
__device__ inline void plan_fwd_body(const LayerDims& L, int esize, const int32_t* counts, const int32_t* offsets,
                                     const FwdPlanArgs& a, PlanLds& S) {
  const int tid = threadIdx.x, lane = tid & 63, d = L.d;
  const size_t es = esize;
  plan_offsets(L, counts, a.kchunk, 1, S);
  __syncthreads();
  if (tid < 64) {
    if (tid < L.N) {
      const int e = L.order[tid], n_e = counts[e], f = L.f[e];
      const size_t hoff = S.hoff[e];
      GemmProblem P = {};
      P.A = cadd(a.Xp, (size_t)offsets[e] * d * es);
      P.B = cadd(a.W1, (size_t)L.foff[e] * d * es);
      P.B2 = cadd(a.W3, (size_t)L.foff[e] * d * es);
      P.C = vadd(a.H, hoff * es);
      P.C2 = vadd(a.dHdA, hoff * es);
      P.C3 = vadd(a.dHdB, hoff * es);
      P.M = n_e; P.N = f; P.K = d;
      P.lda = d; P.ldb = d; P.ldc = f;
      S.tiles[0][tid] = set_tiles(P, a.up_tile.bm, a.up_tile.bn);
      a.up->prob[tid] = P;
    }
  } else {
    for (int p = tid - 64; p < S.first[L.N]; p += blockDim.x - 64) {
      const int i = plan_expert(S, L.N, p), c = p - S.first[i];
      const int e = L.order[i], n_e = counts[e], f = L.f[e];
      const size_t hoff = S.hoff[e];
      const int len = a.kchunk > 0 ? balanced_chunk(f, (f + a.kchunk - 1) / a.kchunk) : f, k0 = min(c * len, f);
      GemmProblem P = {};
      P.A = cadd(a.H, (hoff + k0) * es);
      P.B = cadd(a.W2, ((size_t)L.foff[e] * d + k0) * es);
      if (a.kchunk > 0) P.C = a.Opart + ((size_t)c * L.T * L.k + offsets[e]) * d;  // float32 partial sums
      else P.C = vadd(a.O, (size_t)offsets[e] * d * es);
      P.M = n_e; P.N = d; P.K = min(len, f - k0);
      P.lda = f; P.ldb = f; P.ldc = d;
      S.tiles[1][p] = set_tiles(P, a.down_tile.bm, a.down_tile.bn);
      a.down->prob[p] = P;
    }
  }
  __syncthreads();
  if (tid < 64) finish_plan(a.up, lane, L.N, S.tiles[0]);
  else if (tid < 128) finish_plan(a.down, lane, S.first[L.N], S.tiles[1]);
}

// Problem tables of the three backward GEMMs, by a block of at least 192 threads.
__device__ inline void plan_bwd_body(const LayerDims& L, int esize, const int32_t* counts, const int32_t* offsets,
                                     const BwdPlanArgs& a, PlanLds& S) {
  const int tid = threadIdx.x, lane = tid & 63, d = L.d;
  const size_t es = esize;
  plan_offsets(L, counts, a.dx_kchunk, 2, S);
  __syncthreads();
  if (tid < 64) {
    if (tid < L.N) {  // dh = dO W2 (W2_e is [d, f]: a [K, N] operand), fused SwiGLU backward -> dA, dB
      const int e = L.order[tid], n_e = counts[e], f = L.f[e];
      const size_t hoff = S.hoff[e];
      GemmProblem P = {};
      P.A = cadd(a.dO, (size_t)offsets[e] * d * es);
      P.B = cadd(a.W2, (size_t)L.foff[e] * d * es);
      P.C = vadd(a.dA, hoff * es);
      P.C2 = vadd(a.dB, hoff * es);
      P.E1 = cadd(a.dHdA, hoff * es);
      P.E2 = cadd(a.dHdB, hoff * es);
      P.M = n_e; P.N = f; P.K = d;
      P.lda = d; P.ldb = f; P.ldc = f;
      S.tiles[0][tid] = set_tiles(P, a.dh_tile.bm, a.dh_tile.bn);
      a.dh->prob[tid] = P;
    }
  } else if (tid < 128) {
    // dXp = dA W1 + dB W3 (W1_e, W3_e are [f, d]: [K, N] operands); split: one problem per (expert, operand pair, chunk
    // of K), float32 partial sums
    for (int p = lane; p < S.first[L.N]; p += 64) {
      const int i = plan_expert(S, L.N, p), c = p - S.first[i];
      const int e = L.order[i], n_e = counts[e], f = L.f[e];
      const size_t hoff = S.hoff[e], woff = (size_t)L.foff[e] * d;
      GemmProblem P = {};
      if (a.dx_kchunk > 0) {
        const int nchunk = (f + a.dx_kchunk - 1) / a.dx_kchunk, len = balanced_chunk(f, nchunk);
        const int k0 = min((c % nchunk) * len, f);
        P.A = cadd(c < nchunk ? a.dA : a.dB, (hoff + k0) * es);
        P.B = cadd(c < nchunk ? a.W1 : a.W3, (woff + (size_t)k0 * d) * es);
        P.C = a.dXpart + ((size_t)c * L.T * L.k + offsets[e]) * d;
        P.K = min(len, f - k0);
      } else {
        P.A = cadd(a.dA, hoff * es);
        P.B = cadd(a.W1, woff * es);
        P.A2 = cadd(a.dB, hoff * es);
        P.B2 = cadd(a.W3, woff * es);
        P.C = vadd(a.dXp, (size_t)offsets[e] * d * es);
        P.K = f;
      }
      P.M = n_e; P.N = d;
      P.lda = f; P.ldb = d; P.ldc = d;
      S.tiles[1][p] = set_tiles(P, a.dx_tile.bm, a.dx_tile.bn);
      a.dx->prob[p] = P;
    }
  } else if (tid < 192) {
    // Weight gradients contract over the expert's tokens, so a tile costs n_e K-steps whatever its expert's
    // width: the three GEMMs of one expert are listed together, experts by falling token count.
    if (lane < L.N) {
      const int e = L.order[lane], n_e = counts[e], f = L.f[e];
      const size_t hoff = S.hoff[e], woff = (size_t)L.foff[e] * d, roff = (size_t)offsets[e] * d;
      int rank = 0;
      for (int q = 0; q < L.N; ++q) rank += (counts[q] > n_e || (counts[q] == n_e && q < e)) ? 1 : 0;
      for (int which = 0; which < 3; ++which) {  // dW1 = dA^T Xp, dW3 = dB^T Xp, dW2 = dO^T H
        GemmProblem P = {};
        if (which < 2) {
          P.A = cadd(which ? a.dB : a.dA, hoff * es);  // [K = n_e, M = f]
          P.B = cadd(a.Xp, roff * es);                 // [K = n_e, N = d]
          P.C = (which ? a.dW3 : a.dW1) + woff;
          P.M = f; P.N = d;
        } else {
          P.A = cadd(a.dO, roff * es);  // [K = n_e, M = d]
          P.B = cadd(a.H, hoff * es);   // [K = n_e, N = f]
          P.C = a.dW2 + woff;
          P.M = d; P.N = f;
        }
        P.K = n_e;
        P.lda = P.M; P.ldb = P.N; P.ldc = P.N;
        S.tiles[2][3 * rank + which] = set_tiles(P, a.wg_tile.bm, a.wg_tile.bn);
        a.wg->prob[3 * rank + which] = P;
      }
    }
  }
  __syncthreads();
  if (tid < 64) finish_plan(a.dh, lane, L.N, S.tiles[0]);
  else if (tid < 128) finish_plan(a.dx, lane, S.first[L.N], S.tiles[1]);
  else if (tid < 192) finish_plan(a.wg, lane, 3 * L.N, S.tiles[2]);
}

}  // namespace modse_gemm
