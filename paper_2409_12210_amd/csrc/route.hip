// Router, permutation, combine and the element-wise backward kernels of the MoDSE layer (gfx950).
//
// Router: logits H(x) = x W_gate (+bias), KeepTopK, softmax over the kept logits (Sec. 2 Eq. 2-3 of
// arXiv 2409.12210).  Logits are accumulated in float64: products of bf16 or fp32 inputs are exact in
// float64, so the integer routing decision is taken at the same precision as a float64 reference and
// does not depend on summation order beyond the last bit.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "bwd_dwg.h"
#include "common.h"
#include "gemm_plan.h"

namespace {

constexpr int TPB = MODSE_ROUTE_TOKENS_PER_BLOCK;  // tokens per block
constexpr int ROUTE_THREADS = 256;
constexpr int ROUTER_TOKEN_MAX_T = 4096;  // plain-gate batches up to this size take a token router (one or four per block)
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ inline double shfl_xor_f64(double v, int mask) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __shfl_xor(lo, mask, 64);
  hi = __shfl_xor(hi, mask, 64);
  return __hiloint2double(hi, lo);
}

// Sum each of the V values over the 64 lanes of a wave.  Every halving step sends half of the values to
// the partner lane and keeps the other half, so V values cost V-1 + (6 - log2 V) shuffles.  On return
// lane l (l < V) holds in vals[0] the total of value index bitrev_{log2 V}(l).  (Template recursion, not
// loops: every index into vals is then a constant and the array stays in registers for any V.)
template <int V>
struct Log2 {
  static constexpr int value = 1 + Log2<V / 2>::value;
};
template <>
struct Log2<1> {
  static constexpr int value = 0;
};

template <int W, int I, int BIT, int V>
__device__ inline void halve_one(double (&vals)[V], bool upper) {
  if constexpr (I < W) {
    const double keep = upper ? vals[I + W] : vals[I];
    const double send = upper ? vals[I] : vals[I + W];
    vals[I] = keep + shfl_xor_f64(send, BIT);
    halve_one<W, I + 1, BIT>(vals, upper);
  }
}
template <int LIVE, int BIT, int V>
__device__ inline void halve_all(double (&vals)[V], int lane) {
  if constexpr (LIVE > 1) {
    halve_one<LIVE / 2, 0, BIT>(vals, (lane & BIT) != 0);
    halve_all<LIVE / 2, BIT * 2>(vals, lane);
  }
}
template <int V>
__device__ inline void wave_sum_values(double (&vals)[V], int lane) {
  halve_all<V, 1>(vals, lane);
#pragma unroll
  for (int s = Log2<V>::value; s < 6; ++s) vals[0] += shfl_xor_f64(vals[0], 1 << s);
}

template <int P>
__device__ inline int bitrev(int v) {
  int r = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) r |= ((v >> i) & 1) << (P - 1 - i);
  return r;
}

// NE consecutive elements -> floats, with the widest aligned vector loads
template <int NE, typename T>
__device__ inline void load_row(const T* p, float* out) {
  if constexpr (NE % 8 == 0) {
#pragma unroll
    for (int e = 0; e < NE; e += 8) load8(p + e, out + e);
  } else if constexpr (NE == 4) {
    load4(p, out);
  } else {
#pragma unroll
    for (int e = 0; e < NE; ++e) out[e] = (float)p[e];
  }
}

__device__ inline double softplus_f64(double u) {  // log(1 + exp(u)) without overflow
  return u > 0.0 ? u + log1p(exp(-u)) : log1p(exp(u));
}

// KeepTopK on one token's N logits (Sec. 2 Eq. 3), k <= 2: the two largest and the third largest value.  Strict
// comparisons while scanning upward leave ties with the lower index.  The second pick always differs from the
// first: when no logit besides the first is above -inf (all others masked out by an infinite negative bias) it is
// the lowest other index, as in a stable descending sort.
struct TopPick {
  double m1, m2, m3;
  int i1, i2;
};
__device__ inline TopPick pick_top(const double* logits, int N) {
  TopPick p = {-INFINITY, -INFINITY, -INFINITY, 0, -1};
  for (int e = 0; e < N; ++e) {
    const double l = logits[e];
    if (l > p.m1) {
      p.m3 = p.m2; p.m2 = p.m1; p.i2 = p.i1; p.m1 = l; p.i1 = e;
    } else if (l > p.m2) {
      p.m3 = p.m2; p.m2 = l; p.i2 = e;
    } else if (l > p.m3) {
      p.m3 = l;
    }
  }
  if (p.i2 < 0 || p.i2 == p.i1) p.i2 = p.i1 == 0 ? 1 : 0;
  return p;
}
// Writes token t's expert indices and gate weights (softmax over the kept logits, Eq. 2); returns whether the
// gap that decided the selection is under 1e-6.
__device__ inline bool write_gate(const TopPick& p, int t, int N, int top_k, int32_t* __restrict__ topk_idx,
                                  float* __restrict__ topk_w) {
  if (top_k == 2) {
    const double g1 = 1.0 / (1.0 + exp(p.m2 - p.m1));
    topk_idx[(size_t)t * 2] = p.i1;
    topk_idx[(size_t)t * 2 + 1] = p.i2;
    topk_w[(size_t)t * 2] = (float)g1;
    topk_w[(size_t)t * 2 + 1] = (float)(1.0 - g1);
    return (p.m1 - p.m2 < 1e-6) || (N > 2 && p.m2 - p.m3 < 1e-6);
  }
  topk_idx[t] = p.i1;
  topk_w[t] = 1.f;
  return N > 1 && p.m1 - p.m2 < 1e-6;
}

// ---------------------------------------------------------------- the router's dot products

// Row r of the LDS copy of W_gate that router_stream_kernel keeps: elements of type W (double when the matrix
// fits that way, else float), NE per row; the eight rows of one lane and step lie together, followed by 16
// bytes of padding, so that the 16 lanes which a 128-bit LDS read serves together fall into different banks.
constexpr int rs_group_bytes(int NE, int elem) { return 8 * NE * elem + 16; }
template <typename W, int NE>
struct LdsRows {
  const char* base;
  __device__ void fetch(int r, W (&wf)[NE]) const {
    constexpr int PER = 16 / sizeof(W);  // elements per 128-bit read
    typedef W vec_t __attribute__((ext_vector_type(PER)));
    const char* p = base + (r >> 3) * rs_group_bytes(NE, sizeof(W)) + (r & 7) * NE * (int)sizeof(W);
    if constexpr (NE >= PER) {
#pragma unroll
      for (int e = 0; e < NE; e += PER) {
        const vec_t q = *reinterpret_cast<const vec_t*>(p + e * sizeof(W));
#pragma unroll
        for (int j = 0; j < PER; ++j) wf[e + j] = q[j];
      }
    } else {  // two floats
      const f32x2 q = *reinterpret_cast<const f32x2*>(p);
      wf[0] = q.x; wf[1] = q.y;
    }
  }
};

// Router for large batches of layers with up to 16 experts, without the optional gate parts.  One 512-thread block per CU
// copies W_gate into LDS once (as float64 when that fits RS_W_BYTES, else as float: both exact) and then walks over groups
// of 64 tokens (two histogram blocks of TPB tokens), eight tokens per wave, so that a matrix row costs an LDS read instead
// of a trip through the vector memory pipeline per TOK tokens.
// Lane l of a wave takes the columns 8l..8l+7 of every 512-column step of the token rows: a row is read with one contiguous
// 1 KiB load per wave and step.  A wave holds TOK tokens x NE experts of float64 sums at a time (at most 32, so that sums,
// the row registers and one converted matrix row fit the register file without spilling).
// A wave's work is a flat sequence of steps (group, pass of TOK tokens, 512 columns of the token rows); the loads of the
// step two ahead are issued before the arithmetic of the current step, across pass and group boundaries, and the first two
// steps are under way while W_gate is being copied.
// Sums are float64 FMAs in a fixed order per lane, then wave_sum_values: results do not depend on timing.
constexpr int RS_THREADS = 512, RS_WAVES = RS_THREADS / 64, RS_TOKENS = 64;
constexpr int RS_W_BYTES = 136 * 1024;

template <typename T, int NE, typename W>
__global__ __launch_bounds__(RS_THREADS) void router_stream_kernel(const T* __restrict__ x, const T* __restrict__ Wg,
                                                                  const float* __restrict__ bias, int ntok, int d,
                                                                  int N, int top_k, int32_t* __restrict__ topk_idx,
                                                                  float* __restrict__ topk_w,
                                                                  int32_t* __restrict__ blockhist) {
  constexpr int TOK = 32 / NE < 4 ? 32 / NE : 4;  // (more tokens: their row registers no longer fit)
  constexpr int V = TOK * NE, NPASS = 8 / TOK;
  constexpr int GB = rs_group_bytes(NE, sizeof(W));
  constexpr int HW = MODSE_MAX_EXPERTS + 1;
  __shared__ __attribute__((aligned(16))) char s_w[RS_W_BYTES];
  __shared__ double s_logit[RS_WAVES][TOK][NE];
  __shared__ int s_hist[2 * HW];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ngroups = (ntok + RS_TOKENS - 1) / RS_TOKENS;
  const int nhist = (ntok + TPB - 1) / TPB;
  const int nstep = (d + 511) >> 9;

  // the loader runs two steps ahead of the arithmetic
  Raw8<T> cur[TOK], nx1[TOK], nx2[TOK];
  int l_grp = blockIdx.x, l_pass = 0, l_st = 0;
  auto load_next = [&](Raw8<T> (&dst)[TOK]) {
    if (l_grp < ngroups) {
      const int tbase = l_grp * RS_TOKENS + wave * 8 + l_pass * TOK;
      const int c = min(l_st * 512 + lane * 8, d - 8);
#pragma unroll
      for (int tt = 0; tt < TOK; ++tt)  // rows past the end repeat the last token; never written
        dst[tt].load(x + (size_t)min(tbase + tt, ntok - 1) * d + c);
    }
    if (++l_st == nstep) {
      l_st = 0;
      if (++l_pass == NPASS) {
        l_pass = 0;
        l_grp += gridDim.x;
      }
    }
  };
  load_next(cur);
  load_next(nx1);

  for (int r = tid; r < d; r += RS_THREADS) {  // W_gate -> LDS; columns past N read as zero
    float wf[NE];
    if (N == NE) {
      load_row<NE>(Wg + (size_t)r * N, wf);
    } else {
#pragma unroll
      for (int e = 0; e < NE; ++e) wf[e] = e < N ? (float)Wg[(size_t)r * N + e] : 0.f;
    }
    W* dst = reinterpret_cast<W*>(s_w + (r >> 3) * GB + (r & 7) * NE * (int)sizeof(W));
#pragma unroll
    for (int e = 0; e < NE; ++e) dst[e] = (W)wf[e];
  }
  if (tid < 2 * HW) s_hist[tid] = 0;
  __syncthreads();

  for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    for (int pass = 0; pass < NPASS; ++pass) {
      const int tbase = grp * RS_TOKENS + wave * 8 + pass * TOK;
      const LdsRows<W, NE> rows = {s_w};
      double acc[V];
#pragma unroll
      for (int i = 0; i < V; ++i) acc[i] = 0.0;
      for (int st = 0; st < nstep; ++st) {
        load_next(nx2);
        const int c = st * 512 + lane * 8;
        if (c < d) {
          W wf[NE];
          rows.fetch(c, wf);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            W wn[NE];
            if (i < 7) rows.fetch(c + i + 1, wn);  // the next matrix row is on its way during this row's arithmetic
            double wd[NE];
#pragma unroll
            for (int e = 0; e < NE; ++e) wd[e] = (double)wf[e];
#pragma unroll
            for (int tt = 0; tt < TOK; ++tt) {
              const double xd = (double)cur[tt].get(i);
#pragma unroll
              for (int e = 0; e < NE; ++e) acc[tt * NE + e] = fma(xd, wd[e], acc[tt * NE + e]);
            }
            if (i < 7) {
#pragma unroll
              for (int e = 0; e < NE; ++e) wf[e] = wn[e];
            }
            // keeps the scheduler from fetching and converting all eight rows ahead of the arithmetic, which costs more
            // registers than there are
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int tt = 0; tt < TOK; ++tt) {
          cur[tt] = nx1[tt];
          nx1[tt] = nx2[tt];
        }
      }
      wave_sum_values<V>(acc, lane);
      if (lane < V) {
        const int v = bitrev<Log2<V>::value>(lane);
        s_logit[wave][v / NE][v % NE] = acc[0];
      }
      __syncthreads();
      if (lane < TOK && tbase + lane < ntok) {
        const int t = tbase + lane;
        if (bias)
          for (int e = 0; e < N; ++e) s_logit[wave][lane][e] += (double)bias[e];
        const TopPick p = pick_top(s_logit[wave][lane], N);
        const bool near = write_gate(p, t, N, top_k, topk_idx, topk_w);
        int* hist = s_hist + (wave >> 2) * HW;  // waves 0-3 hold the group's first TPB tokens
        atomicAdd(&hist[p.i1], 1);
        if (top_k == 2) atomicAdd(&hist[p.i2], 1);
        if (near) atomicAdd(&hist[N], 1);
      }
      __syncthreads();
    }
    if (tid < 2 * HW) {  // the thread that writes a counter out also clears it for the next group
      const int h = tid / HW, i = tid % HW, b = grp * 2 + h;
      if (i <= N && b < nhist) blockhist[(size_t)b * (N + 1) + i] = s_hist[tid];
      s_hist[tid] = 0;
    }
  }
}

// The same router on the float64 matrix instruction (v_mfma_f64_4x4x4_4b_f64: four independent 4 x 4 x 4 products
// per wave instruction; 64 float64 TFLOP/s measured on this chip against 50 for v_fma_f64 with two resident waves,
// and the conversions and LDS reads no longer compete with the multiply-adds for issue slots).  Operand lane
// 16 k + 4 b + i holds A_b[i][k] (or B_b[k][i]); result lane 16 i + 4 b + j holds D_b[i][j] (checked with a
// one-hot probe).  Here block b, row i is token 4 b + i of a set of 16, column j is expert 4 g + j of expert group g,
// and k runs over the columns of x: one x value per lane and instruction, converted to float64 (exact; the products
// of two bf16 values and their float64 sums are the same as the vector router's up to the order of the additions).
// One 512-thread block per CU keeps W_gate in LDS as float64 and walks over 64-token groups.  Wave w takes the
// columns [w d/8, (w+1) d/8) of all 64 tokens (four sets of 16), so a W value read from LDS serves four matrix
// instructions; a lane loads 16 bytes of a token row (8 columns) at a time, 16 rows x 64 consecutive bytes per wave
// instruction, two steps of 32 columns ahead, across groups.  The eight waves' partial sums meet in LDS and are added
// in a fixed order; then one thread per token does top-k, gate and the block histogram, as in the vector router.
// Needs d % 256 == 0 and the float64 copy of W_gate (d x NE x 8 bytes, NE = 8 or 16) in RM_W_BYTES.
constexpr int RM_THREADS = 512, RM_WAVES = RM_THREADS / 64, RM_TOKENS = 64, RM_SETS = RM_TOKENS / 16;
constexpr int rm_w_bytes(int NE) { return NE <= 8 ? 128 * 1024 : 112 * 1024; }

template <typename T, int NE>
__global__ __launch_bounds__(RM_THREADS) void router_mfma_kernel(const T* __restrict__ x, const T* __restrict__ Wg,
                                                                const float* __restrict__ bias, int ntok, int d, int N,
                                                                int top_k, int32_t* __restrict__ topk_idx,
                                                                float* __restrict__ topk_w,
                                                                int32_t* __restrict__ blockhist) {
  static_assert(NE == 8 || NE == 16, "expert groups of four; rows of 64 or 128 bytes");
  constexpr int EG = NE / 4;  // expert groups
  constexpr int HW = MODSE_MAX_EXPERTS + 1;
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) double s_w[rm_w_bytes(NE) / 8];  // [column][j][g] = W_gate[column][4 g + j]
  __shared__ double s_part[RM_WAVES / 2][RM_TOKENS][NE];
  __shared__ int s_hist[2 * HW];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, blk = (lane >> 2) & 3, ij = lane & 3;
  const int ngroups = (ntok + RM_TOKENS - 1) / RM_TOKENS;
  const int nhist = (ntok + TPB - 1) / TPB;
  const int wcols = d / RM_WAVES, nstep = wcols / 32;
  const int col0 = wave * wcols + kq * 8;  // this lane's first column

  // the loader runs two steps ahead of the arithmetic
  Raw8<T> cur[RM_SETS], nx1[RM_SETS], nx2[RM_SETS];
  int l_grp = blockIdx.x, l_st = 0;
  auto load_next = [&](Raw8<T> (&dst)[RM_SETS]) {
    if (l_grp < ngroups) {
      const int c = col0 + l_st * 32;
#pragma unroll
      for (int q = 0; q < RM_SETS; ++q) {  // rows past the end repeat the last token; never written
        const int t = min(l_grp * RM_TOKENS + q * 16 + blk * 4 + ij, ntok - 1);
        dst[q].load(x + (size_t)t * d + c);
      }
    }
    if (++l_st == nstep) {
      l_st = 0;
      l_grp += gridDim.x;
    }
  };
  load_next(cur);
  load_next(nx1);

  for (int r = tid; r < d; r += RM_THREADS) {  // W_gate -> LDS; columns past N read as zero
    float wf[NE];
    if (N == NE) {
      load_row<NE>(Wg + (size_t)r * N, wf);
    } else {
#pragma unroll
      for (int e = 0; e < NE; ++e) wf[e] = e < N ? (float)Wg[(size_t)r * N + e] : 0.f;
    }
    double* dst = s_w + (size_t)r * NE;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int g = 0; g < EG; ++g) dst[j * EG + g] = (double)wf[4 * g + j];
  }
  if (tid < 2 * HW) s_hist[tid] = 0;
  __syncthreads();

  for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    double acc[RM_SETS][EG];
#pragma unroll
    for (int q = 0; q < RM_SETS; ++q)
#pragma unroll
      for (int g = 0; g < EG; ++g) acc[q][g] = 0.0;
    for (int st = 0; st < nstep; ++st) {
      load_next(nx2);
      const double* wrow = s_w + (size_t)(col0 + st * 32) * NE + ij * EG;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        double b[EG];
#pragma unroll
        for (int g2 = 0; g2 < EG / 2; ++g2) {
          const f64x2 v = *reinterpret_cast<const f64x2*>(wrow + m * NE + 2 * g2);
          b[2 * g2] = v[0];
          b[2 * g2 + 1] = v[1];
        }
#pragma unroll
        for (int q = 0; q < RM_SETS; ++q) {
          const double a = (double)cur[q].get(m);
#pragma unroll
          for (int g = 0; g < EG; ++g) acc[q][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b[g], acc[q][g], 0, 0, 0);
        }
      }
#pragma unroll
      for (int q = 0; q < RM_SETS; ++q) {
        cur[q] = nx1[q];
        nx1[q] = nx2[q];
      }
    }
    // result lane 16 i + 4 b + j: token 4 b + i of the set, expert 4 g + j.  Waves 4-7 hand their sums to waves
    // 0-3, which add their own and leave four partial sums per logit.
    const int tloc = blk * 4 + kq;
    if (wave >= RM_WAVES / 2) {
#pragma unroll
      for (int q = 0; q < RM_SETS; ++q)
#pragma unroll
        for (int g = 0; g < EG; ++g) s_part[wave - RM_WAVES / 2][q * 16 + tloc][4 * g + ij] = acc[q][g];
    }
    __syncthreads();
    if (wave < RM_WAVES / 2) {
#pragma unroll
      for (int q = 0; q < RM_SETS; ++q)
#pragma unroll
        for (int g = 0; g < EG; ++g) {
          double* p = &s_part[wave][q * 16 + tloc][4 * g + ij];
          *p = acc[q][g] + *p;
        }
    }
    __syncthreads();
    const int tbase = grp * RM_TOKENS;
    if (tid < RM_TOKENS && tbase + tid < ntok) {
      const int t = tbase + tid;
      for (int e = 0; e < N; ++e) {
        double l = (s_part[0][tid][e] + s_part[1][tid][e]) + (s_part[2][tid][e] + s_part[3][tid][e]);
        if (bias) l += (double)bias[e];
        s_part[0][tid][e] = l;
      }
      const TopPick p = pick_top(s_part[0][tid], N);
      const bool near = write_gate(p, t, N, top_k, topk_idx, topk_w);
      int* hist = s_hist + (tid / TPB) * HW;  // the group's first and second TPB tokens
      atomicAdd(&hist[p.i1], 1);
      if (top_k == 2) atomicAdd(&hist[p.i2], 1);
      if (near) atomicAdd(&hist[N], 1);
    }
    __syncthreads();
    if (tid < 2 * HW) {  // the thread that writes a counter out also clears it for the next group
      const int h = tid / HW, i = tid % HW, b = grp * 2 + h;
      if (i <= N && b < nhist) blockhist[(size_t)b * (N + 1) + i] = s_hist[tid];
      s_hist[tid] = 0;
    }
  }
}

// EPL consecutive elements of a router matrix row as loaded, and element i of them as float
template <typename T, int EPL>
struct RawRow;
template <int EPL>
struct RawRow<bf16_t, EPL> {
  typedef std::conditional_t<EPL == 1, uint16_t, std::conditional_t<EPL == 2, uint32_t, uint64_t>> word_t;
  word_t v;
  __device__ void load(const bf16_t* p) { v = *reinterpret_cast<const word_t*>(p); }
  __device__ float get(int i) const { return __uint_as_float((uint32_t)(uint16_t)(v >> (16 * i)) << 16); }
};
template <int EPL>
struct RawRow<float, EPL> {
  typedef float vec_t __attribute__((ext_vector_type(EPL)));
  vec_t v;
  __device__ void load(const float* p) { v = *reinterpret_cast<const vec_t*>(p); }
  __device__ float get(int i) const { return v[i]; }
};
template <>
struct RawRow<float, 1> {
  float v;
  __device__ void load(const float* p) { v = *p; }
  __device__ float get(int) const { return v; }
};

// Top-k of two sets of experts, every expert of a before every expert of b: equal values stay with a.
__device__ inline TopPick merge_top(const TopPick& a, const TopPick& b) {
  TopPick r;
  if (b.m1 > a.m1) {
    r.m1 = b.m1; r.i1 = b.i1;
    if (b.m2 > a.m1) { r.m2 = b.m2; r.i2 = b.i2; r.m3 = fmax(a.m1, b.m3); }
    else { r.m2 = a.m1; r.i2 = a.i1; r.m3 = fmax(a.m2, b.m2); }
  } else {
    r.m1 = a.m1; r.i1 = a.i1;
    if (b.m1 > a.m2) { r.m2 = b.m1; r.i2 = b.i1; r.m3 = fmax(a.m2, b.m2); }
    else { r.m2 = a.m2; r.i2 = a.i2; r.m3 = fmax(a.m3, b.m1); }
  }
  return r;
}

// Logits -> routing of 16 lanes' token (lanes t16 = 0..15 of an aligned group; `on`: the token exists): each lane holds
// PER consecutive logits l[], experts t16 * PER .., and, with the noise term, their x W_n in u[].  All lanes return the
// pick; lane 0 has written topk_idx / topk_w.  Sums over experts run over a fixed tree.
template <int PER, bool NOISE>
__device__ inline TopPick route_token16(double (&l)[PER], double (&u)[PER], int t16, int t, bool on, int N, int top_k,
                                        const GateExtPtrs& G, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                        bool& near) {
  const int e0 = t16 * PER;
  if constexpr (NOISE) {  // H(x)_e += gamma s_e / sqrt(mean_i s_i^2 + eps),  s = softplus(x W_n)
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (e0 + i < N) {
        if (on) G.noise_pre[(size_t)t * N + e0 + i] = (float)u[i];
        u[i] = softplus_f64(u[i]);
        ss += u[i] * u[i];
      }
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) ss += shfl_xor_f64(ss, m);
    const double scale = (double)G.gamma[0] / sqrt(ss / N + (double)G.eps);
#pragma unroll
    for (int i = 0; i < PER; ++i) l[i] += scale * u[i];
  }
  TopPick p = {-INFINITY, -INFINITY, -INFINITY, -1, -1};
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const double v = e0 + i < N ? l[i] : -INFINITY;
    if (v > p.m1) {
      p.m3 = p.m2; p.m2 = p.m1; p.i2 = p.i1; p.m1 = v; p.i1 = e0 + i;
    } else if (v > p.m2) {
      p.m3 = p.m2; p.m2 = v; p.i2 = e0 + i;
    } else if (v > p.m3) {
      p.m3 = v;
    }
  }
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    TopPick o;
    o.m1 = shfl_xor_f64(p.m1, m); o.m2 = shfl_xor_f64(p.m2, m); o.m3 = shfl_xor_f64(p.m3, m);
    o.i1 = __shfl_xor(p.i1, m, 64); o.i2 = __shfl_xor(p.i2, m, 64);
    p = (t16 & m) ? merge_top(o, p) : merge_top(p, o);
  }
  if (p.i1 < 0) p.i1 = 0;                                     // every logit is -inf
  if (p.i2 < 0 || p.i2 == p.i1) p.i2 = p.i1 == 0 ? 1 : 0;     // no second one above -inf (see pick_top)
  near = false;
  if (on && t16 == 0) near = write_gate(p, t, N, top_k, topk_idx, topk_w);
  if (G.probs) {  // p(x) = softmax over all N logits (Sec. 3.2 Eq. 11)
    double ex[PER], den = 0.0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      ex[i] = e0 + i < N ? exp(l[i] - p.m1) : 0.0;
      den += ex[i];
    }
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) den += shfl_xor_f64(den, m);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (on && e0 + i < N) G.probs[(size_t)t * N + e0 + i] = (float)(ex[i] / den);
  }
  return p;
}

// Router for more than 16 experts and for the optional gate parts (noise term: NOISE; probabilities: G.probs), on
// v_mfma_f64_16x16x4_f64.  Operand lane 16 k + i holds A[i][k] (or B[k][i]); result lane 16 q + j, register r holds
// D[4 r + q][j] (checked with a one-hot probe).  Rows are 16 tokens, columns 16 experts (or, up to 8 experts with the
// noise term, 8 experts and their noise columns); the order of the contraction is free, so lane 16 q + i takes the eight
// columns 8q .. 8q+7 of a 32-column step of its token row (one 16-byte load) and the matrix rows that go with them.  A
// lane reads EPL neighbouring experts of a matrix row at once: column j of group g is expert EPL j + g.
// A block of eight waves takes 32 tokens; wave w takes the column steps w, w + 8, ...; the matrices come from L2 (32
// tokens share a read) straight into operand order, and the eight partial sums meet in LDS in a fixed order.
// Bound by the float64 matrix pipe: 73 TFLOP/s of a probe, 29 us for 8192 tokens, d = 2048, 64 experts, where the launch
// takes 46 us; the vector-FMA form before it, which fetched every matrix row for two tokens, took 178.
constexpr int RW_THREADS = 512, RW_WAVES = RW_THREADS / 64, RW_TOKENS = 32;
static_assert(RW_TOKENS == TPB && RW_TOKENS * 16 == RW_THREADS, "one histogram block per group; 16 threads per token");
template <typename T, int NE, bool NOISE>
__global__ __launch_bounds__(RW_THREADS) void router_kernel(const T* __restrict__ x, const T* __restrict__ Wg,
                                                           const float* __restrict__ bias, int ntok, int d, int N,
                                                           int top_k, int32_t* __restrict__ topk_idx,
                                                           float* __restrict__ topk_w, int32_t* __restrict__ blockhist,
                                                           GateExtPtrs G) {
  constexpr int EPL = NE <= 16 ? 1 : NE / 16, PER = EPL;
  constexpr bool SHARE = NOISE && NE <= 8;       // gate and noise columns share one group of 16
  constexpr int NM = NOISE && !SHARE ? 2 : 1;    // passes over the token rows: W_gate, W_noise (both at once do not fit the registers)
  constexpr int NG = EPL;                        // column groups per pass over the token rows
  constexpr int CP = 16 * NM * NG + 1;           // (+1: the rows of a column read start in different banks)
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  __shared__ double s_part[RW_WAVES / 2][RW_TOKENS][CP];
  __shared__ int s_hist[MODSE_MAX_EXPERTS + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, j = lane & 15;
  const int ngroups = (ntok + RW_TOKENS - 1) / RW_TOKENS;
  const int nstep = (d / 32 - wave + RW_WAVES - 1) / RW_WAVES;  // this wave's column steps
  const T* Wn = static_cast<const T*>(G.W_noise);
  // this lane's columns of the matrix rows (lanes without a column repeat one; their results are not used)
  const T* wsrc[NM];
  if constexpr (SHARE) wsrc[0] = j < 8 ? Wg + min(j, NE - 1) : Wn + min(j - 8, NE - 1);
  else {
    wsrc[0] = Wg + min(j * EPL, NE - EPL);
    if constexpr (NM == 2) wsrc[1] = Wn + min(j * EPL, NE - EPL);
  }
  struct Step {
    Raw8<T> x[2];
    RawRow<T, EPL> w[8];
  };
  Step cur, nxt;
  int l_grp = blockIdx.x, l_pass = 0, l_st = 0;
  auto load_next = [&](Step& s) {  // one step ahead of the arithmetic, across groups
    if (l_grp >= ngroups || nstep <= 0) return;
    const int c = (wave + l_st * RW_WAVES) * 32 + q * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h)  // rows past the end repeat the last token; never written
      s.x[h].load(x + (size_t)min(l_grp * RW_TOKENS + h * 16 + j, ntok - 1) * d + c);
    const T* w = NM == 2 && l_pass ? wsrc[NM - 1] : wsrc[0];
#pragma unroll
    for (int m = 0; m < 8; ++m) s.w[m].load(w + (size_t)(c + m) * NE);
    if (++l_st == nstep) {
      l_st = 0;
      if (++l_pass == NM) {
        l_pass = 0;
        l_grp += gridDim.x;
      }
    }
  };
  load_next(cur);
  if (tid <= MODSE_MAX_EXPERTS) s_hist[tid] = 0;

  for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
#pragma unroll 1
    for (int pass = 0; pass < NM; ++pass) {
      f64x4 acc[2][NG];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[h][g] = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int st = 0; st < nstep; ++st) {
        load_next(nxt);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const double a0 = (double)cur.x[0].get(m), a1 = (double)cur.x[1].get(m);
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            const double b = (double)cur.w[m].get(g);
            acc[0][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b, acc[0][g], 0, 0, 0);
            acc[1][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b, acc[1][g], 0, 0, 0);
          }
        }
        cur = nxt;
      }
      // waves 4-7 hand their sums to waves 0-3, which add their own and leave four partial sums per value
      auto part = [&](int w, int h, int g, int r) -> double& {
        return s_part[w][h * 16 + 4 * r + q][(pass * NG + g) * 16 + j];
      };
      if (wave >= RW_WAVES / 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) part(wave - RW_WAVES / 2, h, g, r) = acc[h][g][r];
      }
      __syncthreads();
      if (wave < RW_WAVES / 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) part(wave, h, g, r) = acc[h][g][r] + part(wave, h, g, r);
      }
    }
    __syncthreads();
    // sixteen threads per token
    const int t16 = tid & 15, tl = tid >> 4, t = grp * RW_TOKENS + tl;
    double l[PER], u[PER];
    auto total = [&](int c) { return (s_part[0][tl][c] + s_part[1][tl][c]) + (s_part[2][tl][c] + s_part[3][tl][c]); };
#pragma unroll
    for (int i = 0; i < PER; ++i) {  // expert t16 * EPL + i: column t16 of group i
      const int e = t16 * PER + i;
      l[i] = total(i * 16 + t16) + ((bias && e < N) ? (double)bias[e] : 0.0);
      u[i] = NOISE ? total(SHARE ? 8 + (t16 & 7) : (EPL * (NM - 1) + i) * 16 + t16) : 0.0;
    }
    bool near;
    const TopPick p = route_token16<PER, NOISE>(l, u, t16, t, t < ntok, N, top_k, G, topk_idx, topk_w, near);
    if (t16 == 0 && t < ntok) {
      atomicAdd(&s_hist[p.i1], 1);
      if (top_k == 2) atomicAdd(&s_hist[p.i2], 1);
      if (near) atomicAdd(&s_hist[N], 1);
    }
    __syncthreads();
    if (tid <= N) {  // the thread that writes a counter out also clears it for the next group
      blockhist[(size_t)grp * (N + 1) + tid] = s_hist[tid];
      s_hist[tid] = 0;
    }
  }
}

// ---------------------------------------------------------------- screened router
// Plain gate, bf16, more than 16 experts: of a token's logits only the top k and their rivals matter in float64.  A first
// launch takes all logits on the bf16 matrix pipe with a bound of their error and keeps, per token, the experts that can
// be among the top k or within the near-tie distance of them; a second one takes those experts' dot products in
// float64 and decides as the other routers do.  The decision and the gate weights are therefore the same float64 results.
//
// Bound of the error: a product of two bf16 values is exact in float32, and whatever the order in which the matrix pipe adds
// up n terms, and if it truncates, each of the additions is off by at most 2^-23 of the sum of the terms' magnitudes.  That
// sum is at most |x| |w|, the lengths of the token's row and the expert's column.  A wave adds d / 8 terms (and the
// accumulator, once per 32), so gamma = 1.1 (d / 8 + 64) 2^-23 times |x| |w| covers it (4e-5 of it at d = 2048, 1.5e-3
// for logits of deviation 0.9: a few of a hundred tokens get more than k candidates).  What the lengths lose of values
// below 2^-63, whose squares are subnormal, and the matrix pipe of subnormal inputs is less than d 2^-32 of |x| |w| as
// long as no length exceeds 2^30; of a longer row, of one with an infinity or no number, and of all rows if a column is such,
// all experts are left to the second launch.  The logits of a row of zeros are the bias: its top k + 1 are found here.
//
// 64 experts, d = 2048, 8192 tokens: the launches take 12.7 and 11.5 us, the general router 46.9 (float64 matrix pipe); routing
// call 55.0 -> 35.1.  The first is a chain of latencies (loads, then the sums and bounds of a token: 8 + 4 us), the second
// half float64 arithmetic, half the same.  Tried on the first without gain: sixteen waves of half as many steps, blocks
// that start at different columns, loops that are not unrolled (14.7).
// The second launch's time depends on the candidates.  Routing call at d = 2048, ordinary values / every tenth row zero / W_gate = 0 (all
// experts of all tokens, see exact_crowd) / the general router: 64 experts 8192 tokens 33 / 39 / 63 / 56 us, 32768 tokens 86 / 96 /
// 205 / 187; 32 experts 8192 tokens 29 / 35 / 43 / 36.  (With the candidates two at a time whatever their number and rows of zeros
// like the others 33 / 151 / 174, 86 / 357 / 612, 29 / 101 / 97.)
constexpr int SC_THREADS = 512, SC_WAVES = SC_THREADS / 64, SC_TOKENS = 32, SC_TRANSPOSE_ROWS = 64;
constexpr int SC_CROWD = 12;
constexpr double SC_NEAR = 1.1e-6;  // (the near-tie distance of write_gate, and some)
constexpr float SC_LARGE = 0x1p60f;  // square of the largest length
// Columns of W_gate as rows (the second launch reads them): 64 rows of W_gate per block.
__device__ inline void transpose_block(const bf16_t* __restrict__ W, int d, int N, int k0, bf16_t* __restrict__ Wt,
                                       bf16_t (*tile)[SC_TRANSPOSE_ROWS + 8]) {
  static_assert(SC_THREADS == 8 * MODSE_MAX_EXPERTS && SC_TRANSPOSE_ROWS == 64, "an expert per eight threads, a row per wave and round");
  const int rows = min(SC_TRANSPOSE_ROWS, d - k0), col = threadIdx.x & 63;
  bf16_t v[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int k = (threadIdx.x >> 6) + 8 * r;
    v[r] = col < N && k < rows ? W[(size_t)(k0 + k) * N + col] : (bf16_t)0.f;
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) tile[col][(threadIdx.x >> 6) + 8 * r] = v[r];
  __syncthreads();
  const int e = threadIdx.x >> 3, c = (threadIdx.x & 7) * 8;
  if (e < N && c < rows) *reinterpret_cast<bf16x8*>(Wt + (size_t)e * d + k0 + c) = *reinterpret_cast<const bf16x8*>(&tile[e][c]);
}
// cand_lo / cand_hi [t * top_k]: bits of token t's candidates.  crowd: a byte per four tokens, whose lowest bits say which have
// more than SC_CROWD of them.  The first nscreen blocks take 32 tokens each, the others transpose W (rows of N; Wg: the same in
// rows of NE).  blockhist (may be null) is cleared for the second launch.
template <int NE>
__global__ __launch_bounds__(SC_THREADS, 4) void router_screen_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wg,
                                                                   const bf16_t* __restrict__ W, const float* __restrict__ bias,
                                                                   int ntok, int d, int N, int top_k, int nscreen,
                                                                   uint32_t* __restrict__ cand_lo, uint32_t* __restrict__ cand_hi,
                                                                   uint8_t* __restrict__ crowd, bf16_t* __restrict__ Wt,
                                                                   int32_t* __restrict__ blockhist) {
  // A lane reads EPL neighbouring experts of eight matrix rows; column j of group g is expert EPL j + g.  TRADE: it reads
  // twice as many of four rows and trades half of them with lane j ^ 8, which has the next four rows (half as many loads; 64
  // experts 13.8 -> 12.7 us, but with 32 9.7 -> 11.0); column j of group g is then expert 2 EPL (j & 7) + EPL (j >> 3) + g.
  constexpr int EPL = NE / 16, WORDS = EPL / 2;
  constexpr bool TRADE = NE == 64;
  constexpr int LROWS = TRADE ? 4 : 8, LWORDS = TRADE ? 2 * WORDS : WORDS;
  struct Sums {
    float l[SC_WAVES / 2][SC_TOKENS][NE + 1];
    float x2[SC_WAVES][SC_TOKENS], w2[SC_WAVES][NE];  // squares of the lengths
  };
  __shared__ union {
    Sums part;
    bf16_t tile[MODSE_MAX_EXPERTS][SC_TRANSPOSE_ROWS + 8];
  } s;
  __shared__ int s_large;
  if ((int)blockIdx.x >= nscreen) {
    transpose_block(W, d, N, ((int)blockIdx.x - nscreen) * SC_TRANSPOSE_ROWS, Wt, s.tile);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, j = lane & 15, t0 = blockIdx.x * SC_TOKENS;
  if (tid == 0) s_large = 0;
  if (blockhist && tid <= N) blockhist[(size_t)blockIdx.x * (N + 1) + tid] = 0;
  const int nstep = (d / 32 - wave + SC_WAVES - 1) / SC_WAVES;  // this wave's steps of 32 columns: wave, wave + 8, ...
  struct Step {
    u32x4 x[2];
    uint32_t w[LROWS][LWORDS];
  };
  int xoff[2];  // (rows past the end repeat the last one; never written)
#pragma unroll
  for (int h = 0; h < 2; ++h) xoff[h] = min(h * 16 + j, ntok - 1 - t0) * d + q * 8;
  const int woff = TRADE ? (q * 8 + (j >> 3) * 4) * NE + (j & 7) * 2 * EPL : q * 8 * NE + j * EPL;
  auto load = [&](Step& st, int i) {
    const int c = (wave + min(i, nstep - 1) * SC_WAVES) * 32;
    const bf16_t* const xc = x + (size_t)t0 * d + c;
    const bf16_t* const wc = Wg + (size_t)c * NE;
#pragma unroll
    for (int h = 0; h < 2; ++h) st.x[h] = *reinterpret_cast<const u32x4*>(xc + xoff[h]);
#pragma unroll
    for (int m = 0; m < LROWS; ++m) {
      typedef uint32_t vec_t __attribute__((ext_vector_type(LWORDS)));
      const vec_t v = *reinterpret_cast<const vec_t*>(wc + woff + m * NE);
#pragma unroll
      for (int w = 0; w < LWORDS; ++w) st.w[m][w] = v[w];
    }
  };
  f32x4 acc[2][EPL];
  float x2[2] = {0.f, 0.f}, w2[EPL] = {};
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int g = 0; g < EPL; ++g) acc[h][g] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto add_squares = [](u32x4 v, float sum) {
    typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16x2 p = __builtin_bit_cast(bf16x2, (uint32_t)v[i]);
      sum = __builtin_amdgcn_fdot2_f32_bf16(p, p, sum, false);
    }
    return sum;
  };
  auto bf = [](u32x4 v) { return __builtin_bit_cast(bf16x8, v); };
  auto multiply = [&](const Step& st) {
#pragma unroll
    for (int h = 0; h < 2; ++h) x2[h] = add_squares(st.x[h], x2[h]);
    uint32_t row[8][WORDS];
#pragma unroll
    for (int m = 0; m < LROWS; ++m)
#pragma unroll
      for (int w = 0; w < WORDS; ++w) {
        if constexpr (TRADE) {  // row_ror:8, into lanes 8-15 of sixteen the upper experts of rows 0-3, into lanes 0-7 the lower ones of rows 4-7
          row[m][w] = __builtin_amdgcn_update_dpp(st.w[m][w], st.w[m][WORDS + w], 0x128, 0xf, 0xc, false);
          row[4 + m][w] = __builtin_amdgcn_update_dpp(st.w[m][WORDS + w], st.w[m][w], 0x128, 0xf, 0x3, false);
        } else {
          row[m][w] = st.w[m][w];
        }
      }
#pragma unroll
    for (int g = 0; g < EPL; ++g) {
      u32x4 w;  // eight rows of column j of group g
#pragma unroll
      for (int m = 0; m < 4; ++m)
        w[m] = __builtin_amdgcn_perm(row[2 * m + 1][g / 2], row[2 * m][g / 2], (g & 1) ? 0x07060302u : 0x05040100u);
      w2[g] = add_squares(w, w2[g]);
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[h][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf(st.x[h]), bf(w), acc[h][g], 0, 0, 0);
    }
  };
  if (nstep > 0) {  // two steps ahead (the fences keep the compiler from moving the loads to their uses)
    Step buf[3];
    load(buf[0], 0);
    load(buf[1], 1);
    int i = 0;
#pragma unroll 1
    for (; i + 3 <= nstep; i += 3) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        load(buf[(b + 2) % 3], i + b + 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(buf[b]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (i < nstep) multiply(buf[0]);
    if (i + 1 < nstep) multiply(buf[1]);
  }
  // result lane 16 q + j, register r: token 4 q + r of the half, column j.  Waves 4-7 hand their sums to waves 0-3.
  auto put = [&](int w, auto add) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int g = 0; g < EPL; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float& l = s.part.l[w][h * 16 + 4 * q + r][g * 16 + j];
          l = acc[h][g][r] + (decltype(add)::value ? l : 0.f);
        }
  };
  if (wave >= SC_WAVES / 2) put(wave - SC_WAVES / 2, std::false_type{});
  auto over_quarters = [](float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
  };
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float v = over_quarters(x2[h]);
    if (q == h) s.part.x2[wave][h * 16 + j] = v;
  }
#pragma unroll
  for (int g = 0; g < EPL; ++g) {
    const float v = over_quarters(w2[g]);
    if (q == g) s.part.w2[wave][g * 16 + j] = v;
  }
  __syncthreads();
  if (wave < SC_WAVES / 2) put(wave, std::true_type{});
  // the lengths: of token tid, of column tid - 32
  float len = 0.f;
  const bool is_x = tid < SC_TOKENS;
  if (tid < SC_TOKENS + NE) {
#pragma unroll
    for (int w = 0; w < SC_WAVES; ++w) len += is_x ? s.part.x2[w][tid] : s.part.w2[w][tid - SC_TOKENS];
    if (!is_x && !(len <= SC_LARGE)) s_large = 1;
  }
  __syncthreads();
  if (is_x) s.part.x2[0][tid] = len <= SC_LARGE ? sqrtf(len) : INFINITY;
  else if (tid < SC_TOKENS + NE) s.part.w2[0][tid - SC_TOKENS] = sqrtf(len);
  __syncthreads();
  // sixteen threads per token, EPL experts each
  const int tl = tid >> 4, t16 = tid & 15, t = t0 + tl;
  auto expert = [&](int i) { return TRADE ? 2 * EPL * (t16 & 7) + EPL * (t16 >> 3) + i : EPL * t16 + i; };
  const float xlen = s.part.x2[0][tl];
  const bool large = s_large || xlen == INFINITY;
  const double gamma = 1.1 * (d / 8 + 64) * 0x1p-23;
  double hi[EPL], m1 = -INFINITY, m2 = -INFINITY;  // m1, m2: the largest lower bounds
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = expert(i), c = i * 16 + t16;
    double l = 0.0;
#pragma unroll
    for (int w = 0; w < SC_WAVES / 2; ++w) l += (double)s.part.l[w][tl][c];
    const double err = gamma * ((double)(xlen * s.part.w2[0][c]) + d * 0x1p-32) + 1e-12;
    double lo = l - err;
    hi[i] = l + err;
    if (bias) {  // (rounded as the exact logit will be: a bias may be so large that this matters)
      const double b = e < N ? (double)bias[e] : 0.0;
      lo += b;
      hi[i] += b;
    }
    if (e >= N) lo = -INFINITY;
    if (lo > m1) {
      m2 = m1;
      m1 = lo;
    } else if (lo > m2) {
      m2 = lo;
    }
  }
#pragma unroll
  for (int b = 1; b < 16; b <<= 1) {
    const double o1 = shfl_xor_f64(m1, b), o2 = shfl_xor_f64(m2, b);
    m2 = o1 > m1 ? fmax(m1, o2) : fmax(o1, m2);
    m1 = fmax(m1, o1);
  }
  const double least = (top_k == 2 ? m2 : m1) - SC_NEAR;
  uint64_t mask = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = expert(i);
    if (e < N && (large || hi[i] >= least)) mask |= 1ull << e;
  }
  if (xlen == 0.f && !large) {  // a row of zeros, or of values whose squares are
    const bf16_t* const row = x + (size_t)min(t, ntok - 1) * d;
    uint32_t bits = 0;
#pragma unroll 4
    for (int c = t16 * 8; c < d; c += 128) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(row + c);
      bits |= v[0] | v[1] | v[2] | v[3];
    }
#pragma unroll
    for (int b = 1; b < 16; b <<= 1) bits |= __shfl_xor(bits, b, 64);
    if ((bits & 0x7fff7fffu) == 0) {  // its logits are the bias: the first top_k + 1 decide (most often all experts tie)
      mask = 0;
#pragma unroll
      for (int i = 0; i < EPL; ++i) hi[i] = bias && expert(i) < N ? (double)bias[expert(i)] : 0.0;
#pragma unroll 1
      for (int r = 0; r <= top_k; ++r) {
        double best = -INFINITY;
        int at = N;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const int e = expert(i);
          if (e < N && !(mask >> e & 1) && hi[i] > best) {
            best = hi[i];
            at = e;
          }
        }
#pragma unroll
        for (int b = 1; b < 16; b <<= 1) {
          const double o = shfl_xor_f64(best, b);
          const int oe = __shfl_xor(at, b, 64);
          if (o > best || (o == best && oe < at)) {
            best = o;
            at = oe;
          }
        }
        if (at < N) mask |= 1ull << at;
      }
    }
  }
#pragma unroll
  for (int b = 1; b < 16; b <<= 1) {
    const uint32_t lo32 = __shfl_xor((uint32_t)mask, b, 64), hi32 = __shfl_xor((uint32_t)(mask >> 32), b, 64);
    mask |= ((uint64_t)hi32 << 32) | lo32;
  }
  if (t16 == 0 && t < ntok) {
    cand_lo[(size_t)t * top_k] = (uint32_t)mask;
    cand_hi[(size_t)t * top_k] = (uint32_t)(mask >> 32);
  }
  const uint64_t crowded = __ballot(t16 == 0 && t < ntok && __popcll(mask) > SC_CROWD);  // bits 0, 16, 32 and 48
  if (lane == 0) crowd[blockIdx.x * SC_WAVES + wave] = (crowded | crowded >> 15 | crowded >> 30 | crowded >> 45) & 15;
}

// The candidates' dot products in float64, top-k and gate: 32 threads per token, two candidates at a time, in ascending
// order.  topk_idx and topk_w hold the token's candidates when the launch starts.  A sum runs over a thread's columns and then
// over a fixed tree.
// A round of two takes 4.7 us at 8192 tokens, d = 2048, and a token may have all experts for candidates (columns of W_gate that
// are equal or zero, rows and columns beyond the error bound).  Tokens of more than SC_CROWD candidates therefore take all logits,
// from the float64 matrix pipe (exact_crowd), which is as long as six or seven rounds.  Which way a token goes depends on its row,
// W_gate and the bias alone, and so do the bits of its gate weights.
constexpr int EX_LANES = 32, EX_TOKENS = 8, EX_THREADS = EX_LANES * EX_TOKENS, EX_CROWD_TOKENS = 2 * EX_TOKENS;
template <int NE>
struct CrowdLds {
  double part[2][EX_CROWD_TOKENS][NE + 1];
};
// Decides for those of the sixteen tokens from t0 on that are in `crowd` (a byte per four tokens).  Operand lanes as in
// router_kernel; a wave takes every fourth step of 32 columns.  (The instruction of router_mfma_kernel would fit a block's eight
// tokens, but then W_gate is read for every eight: 32768 tokens with W_gate = 0, 64 experts 327 us, this 205.)
template <int NE>
__device__ inline void exact_crowd(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wt, const float* __restrict__ bias,
                                   uint32_t crowd, int t0, int ntok, int d, int N, int top_k, int32_t* topk_idx, float* topk_w,
                                   int32_t* __restrict__ blockhist, int32_t* __restrict__ near_flag, CrowdLds<NE>& s) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  constexpr int NG = NE / 16, WAVES = EX_THREADS / 64;
  static_assert(EX_CROWD_TOKENS == 16 && EX_THREADS == 16 * 16 && WAVES == 4, "sixteen threads per token, two pairs of waves");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, j = lane & 15, nstep = (d / 32 - wave + WAVES - 1) / WAVES;
  // (tokens and experts that are not there repeat the last; not used)
  const bf16_t* const row = x + (size_t)min(t0 + j, ntok - 1) * d + q * 8;
  const bf16_t* col[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) col[g] = Wt + (size_t)min(g * 16 + j, N - 1) * d + q * 8;
  f64x4 acc[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) acc[g] = f64x4{0.0, 0.0, 0.0, 0.0};
  struct Step {
    Raw8<bf16_t> x, w[NG];
  };
  auto load = [&](Step& st, int i) {
    const int c = (wave + min(i, nstep - 1) * WAVES) * 32;
    st.x.load(row + c);
#pragma unroll
    for (int g = 0; g < NG; ++g) st.w[g].load(col[g] + c);
  };
  if (nstep > 0) {
    Step cur, nxt;
    load(cur, 0);
#pragma unroll 1
    for (int i = 0; i < nstep; ++i) {
      load(nxt, i + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const double a = (double)cur.x.get(m);
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)cur.w[g].get(m), acc[g], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      cur = nxt;
    }
  }
#pragma unroll
  for (int half = 0; half < 2; ++half) {  // waves 2 and 3 hand their sums to waves 0 and 1
    if ((wave >= 2) == (half == 0)) {
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double& v = s.part[wave & 1][4 * r + q][g * 16 + j];
          v = half == 0 ? acc[g][r] : acc[g][r] + v;
        }
    }
    __syncthreads();
  }
  const int tl = tid >> 4, t16 = tid & 15, t = t0 + tl;
  const bool on = (crowd >> (8 * (tl >> 2) + (tl & 3)) & 1) != 0;
  double l[NG], u[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int e = t16 * NG + i;
    l[i] = s.part[0][tl][e] + s.part[1][tl][e] + (bias && e < N ? (double)bias[e] : 0.0);
    u[i] = 0.0;
  }
  bool near;
  const TopPick p = route_token16<NG, false>(l, u, t16, t, on, N, top_k, GateExtPtrs{}, topk_idx, topk_w, near);
  if (on && t16 == 0) {
    if (near_flag) {
      near_flag[t] = near ? 1 : 0;
    } else {
      int32_t* const hist = blockhist + (size_t)(t / TPB) * (N + 1);
      atomicAdd(&hist[p.i1], 1);
      if (top_k == 2) atomicAdd(&hist[p.i2], 1);
      if (near) atomicAdd(&hist[N], 1);
    }
  }
}
template <int NE>
__global__ __launch_bounds__(EX_THREADS, 4) void router_exact_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wt,
                                                                     const float* __restrict__ bias,
                                                                     const uint32_t* __restrict__ crowd_words, int ntok, int d, int N,
                                                                     int top_k, int32_t* topk_idx, float* topk_w,
                                                                     int32_t* __restrict__ blockhist,
                                                                     int32_t* __restrict__ near_flag) {
  __shared__ int s_hist[MODSE_MAX_EXPERTS + 1];
  __shared__ CrowdLds<NE> s_crowd;
  const int tid = threadIdx.x, tl = tid / EX_LANES, ln = tid % EX_LANES, t = blockIdx.x * EX_TOKENS + tl;
  if (tid <= MODSE_MAX_EXPERTS) s_hist[tid] = 0;
  // My own tokens' byte pair, and the sixteen tokens whose crowded ones are mine: those of the first half of the grid, which share
  // out evenly to the CUs (32768 tokens, W_gate = 0: 204 us, as tasks of every other block 349).
  const uint32_t crowd = crowd_words[blockIdx.x >> 1] >> (blockIdx.x & 1) * 16;
  const uint32_t task = blockIdx.x < (gridDim.x + 1) / 2 ? crowd_words[blockIdx.x] : 0;
  const size_t at = (size_t)min(t, ntok - 1) * top_k;
  uint64_t mask = ((uint64_t)__float_as_uint(topk_w[at]) << 32) | (uint32_t)topk_idx[at];  // (of a crowded token: anything)
  __syncthreads();
  if (task)
    exact_crowd<NE>(x, Wt, bias, task, blockIdx.x * EX_CROWD_TOKENS, ntok, d, N, top_k, topk_idx, topk_w, blockhist, near_flag, s_crowd);
  if (t < ntok && !(crowd >> (8 * (tl >> 2) + (tl & 3)) & 1)) {
    const bf16_t* const row = x + (size_t)t * d;
    TopPick p = {-INFINITY, -INFINITY, -INFINITY, -1, -1};
    auto consider = [&](double dot, int e) {
      const double l = dot + (bias ? (double)bias[e] : 0.0);
      if (l > p.m1) {
        p.m3 = p.m2; p.m2 = p.m1; p.i2 = p.i1; p.m1 = l; p.i1 = e;
      } else if (l > p.m2) {
        p.m3 = p.m2; p.m2 = l; p.i2 = e;
      } else if (l > p.m3) {
        p.m3 = l;
      }
    };
    while (mask) {
      int e[2];
      e[0] = __builtin_ctzll(mask);
      mask &= mask - 1;
      const bool two = mask != 0;
      e[1] = two ? __builtin_ctzll(mask) : e[0];
      mask &= mask - 1;  // (0 stays 0)
      const bf16_t* const w0 = Wt + (size_t)e[0] * d;
      const bf16_t* const w1 = Wt + (size_t)e[1] * d;
      double sum[2] = {0.0, 0.0};
      // `n` pieces of 256 columns from column c0 on, all their loads in flight at once (the fence keeps them there)
      auto pieces = [&](auto n, int c0) {
        constexpr int P = decltype(n)::value;
        Raw8<bf16_t> xv[P], wv[2][P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const int c = c0 + (i * EX_LANES + ln) * 8;
          xv[i].load(row + c);
          wv[0][i].load(w0 + c);
          wv[1][i].load(w1 + c);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
          for (int m = 0; m < 8; ++m) {
            const double xd = (double)xv[i].get(m);
            sum[0] = fma(xd, (double)wv[0][i].get(m), sum[0]);
            sum[1] = fma(xd, (double)wv[1][i].get(m), sum[1]);
          }
      };
      int c0 = 0;
      for (; c0 + 4 * EX_LANES * 8 <= d; c0 += 4 * EX_LANES * 8) pieces(std::integral_constant<int, 4>{}, c0);
      for (; c0 + ln * 8 < d; c0 += EX_LANES * 8) pieces(std::integral_constant<int, 1>{}, c0);
#pragma unroll
      for (int b = 1; b < EX_LANES; b <<= 1) {
        sum[0] += shfl_xor_f64(sum[0], b);
        sum[1] += shfl_xor_f64(sum[1], b);
      }
      consider(sum[0], e[0]);
      if (two) consider(sum[1], e[1]);
    }
    if (p.i1 < 0) p.i1 = 0;                                  // every logit is -inf
    if (p.i2 < 0 || p.i2 == p.i1) p.i2 = p.i1 == 0 ? 1 : 0;  // no second one above -inf (see pick_top)
    if (ln == 0) {
      const bool near = write_gate(p, t, N, top_k, topk_idx, topk_w);
      if (near_flag) near_flag[t] = near ? 1 : 0;
      atomicAdd(&s_hist[p.i1], 1);
      if (top_k == 2) atomicAdd(&s_hist[p.i2], 1);
      if (near) atomicAdd(&s_hist[N], 1);
    }
  }
  if (near_flag) return;  // (the permutation of a small batch counts by itself)
  __syncthreads();
  static_assert(TPB % EX_TOKENS == 0, "the tokens of a block belong to one histogram");
  if (tid <= N && s_hist[tid]) atomicAdd(&blockhist[(size_t)(blockIdx.x * EX_TOKENS / TPB) * (N + 1) + tid], s_hist[tid]);
}

// Router without the optional gate parts: one block per G tokens, the 256 threads split the d columns, so
// a token row and the router matrix are read once with 16-byte loads and the whole dot product is one or
// two rounds of memory latency.  Every thread leaves its G x N float64 partial sums in LDS; they are added
// in two fixed-order steps (8 groups of 32 threads, then the 8 group sums), so the result does not depend
// on timing; one thread per token then does top-k and gate.  The block histograms that the permutation
// needs are counted by the permutation itself from topk_idx and near_flag.
template <typename T, int NE, int G>
__global__ __launch_bounds__(ROUTE_THREADS, 2) void router_token_kernel(const T* __restrict__ x,
                                                                       const T* __restrict__ Wg,
                                                                       const float* __restrict__ bias, int ntok, int d,
                                                                       int N, int top_k,
                                                                       int32_t* __restrict__ topk_idx,
                                                                       float* __restrict__ topk_w,
                                                                       int32_t* __restrict__ near_flag) {
  constexpr int V = G * NE;
  static_assert(V <= 32, "one thread per value and group in the second reduction step");
  __shared__ double s_part[ROUTE_THREADS][V + 1];  // (+1: rows start in different banks)
  __shared__ double s_group[8][V];
  __shared__ double s_logit[G][NE];
  const int tid = threadIdx.x, t0 = blockIdx.x * G;
  double acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0.0;
  for (int c = tid * 8; c < d; c += ROUTE_THREADS * 8) {
    float xv[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) load8(x + (size_t)min(t0 + g, ntok - 1) * d + c, xv[g]);  // (clamped rows: never written)
    float wf[NE];
    load_row<NE>(Wg + (size_t)c * NE, wf);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float wn[NE];
      if (i < 7) load_row<NE>(Wg + (size_t)(c + i + 1) * NE, wn);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const double wd = (double)wf[e];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g * NE + e] = fma((double)xv[g][i], wd, acc[g * NE + e]);
      }
      if (i < 7) {
#pragma unroll
        for (int e = 0; e < NE; ++e) wf[e] = wn[e];
      }
      __builtin_amdgcn_sched_barrier(0);  // (as in router_stream_kernel: one row ahead, no more)
    }
  }
#pragma unroll
  for (int v = 0; v < V; ++v) s_part[tid][v] = acc[v];
  __syncthreads();
  {
    const int v = tid & 31, grp = tid >> 5;
    if (v < V) {
      double sum = 0.0;
      for (int i = 0; i < 32; ++i) sum += s_part[grp * 32 + i][v];
      s_group[grp][v] = sum;
    }
  }
  __syncthreads();
  if (tid < V) {
    double sum = 0.0;
    for (int q = 0; q < 8; ++q) sum += s_group[q][tid];
    const int e = tid % NE;
    s_logit[tid / NE][e] = sum + ((bias && e < N) ? (double)bias[e] : 0.0);
  }
  __syncthreads();
  if (tid < G && t0 + tid < ntok) {
    const int t = t0 + tid;
    const TopPick p = pick_top(s_logit[tid], N);
    near_flag[t] = write_gate(p, t, N, top_k, topk_idx, topk_w) ? 1 : 0;
  }
}

// The one-block-per-token(s) router for more than 16 experts: sixteen threads share a matrix row (EPL = NE / 16
// neighbouring experts each), the block's sixteen such groups share the columns of d, eight consecutive ones at a time.
// A matrix row read serves the block's G tokens.  Sums are added in a fixed order: four groups of a wave by shuffles,
// then the four waves through LDS.
template <typename T, int NE, int G>
__global__ __launch_bounds__(ROUTE_THREADS) void router_token_wide_kernel(const T* __restrict__ x, const T* __restrict__ Wg,
                                                                         const float* __restrict__ bias, int ntok, int d,
                                                                         int N, int top_k, int32_t* __restrict__ topk_idx,
                                                                         float* __restrict__ topk_w,
                                                                         int32_t* __restrict__ near_flag) {
  constexpr int EPL = NE / 16;
  static_assert(G * 16 <= ROUTE_THREADS, "sixteen threads per token in the last step");
  __shared__ double s_part[ROUTE_THREADS / 64][G][NE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, t16 = tid & 15, t0 = blockIdx.x * G;
  double acc[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.0;
  const T* row[G];
#pragma unroll
  for (int g = 0; g < G; ++g) row[g] = x + (size_t)min(t0 + g, ntok - 1) * d;  // (clamped rows: never written)
#pragma unroll 2
  for (int c = (tid >> 4) * 8; c < d; c += ROUTE_THREADS / 16 * 8) {
    RawRow<T, EPL> w[8];
    Raw8<T> xv[G];
#pragma unroll
    for (int m = 0; m < 8; ++m) w[m].load(Wg + (size_t)(c + m) * NE + t16 * EPL);
#pragma unroll
    for (int g = 0; g < G; ++g) xv[g].load(row[g] + c);
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const double wd = (double)w[m].get(e);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g][e] = fma((double)xv[g].get(m), wd, acc[g][e]);
      }
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      double v = acc[g][e];
      v += shfl_xor_f64(v, 16);
      v += shfl_xor_f64(v, 32);
      if (lane < 16) s_part[wave][g][t16 * EPL + e] = v;
    }
  __syncthreads();
  const int g = tid >> 4, t = t0 + g;
  if (g < G) {
    double l[EPL], u[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int e = t16 * EPL + i;
      l[i] = (s_part[0][g][e] + s_part[1][g][e]) + (s_part[2][g][e] + s_part[3][g][e]) + ((bias && e < N) ? (double)bias[e] : 0.0);
      u[i] = 0.0;
    }
    bool near;
    route_token16<EPL, false>(l, u, t16, t, t < ntok, N, top_k, GateExtPtrs{}, topk_idx, topk_w, near);
    if (t16 == 0 && t < ntok) near_flag[t] = near ? 1 : 0;
  }
}

// Single block.  Turns blockhist[b][e] into the exclusive prefix over blocks (in place), writes counts, offsets
// and the near-tie total and, when a forward pass follows, the tile plans of its two GEMMs (from the counts
// still in LDS: no second launch, no round trip through memory).  The launch is a chain of memory latencies and nothing
// else.  The table lies [block][column]: a thread owns one column and a run of blocks, neighbours own neighbouring
// columns, so that a step reads whole lines, and up to SCAN_NB blocks of a thread are loaded at once and stay in registers
// for the second pass.  64 experts, 8192 tokens (65 columns of 256 blocks): 7 us in place of 46 with 16 columns per
// pass; 8 experts, 16384 tokens: 7 to 11 in place of 12 to 19.
constexpr int SCAN_THREADS = 1024, SCAN_NB = 20;
__global__ __launch_bounds__(SCAN_THREADS) void route_scan_kernel(int32_t* __restrict__ blockhist, int nb, int N,
                                                                  int32_t* __restrict__ counts,
                                                                  int32_t* __restrict__ offsets,
                                                                  int32_t* __restrict__ near_tie_count, LayerDims L,
                                                                  int esize, FwdPlanArgs plan, int with_plan) {
  __shared__ int s_part[SCAN_THREADS];  // [run][column]
  __shared__ int s_total[MODSE_MAX_EXPERTS + 1];
  __shared__ int s_counts[MODSE_MAX_EXPERTS], s_offsets[MODSE_MAX_EXPERTS];
  __shared__ modse_gemm::PlanLds s_plan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = N + 1, nrun = SCAN_THREADS / W, per = (nb + nrun - 1) / nrun;
  const int c = tid % W, run_of = tid / W;
  const int b0 = run_of < nrun ? min(run_of * per, nb) : nb, b1 = min(b0 + per, nb);
  int32_t* const col = blockhist + c;
  int v[SCAN_NB], sum = 0;
  for (int b = b0; b < b1; b += SCAN_NB) {
#pragma unroll
    for (int q = 0; q < SCAN_NB; ++q) v[q] = b + q < b1 ? col[(size_t)(b + q) * W] : 0;
#pragma unroll
    for (int q = 0; q < SCAN_NB; ++q) sum += v[q];
  }
  if (run_of < nrun) s_part[run_of * W + c] = sum;
  __syncthreads();
  for (int j = wave; j < W; j += SCAN_THREADS / 64) {  // exclusive scan of column j's run totals (at most 512: W >= 2)
    constexpr int PER = 8;
    const int n = (nrun + 63) / 64;
    int p[PER], local = 0, total;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int r = lane * n + i;
      p[i] = i < n && r < nrun ? s_part[r * W + j] : 0;
      local += p[i];
    }
    int run = modse_gemm::wave_exclusive(local, lane, total);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int r = lane * n + i;
      if (i < n && r < nrun) s_part[r * W + j] = run;
      run += p[i];
    }
    if (lane == 0) s_total[j] = total;
  }
  __syncthreads();
  if (c < N && run_of < nrun) {  // (the near-tie column, c == N, keeps its counts)
    int run = s_part[run_of * W + c];
    for (int b = b0; b < b1; b += SCAN_NB) {
      if (per > SCAN_NB) {
#pragma unroll
        for (int q = 0; q < SCAN_NB; ++q) v[q] = b + q < b1 ? col[(size_t)(b + q) * W] : 0;
      }
#pragma unroll
      for (int q = 0; q < SCAN_NB; ++q)
        if (b + q < b1) {
          col[(size_t)(b + q) * W] = run;
          run += v[q];
        }
    }
  }
  if (wave == 0) {
    const int n = lane < N ? s_total[lane] : 0;
    int total;
    const int o = modse_gemm::wave_exclusive(n, lane, total);
    if (lane < N) {
      counts[lane] = s_counts[lane] = n;
      offsets[lane] = s_offsets[lane] = o;
    }
    if (lane == 0) {
      offsets[N] = total;
      near_tie_count[0] = s_total[N];
    }
  }
  if (with_plan) {
    __syncthreads();
    modse_gemm::plan_fwd_body(L, esize, s_counts, s_offsets, plan, s_plan);
  }
}

// Auxiliary load-balance loss (Sec. 3.2 Eq. 9-12), single block: f_i = share of tokens whose first choice is
// expert i, P_i = mean of p_i, L_a = alpha N sum_i f_i P_i.  A thread sums one column over every nrow-th token (threads
// side by side read whole lines of p, sixteen loads in flight), the threads' sums of a column are added in a fixed tree,
// so the result does not depend on timing.  The sums over batches of sixteen are float64: a thread adds up to ntok N / 1024
// values in a row, which in float32 put P off by 7e-7 at 2^20 tokens and 64 experts.  8192 tokens, 8 experts: 8 to 12 us in
// place of 61 to 83 with one pass over all tokens per expert.
constexpr int AUX_THREADS = 1024;
__global__ __launch_bounds__(AUX_THREADS) void aux_finish_kernel(const float* __restrict__ probs,
                                                                 const int32_t* __restrict__ topk_idx, int ntok, int N,
                                                                 int top_k, float alpha, float* __restrict__ f_out,
                                                                 float* __restrict__ P_out, float* __restrict__ loss) {
  __shared__ double s_p[AUX_THREADS];
  __shared__ int s_c[MODSE_MAX_EXPERTS];
  const int tid = threadIdx.x;
  if (tid < N) s_c[tid] = 0;
  const int nrow = AUX_THREADS / N, e = tid % N, r0 = tid / N;
  double acc = 0.0;
  if (r0 < nrow) {
    int t = r0;
    for (; (long)t + 15L * nrow < ntok; t += 16 * nrow) {
      float v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = probs[(size_t)(t + q * nrow) * N + e];
#pragma unroll
      for (int half = 8; half >= 2; half >>= 1)
#pragma unroll
        for (int q = 0; q < half; ++q) v[q] += v[q + half];
      acc += (double)v[0] + (double)v[1];
    }
#pragma unroll 16
    for (; t < ntok; t += nrow) acc += (double)probs[(size_t)t * N + e];
  }
  s_p[tid] = acc;
  __syncthreads();
#pragma unroll 8
  for (int t = tid; t < ntok; t += AUX_THREADS) atomicAdd(&s_c[topk_idx[(size_t)t * top_k]], 1);
  for (int n = nrow; n > 1;) {  // rows r and r + half of the table [nrow][N]
    const int half = (n + 1) / 2;
    if (r0 < n - half) s_p[tid] += s_p[tid + half * N];
    n = half;
    __syncthreads();
  }
  if (tid < 64) {
    double l = 0.0;
    if (tid < N) {
      const double P = s_p[tid] / ntok, f = (double)s_c[tid] / ntok;
      f_out[tid] = (float)f;
      P_out[tid] = (float)P;
      l = f * P;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) l += shfl_xor_f64(l, m);
    if (tid == 0) loss[0] = (float)((double)alpha * N * l);
  }
}

// Routing statistics in the shape of the paper's Appendix A tables, single block: slot_counts[j][i] = tokens
// whose j-th choice is expert i; summary[j] = max/min of row j, summary[k] = max/min of the per-expert
// totals, summary[k+1] = average hidden width of the chosen experts (Sec. 4.3).
__global__ __launch_bounds__(256) void routing_stats_kernel(const int32_t* __restrict__ topk_idx, int ntok, int N,
                                                            int top_k, LayerDims L, int32_t* __restrict__ slot_counts,
                                                            float* __restrict__ summary) {
  __shared__ int s_cnt[2][MODSE_MAX_EXPERTS];
  const int tid = threadIdx.x;
  if (tid < 2 * MODSE_MAX_EXPERTS) (&s_cnt[0][0])[tid] = 0;
  __syncthreads();
  for (int i = tid; i < ntok * top_k; i += 256) atomicAdd(&s_cnt[i % top_k][topk_idx[i]], 1);
  __syncthreads();
  for (int i = tid; i < top_k * N; i += 256) slot_counts[i] = s_cnt[i / N][i % N];
  if (tid == 0) {
    double wsum = 0.0;
    long tot_all = 0;
    int tmax = 0, tmin = INT_MAX;
    for (int e = 0; e < N; ++e) {
      const int tot = s_cnt[0][e] + (top_k == 2 ? s_cnt[1][e] : 0);
      tmax = max(tmax, tot);
      tmin = min(tmin, tot);
      wsum += (double)tot * L.f[e];
      tot_all += tot;
    }
    for (int j = 0; j < top_k; ++j) {
      int mx = 0, mn = INT_MAX;
      for (int e = 0; e < N; ++e) {
        mx = max(mx, s_cnt[j][e]);
        mn = min(mn, s_cnt[j][e]);
      }
      summary[j] = mn > 0 ? (float)mx / (float)mn : INFINITY;
    }
    summary[top_k] = tmin > 0 ? (float)tmax / (float)tmin : INFINITY;
    summary[top_k + 1] = tot_all > 0 ? (float)(wsum / (double)tot_all) : 0.f;
  }
}

// Stable scatter: permuted row = offsets[e] + (assignments to e in earlier blocks) + (earlier tokens of this
// block routed to e).  Also copies the token rows into expert-contiguous order when Xp is given.
template <typename T>
__global__ __launch_bounds__(ROUTE_THREADS) void scatter_kernel(const T* __restrict__ x, int ntok, int d, int N,
                                                                int top_k, const int32_t* __restrict__ topk_idx,
                                                                const int32_t* __restrict__ offsets,
                                                                const int32_t* __restrict__ blockbase,
                                                                int32_t* __restrict__ row_of,
                                                                int32_t* __restrict__ src_of, T* __restrict__ Xp,
                                                                int parts) {
  __shared__ int s_row[TPB][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int block = blockIdx.x / parts, part = blockIdx.x % parts;  // parts: blocks that share the copies of TPB tokens
  const int t0 = block * TPB;
  if (wave == 0) {
    const int t = t0 + lane;
    const bool valid = lane < TPB && t < ntok;
    int e0 = -1, e1 = -1;
    if (valid) {
      e0 = topk_idx[(size_t)t * top_k];
      if (top_k == 2) e1 = topk_idx[(size_t)t * top_k + 1];
    }
    int r0 = 0, r1 = 0;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int e = 0; e < N; ++e) {
      const unsigned long long m = __ballot(e0 == e || e1 == e);
      const int rank = __popcll(m & below);
      if (e0 == e) r0 = rank;
      if (e1 == e) r1 = rank;
    }
    if (valid) {
      const int32_t* bb = blockbase + (size_t)block * (N + 1);
      const int row0 = offsets[e0] + bb[e0] + r0;
      if (part == 0) {
        row_of[(size_t)t * top_k] = row0;
        src_of[row0] = t * top_k;
      }
      s_row[lane][0] = row0;
      if (top_k == 2) {
        const int row1 = offsets[e1] + bb[e1] + r1;
        if (part == 0) {
          row_of[(size_t)t * top_k + 1] = row1;
          src_of[row1] = t * top_k + 1;
        }
        s_row[lane][1] = row1;
      }
    }
  }
  __syncthreads();
  if (Xp == nullptr) return;
  for (int tl = part * 4 + wave; tl < TPB; tl += parts * 4) {
    const int t = t0 + tl;
    if (t >= ntok) break;
    const int row0 = s_row[tl][0];
    const int row1 = top_k == 2 ? s_row[tl][1] : -1;
    constexpr int VEC = 16 / sizeof(T);
    for (int c = lane * VEC; c < d; c += 64 * VEC) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(x + (size_t)t * d + c);
      *reinterpret_cast<f32x4*>(Xp + (size_t)row0 * d + c) = v;
      if (row1 >= 0) *reinterpret_cast<f32x4*>(Xp + (size_t)row1 * d + c) = v;
    }
  }
}

// Decode-sized batches of layers with few experts, one token per lane of a wave: histogram, offsets, stable scatter and, when
// a forward pass follows, the tile plans of its two GEMMs in one launch of small blocks.  Wave 0 of every block ranks all
// tokens with one ballot per expert (the same rows as scatter_kernel: tokens of an expert in token order).  The first block
// writes the routing outputs and makes the plans, block 1 + t copies token t's row (no such blocks when there is no Xp).
// Near-tie total: from near_flag (the routers with one or four tokens per block) or, when that is null, from the last
// column of the router's block histograms.
// Bound by latency: 4 barriers and 16 waves less than permute_fused_kernel, but a step per expert.  The routing call, replayed
// from a graph: one token, 8 experts, d = 256: 5.3 us in place of 7.1; 64 tokens, 16 experts: 7.4 / 8.9, but 64 experts
// 10.0 / 9.0; a forward pass of 64 tokens with 32 or 64 experts is 1 to 2.5 us slower with it, with 8 to 16 0.2 to 0.7 faster.
constexpr int PS_THREADS = 256, PS_EXPERTS = 16;
static_assert(MODSE_PERMUTE_SMALL_MAX_T <= 64, "a token per lane");
template <typename T>
__global__ __launch_bounds__(PS_THREADS) void permute_small_kernel(const T* __restrict__ x, int ntok, int d, int N, int top_k,
                                                                   const int32_t* __restrict__ topk_idx,
                                                                   const int32_t* __restrict__ near_flag,
                                                                   const int32_t* __restrict__ blockhist, RoutingPtrs R,
                                                                   T* __restrict__ Xp, LayerDims L, int esize,
                                                                   FwdPlanArgs plan, int with_plan) {
  __shared__ int s_row[2];  // of the block's token
  __shared__ int s_counts[MODSE_MAX_EXPERTS], s_offsets[MODSE_MAX_EXPERTS];
  __shared__ modse_gemm::PlanLds s_plan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool planner = blockIdx.x == 0;
  const int mine = (int)blockIdx.x - 1;
  if (wave == 0) {
    const int t = lane;
    const bool valid = t < ntok;
    const int e0 = valid ? topk_idx[(size_t)t * top_k] : -1;
    const int e1 = valid && top_k == 2 ? topk_idx[(size_t)t * top_k + 1] : -1;
    const unsigned long long below = (1ull << lane) - 1ull;
    int run = 0, row0 = 0, row1 = 0, my_count = 0, my_offset = 0;
#pragma unroll 4
    for (int e = 0; e < N; ++e) {
      const unsigned long long m = __ballot(e0 == e || e1 == e);
      const int rank = __popcll(m & below), c = __popcll(m);
      if (e0 == e) row0 = run + rank;
      if (e1 == e) row1 = run + rank;
      if (lane == e) {
        my_count = c;
        my_offset = run;
      }
      run += c;
    }
    if (t == mine) {
      s_row[0] = row0;
      s_row[1] = row1;
    }
    if (planner) {
      int near = 0;
      if (near_flag) {
        near = __popcll(__ballot(valid && near_flag[valid ? t : 0] != 0));
      } else {
        for (int b = 0; b * TPB < ntok; ++b) near += blockhist[(size_t)b * (N + 1) + N];
      }
      if (lane < N) {
        R.counts[lane] = s_counts[lane] = my_count;
        R.offsets[lane] = s_offsets[lane] = my_offset;
      }
      if (lane == 0) {
        R.offsets[N] = run;
        R.near_tie_count[0] = near;
      }
      if (valid) {
        R.row_of[(size_t)t * top_k] = row0;
        R.src_of[row0] = t * top_k;
        if (top_k == 2) {
          R.row_of[(size_t)t * top_k + 1] = row1;
          R.src_of[row1] = t * top_k + 1;
        }
      }
    }
  }
  __syncthreads();
  if (planner) {
    if (with_plan) modse_gemm::plan_fwd_body(L, esize, s_counts, s_offsets, plan, s_plan);
    return;
  }
  const int row0 = s_row[0], row1 = top_k == 2 ? s_row[1] : -1;
  constexpr int VEC = 16 / sizeof(T);
  for (int c = tid * VEC; c < d; c += PS_THREADS * VEC) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(x + (size_t)mine * d + c);
    *reinterpret_cast<f32x4*>(Xp + (size_t)row0 * d + c) = v;
    if (row1 >= 0) *reinterpret_cast<f32x4*>(Xp + (size_t)row1 * d + c) = v;
  }
}

// Larger batches, of at most MODSE_PERMUTE_FUSED_MAX_T tokens: the same in one launch instead of three; at these sizes a
// launch costs more than its work.
// Every block counts all tokens' choices by itself (at most 32 KiB from the L2), those of the tokens before its own
// sixteen apart from the rest, so no block waits for another.  A counter has 32 copies side by side, lane l of a wave adding
// to copy l mod 32: at most two additions of a wave meet in a word.  The first block writes the routing totals and makes the
// plans, the others rank their tokens (the same rows as scatter_kernel: tokens of an expert in token order) and copy their
// rows.
// Near-tie total: from near_flag (the routers with one or four tokens per block) or, when that is null, from the last
// column of the router's block histograms.
// d = 2048, 389 / 2048 tokens: 7 / 11 us in place of 5 + 13 + 13 (15) and two launch gaps (blocks of 256 threads and eight
// tokens: 8 / 15).
constexpr int PF_TOKENS = 16, PF_THREADS = 1024;
template <typename T>
__global__ __launch_bounds__(PF_THREADS) void permute_fused_kernel(const T* __restrict__ x, int ntok, int d, int N, int top_k,
                                                            const int32_t* __restrict__ topk_idx,
                                                            const int32_t* __restrict__ near_flag,
                                                            const int32_t* __restrict__ blockhist, RoutingPtrs R,
                                                            T* __restrict__ Xp, LayerDims L, int esize,
                                                            FwdPlanArgs plan, int with_plan) {
  constexpr int COPIES = 32;
  __shared__ int s_cnt[2 * MODSE_MAX_EXPERTS * COPIES];  // [before my tokens, from them on][expert][copy]
  __shared__ int s_sum[2 * MODSE_MAX_EXPERTS];
  __shared__ int s_base[MODSE_MAX_EXPERTS];  // first row of my tokens' rows of an expert
  __shared__ int s_counts[MODSE_MAX_EXPERTS], s_offsets[MODSE_MAX_EXPERTS];
  __shared__ int s_row[PF_TOKENS][2], s_near;
  __shared__ modse_gemm::PlanLds s_plan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool planner = blockIdx.x == 0;
  const int t0 = planner ? ntok : (int)(blockIdx.x - 1) * PF_TOKENS;
  for (int i = tid; i < 2 * N * COPIES; i += PF_THREADS) s_cnt[i] = 0;
  if (tid == 0) s_near = 0;
  __syncthreads();
  const int n = ntok * top_k, before = t0 * top_k;
#pragma unroll 8
  for (int i = tid; i < n; i += PF_THREADS) atomicAdd(&s_cnt[((i < before ? 0 : N) + topk_idx[i]) * COPIES + (tid & (COPIES - 1))], 1);
  if (planner) {
    int near = 0;
    if (near_flag) {
      for (int t = tid; t < ntok; t += PF_THREADS) near += near_flag[t] != 0 ? 1 : 0;
    } else {
      for (int b = tid; b * TPB < ntok; b += PF_THREADS) near += blockhist[(size_t)b * (N + 1) + N];
    }
    if (near) atomicAdd(&s_near, near);
  }
  __syncthreads();
  for (int i = tid; i < 2 * N * 8; i += PF_THREADS) {  // eight threads add up a counter's copies (whole groups of lanes run)
    int sum = 0;
#pragma unroll
    for (int q = 0; q < COPIES / 8; ++q) sum += s_cnt[i / 8 * COPIES + q * 8 + (i & 7)];
#pragma unroll
    for (int m = 4; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
    if ((i & 7) == 0) s_sum[i / 8] = sum;
  }
  __syncthreads();
  if (wave == 0) {
    const int b = lane < N ? s_sum[lane] : 0, c = lane < N ? b + s_sum[N + lane] : 0;
    int total;
    const int o = modse_gemm::wave_exclusive(c, lane, total);
    if (lane < N) {
      s_base[lane] = o + b;
      s_counts[lane] = c;
      s_offsets[lane] = o;
      if (planner) {
        R.counts[lane] = c;
        R.offsets[lane] = o;
      }
    }
    if (planner && lane == 0) {
      R.offsets[N] = total;
      R.near_tie_count[0] = s_near;
    }
  }
  __syncthreads();
  if (planner) {
    if (with_plan) modse_gemm::plan_fwd_body(L, esize, s_counts, s_offsets, plan, s_plan);
    return;
  }
  if (wave == 0) {
    const int t = t0 + lane;
    const bool valid = lane < PF_TOKENS && t < ntok;
    const int e0 = valid ? topk_idx[(size_t)t * top_k] : -1;
    const int e1 = valid && top_k == 2 ? topk_idx[(size_t)t * top_k + 1] : -1;
    int r0 = 0, r1 = 0;  // my block's earlier tokens with the same expert
#pragma unroll 5
    for (int i = 0; i < PF_TOKENS - 1; ++i) {
      const int a = __shfl(e0, i, 64), b = __shfl(e1, i, 64);
      if (i < lane) {
        r0 += a == e0 || b == e0 ? 1 : 0;
        r1 += a == e1 || b == e1 ? 1 : 0;
      }
    }
    if (valid) {
      const int row0 = s_base[e0] + r0;
      R.row_of[(size_t)t * top_k] = row0;
      R.src_of[row0] = t * top_k;
      s_row[lane][0] = row0;
      if (top_k == 2) {
        const int row1 = s_base[e1] + r1;
        R.row_of[(size_t)t * top_k + 1] = row1;
        R.src_of[row1] = t * top_k + 1;
        s_row[lane][1] = row1;
      }
    }
  }
  __syncthreads();
  if (Xp == nullptr) return;
  constexpr int VEC = 16 / sizeof(T);
  static_assert(PF_TOKENS == PF_THREADS / 64, "a wave copies one token");
  const int tl = wave;
  if (t0 + tl < ntok) {
    const int row0 = s_row[tl][0], row1 = top_k == 2 ? s_row[tl][1] : -1;
    const T* const src = x + (size_t)(t0 + tl) * d;
#pragma unroll 4
    for (int c = lane * VEC; c < d; c += 64 * VEC) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + c);
      *reinterpret_cast<f32x4*>(Xp + (size_t)row0 * d + c) = v;
      if (row1 >= 0) *reinterpret_cast<f32x4*>(Xp + (size_t)row1 * d + c) = v;
    }
  }
}

// Batches beyond that: the same over the router's block histograms, whose rows of W = N + 1 counters every block adds up by itself,
// those of the blocks before its own apart (PERMUTE_HIST_MAX counters, 128 KiB from the L2, at most), so that no scan has to come
// before.  The first block writes the totals and makes the plans, block 1 + b ranks and copies the tokens of histogram b.  What
// that costs grows with the square of the batch: see permute_by_hist for the batches that take it.
constexpr int PH_THREADS = 1024, PH_RUNS = 32;
template <typename T>
__global__ __launch_bounds__(PH_THREADS) void permute_hist_kernel(const T* __restrict__ x, int ntok, int d, int N, int top_k,
                                                                  const int32_t* __restrict__ topk_idx,
                                                                  const int32_t* __restrict__ blockhist, int nb, RoutingPtrs R,
                                                                  T* __restrict__ Xp, LayerDims L, int esize, FwdPlanArgs plan,
                                                                  int with_plan) {
  __shared__ int s_part[2][PH_THREADS];  // [before my block, all][run of blocks][column]
  __shared__ int s_sum[2][MODSE_MAX_EXPERTS + 1];
  __shared__ int s_base[MODSE_MAX_EXPERTS];  // first row of my tokens' rows of an expert
  __shared__ int s_counts[MODSE_MAX_EXPERTS], s_offsets[MODSE_MAX_EXPERTS];
  __shared__ int s_row[TPB][2];
  __shared__ modse_gemm::PlanLds s_plan;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool planner = blockIdx.x == 0;
  const int mine = planner ? nb : (int)blockIdx.x - 1, t0 = mine * TPB;
  const int W = N + 1, nrun = min(PH_THREADS / W, PH_RUNS), c = tid % W, run = tid / W;
  int before = 0, all = 0;
  if (run < nrun) {
#pragma unroll 8
    for (int b = run; b < nb; b += nrun) {
      const int v = blockhist[(size_t)b * W + c];
      all += v;
      before += b < mine ? v : 0;
    }
  }
  s_part[0][tid] = before;
  s_part[1][tid] = all;
  __syncthreads();
  if (tid < 2 * W) {
    const int which = tid / W, col = tid % W;
    int sum = 0;
#pragma unroll 8
    for (int r = 0; r < nrun; ++r) sum += s_part[which][r * W + col];
    s_sum[which][col] = sum;
  }
  __syncthreads();
  if (wave == 0) {
    const int n = lane < N ? s_sum[1][lane] : 0;
    int total;
    const int o = modse_gemm::wave_exclusive(n, lane, total);
    if (lane < N) {
      s_base[lane] = o + s_sum[0][lane];
      s_counts[lane] = n;
      s_offsets[lane] = o;
      if (planner) {
        R.counts[lane] = n;
        R.offsets[lane] = o;
      }
    }
    if (planner && lane == 0) {
      R.offsets[N] = total;
      R.near_tie_count[0] = s_sum[1][N];
    }
  }
  __syncthreads();
  if (planner) {
    if (with_plan) modse_gemm::plan_fwd_body(L, esize, s_counts, s_offsets, plan, s_plan);
    return;
  }
  if (wave == 0) {
    const int t = t0 + lane;
    const bool valid = lane < TPB && t < ntok;
    const int e0 = valid ? topk_idx[(size_t)t * top_k] : -1;
    const int e1 = valid && top_k == 2 ? topk_idx[(size_t)t * top_k + 1] : -1;
    int r0 = 0, r1 = 0;  // my block's earlier tokens with the same expert
#pragma unroll 8
    for (int i = 0; i < TPB - 1; ++i) {
      const int a = __builtin_amdgcn_readlane(e0, i), b = __builtin_amdgcn_readlane(e1, i);
      if (i < lane) {
        r0 += a == e0 || b == e0 ? 1 : 0;
        r1 += a == e1 || b == e1 ? 1 : 0;
      }
    }
    if (valid) {
      const int row0 = s_base[e0] + r0;
      R.row_of[(size_t)t * top_k] = row0;
      R.src_of[row0] = t * top_k;
      s_row[lane][0] = row0;
      if (top_k == 2) {
        const int row1 = s_base[e1] + r1;
        R.row_of[(size_t)t * top_k + 1] = row1;
        R.src_of[row1] = t * top_k + 1;
        s_row[lane][1] = row1;
      }
    }
  }
  __syncthreads();
  if (Xp == nullptr) return;
  constexpr int VEC = 16 / sizeof(T);
  for (int tl = wave; tl < TPB && t0 + tl < ntok; tl += PH_THREADS / 64) {
    const int row0 = s_row[tl][0], row1 = top_k == 2 ? s_row[tl][1] : -1;
    const T* const src = x + (size_t)(t0 + tl) * d;
#pragma unroll 4
    for (int q = lane * VEC; q < d; q += 64 * VEC) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + q);
      *reinterpret_cast<f32x4*>(Xp + (size_t)row0 * d + q) = v;
      if (row1 >= 0) *reinterpret_cast<f32x4*>(Xp + (size_t)row1 * d + q) = v;
    }
  }
}

// y[t] = sum_j g[t,j] * O[row_of[t,j]]   (Eq. 1 on permuted expert outputs; one wave per token, fp32 math)
template <typename T>
__global__ __launch_bounds__(256) void combine_kernel(const T* __restrict__ O, int ntok, int d, int top_k,
                                                      const int32_t* __restrict__ row_of,
                                                      const float* __restrict__ topk_w, T* __restrict__ y) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= ntok) return;
  const int lane = threadIdx.x & 63;
  const int r0 = row_of[(size_t)t * top_k];
  const float g0 = topk_w[(size_t)t * top_k];
  const int r1 = top_k == 2 ? row_of[(size_t)t * top_k + 1] : 0;
  const float g1 = top_k == 2 ? topk_w[(size_t)t * top_k + 1] : 0.f;
  for (int c = lane * 8; c < d; c += 64 * 8) {
    float a[8], b[8], o[8];
    load8(O + (size_t)r0 * d + c, a);
    if (top_k == 2) {
      load8(O + (size_t)r1 * d + c, b);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = g0 * a[i] + g1 * b[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = g0 * a[i];
    }
    store8(y + (size_t)t * d + c, o);
  }
}

// acc[j] = the sum of the n[j] slabs at src[j], added in ascending order; the loads of the K rows go out side by side
template <int K>
__device__ inline void sum_slabs8(const float* const (&src)[K], size_t slab, const int (&n)[K], float (&acc)[K][8]) {
  int most = n[0];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    most = max(most, n[j]);
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[j][q] = 0.f;
  }
#pragma unroll 4
  for (int s = 0; s < most; ++s) {
    float v[K][8];
#pragma unroll
    for (int j = 0; j < K; ++j) load8(src[j] + min(s, n[j] - 1) * slab, v[j]);  // (a row with fewer slabs repeats its last)
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[j][q] = s < n[j] ? acc[j][q] + v[j][q] : acc[j][q];
  }
}

// Combine after a split-K down-projection: expert e's output rows are the sum of ceil(f_e / kchunk) float32
// partial slabs Opart[c] ([T*k, d] each), added in ascending c.  One thread per token and 8 columns.  O (may be null)
// receives the summed rows.
template <typename T>
__global__ __launch_bounds__(256) void combine_split_kernel(const float* __restrict__ Opart, int ntok, int d,
                                                            int top_k, LayerDims L, int kchunk,
                                                            const int32_t* __restrict__ topk_idx,
                                                            const int32_t* __restrict__ row_of,
                                                            const float* __restrict__ topk_w, T* __restrict__ O,
                                                            T* __restrict__ y) {
  const int per_tok = d / 8;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)ntok * per_tok) return;
  const int t = (int)(i / per_tok), c = (int)(i % per_tok) * 8;
  const size_t slab = (size_t)ntok * top_k * d;
  auto row = [&](auto two_tag) {
    constexpr int K = decltype(two_tag)::value ? 2 : 1;
    const float* src[K];
    int n[K];
    size_t at[K];
    float g[K], acc[K][8], o[8];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      n[j] = (L.f[topk_idx[(size_t)t * K + j]] + kchunk - 1) / kchunk;
      at[j] = (size_t)row_of[(size_t)t * K + j] * d + c;
      g[j] = topk_w[(size_t)t * K + j];
      src[j] = Opart + at[j];
    }
    sum_slabs8(src, slab, n, acc);
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = 0.f;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      if (O) store8(O + at[j], acc[j]);
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = fmaf(g[j], acc[j][q], o[q]);
    }
    store8(y + (size_t)t * d + c, o);
  };
  if (top_k == 2) row(std::true_type{});
  else row(std::false_type{});
}

// One thread per permuted row and 8 columns.
template <typename T>
__global__ __launch_bounds__(256) void sum_slabs_kernel(const float* __restrict__ slabs, int nrows, int d, LayerDims L,
                                                        int kchunk, int passes, const int32_t* __restrict__ topk_idx,
                                                        const int32_t* __restrict__ src_of, T* __restrict__ out) {
  const int per_row = d / 8;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)nrows * per_row) return;
  const int r = (int)(i / per_row), c = (int)(i % per_row) * 8;
  const int e = topk_idx[src_of[r]];
  const size_t at = (size_t)r * d + c;
  const float* const src[1] = {slabs + at};
  const int n[1] = {passes * ((L.f[e] + kchunk - 1) / kchunk)};
  float acc[1][8];
  sum_slabs8(src, (size_t)nrows * d, n, acc);
  store8(out + at, acc[0]);
}

// Backward of the combine, one wave per token: for its permuted rows r_j
//   dO[r_j] = g_j * dY[t]      d g_j = <dY[t], O[r_j]>
// and, where the gate has none of its optional parts (GATE), the gradient of the logits in the same breath:
//   dl_j = g_j (dg_j - sum_m g_m dg_m) on the kept logits (softmax over KeepTopK), 0 elsewhere.
// The first block makes the tile plans of the backward GEMMs beside the others, the blocks behind the tokens' (GATE) copy
// W_gate [d, N] to Wt [N, d] for bwd_gate_rows_kernel, 256 rows each.
// Bound by memory; dY is read once per token, not once per row, and the gate's gradient needs no launch.  d = 2048, 32768
// tokens: 131 -> 122 us; the launch of the gate's gradient took 4 to 6 us.
constexpr int PREP_TOKENS = 4;
template <typename T, bool GATE>
__global__ __launch_bounds__(256) void bwd_prep_plan_bwd_kernel(const T* __restrict__ dY, const T* __restrict__ O, RoutingPtrs R,
                                                                T* __restrict__ dO, float* __restrict__ dg,
                                                                LayerDims L, int esize, BwdPlanArgs plan,
                                                                float* __restrict__ dl, const T* __restrict__ Wg,
                                                                T* __restrict__ Wt) {
  __shared__ modse_gemm::PlanLds s_plan;
  __shared__ int s_counts[MODSE_MAX_EXPERTS], s_offsets[MODSE_MAX_EXPERTS];
  const int d = L.d, N = L.N, ntok = L.T, top_k = L.k;
  if (blockIdx.x == 0) {
    if (threadIdx.x < N) {
      s_counts[threadIdx.x] = R.counts[threadIdx.x];
      s_offsets[threadIdx.x] = R.offsets[threadIdx.x];
    }
    __syncthreads();
    modse_gemm::plan_bwd_body(L, esize, s_counts, s_offsets, plan, s_plan);
    return;
  }
  const int nbt = (ntok + PREP_TOKENS - 1) / PREP_TOKENS;
  if (GATE && (int)blockIdx.x > nbt) {
    const int c = ((int)blockIdx.x - 1 - nbt) * 256 + threadIdx.x;
    if (c < d)
#pragma unroll 8
      for (int e = 0; e < N; ++e) Wt[(size_t)e * d + c] = Wg[(size_t)c * N + e];
    return;
  }
  const int t = (blockIdx.x - 1) * PREP_TOKENS + (threadIdx.x >> 6);
  if (t >= ntok) return;
  const int lane = threadIdx.x & 63;
  auto rows = [&](auto two_tag) {
    constexpr int K = decltype(two_tag)::value ? 2 : 1;
    int r[K];
    float g[K], dot[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      r[j] = R.row_of[(size_t)t * K + j];
      g[j] = R.topk_w[(size_t)t * K + j];
      dot[j] = 0.f;
    }
#pragma unroll 2
    for (int c = lane * 8; c < d; c += 64 * 8) {
      float a[8], o[K][8], w[8];
      load8(dY + (size_t)t * d + c, a);
#pragma unroll
      for (int j = 0; j < K; ++j) load8(O + (size_t)r[j] * d + c, o[j]);
#pragma unroll
      for (int j = 0; j < K; ++j) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          dot[j] = fmaf(a[i], o[j][i], dot[j]);
          w[i] = g[j] * a[i];
        }
        store8(dO + (size_t)r[j] * d + c, w);
      }
    }
    float mean = 0.f;
#pragma unroll
    for (int j = 0; j < K; ++j) {
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) dot[j] += __shfl_xor(dot[j], m, 64);
      mean += g[j] * dot[j];
    }
    if constexpr (GATE) {
      float v = 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j)
        if (R.topk_idx[(size_t)t * K + j] == lane) v = g[j] * (dot[j] - mean);
      if (lane < N) dl[(size_t)t * N + lane] = v;
    } else if (lane == 0) {
#pragma unroll
      for (int j = 0; j < K; ++j) dg[r[j]] = dot[j];
    }
  };
  if (top_k == 2) rows(std::true_type{});
  else rows(std::false_type{});
}

// Backward through a gate with optional parts, one thread per token: the dense gradient of the logits H(x),
//   dl_j = g_j (dg_j - sum_m g_m dg_m) on the kept logits (softmax over KeepTopK), 0 elsewhere,
//   + aux_coef p_i (f_i - sum_m f_m p_m)  when the auxiliary loss is on (Sec. 3.2 Eq. 9-12 with f constant;
//     aux_coef = dLoss/dL_a * alpha N / T),
// and, when the noise term is on (z = gamma s / r, s = softplus(u), r = sqrt(mean s^2 + eps), Sec. 2
// Eq. 4-5), the gradient of u = x W_n and this block's share of d gamma:
//   du_i = gamma (dl_i / r - s_i <s, dl> / (N r^3)) sigmoid(u_i),   dgamma = sum_t <dl, s> / r.
constexpr int GB_THREADS = 64;  // (blocks of 256 threads left most CUs idle: 24 us at 8192 tokens with both gate extensions, now 11)
__global__ __launch_bounds__(GB_THREADS) void gate_bwd_kernel(const float* __restrict__ dg, int ntok, int N, int top_k,
                                                              const int32_t* __restrict__ topk_idx,
                                                              const float* __restrict__ topk_w,
                                                              const int32_t* __restrict__ row_of, GateExtPtrs G,
                                                              float aux_coef, float* __restrict__ dl, float* __restrict__ du,
                                                              float* __restrict__ dgamma_part) {
  const int tid = threadIdx.x;
  // (a token's row of dl is put together in LDS: in memory every step would wait for the one before)
  __shared__ float s_row[MODSE_MAX_EXPERTS][GB_THREADS], s_sp[MODSE_MAX_EXPERTS][GB_THREADS];
  const int t = blockIdx.x * GB_THREADS + tid;
  float dgam = 0.f;
  if (t < ntok) {
    if (G.probs && aux_coef != 0.f) {
      const float* p = G.probs + (size_t)t * N;
      float fp = 0.f;
#pragma unroll 8
      for (int e = 0; e < N; ++e) {
        const float v = p[e];
        s_row[e][tid] = v;
        fp = fmaf(G.aux_f[e], v, fp);
      }
#pragma unroll 8
      for (int e = 0; e < N; ++e) s_row[e][tid] = aux_coef * s_row[e][tid] * (G.aux_f[e] - fp);
    } else {
      for (int e = 0; e < N; ++e) s_row[e][tid] = 0.f;
    }
    float g[2] = {0.f, 0.f}, dgv[2] = {0.f, 0.f};
    float mean = 0.f;
    for (int j = 0; j < top_k; ++j) {
      g[j] = topk_w[(size_t)t * top_k + j];
      dgv[j] = dg[row_of[(size_t)t * top_k + j]];
      mean += g[j] * dgv[j];
    }
    for (int j = 0; j < top_k; ++j) s_row[topk_idx[(size_t)t * top_k + j]][tid] += g[j] * (dgv[j] - mean);
#pragma unroll 8
    for (int e = 0; e < N; ++e) dl[(size_t)t * N + e] = s_row[e][tid];
    if (G.W_noise) {
      const float* u = G.noise_pre + (size_t)t * N;
      float ss = 0.f, sd = 0.f;
#pragma unroll 8
      for (int e = 0; e < N; ++e) {
        const float v = u[e], sp = v > 15.f ? v : log1pf(__expf(v));
        s_sp[e][tid] = sp;
        ss = fmaf(sp, sp, ss);
        sd = fmaf(sp, s_row[e][tid], sd);
      }
      const float r = sqrtf(ss / (float)N + G.eps), gam = G.gamma[0];
      const float k1 = gam / r, k2 = gam * sd / ((float)N * r * r * r);
#pragma unroll 8
      for (int e = 0; e < N; ++e)
        du[(size_t)t * N + e] = (k1 * s_row[e][tid] - k2 * s_sp[e][tid]) / (1.f + __expf(-u[e]));
      dgam = sd / r;
    }
  }
  if (dgamma_part) {  // fixed-order sum over the block
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dgam += __shfl_xor(dgam, m, 64);
    if (tid == 0) dgamma_part[blockIdx.x] = dgam;
  }
}

// ---- backward through the router matrices.  "Column" e < N means W_gate with dl, e >= N (noise term on) W_noise with du.
// All bound by memory.  (One kernel for dX and the partial gradients, a block of 256 threads per 32 tokens that walked
// them four at a time, eight expert columns per launch, took 29 us at 1021 tokens and 8 experts, 129 at 32768, and 300 us
// for the whole stage at 1021 tokens with 64 experts, where every launch read x and dX again.  The stage now takes 37 us
// with 64 experts; at 32768 tokens and 8 experts 139 in place of 157, with both gate extensions at 8192 tokens 101 in
// place of 146.)

// The router's weight gradients (+)= the sum of the chunks' partials, in a fixed order (deterministic): 64 outputs per
// block, the partials are split over the 4 waves and combined through LDS.  Outputs: dW_gate, then (noise term on)
// dW_noise and dgamma, whose partials lie in an array of their own.
struct DwgReduceArgs {
  const float* partial;
  int nchunk, n, nmat;  // chunks; elements of a matrix; matrices
  const float* dgamma_part;
  int ngamma, accumulate;
  float *dWg, *dWn, *dgamma;
};
inline int dwg_reduce_blocks(const DwgReduceArgs& a) { return (a.n * a.nmat + 63) / 64 + (a.nmat == 2 ? 1 : 0); }
__device__ inline void dwg_reduce(const DwgReduceArgs& a, int block, int nblock, float (&s_part)[4][64]) {
  const int li = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int i = block * 64 + li, total = a.n * a.nmat;
  const bool gamma = a.nmat == 2 && block == nblock - 1 && li == 63 && i >= total;
  float acc = 0.f;
  if (i < total) {
#pragma unroll 8
    for (int b = part; b < a.nchunk; b += 4) acc += a.partial[(size_t)b * total + i];  // unrolled: several loads in flight
  } else if (gamma) {
    double sum = 0.0;  // (T / 256 values in a row)
#pragma unroll 8
    for (int b = part; b < a.ngamma; b += 4) sum += (double)a.dgamma_part[b];
    acc = (float)sum;
  }
  s_part[part][li] = acc;
  __syncthreads();
  if (part != 0) return;
  float* const out = i < a.n ? a.dWg + i : i < total ? a.dWn + (i - a.n) : gamma ? a.dgamma : nullptr;
  if (!out) return;
  const float v = (s_part[0][li] + s_part[1][li]) + (s_part[2][li] + s_part[3][li]);
  *out = a.accumulate ? *out + v : v;
}
__global__ __launch_bounds__(256) void dwg_reduce_kernel(DwgReduceArgs a) {
  __shared__ float s_part[4][64];
  dwg_reduce(a, blockIdx.x, gridDim.x, s_part);
}

// Plain gate: dl is zero except for the chosen experts, so
//   dX[t] = sum_j (dXp[row_of[t, j]] + W_gate[:, e_j] dl[t, e_j])
// with W_gate's columns as rows of Wt: one thread per token and eight columns of d, four row reads and a write.  SPLIT: a
// row of dXp is still the passes * ceil(f_e / kchunk) float32 slabs of the split product.
// The first `nreduce` blocks finish the router's weight gradient, which as a launch of its own took 4 to 5 us.  Stage of the
// router's backward pass without that launch and the gate's: d = 256, 512 tokens 18.7 -> 12.4 us; d = 2048, 1021 tokens 45 -> 37
// (and the slabs of a token's two rows fetched side by side), 32768 tokens 135 -> 122.
template <typename T, bool SPLIT>
__global__ __launch_bounds__(256) void bwd_gate_rows_kernel(const T* __restrict__ dXp, const float* __restrict__ slabs,
                                                            LayerDims L, int kchunk, const T* __restrict__ Wt,
                                                            const float* __restrict__ dl,
                                                            const int32_t* __restrict__ topk_idx,
                                                            const int32_t* __restrict__ row_of, T* __restrict__ dX,
                                                            DwgReduceArgs reduce, int nreduce) {
  __shared__ float s_part[4][64];
  if ((int)blockIdx.x < nreduce) {
    dwg_reduce(reduce, blockIdx.x, nreduce, s_part);
    return;
  }
  const int d = L.d, per_tok = d / 8;
  const long i = (long)((int)blockIdx.x - nreduce) * 256 + threadIdx.x;
  if (i >= (long)L.T * per_tok) return;
  const int t = (int)(i / per_tok), c = (int)(i % per_tok) * 8;
  auto row = [&](auto two_tag) {
    constexpr int K = decltype(two_tag)::value ? 2 : 1;
    int e[K];
    size_t at[K];
    float g[K], v[K][8], w[K][8], o[8];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      e[j] = topk_idx[(size_t)t * K + j];
      at[j] = (size_t)row_of[(size_t)t * K + j] * d + c;
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
      g[j] = dl[(size_t)t * L.N + e[j]];
      load8(Wt + (size_t)e[j] * d + c, w[j]);
    }
    if constexpr (SPLIT) {
      const float* src[K];
      int n[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        src[j] = slabs + at[j];
        n[j] = 2 * ((L.f[e[j]] + kchunk - 1) / kchunk);
      }
      sum_slabs8(src, (size_t)L.T * L.k * d, n, v);
    } else {
#pragma unroll
      for (int j = 0; j < K; ++j) load8(dXp + at[j], v[j]);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = 0.f;
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = fmaf(w[j][q], g[j], o[q] + v[j][q]);
    store8(dX + (size_t)t * d + c, o);
  };
  if (L.k == 2) row(std::true_type{});
  else row(std::false_type{});
}

static_assert(BR_TOK == MODSE_ROUTE_TOKENS_PER_BLOCK, "the workspace holds one partial gradient per 32-token block");
struct BwdRouterArgs {
  const void *Wg, *Wn;        // [d, N]; Wn null: no noise term
  const float *dl, *du;       // [T, N]
  int ntok, d, N, NP, top_k;  // NP: N, or 2 N with the noise term
  const int32_t *row_of;
};

// Gate extensions: dX[t] = sum_j dXp[row_of[t, j]] + W_gate dl[t] (+ W_noise du[t]).  A block owns a slab of 512 columns of
// d and `rounds` groups of 32 tokens, eight per wave; all rows of a batch are loaded before any arithmetic.  The matrices
// lie in LDS as [column e][512 columns of d], EMAX columns e at a time.
template <typename T>
__global__ __launch_bounds__(256) void bwd_gate_rows_ext_kernel(BwdRouterArgs a, const T* __restrict__ dXp, int rounds,
                                                                T* __restrict__ dX) {
  constexpr int TB = sizeof(T) == 2 ? 8 : 4;  // tokens per batch
  constexpr int EMAX = 64 * 1024 / (BR_SLAB * sizeof(T));
  __shared__ __attribute__((aligned(16))) T s_w[EMAX * BR_SLAB];  // [column e][column of d]
  __shared__ __attribute__((aligned(16))) float s_dl[EMAX * BR_TOK];  // [column e][token]
  __shared__ int s_row[BR_TOK][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = a.d, N = a.N, c0 = blockIdx.y * BR_SLAB, c = c0 + lane * 8;
  const int cl = min(c, d - 8);  // (lanes beyond the matrix repeat its last columns and store nothing)
  const int npass = (a.NP + EMAX - 1) / EMAX;
  auto stage_w = [&](int e0, int ne) {  // two columns of d per thread
    const int cg = min(c0 + 2 * tid, d - 2);
    for (int e = 0; e < ne; ++e) {
      const int eg = e0 + e;
      const T* const W = static_cast<const T*>(eg < N ? a.Wg : a.Wn) + (eg < N ? eg : eg - N);
      s_w[e * BR_SLAB + 2 * tid] = W[(size_t)cg * N];
      s_w[e * BR_SLAB + 2 * tid + 1] = W[(size_t)(cg + 1) * N];
    }
  };
  auto stage_dl = [&](int t0, int e0, int ne) {
    for (int i = tid; i < ne * BR_TOK; i += 256) {
      const int t = i / ne, e = i % ne, eg = e0 + e;
      s_dl[e * BR_TOK + t] = t0 + t < a.ntok ? (eg < N ? a.dl[(size_t)(t0 + t) * N + eg] : a.du[(size_t)(t0 + t) * N + eg - N]) : 0.f;
    }
  };
  if (npass == 1) stage_w(0, a.NP);
  for (int r = 0; r < rounds; ++r) {
    const int t0 = (blockIdx.x * rounds + r) * BR_TOK;
    if (t0 >= a.ntok) break;
    const int nt = min(BR_TOK, a.ntok - t0);
    __syncthreads();  // the round before has been read
    if (tid < 2 * BR_TOK)
      s_row[tid >> 1][tid & 1] = a.row_of[(size_t)(t0 + min(tid >> 1, nt - 1)) * a.top_k + min(tid & 1, a.top_k - 1)];
    if (npass == 1) stage_dl(t0, 0, a.NP);
    __syncthreads();
    const float use_b = a.top_k == 2 ? 1.f : 0.f;
#pragma unroll 1
    for (int b = 0; b < BR_TOK / 4 / TB; ++b) {
      const int tw = wave * (BR_TOK / 4) + b * TB;
      float go[TB][8], bv[TB][8];
#pragma unroll
      for (int u = 0; u < TB; ++u) {  // (no branch between the loads: a missing row is a repeated one)
        load8(dXp + (size_t)s_row[tw + u][0] * d + cl, go[u]);
        load8(dXp + (size_t)s_row[tw + u][1] * d + cl, bv[u]);
      }
#pragma unroll
      for (int u = 0; u < TB; ++u)
#pragma unroll
        for (int q = 0; q < 8; ++q) go[u][q] = fmaf(use_b, bv[u][q], go[u][q]);
      for (int p = 0; p < npass; ++p) {
        const int e0 = p * EMAX, ne = min(EMAX, a.NP - e0);
        if (npass > 1) {
          __syncthreads();
          stage_w(e0, ne);
          stage_dl(t0, e0, ne);
          __syncthreads();
        }
        for (int e = 0; e < ne; ++e) {
          float w[8], dv[TB];
          load8(s_w + e * BR_SLAB + lane * 8, w);
#pragma unroll
          for (int u = 0; u < TB; u += 4) load4(s_dl + e * BR_TOK + tw + u, dv + u);
#pragma unroll
          for (int u = 0; u < TB; ++u)
#pragma unroll
            for (int q = 0; q < 8; ++q) go[u][q] = fmaf(w[q], dv[u], go[u][q]);
        }
      }
      if (c < d) {
#pragma unroll
        for (int u = 0; u < TB; ++u)
          if (tw + u < nt) store8(dX + (size_t)(t0 + tw + u) * d + c, go[u]);
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256, 3) void bwd_dwg_kernel(DwgArgs a) {
  __shared__ DwgSums s_sum;
  bwd_dwg_block<T, sizeof(T) == 2 ? 8 : 4>(a, blockIdx.x, s_sum);
}

// [d, N] -> [d, NE] with zero columns behind the N real ones
template <typename T>
__global__ __launch_bounds__(256) void pad_rows_kernel(const T* __restrict__ W, int d, int N, int NE,
                                                       T* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d * NE) return;
  const int r = i / NE, e = i % NE;
  out[i] = e < N ? W[(size_t)r * N + e] : (T)0.f;
}

template <typename T, int NE>
hipError_t run_router(const LayerDims& L, const T* x, const T* Wg, const float* bias, const RoutingPtrs& R,
                      int32_t* blockhist, const GateExtPtrs* G, hipStream_t s) {
  const dim3 grid(std::min((L.T + RW_TOKENS - 1) / RW_TOKENS, 256)), blk(RW_THREADS);
  if (G && G->W_noise)
    hipLaunchKernelGGL((router_kernel<T, NE, true>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k, R.topk_idx,
                       R.topk_w, blockhist, *G);
  else
    hipLaunchKernelGGL((router_kernel<T, NE, false>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k, R.topk_idx,
                       R.topk_w, blockhist, G ? *G : GateExtPtrs{});
  return hipGetLastError();
}

// whether the router (token-wise or screened) leaves flags and no block histograms
bool router_leaves_flags(const LayerDims& L, const GateExtPtrs* G) { return !G && L.T <= ROUTER_TOKEN_MAX_T; }
enum RouterKind { ROUTER_TOKEN, ROUTER_STREAM, ROUTER_SCREEN, ROUTER_BLOCK };
// Which router a layer takes.  Plain gate, small and medium batches: one block per token (or four) keeps the chip busy
// where 32-token blocks would leave most CUs idle.  Larger plain batches of up to 16 experts: router_stream_kernel (or
// its matrix-instruction form) when W_gate fits its LDS area.  Otherwise, and with the optional gate parts,
// router_kernel.  bf16 with more than 16 experts, and room for W_gate's columns: the screened router as soon as its two
// launches beat the token router's rounds (four tokens per block): routing call at d = 2048, token router / screened, 64
// experts 1024 tokens 19.9 / 21.4 us, 1536 27.8 / 21.8, 4096 47.6 / 28.1; 32 experts 1536 20.6 / 20.5, 3072 26.4 / 22.3 (d =
// 1024, 2048 tokens: 19.8 / 20.1 and 15.5 / 18.0).
RouterKind router_kind(const LayerDims& L, modse_dtype dt, const GateExtPtrs* G, const RouteBufs& B) {
  if (G) return ROUTER_BLOCK;
  if (dt == MODSE_BF16 && L.N > 16 && L.T > (L.N > 32 ? 1535 : 2048) && B.wt && route_wt_bytes(L, 2) <= ROUTE_WT_MAX)
    return ROUTER_SCREEN;
  if (L.T <= ROUTER_TOKEN_MAX_T) return ROUTER_TOKEN;
  if (L.N <= 16 && (size_t)(L.d / 8) * rs_group_bytes(padded_experts(L.N), 4) <= (size_t)RS_W_BYTES) return ROUTER_STREAM;
  return ROUTER_BLOCK;
}

// whether a layer that takes the streaming router can take its matrix-instruction form
bool router_on_mfma(const LayerDims& L) {
  const int NE = L.N <= 8 ? 8 : 16;
  return L.N <= 16 && L.d % 256 == 0 && (size_t)L.d * NE * 8 <= (size_t)rm_w_bytes(NE);
}

// logits, top-k, gate (and the block histograms, or the flags of router_leaves_flags)
template <typename T>
hipError_t router_typed(const LayerDims& L, const void* xv, const void* Wgv, const float* bias, const RoutingPtrs& R,
                        const RouteBufs& B, const GateExtPtrs* G, hipStream_t s) {
  const T* x = static_cast<const T*>(xv);
  const T* Wg = static_cast<const T*>(Wgv);
  hipError_t e;
  const RouterKind kind = router_kind(L, std::is_same_v<T, float> ? MODSE_F32 : MODSE_BF16, G, B);
  const int NE = padded_experts(L.N);
  GateExtPtrs Gp;
  if (G) Gp = *G;
  if (kind != ROUTER_STREAM && NE != L.N) {  // these kernels want matrix rows of NE elements
    T* pad = static_cast<T*>(B.wpad);
    const int nblk = (L.d * NE + 255) / 256;
    hipLaunchKernelGGL((pad_rows_kernel<T>), dim3(nblk), dim3(256), 0, s, Wg, L.d, L.N, NE, pad);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    Wg = pad;
    if (G && G->W_noise) {
      T* pad2 = pad + (size_t)L.d * NE;
      hipLaunchKernelGGL((pad_rows_kernel<T>), dim3(nblk), dim3(256), 0, s, static_cast<const T*>(G->W_noise), L.d,
                         L.N, NE, pad2);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      Gp.W_noise = pad2;
    }
  }
  if (kind == ROUTER_TOKEN) {
    const dim3 grid(L.T), blk(ROUTE_THREADS);
#define MODSE_LAUNCH_TOKEN_ROUTER(NE_)                                                                           \
  hipLaunchKernelGGL((router_token_kernel<T, NE_, 1>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k, R.topk_idx, \
                     R.topk_w, B.near_flag)
    if (NE == 2) MODSE_LAUNCH_TOKEN_ROUTER(2);
    else if (NE == 4) MODSE_LAUNCH_TOKEN_ROUTER(4);
    else if (NE == 8) MODSE_LAUNCH_TOKEN_ROUTER(8);
    else if (NE == 16) MODSE_LAUNCH_TOKEN_ROUTER(16);
#define MODSE_LAUNCH_TOKEN_WIDE(NE_, G_)                                                                             \
  hipLaunchKernelGGL((router_token_wide_kernel<T, NE_, G_>), dim3((L.T + G_ - 1) / G_), blk, 0, s, x, Wg, bias, L.T, \
                     L.d, L.N, L.k, R.topk_idx, R.topk_w, B.near_flag)
    else if (L.T <= 512) {  // one token per block until they fill the chip twice
      if (NE == 32) MODSE_LAUNCH_TOKEN_WIDE(32, 1);
      else MODSE_LAUNCH_TOKEN_WIDE(64, 1);
    } else {
      if (NE == 32) MODSE_LAUNCH_TOKEN_WIDE(32, 4);
      else MODSE_LAUNCH_TOKEN_WIDE(64, 4);
    }
#undef MODSE_LAUNCH_TOKEN_WIDE
#undef MODSE_LAUNCH_TOKEN_ROUTER
    e = hipGetLastError();
  } else if (kind == ROUTER_SCREEN) {
    if constexpr (std::is_same_v<T, bf16_t>) {
      const int nscreen = (L.T + SC_TOKENS - 1) / SC_TOKENS;
      const dim3 grid(nscreen + (L.d + SC_TRANSPOSE_ROWS - 1) / SC_TRANSPOSE_ROWS);
      uint32_t* const lo = reinterpret_cast<uint32_t*>(R.topk_idx);
      uint32_t* const hi = reinterpret_cast<uint32_t*>(R.topk_w);
      bf16_t* const wt = static_cast<bf16_t*>(B.wt);
      uint8_t* const crowd = reinterpret_cast<uint8_t*>(R.src_of);  // (written by the permutation only; T k words for T / 4 bytes)
      int32_t* const hist = router_leaves_flags(L, G) ? nullptr : B.blockhist;
      if (NE == 32)
        hipLaunchKernelGGL((router_screen_kernel<32>), grid, dim3(SC_THREADS), 0, s, x, Wg, static_cast<const T*>(Wgv), bias, L.T, L.d,
                           L.N, L.k, nscreen, lo, hi, crowd, wt, hist);
      else
        hipLaunchKernelGGL((router_screen_kernel<64>), grid, dim3(SC_THREADS), 0, s, x, Wg, static_cast<const T*>(Wgv), bias, L.T, L.d,
                           L.N, L.k, nscreen, lo, hi, crowd, wt, hist);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      hipLaunchKernelGGL((NE == 32 ? router_exact_kernel<32> : router_exact_kernel<64>), dim3((L.T + EX_TOKENS - 1) / EX_TOKENS),
                         dim3(EX_THREADS), 0, s, x, wt, bias, reinterpret_cast<const uint32_t*>(crowd), L.T, L.d, L.N, L.k, R.topk_idx, R.topk_w, hist,
                         hist ? nullptr : B.near_flag);
    }
    e = hipGetLastError();
  } else if (kind == ROUTER_STREAM && router_on_mfma(L)) {
    const int ngroups = (L.T + RM_TOKENS - 1) / RM_TOKENS;
    const dim3 grid(std::min(ngroups, 256)), blk(RM_THREADS);  // one block per CU holds the LDS copy of W_gate
    if (L.N <= 8)
      hipLaunchKernelGGL((router_mfma_kernel<T, 8>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k, R.topk_idx,
                         R.topk_w, B.blockhist);
    else
      hipLaunchKernelGGL((router_mfma_kernel<T, 16>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k, R.topk_idx,
                         R.topk_w, B.blockhist);
    e = hipGetLastError();
  } else if (kind == ROUTER_STREAM) {
    const int ngroups = (L.T + RS_TOKENS - 1) / RS_TOKENS;
    const dim3 grid(std::min(ngroups, 256)), blk(RS_THREADS);  // one block per CU holds the LDS copy of W_gate
    const bool w64 = (size_t)(L.d / 8) * rs_group_bytes(NE, 8) <= (size_t)RS_W_BYTES;  // W_gate fits as float64
#define MODSE_LAUNCH_STREAM_ROUTER(NE_)                                                                            \
  do {                                                                                                            \
    if (w64)                                                                                                      \
      hipLaunchKernelGGL((router_stream_kernel<T, NE_, double>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k, \
                         R.topk_idx, R.topk_w, B.blockhist);                                                      \
    else                                                                                                          \
      hipLaunchKernelGGL((router_stream_kernel<T, NE_, float>), grid, blk, 0, s, x, Wg, bias, L.T, L.d, L.N, L.k,  \
                         R.topk_idx, R.topk_w, B.blockhist);                                                      \
  } while (0)
    switch (NE) {
      case 2: MODSE_LAUNCH_STREAM_ROUTER(2); break;
      case 4: MODSE_LAUNCH_STREAM_ROUTER(4); break;
      case 8: MODSE_LAUNCH_STREAM_ROUTER(8); break;
      default: MODSE_LAUNCH_STREAM_ROUTER(16); break;
    }
#undef MODSE_LAUNCH_STREAM_ROUTER
    e = hipGetLastError();
  } else {
    const GateExtPtrs* g = G ? &Gp : nullptr;
    switch (NE) {
      case 2: e = run_router<T, 2>(L, x, Wg, bias, R, B.blockhist, g, s); break;
      case 4: e = run_router<T, 4>(L, x, Wg, bias, R, B.blockhist, g, s); break;
      case 8: e = run_router<T, 8>(L, x, Wg, bias, R, B.blockhist, g, s); break;
      case 16: e = run_router<T, 16>(L, x, Wg, bias, R, B.blockhist, g, s); break;
      case 32: e = run_router<T, 32>(L, x, Wg, bias, R, B.blockhist, g, s); break;
      default: e = run_router<T, 64>(L, x, Wg, bias, R, B.blockhist, g, s); break;
    }
  }
  if (e != hipSuccess) return e;
  if (G && G->probs) {
    hipLaunchKernelGGL(aux_finish_kernel, dim3(1), dim3(AUX_THREADS), 0, s, G->probs, R.topk_idx, L.T, L.N, L.k, G->alpha,
                       G->aux_f, G->aux_P, G->aux_loss);
    e = hipGetLastError();
  }
  return e;
}

// The permutation (and the forward tile plans when `plan` is given).  Up to MODSE_PERMUTE_FUSED_MAX_T tokens: one launch for all of it, whose
// blocks count the choices themselves, which grows with the square of the batch; beyond that one over the router's block
// histograms (permute_by_hist), or a scan over them, then the scatter.
template <typename T>
hipError_t permute_typed(const LayerDims& L, modse_dtype dt, const void* xv, const RoutingPtrs& R, const RouteBufs& B,
                         void* Xpv, const GateExtPtrs* G, const FwdPlanArgs* plan, hipStream_t s) {
  const T* x = static_cast<const T*>(xv);
  const int nb = (L.T + TPB - 1) / TPB;
  static_assert(ROUTER_TOKEN_MAX_T == MODSE_PERMUTE_FUSED_MAX_T, "the routers of small batches make no block histograms");
  const int32_t* const near_flag = router_leaves_flags(L, G) ? B.near_flag : nullptr;
  if (L.T <= MODSE_PERMUTE_SMALL_MAX_T && L.N <= PS_EXPERTS) {
    hipLaunchKernelGGL((permute_small_kernel<T>), dim3(Xpv ? L.T + 1 : 1), dim3(PS_THREADS), 0, s, x, L.T, L.d, L.N, L.k,
                       R.topk_idx, near_flag, B.blockhist, R, static_cast<T*>(Xpv), L, dt == MODSE_F32 ? 4 : 2,
                       plan ? *plan : FwdPlanArgs{}, plan ? 1 : 0);
    return hipGetLastError();
  }
  if (L.T <= MODSE_PERMUTE_FUSED_MAX_T) {
    hipLaunchKernelGGL((permute_fused_kernel<T>), dim3((L.T + PF_TOKENS - 1) / PF_TOKENS + 1), dim3(PF_THREADS), 0, s, x, L.T,
                       L.d, L.N, L.k, R.topk_idx, near_flag, B.blockhist, R, static_cast<T*>(Xpv), L, dt == MODSE_F32 ? 4 : 2,
                       plan ? *plan : FwdPlanArgs{}, plan ? 1 : 0);
    return hipGetLastError();
  }
  if (permute_by_hist(L, sizeof(T), Xpv != nullptr)) {
    hipLaunchKernelGGL((permute_hist_kernel<T>), dim3(nb + 1), dim3(PH_THREADS), 0, s, x, L.T, L.d, L.N, L.k, R.topk_idx, B.blockhist, nb,
                       R, static_cast<T*>(Xpv), L, dt == MODSE_F32 ? 4 : 2, plan ? *plan : FwdPlanArgs{}, plan ? 1 : 0);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(route_scan_kernel, dim3(1), dim3(SCAN_THREADS), 0, s, B.blockhist, nb, L.N, R.counts, R.offsets,
                     R.near_tie_count, L, dt == MODSE_F32 ? 4 : 2, plan ? *plan : FwdPlanArgs{}, plan ? 1 : 0);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // two blocks share the copies of a histogram block's tokens while those blocks are few
  const int parts = Xpv && nb < 512 ? 2 : 1;
  hipLaunchKernelGGL((scatter_kernel<T>), dim3(nb * parts), dim3(ROUTE_THREADS), 0, s, x, L.T, L.d, L.N, L.k, R.topk_idx,
                     R.offsets, B.blockhist, R.row_of, R.src_of, static_cast<T*>(Xpv), parts);
  return hipGetLastError();
}

// dLoss/dL_a * alpha N / T, the factor of the auxiliary loss in the gradient of the logits
float aux_coefficient(const LayerDims& L, const GateExtPtrs& G, float aux_grad) {
  return G.probs ? aux_grad * G.alpha * (float)L.N / (float)L.T : 0.f;
}
// neither optional part of the gate takes part in the backward pass
bool gate_is_plain(const GateExtPtrs& G, float aux_coef) { return !G.W_noise && aux_coef == 0.f; }

template <typename T>
hipError_t bwd_prep_typed(const LayerDims& L, const void* dY, const void* O, const RoutingPtrs& R, void* dO, float* dg,
                          const BwdPlanArgs& plan, bool plain, const void* Wg, const BwdRouterBufs& B, hipStream_t s) {
  const dim3 grid(1 + (L.T + PREP_TOKENS - 1) / PREP_TOKENS + (plain ? (L.d + 255) / 256 : 0));
  const T *dYt = static_cast<const T*>(dY), *Ot = static_cast<const T*>(O), *Wt = static_cast<const T*>(Wg);
  if (plain)
    hipLaunchKernelGGL((bwd_prep_plan_bwd_kernel<T, true>), grid, dim3(256), 0, s, dYt, Ot, R, static_cast<T*>(dO), dg, L,
                       (int)sizeof(T), plan, B.dl, Wt, static_cast<T*>(B.Wt));
  else
    hipLaunchKernelGGL((bwd_prep_plan_bwd_kernel<T, false>), grid, dim3(256), 0, s, dYt, Ot, R, static_cast<T*>(dO), dg, L,
                       (int)sizeof(T), plan, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

template <typename T>
hipError_t bwd_router_typed(const LayerDims& L, const GateExtPtrs& G, float aux_coef, const void* xv, const void* Wv,
                            const DxRows& rows, const float* dg, const RoutingPtrs& R, const BwdRouterBufs& B, void* dXv,
                            float* dW_gate, float* dW_noise, float* dgamma, int accumulate, bool dwg_done, hipStream_t s) {
  const T *x = static_cast<const T*>(xv), *W = static_cast<const T*>(Wv), *dXp = static_cast<const T*>(rows.dXp);
  T* const dX = static_cast<T*>(dXv);
  const bool noise = G.W_noise != nullptr, sparse = gate_is_plain(G, aux_coef);  // dl is zero but for the chosen experts
  const int nbt = (L.T + GB_THREADS - 1) / GB_THREADS;
  hipError_t e;
  if (!sparse) {  // (otherwise launch_bwd_prep has seen to dl and Wt)
    hipLaunchKernelGGL(gate_bwd_kernel, dim3(nbt), dim3(GB_THREADS), 0, s, dg, L.T, L.N, L.k, R.topk_idx, R.topk_w, R.row_of, G,
                       aux_coef, B.dl, noise ? B.du : nullptr, noise ? B.dgamma_part : nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int nmat = noise ? 2 : 1, slabs = (L.d + BR_SLAB - 1) / BR_SLAB, nb = (L.T + BR_TOK - 1) / BR_TOK;
  const BwdRouterArgs a = {W, G.W_noise, B.dl, B.du, L.T, L.d, L.N, nmat * L.N, L.k, R.row_of};
  // dX comes last: its buffer may be x's (nothing after the weight gradients reads x).
  const DwgArgs w = dwg_args(L, x, B, nmat);
  if (!dwg_done) {
    hipLaunchKernelGGL((bwd_dwg_kernel<T>), dim3(dwg_blocks(w)), dim3(256), 0, s, w);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const DwgReduceArgs red = {B.dW_partial, w.nchunk, L.d * L.N, nmat, B.dgamma_part, nbt, accumulate, dW_gate, dW_noise, dgamma};
  const int nred = dwg_reduce_blocks(red);
  if (sparse) {
    const dim3 grid((unsigned)(((long)L.T * (L.d / 8) + 255) / 256 + nred));
    if (rows.kchunk)
      hipLaunchKernelGGL((bwd_gate_rows_kernel<T, true>), grid, dim3(256), 0, s, dXp, rows.slabs, L, rows.kchunk,
                         static_cast<const T*>(B.Wt), B.dl, R.topk_idx, R.row_of, dX, red, nred);
    else
      hipLaunchKernelGGL((bwd_gate_rows_kernel<T, false>), grid, dim3(256), 0, s, dXp, nullptr, L, 0,
                         static_cast<const T*>(B.Wt), B.dl, R.topk_idx, R.row_of, dX, red, nred);
  } else {
    hipLaunchKernelGGL(dwg_reduce_kernel, dim3(nred), dim3(256), 0, s, red);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (rows.kchunk) {
      const long chunks = (long)L.T * L.k * (L.d / 8);
      hipLaunchKernelGGL((sum_slabs_kernel<T>), dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, rows.slabs, L.T * L.k, L.d,
                         L, rows.kchunk, 2, R.topk_idx, R.src_of, static_cast<T*>(rows.dXp));
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // several groups of tokens per block once there are four blocks per CU without
    const int rounds = std::max(1, std::min(8, nb * slabs / 1024));
    hipLaunchKernelGGL((bwd_gate_rows_ext_kernel<T>), dim3((nb + rounds - 1) / rounds, slabs), dim3(256), 0, s, a, dXp, rounds,
                       dX);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_router(const LayerDims& L, modse_dtype dt, const void* x, const void* W_gate, const float* bias,
                         const RoutingPtrs& R, const RouteBufs& B, const GateExtPtrs* G, hipStream_t s) {
  return dt == MODSE_F32 ? router_typed<float>(L, x, W_gate, bias, R, B, G, s)
                         : router_typed<bf16_t>(L, x, W_gate, bias, R, B, G, s);
}

hipError_t launch_permute(const LayerDims& L, modse_dtype dt, const void* x, const RoutingPtrs& R, const RouteBufs& B,
                          void* Xp, const GateExtPtrs* G, const FwdPlanArgs* plan, hipStream_t s) {
  return dt == MODSE_F32 ? permute_typed<float>(L, dt, x, R, B, Xp, G, plan, s)
                         : permute_typed<bf16_t>(L, dt, x, R, B, Xp, G, plan, s);
}

hipError_t launch_route(const LayerDims& L, modse_dtype dt, const void* x, const void* W_gate, const float* bias,
                        const RoutingPtrs& R, const RouteBufs& B, void* Xp, const GateExtPtrs* G, hipStream_t s) {
  const hipError_t e = launch_router(L, dt, x, W_gate, bias, R, B, G, s);
  return e != hipSuccess ? e : launch_permute(L, dt, x, R, B, Xp, G, nullptr, s);
}

hipError_t launch_routing_stats(const LayerDims& L, const int32_t* topk_idx, int32_t* slot_counts, float* summary,
                                hipStream_t s) {
  hipLaunchKernelGGL(routing_stats_kernel, dim3(1), dim3(256), 0, s, topk_idx, L.T, L.N, L.k, L, slot_counts, summary);
  return hipGetLastError();
}

hipError_t launch_combine(const LayerDims& L, modse_dtype dt, const void* O, const RoutingPtrs& R, void* y,
                          hipStream_t s) {
  const int nb = (L.T + 3) / 4;
  if (dt == MODSE_F32)
    hipLaunchKernelGGL((combine_kernel<float>), dim3(nb), dim3(256), 0, s, static_cast<const float*>(O), L.T, L.d, L.k,
                       R.row_of, R.topk_w, static_cast<float*>(y));
  else
    hipLaunchKernelGGL((combine_kernel<bf16_t>), dim3(nb), dim3(256), 0, s, static_cast<const bf16_t*>(O), L.T, L.d,
                       L.k, R.row_of, R.topk_w, static_cast<bf16_t*>(y));
  return hipGetLastError();
}

hipError_t launch_combine_split(const LayerDims& L, modse_dtype dt, const float* Opart, int kchunk, const RoutingPtrs& R,
                                void* O, void* y, hipStream_t s) {
  const int nb = (int)(((long)L.T * (L.d / 8) + 255) / 256);
  if (dt == MODSE_F32)
    hipLaunchKernelGGL((combine_split_kernel<float>), dim3(nb), dim3(256), 0, s, Opart, L.T, L.d, L.k, L, kchunk,
                       R.topk_idx, R.row_of, R.topk_w, static_cast<float*>(O), static_cast<float*>(y));
  else
    hipLaunchKernelGGL((combine_split_kernel<bf16_t>), dim3(nb), dim3(256), 0, s, Opart, L.T, L.d, L.k, L, kchunk,
                       R.topk_idx, R.row_of, R.topk_w, static_cast<bf16_t*>(O), static_cast<bf16_t*>(y));
  return hipGetLastError();
}

bool bwd_gate_is_plain(const LayerDims& L, const GateExtPtrs* G, float aux_grad) {
  return !G || gate_is_plain(*G, aux_coefficient(L, *G, aux_grad));
}

hipError_t launch_bwd_prep(const LayerDims& L, modse_dtype dt, const void* dY, const void* O, const RoutingPtrs& R,
                           void* dO, float* dg, const BwdPlanArgs& plan, const GateExtPtrs* G, float aux_grad,
                           const void* W_gate, const BwdRouterBufs& B, hipStream_t s) {
  const bool plain = bwd_gate_is_plain(L, G, aux_grad);
  return dt == MODSE_F32 ? bwd_prep_typed<float>(L, dY, O, R, dO, dg, plan, plain, W_gate, B, s)
                         : bwd_prep_typed<bf16_t>(L, dY, O, R, dO, dg, plan, plain, W_gate, B, s);
}

hipError_t launch_bwd_router(const LayerDims& L, modse_dtype dt, const void* x, const void* W_gate, const DxRows& rows,
                             const float* dg, const RoutingPtrs& R, const GateExtPtrs* G, float aux_grad,
                             const BwdRouterBufs& B, void* dX, float* dW_gate, float* dW_noise, float* dgamma,
                             int accumulate, bool dwg_done, hipStream_t s) {
  const GateExtPtrs none = {};
  const GateExtPtrs& g = G ? *G : none;
  const float aux_coef = aux_coefficient(L, g, aux_grad);
  return dt == MODSE_F32 ? bwd_router_typed<float>(L, g, aux_coef, x, W_gate, rows, dg, R, B, dX, dW_gate, dW_noise, dgamma,
                                                   accumulate, dwg_done, s)
                         : bwd_router_typed<bf16_t>(L, g, aux_coef, x, W_gate, rows, dg, R, B, dX, dW_gate, dW_noise, dgamma,
                                                    accumulate, dwg_done, s);
}
