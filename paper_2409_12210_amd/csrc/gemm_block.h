// Grouped GEMM with small tiles for gfx950: 128 x 128 down to 32 x 128 (float32: 32 x 32) tiles, one per workgroup of four
// waves, float32 and bf16, every layout and epilogue of the layer.
//
// Where the 256 x 256 kernel of gemm_bf16.h wants tall problems (one workgroup per CU, a ring of five panels), this one
// serves problems that do not fill such tiles: the workgroup is small enough (80 KiB of LDS) that two of them share a
// CU, so one multiplies while the other waits at its barrier or stores its result, and the tiles are numerous enough to
// go round.  The grid has one workgroup per tile; workgroups beyond the tile list
// (its length is known on the device only) leave at once.
//
// An LDS row of a K-contiguous operand is 128 bytes whatever the element type: 64 bf16 or 32 float32 along K, which is
// one K step.  The 16-byte chunk index of a row is XOR-ed with ((row >> 1) & 7), so that the lanes a 128-bit LDS read
// serves together fall into different banks.  A lane of the upper half takes the odd chunk of a pair, one of the lower
// half the even one.  For bf16 that is the operand layout of v_mfma_f32_32x32x16_bf16; for float32 the four values of
// the chunk feed four v_mfma_f32_32x32x2_f32 (K index s of the even chunk with K index s of the odd one: the order of
// the contraction is free as long as both operands agree).
// An operand stored [K, X] keeps its memory order in LDS; bf16 fragments are read with ds_read_b64_tr_b16 (16-byte chunk
// index XOR-ed so that the four K rows a read covers start in different banks), float32 ones with 32-bit reads: the
// float32 matrix instruction takes 64 cycles, so LDS has time to spare.
//
// bf16 at few rows per expert is bound by the weight stream, so what counts is bytes in flight: LDS is a ring of as many
// operand panels as fit (five of 16 KiB for 128 x 128, four stages of 20 KiB for 32 x 128), refilled one step behind the
// reads, with counted waits.  Weights that meet one row block are loaded with the non-temporal hint: they are read once,
// and behind a backward pass, whose weight gradients have just filled the caches, the up-projection of 130 tokens took
// 143 us without and 83 with it (with it, weights that several row blocks read were slower: 117 -> 160 us at 600 tokens).
// At d = 2048, eight experts of mean width 5632, in place of 256-row tiles (up / down + combine): 389 tokens 117 / 170 ->
// 91 / 60 us; at d = 4096, one token, in place of 64-row tiles of 512 columns that left half of the CUs without one: 131 /
// 79 -> 69 / 44 us, weights at 6.5 TB/s.  At many rows it is bound by LDS reads and load issue
// (0.87 PFLOP/s against 1.1 to 1.2 of the 256 x 256 kernel): gemm_choice picks.
//
// float32 is bound by the matrix pipe (157 TFLOP/s; a library product of 8192^3 reaches 153).  Measured in place of
// vector-FMA tiles of 64 x 64 x 16: the five GEMMs of a training step at d = 1024, 4096 tokens, 8 experts of mean width
// 2816 took 3.9 ms instead of 7.0 (60 -> 109 TFLOP/s; 3.4 by now, 122 over the whole pass); at d = 256, 512 tokens 46 us
// instead of 174.
#pragma once
#include "bwd_dwg.h"
#include "gemm_bf16.h"

namespace modse_gemm {

// Consecutive workgroups go to the 8 XCDs in turn.  Runs of TILE_RUN tiles (row blocks of the same weight columns come
// first in the list) stay on one XCD, so that they read the weights through the same L2, and the runs are dealt out to
// the XCDs in turn: the list is sorted by falling cost, and contiguous eighths of it would leave the last XCDs idle.
constexpr int TILE_RUN = 8;
__device__ inline int tile_of_workgroup(int b) {
  const int i = b / NUM_XCD;
  return ((i / TILE_RUN) * NUM_XCD + b % NUM_XCD) * TILE_RUN + i % TILE_RUN;
}

// BN: columns of C per tile.  NB = 2: two B matrices that share A (the up-projection's W1 and W3), BN columns of each.
// KG > 1: KG groups of waves share the tile, each takes every KG-th of a step's four K slices, and the sums meet in LDS.
// block: of the launch's workgroups that work on this plan.  ring: ring_bytes(BM, NB * BN, NSLOT) of LDS.
constexpr int ring_bytes(int bm, int br, int nslot) { return bm == br ? nslot * bm * 128 : nslot / 2 * (bm + br) * 128; }
template <typename T, int BM, int BN, int NB, int WAVES_M, int WAVES_N, int NSLOT, int EPI, int LAYOUT, int KG = 1>
__device__ __forceinline__ void gg_block(const GemmPlan* __restrict__ plan, int n_prob, int accumulate, int option, int block,
                                         char* const ring) {
  constexpr int ES = sizeof(T), CE = 16 / ES, BK = 128 / ES;
  constexpr bool A_T = (LAYOUT & 1) != 0, B_T = (LAYOUT & 2) != 0, F32 = ES == 4;
  constexpr int BR = NB * BN;               // B rows of a stage
  constexpr int STAGE = (BM + BR) * 128;
  constexpr int NW = WAVES_M * WAVES_N * KG;
  constexpr int UA = BM / 8 / NW, UB = BR / 8 / NW;  // 1 KiB load units per wave and step
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, MI = WM / 32, NI = WN / 32;
  static_assert(BM % (32 * WAVES_M) == 0 && BN % (32 * WAVES_N) == 0 && UA >= 1, "wave tiles of 32 x 32 blocks");
  static_assert(!(B_T && NB != 1), "a [K, N] operand is a single matrix");
  // Panels are numbered in the order in which they are loaded: 2 g is step g's B panel, 2 g + 1 its A panel.  Panel i lies
  // in slot i mod NSLOT.  Panels of different sizes come in whole stages (an even NSLOT).
  constexpr bool EQUAL = BM == BR;
  static_assert(EQUAL || NSLOT % 2 == 0, "panels of different sizes: whole stages");
  static_assert(KG == 1 || (KG == 4 && MI * NI == 1), "a slice and a block per wave");
  static_assert((NSLOT % 2 == 0 ? STAGE : BM * 128) >= NW / KG * 4096, "epilogue: 4 KiB per wave in the slots of one step");
  auto slot_byte = [](int slot) { return EQUAL ? slot * (BM * 128) : (slot >> 1) * STAGE + (slot & 1) * (BR * 128); };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (WAVES_M * WAVES_N);
  const int wm = wave % (WAVES_M * WAVES_N) / WAVES_N, wn = wave % WAVES_N;
  const int tile = tile_of_workgroup(block);
  // The tile's problem: the last one that starts at or before it.  Every lane looks at the first tile of up to four problems
  // and touches their entries, all in one round trip: a launch's first workgroups find the lists in no cache, and one load
  // after the other (number of problems, their list, the tile's, its entry) took them about a microsecond more: training pass of
  // 512 tokens, d = 256, float32 75.5 -> 72.2 us, 389 tokens, d = 2048 154 -> 151.
  constexpr int CHUNKS = MODSE_MAX_PROBLEMS / 64;
  const int total = plan->tile_start[n_prob];
  int starts[CHUNKS], touch[CHUNKS];
#pragma unroll
  for (int j = 0; j < CHUNKS; ++j) {
    if (j > 0 && j * 64 >= n_prob) break;
    starts[j] = plan->tile_start[min(j * 64 + lane, n_prob)];
    touch[j] = plan->prob[min(j * 64 + lane, n_prob - 1)].M;
  }
  if (tile >= total) return;
  int p = -1, start = 0;
#pragma unroll
  for (int j = 0; j < CHUNKS; ++j) {
    if (j > 0 && j * 64 >= n_prob) break;
    asm volatile("" ::"v"(touch[j]));
    const unsigned long long at = __ballot(j * 64 + lane < n_prob && starts[j] <= tile);
    if (at == 0) break;
    start = __builtin_amdgcn_readlane(starts[j], 63 - __builtin_clzll(at));
    p += __popcll(at);
  }
  p = uniform_int(p);
  ProblemRegs P;
  P.load(plan->prob + p);
  const int M = P.M(), N = P.N(), K = P.K();
  int mt, nt;
  decode_local(tile - uniform_int(start), P.mtiles(), P.ntiles(), P.magic_group(), P.magic_tail(), mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int nk = (K + BK - 1) / BK;
  const bool stream_b = !A_T && P.mtiles() == 1;  // weights that meet a single row block are read once in the whole launch
  // Where most problems have one row block, the weight stream is what bounds the launch.  Their rows usually lie a power of
  // two apart, so what the workgroups of a launch read at the same K step shares the low bits of its address, and few memory
  // channels serve it: a bare loader of these tiles reaches 5.3 TB/s, and 6.3 when the workgroups start their K loops at
  // different places.  So they do (GEMM_SPREAD_K), at 32 of them: 64 tokens at d = 4096 493 -> 470 us for the layer, 389 tokens
  // at d = 2048 169 -> 155.  The place goes by problem and column alone, and the launch by the batch's size: a row's result
  // then depends neither on the other rows nor on its place among them.
  constexpr bool ROTATE = !F32 && !A_T;
  const int first_k = ROTATE && (option & GEMM_SPREAD_K) ? (nk * ((nt * 5 + p) & 31)) >> 5 : 0;  // K step to start with
  const int nsteps = (EPI == EPI_STORE_DUALK) ? 2 * nk : nk;
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane(lds_address(ring));

  // ---- loads.  Which 16-byte chunk a lane fetches is chosen so that the data lands swizzled: unit u of a K-contiguous
  // panel is rows 8u .. 8u+7; of a [K, X] panel 1024 / (X * ES) rows of K.
  auto tr_swz = [](int k, int row_bytes) { return F32 ? 0 : row_bytes >= 256 ? 4 * (k & 3) : 4 * ((k >> 1) & 1); };
  // Offset (bytes) of this lane's chunk of unit u from the unit's first row (`unit`: that row's offset from the tile's first element),
  // and its K index.  (bf16 tiles stay below 2^32 bytes and count from the tile's first element; of float32 ones that holds for
  // the few rows of a unit.)
  auto chunk_offset = [&](bool tr, int X, int u, int x0, int rows, int ld, int& kfirst, size_t& unit) -> uint32_t {
    if (tr) {
      const int rb = X * ES, byte = lane * 16, k0 = u * (1024 / rb);
      const int k = k0 + byte / rb;
      const int c = ((byte % rb) >> 4) ^ tr_swz(k, rb);
      kfirst = k;
      unit = F32 ? (size_t)k0 * ld * ES : 0;
      return (uint32_t)((F32 ? k - k0 : k) * ld + (min(x0 + c * CE, rows - CE) - x0)) * ES;  // columns past the end repeat the last chunk
    }
    const int r = u * 8 + (lane >> 3), first = F32 ? min(x0 + u * 8 % X, rows - 1) : x0;
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    kfirst = c * CE;
    unit = (size_t)(first - x0) * ld * ES;
    return (uint32_t)((min(x0 + r % X, rows - 1) - first) * ld + c * CE) * ES;
  };
  uint32_t offa[UA], offb[UB];
  size_t unita[UA], unitb[UB];
  int ka[UA], kb[UB];
#pragma unroll
  for (int i = 0; i < UA; ++i) offa[i] = chunk_offset(A_T, BM, wave * UA + i, m0, M, P.lda(), ka[i], unita[i]);
#pragma unroll
  for (int i = 0; i < UB; ++i) offb[i] = chunk_offset(B_T, BN, wave * UB + i, n0, N, P.ldb(), kb[i], unitb[i]);
  const size_t a_org = (A_T ? (size_t)m0 : (size_t)m0 * P.lda()) * ES;
  const size_t b_org = (B_T ? (size_t)n0 : (size_t)n0 * P.ldb()) * ES;
  const size_t a_step = A_T ? (size_t)128 * P.lda() : 128, b_step = B_T ? (size_t)128 * P.ldb() : 128;
  const bool second = NB == 2 && wave * UB * 8 >= BN;  // this wave's B units belong to the second matrix
  // an operand of a pass at K step k
  auto at_k = [&](bool is_a, bool pass2, int k) {
    const char* const b = is_a ? (pass2 ? P.A2() : P.A()) : (second || pass2 ? P.B2() : P.B());
    return static_cast<const char*>(uniform_ptr(b + (is_a ? a_org + k * a_step : b_org + k * b_step)));
  };
  const char* sa = at_k(true, false, first_k);
  const char* sb = at_k(false, false, first_k);
  // the loads of one operand's next panel into ring slot `slot`; the operand then moves on to its next K step
  struct Walk {
    int step = 0, kstep;  // of all steps; along K
  } wa, wb;
  wa.kstep = wb.kstep = first_k;
  auto issue = [&](auto is_a, Walk& w, const char*& src, int slot) {
    constexpr bool IS_A = decltype(is_a)::value;
    constexpr int U = IS_A ? UA : UB;
    if (w.step >= nsteps) return;
    const uint32_t dst = lds_base + slot_byte(slot) + wave * U * 1024;
    auto off = [&](int i) { if constexpr (IS_A) return offa[i]; else return offb[i]; };
    auto unit = [&](int i) -> size_t { if constexpr (!F32) return 0; else if constexpr (IS_A) return unita[i]; else return unitb[i]; };
    auto kfirst = [&](int i) { if constexpr (IS_A) return ka[i]; else return kb[i]; };
    if ((w.kstep + 1) * BK <= K) {
#pragma unroll
      for (int i = 0; i < U; ++i) {
        if (!F32 && !IS_A && stream_b) dma_b128_s<true>(src, off(i), dst + i * 1024);
        else dma_b128_s(src + unit(i), off(i), dst + i * 1024);
      }
    } else {  // the last step of a pass: what lies beyond K reads zeros
#pragma unroll
      for (int i = 0; i < U; ++i)
        dma_b128(w.kstep * BK + kfirst(i) < K ? src + unit(i) + off(i) : reinterpret_cast<const char*>(g_zero_chunk), dst + i * 1024);
    }
    src += IS_A ? a_step : b_step;
    ++w.step;
    ++w.kstep;
    if (ROTATE && w.kstep == nk && first_k != 0) {  // from the end of K back to its beginning
      w.kstep = 0;
      src = at_k(IS_A, EPI == EPI_STORE_DUALK && w.step > nk, 0);
    }
    if (EPI == EPI_STORE_DUALK && w.step == nk) {
      w.kstep = first_k;
      src = at_k(IS_A, true, first_k);
    }
  };
  auto issue_a = [&](int slot) { issue(std::true_type{}, wa, sa, slot); };
  auto issue_b = [&](int slot) { issue(std::false_type{}, wb, sb, slot); };

  // ---- fragments: K slice kk (two chunks of every row)
  typedef std::conditional_t<F32, f32x4, bf16x8> frag_t;
  const int khalf = lane >> 5, lsw = (lane >> 1) & 7;
  const int blk = lane >> 4, sl = lane & 15, kq = sl >> 2;
  auto load_frag = [&](bool tr, const char* panel, int X, int row, int kk) -> frag_t {  // row: first of the 32 (or, [K, X], column)
    if (!tr) return *reinterpret_cast<const frag_t*>(panel + (row + (lane & 31)) * 128 + (((kk * 2 + khalf) ^ lsw) << 4));
    const int rb = X * ES;
    if constexpr (F32) {
      frag_t v;
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = *reinterpret_cast<const float*>(panel + (kk * 8 + khalf * 4 + s) * rb + (row + (lane & 31)) * 4);
      return v;
    } else {
      // lane 16 blk + sl reads 8 bytes at K row kk*16 + (blk >> 1)*8 + h*4 + (sl >> 2), column row + (blk & 1)*16 +
      // 4 (sl & 3) and receives four consecutive K of column row + (blk & 1)*16 + sl
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
      const int c16 = (row + (blk & 1) * 16) / 8 + ((sl & 3) >> 1);
      const char* q = panel + (kk * 16 + (blk >> 1) * 8 + kq) * rb + ((c16 ^ tr_swz(kq, rb)) << 4) + (sl & 1) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(q));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(q + 4 * rb));
      const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(frag_t, v);
    }
  };
  frag_t af[2][MI], bf[2][NB][NI];
  auto load_frags = [&](const char* pa, const char* pb, int kk, int set) {
#pragma unroll
    for (int i = 0; i < MI; ++i) af[set][i] = load_frag(A_T, pa, BM, wm * WM + i * 32, kk);
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int j = 0; j < NI; ++j) bf[set][q][j] = load_frag(B_T, pb, BN, q * BN + wn * WN + j * 32, kk);
  };
  f32x16 acc[NB][MI][NI];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][i][j][r] = 0.f;
  // (the B fragment is the instruction's first operand: a lane's accumulator then holds four consecutive columns of C)
  auto mfma_slice = [&](int set, auto behind_first) {  // behind_first(): called behind the slice's first MFMA
    if constexpr (F32) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
              acc[q][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bf[set][q][j][s], af[set][i][s], acc[q][i][j], 0, 0, 0);
              if (s + q + i + j == 0) behind_first();
            }
    } else {
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[q][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[set][q][j], af[set][i], acc[q][i][j], 0, 0, 0);
    }
  };

  int rb = 0;  // slot of step g's B panel; its A panel is in the next one
  auto slot_add = [](int slot, int d) { return slot + d >= NSLOT ? slot + d - NSLOT : slot + d; };
  if constexpr (F32 && KG == 1) {
    // The matrix pipe is the bound, so nothing may stand between two MFMAs of a wave but what runs in their shadow.  Everybody meets
    // before the last slice of a step, whose fragments are in registers: the first ones of the next step are then read behind its
    // MFMAs, and the step's own panels, which nobody reads any more, are refilled behind them, a step and a quarter ahead.
    // Against meeting between two steps, with the loads in front of the first MFMA: training pass of 4096 tokens, d = 1024, 3775 ->
    // 3738 us; with a scalar base per load unit and 32-bit lane offsets, which issue faster than 64-bit addresses, 3492.
    // (Loads spread one by one over the step's MFMAs: 128 x 128 tiles no better than before.)
    static_assert(NSLOT == 4, "two stages");
    auto meet = [&](bool one_stage_behind) {  // my LDS reads have returned and my loads have landed (but the youngest stage's)
      __builtin_amdgcn_sched_barrier(0);
      if (one_stage_behind) __builtin_amdgcn_s_waitcnt(0x0070 | (UA + UB));
      else __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    static_assert(UA + UB < 16, "vmcnt field");
#pragma unroll 1
    for (int slot = 0; slot < NSLOT; slot += 2) {
      issue_b(slot);
      issue_a(slot + 1);
    }
    if (nsteps > 0) {
      meet(nsteps > 1);
      load_frags(ring + slot_byte(1), ring + slot_byte(0), 0, 0);
    }
#pragma unroll 1
    for (int g = 0; g < nsteps; ++g) {
      const int next = slot_add(rb, 2);
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        load_frags(ring + slot_byte(slot_add(rb, 1)), ring + slot_byte(rb), kk + 1, (kk + 1) & 1);
        mfma_slice(kk & 1, [] {});
      }
      meet(false);
      if (g + 1 < nsteps) load_frags(ring + slot_byte(slot_add(next, 1)), ring + slot_byte(next), 0, 0);
      mfma_slice(1, [&] {
        __builtin_amdgcn_sched_barrier(0);
        issue_b(rb);
        issue_a(slot_add(rb, 1));
        __builtin_amdgcn_sched_barrier(0);
      });
      rb = next;
    }
  } else {
#pragma unroll
    for (int i = 0; i < NSLOT - 2; ++i) {
      if (i % 2 == 0) issue_b(i);
      else issue_a(i);
    }
#pragma unroll 1
    for (int g = 0; g < nsteps; ++g) {
      // my loads of step g have landed (those of the NSLOT - 4 panels behind it may still be on their way; s_waitcnt simm16:
      // vmcnt in bits [3:0] and [15:14]) and my LDS reads of step g - 1 have returned; then everybody meets: the panels of
      // step g may be read and those of step g - 1 refilled
      __builtin_amdgcn_sched_barrier(0);
      constexpr int AHEAD = (NSLOT - 4) / 2 * UA + (NSLOT - 3) / 2 * UB;
      static_assert(AHEAD < 64, "vmcnt field");
      if (2 * g + NSLOT - 2 <= 2 * nsteps) __builtin_amdgcn_s_waitcnt(0x0070 | (AHEAD & 15) | (AHEAD >> 4) << 14);  // lgkmcnt(0)
      else __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      const char* pb = ring + slot_byte(rb);
      const char* pa = ring + slot_byte(slot_add(rb, 1));
      load_frags(pa, pb, KG > 1 ? kg : 0, 0);
      if constexpr (NSLOT % 2 == 0) {
        issue_b(slot_add(rb, NSLOT - 2));
        issue_a(slot_add(rb, NSLOT - 1));
      } else {
        issue_a(slot_add(rb, NSLOT - 2));
        issue_b(slot_add(rb, NSLOT - 1));
      }
      rb = slot_add(rb, 2);
#pragma unroll
      for (int kk = 0; kk < 4 / KG; ++kk) {
        if (kk < 4 / KG - 1) load_frags(pa, pb, kk + 1, (kk + 1) & 1);
        mfma_slice(kk & 1, [] {});
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (KG > 1) {  // (nothing is on its way into LDS any more, and behind the barrier nobody reads a panel)
    char* const sums = ring + lane * 16;
    auto part = [&](int g, int q, int r) { return reinterpret_cast<f32x4*>(sums + (((g - 1) * NB + q) * 4 + r) * 1024); };
    static_assert(ring_bytes(BM, BR, NSLOT) >= (KG - 1) * NB * 4096, "the groups' sums");
    __syncthreads();
    if (kg > 0) {
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *part(kg, q, r) = f32x4{acc[q][0][0][4 * r], acc[q][0][0][4 * r + 1], acc[q][0][0][4 * r + 2], acc[q][0][0][4 * r + 3]};
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g)
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const f32x4 v = *part(g, q, r);
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[q][0][0][4 * r + c] += v[c];
        }
  }

  // ---- epilogue.  For register group r of block (i, j) the lane holds columns 8 r + 4 khalf .. + 3 of row lane & 31.
  // A wave stages units of 32 rows x 128 bytes (64 for a 32-column bf16 tile) through LDS, so that global memory sees
  // whole lines: written in accumulator order, read back row-wise.  The staging area lies in the slots that the step
  // after the last one would use: nobody reads them any more and no load is on its way into them.
  typedef std::conditional_t<F32 || EPI == EPI_STORE_F32, float, bf16_t> out_t;
  constexpr int OS = sizeof(out_t), UC = OS == 4 ? 32 : (WN < 64 ? WN : 64);  // columns of a unit
  constexpr int CPR = UC * OS / 16, ITS = 32 * CPR / 64, NJU = WN / UC, JPU = UC / 32;
  typedef std::conditional_t<OS == 4, f32x4, bf16x8> chunk_t;
  char* const slot = ring + slot_byte(rb) + wave * 4096;
  const int er = lane & 31, esw = (er >> 1) & 7;
  const int ldc = P.ldc();
  auto stage = [&](auto value) {  // value(jj, idx): element idx of the accumulator of the unit's block jj
#pragma unroll
    for (int jj = 0; jj < JPU; ++jj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (OS == 4) {
          const f32x4 v = {value(jj, 4 * r), value(jj, 4 * r + 1), value(jj, 4 * r + 2), value(jj, 4 * r + 3)};
          *reinterpret_cast<f32x4*>(slot + er * 128 + (((2 * r + khalf) ^ esw) << 4)) = v;
        } else {
          bf16x4 v;
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = (bf16_t)value(jj, 4 * r + q);
          *reinterpret_cast<bf16x4*>(slot + er * 128 + (((jj * 4 + r) ^ esw) << 4) + khalf * 8) = v;
        }
      }
  };
  auto row_of = [&](int it) { return it * (64 / CPR) + lane / CPR; };
  auto chunk = [&](int it) -> chunk_t* {
    const int rr = row_of(it);
    return reinterpret_cast<chunk_t*>(slot + rr * 128 + (((lane % CPR) ^ ((rr >> 1) & 7)) << 4));
  };
  typedef __attribute__((address_space(1))) chunk_t global_chunk_t;
  // element offset of this lane's chunk `it` of unit (i, ju) in C, or -1 outside the matrix
  auto offset = [&](int i, int ju, int it) -> long {
    const int m = m0 + wm * WM + i * 32 + row_of(it), n = n0 + wn * WN + ju * UC + (lane % CPR) * (16 / OS);
    return (m < M && n < N) ? (long)m * ldc + n : -1;
  };
  auto at = [&](const void* base, long o) { return (global_chunk_t*)(uintptr_t)(static_cast<const out_t*>(base) + o); };
  auto put = [&](void* C, long o, chunk_t v) {
    if (A_T && (option & GEMM_STREAM_C)) __builtin_nontemporal_store(v, at(C, o));
    else *at(C, o) = v;
  };
  auto get = [&](const void* C, long o) -> chunk_t {  // old values of C that are added to
    return option & GEMM_STREAM_C ? __builtin_nontemporal_load(at(C, o)) : *at(C, o);
  };
  auto store_unit = [&](int i, int ju, void* C) {
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const chunk_t v = *chunk(it);
      const long o = offset(i, ju, it);
      if (o >= 0) put(C, o, v);
    }
  };
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (m0 + wm * WM + i * 32 >= M) break;
#pragma unroll
    for (int ju = 0; ju < NJU; ++ju) {
      const int j0 = ju * JPU;
      if constexpr (EPI == EPI_SWIGLU) {
        stage([&](int jj, int x) {
          const float a = acc[0][i][j0 + jj][x], b = acc[NB - 1][i][j0 + jj][x];
          float h, pd, qd;
          swiglu_terms(a, b, F32 ? 1.f / (1.f + __expf(-a)) : sigmoid_fast(a), h, pd, qd);
          acc[0][i][j0 + jj][x] = pd;
          acc[NB - 1][i][j0 + jj][x] = qd;
          return h;
        });
        store_unit(i, ju, P.C());
        if (option & GEMM_SAVE_TERMS) {
          stage([&](int jj, int x) { return acc[0][i][j0 + jj][x]; });
          store_unit(i, ju, P.C2());
          stage([&](int jj, int x) { return acc[NB - 1][i][j0 + jj][x]; });
          store_unit(i, ju, P.C3());
        }
      } else {
        if constexpr (EPI == EPI_SWIGLU_BWD) {
          // the saved terms dh/da and dh/db come in row-wise, are multiplied by dh in accumulator order where they lie
          // in LDS, and leave row-wise
          chunk_t e[2][ITS];
#pragma unroll
          for (int w = 0; w < 2; ++w)
#pragma unroll
            for (int it = 0; it < ITS; ++it) {
              const long o = offset(i, ju, it);
              e[w][it] = o >= 0 ? *at(w ? P.E2() : P.E1(), o) : chunk_t{};
            }
#pragma unroll
          for (int w = 0; w < 2; ++w) {
#pragma unroll
            for (int it = 0; it < ITS; ++it) *chunk(it) = e[w][it];
#pragma unroll
            for (int jj = 0; jj < JPU; ++jj)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                typedef std::conditional_t<OS == 4, f32x4, bf16x4> quad_t;
                quad_t& v = *reinterpret_cast<quad_t*>(OS == 4 ? slot + er * 128 + (((2 * r + khalf) ^ esw) << 4)
                                                               : slot + er * 128 + (((jj * 4 + r) ^ esw) << 4) + khalf * 8);
                quad_t o = v;
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = (out_t)(acc[0][i][j0 + jj][4 * r + q] * (float)o[q]);
                v = o;
              }
            store_unit(i, ju, w ? P.C2() : P.C());
          }
          continue;
        }
        stage([&](int jj, int x) { return acc[0][i][j0 + jj][x]; });
        if constexpr (EPI == EPI_STORE_F32) {
          if (accumulate) {
            chunk_t old[ITS];
#pragma unroll
            for (int it = 0; it < ITS; ++it) {
              const long o = offset(i, ju, it);
              old[it] = o >= 0 ? get(P.C(), o) : chunk_t{};
            }
#pragma unroll
            for (int it = 0; it < ITS; ++it) {
              const chunk_t v = *chunk(it) + old[it];
              const long o = offset(i, ju, it);
              if (o >= 0) put(P.C(), o, v);
            }
            continue;
          }
        }
        store_unit(i, ju, P.C());
      }
    }
  }
}

#define MODSE_RING(BM, BR, NSLOT) __shared__ __attribute__((aligned(1024))) char ring[ring_bytes(BM, BR, NSLOT)]
template <int BM, int BN, int NB, int EPI, int LAYOUT>
__global__ __launch_bounds__(256, 2) void gg_f32_kernel(const GemmPlan* __restrict__ plan, int n_prob, int accumulate, int option) {
  MODSE_RING(BM, NB * BN, 4);
  gg_block<float, BM, BN, NB, 2, 2, 4, EPI, LAYOUT>(plan, n_prob, accumulate, option, blockIdx.x, ring);
}
// Launches of few tiles.  Bound by latency: of the workgroup's start, of the loads of a K step, of the dependent matrix
// instructions of a wave.  So the tile is small (32 x 32), its four waves take one K slice of a step each and add up through
// LDS, and 32 to 36 KiB of ring let four workgroups of a CU wait at a time.  d = 256, 512 tokens: up-projection 14 -> 11 us,
// dX 19 -> 11; with twice the ring and two workgroups per CU the same there, but up to 6 % slower for whole layers of more tiles.
constexpr int small_slots(int nb) { return nb == 1 ? 8 : 6; }
template <int NB, int EPI, int LAYOUT>
__global__ __launch_bounds__(256, 4) void gg_f32_small_kernel(const GemmPlan* __restrict__ plan, int n_prob, int accumulate, int option) {
  MODSE_RING(32, NB * 32, small_slots(NB));
  gg_block<float, 32, 32, NB, 1, 1, small_slots(NB), EPI, LAYOUT, 4>(plan, n_prob, accumulate, option, blockIdx.x, ring);
}
// What follows dH in one launch: the first n_dwg workgroups take the router's weight gradient (of a plain gate), the next `dx_blocks` dX (tiles
// of DX_TILE), the others the weight gradients.  None needs another, and in a layer of few tiles each leaves most of the chip
// idle and takes as long as its chain of latencies: 512 tokens, d = 256 6.8 + 10.9 + 9.6 us in launches of their own, 14.6 in
// one; training pass 72.3 -> 59.6 us.  Backward passes of 24 drawn layers, 38 to 11597 tokens, d = 128 to 1024: 0.996 to 1.47 times
// as fast, on average 1.21.  (The router's tokens come in batches of two: 128 registers.)
template <int DX_TILE, int DX_EPI>
__global__ __launch_bounds__(256, 4) void gg_f32_dx_wgrad_kernel(DwgArgs dwg, int n_dwg, const GemmPlan* __restrict__ dx, int n_dx,
                                                                 int dx_blocks, const GemmPlan* __restrict__ wg, int n_wg,
                                                                 int accumulate, int option) {
  static_assert(ring_bytes(32, 32, 8) == ring_bytes(64, 64, 4) && sizeof(DwgSums) == ring_bytes(64, 64, 4), "one piece of LDS for all");
  MODSE_RING(64, 64, 4);
  const int block = (int)blockIdx.x - n_dwg;
  if (block < 0)
    bwd_dwg_block<float, 2>(dwg, blockIdx.x, *reinterpret_cast<DwgSums*>(ring));
  else if (block >= dx_blocks)
    gg_block<float, 64, 64, 1, 2, 2, 4, EPI_STORE_F32, LAYOUT_AB_K>(wg, n_wg, accumulate, option, block - dx_blocks, ring);
  else if constexpr (DX_TILE == 32)
    gg_block<float, 32, 32, 1, 1, 1, small_slots(1), DX_EPI, LAYOUT_B_KN, 4>(dx, n_dx, 0, 0, block, ring);
  else
    gg_block<float, 64, 64, 1, 2, 2, 4, DX_EPI, LAYOUT_B_KN>(dx, n_dx, 0, 0, block, ring);
}
// as many ring slots as leave room for eight waves per CU
constexpr int ring_slots(int bm, int br, int waves) {
  const int lds = 160 * 1024 / 8 * waves;
  return bm == br ? lds / (bm * 128) : lds / ((bm + br) * 128) * 2;
}
template <int BM, int BN, int NB, int WAVES_M, int WAVES_N, int EPI, int LAYOUT>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, 2) void gg_bf16_block_kernel(const GemmPlan* __restrict__ plan, int n_prob,
                                                                               int accumulate, int option) {
  constexpr int NSLOT = ring_slots(BM, NB * BN, WAVES_M * WAVES_N);
  MODSE_RING(BM, NB * BN, NSLOT);
  gg_block<bf16_t, BM, BN, NB, WAVES_M, WAVES_N, NSLOT, EPI, LAYOUT>(plan, n_prob, accumulate, option, blockIdx.x, ring);
}
// tiles of 32 or 64 rows (decode-sized batches and experts with few tokens), under a name of their own for profiles
template <int BM, int BN, int NB, int WAVES_M, int WAVES_N, int EPI, int LAYOUT>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, 2) void gg_bf16_skinny_kernel(const GemmPlan* __restrict__ plan, int n_prob,
                                                                                int accumulate, int option) {
  constexpr int NSLOT = ring_slots(BM, NB * BN, WAVES_M * WAVES_N);
  MODSE_RING(BM, NB * BN, NSLOT);
  gg_block<bf16_t, BM, BN, NB, WAVES_M, WAVES_N, NSLOT, EPI, LAYOUT>(plan, n_prob, accumulate, option, blockIdx.x, ring);
}
// The same for bf16, dX in tiles of 64 or 128 rows: the n_dwg workgroups behind its `dx_blocks` take the router's weight gradient (of a
// plain gate; by itself worth a launch, which at two micro-batches of 1021 tokens is less than the runs differ), and if the weight
// gradients have 128-row tiles, too, they follow: training passes at d = 1024, eight experts of mean width 1024, 512 / 2048 tokens
// 113 -> 108 / 207 -> 191 us; d = 2048, four experts of 1408, 1024 tokens 243 -> 212.  Backward passes of 34 drawn layers with
// such tiles, 33 to 14313 tokens, d = 512 to 4096: 1.02 to 1.30 times as fast, on average 1.10.
template <int BM, int EPI>
__global__ __launch_bounds__(256, 2) void gg_bf16_dx_kernel(const GemmPlan* __restrict__ dx, int n_dx, int dx_option, int dx_blocks,
                                                            DwgArgs dwg, int n_dwg, const GemmPlan* __restrict__ wg, int n_wg,
                                                            int accumulate, int wg_option) {
  constexpr int NSLOT = ring_slots(BM, 128, 4), WG_SLOTS = ring_slots(128, 128, 4);
  MODSE_RING(128, 128, WG_SLOTS);
  static_assert(sizeof(DwgSums) <= sizeof(ring) && ring_bytes(BM, 128, NSLOT) <= sizeof(ring), "one piece of LDS for all");
  const int block = (int)blockIdx.x - dx_blocks;
  if (block < 0)
    gg_block<bf16_t, BM, 128, 1, 2, 2, NSLOT, EPI, LAYOUT_B_KN>(dx, n_dx, 0, dx_option, blockIdx.x, ring);
  else if (block < n_dwg)
    bwd_dwg_block<bf16_t, 8>(dwg, block, *reinterpret_cast<DwgSums*>(ring));
  else
    gg_block<bf16_t, 128, 128, 1, 2, 2, WG_SLOTS, EPI_STORE_F32, LAYOUT_AB_K>(wg, n_wg, accumulate, wg_option, block - n_dwg, ring);
}
#undef MODSE_RING

}  // namespace modse_gemm
