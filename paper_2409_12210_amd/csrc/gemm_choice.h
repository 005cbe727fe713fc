// Host code: which tiles a GEMM of the layer takes, and whether its K is split.  Pure functions of their arguments: the
// workspace sizes follow from them, and they have to be the same in every process, on every thread and without a device.
#pragma once
#include <algorithm>
#include <cmath>

#include "common.h"

namespace modse_gemm {

constexpr int GEMM_CUS = 256;  // compute units of the chip that the choices are made for

struct GemmChoice {
  TileShape tile;
  int32_t kchunk;  // the product's K = f_e is cut into ceil(f_e / kchunk) chunks (per operand pair); 0 = not split
};

// The realised token counts are known on the device only, so the choice goes by the mean number of rows r = T k / N of an
// expert, with loads spread evenly over r (1 - s) .. r (1 + s): s = 0.1 for up to a dozen experts and more for more, which
// are balanced less well.

// expected number of row blocks of an expert
inline double row_blocks(const LayerDims& L, int bm) {
  const double r = (double)L.T * L.k / L.N, s = std::max(0.1, std::min(0.5, L.N / 128.0)), most = r * (1 + s);
  // 1 + the sum over j >= 1, j bm < most, of min(1, (most - j bm) / (2 s r))
  const double last = std::max(0.0, std::ceil(most / bm) - 1), full = std::max(0.0, std::min(last, std::floor((most - 2 * s * r) / bm)));
  return 1 + full + (r > 0 ? (last - full) * (most - bm * (full + 1 + last) / 2) / (2 * s * r) : 0);
}

// Whether the K loops of a product that reads weights start at different places: where most experts have one row block.
// (With more of them per expert the row blocks that share weights find them in L2, and starting by column took 3 % longer.)
// By the batch's size, not by the realised counts: the order of a row's sums must not depend on the other rows.
inline bool spread_k(const LayerDims& L, modse_dtype dt, TileShape t) {
  return dt == MODSE_BF16 && t.bm <= 128 && row_blocks(L, t.bm) < 1.5;
}

// One product with output tiles of all experts: `tiles` of them with K steps of 64 each
struct Work {
  double tiles = 0, steps = 0;  // totals (steps: over all tiles)
  double longest = 0;           // K steps of the longest tile
  void add(double t, double k) {
    tiles += t;
    steps += t * k;
    longest = std::max(longest, k);
  }
};
inline Work gemm_work(const LayerDims& L, int epilogue, TileShape t) {
  const double mb = row_blocks(L, t.bm);
  auto blocks = [](int n, int b) { return (double)((n + b - 1) / b); };
  Work w;
  for (int e = 0; e < L.N; ++e) {
    const int f = L.f[e], d = L.d;
    switch (epilogue) {
      case EPI_SWIGLU:
      case EPI_SWIGLU_BWD: w.add(mb * blocks(f, t.bn), blocks(d, 64)); break;
      case EPI_STORE: w.add(mb * blocks(d, t.bn), blocks(f, 64)); break;
      case EPI_STORE_DUALK: w.add(mb * blocks(d, t.bn), 2 * blocks(f, 64)); break;
      case EPI_STORE_F32:
        w.add(2 * blocks(f, t.bm) * blocks(d, t.bn) + blocks(d, t.bm) * blocks(f, t.bn), row_blocks(L, 64));
        break;
    }
  }
  return w;
}

// Estimated time in us of a bf16 product (chunk: K steps of a split product's problems, 0 = not split), fitted to the
// measured times of all five GEMMs at d = 1024 ... 4096, 4 ... 64 experts and 16 ... 8192 tokens.  A step of a tile takes
// 1.6 us in the 256 x 256 kernel (one workgroup per CU), 1.1 us (weight gradients: 1.85, dH: 1.15) with 128-row tiles and
// 0.8 us (dH: 1.0) with 64-row ones
// (two workgroups per CU); a tile pays for its opening and its epilogue with `fix` further steps, and the float32 slabs of
// a split product are written and read at 4 TB/s.
inline double gemm_cost(const LayerDims& L, int epilogue, TileShape t, int chunk) {
  const double cus = GEMM_CUS;
  Work w = gemm_work(L, epilogue, t);
  if (w.tiles < 1) return 0;
  const bool wgrad = epilogue == EPI_STORE_F32;
  const bool same = wgrad || epilogue == EPI_SWIGLU || epilogue == EPI_SWIGLU_BWD;  // tiles of one length
  if (t.bm == 256) {
    const double fix = wgrad ? 6.8 : 4;
    const double mean = w.steps / w.tiles + fix;
    const double rounds = w.tiles / cus;
    if (wgrad) return (std::ceil(rounds) + 0.3) * mean * 1.67;  // (their number does not depend on the routing)
    if (same) return (rounds < 0.9 ? 1 : rounds + 0.7) * mean * 1.58;  // whole rounds, of a number that is only expected
    // (a lone workgroup's steps are shorter when other CUs stand idle)
    return std::max((rounds + 0.2) * mean, (0.75 + 0.1 * std::min(1.0, w.tiles / cus)) * (w.longest + fix)) * 1.67;
  }
  const double fix = 2.5, slots = 2 * cus;
  const double us = wgrad ? 1.85 : epilogue == EPI_SWIGLU_BWD ? (t.bm == 128 ? 1.15 : 1.0) : t.bm == 128 ? 1.1 : 0.8;
  double mean = w.steps / w.tiles + fix, chain = w.longest + fix, slabs = 0;
  if (chunk) {
    const double n = std::max(1.0, w.steps / w.tiles / chunk);
    slabs = 2 + n * L.T * L.k * L.d * (8 / 4e6);
    w.tiles *= n;
    mean = chain = chunk + fix;
  }
  // a workgroup that has its CU for itself runs faster
  const double alone = 0.62 + 0.38 * std::min(1.0, std::max(0.0, (w.tiles - cus) / cus));
  const double rounds = wgrad ? w.tiles / slots : !same ? w.tiles / slots + 0.35 : w.tiles > slots ? w.tiles / slots + 0.6 : 0;
  return std::max(rounds * mean, chain * alone) * us + slabs;
}

// Chunk length of a split K = f_e (a multiple of 64), or 0.  A batch with few rows has too few output tiles (d / bn per
// expert and row block) to fill the chip, and K loops of up to f_e / 64 (dX: twice that) steps in a row; cut into chunks
// that become problems of their own it fills the workgroup slots.  Each chunk costs a float32 slab of rows x d, written
// and read once, so chunks are not made shorter than 640 columns.
// Decode-sized batches, whose slabs are small, take more and shorter chunks: they are bound by the weight stream, which
// runs better the more loads are in flight (d = 4096, 64 tokens: 512 / 1024 / 1536 tiles 180 / 183 / 178 us; 16 tokens
// 177 / 173 / 164).
inline int split_chunk(const LayerDims& L, modse_dtype dt, TileShape t, int passes) {
  const int64_t rows = ((int64_t)L.T * L.k + L.N - 1) / L.N;
  const int64_t tiles = ((rows + t.bm - 1) / t.bm) * ((L.d + t.bn - 1) / t.bn);  // of one expert
  const int64_t cus = GEMM_CUS, target = dt == MODSE_F32 ? (t.bm == 64 ? 4 : 2) * cus
                                          : t.bm == 32    ? 6 * cus
                                          : passes == 1     ? (t.bm == 64 ? 4 : 3) * cus : 2 * cus;
  if (t.bm > 128 || t.bn > 128 || tiles == 0 || 4 * L.N * tiles > 3 * target) return 0;
  int64_t F = 0, fmax = 0;
  for (int e = 0; e < L.N; ++e) {
    F += passes * (int64_t)L.f[e];
    fmax = std::max<int64_t>(fmax, L.f[e]);
  }
  const int64_t want = (target + tiles - 1) / tiles, most = MODSE_MAX_PROBLEMS - passes * L.N;
  // passes * sum_e ceil(f_e / chunk) <= F / chunk + passes * N, which has to be at most MODSE_MAX_PROBLEMS
  int64_t chunk = std::min<int64_t>(std::max<int64_t>((F + want - 1) / want, 640), 4096);
  chunk = (int64_t)align_up((size_t)std::max<int64_t>(chunk, (F + most - 1) / most), 64);
  return fmax > 2 * chunk ? (int)chunk : 0;
}
// bf16 products with d columns: mean rows of an expert up to which they take the tiles of 32 and 64 rows
constexpr int split_rows_max(int bm) { return bm == 32 ? 28 : 58; }

inline GemmChoice gemm_choice(const LayerDims& L, modse_dtype dt, int epilogue) {
  const int passes = epilogue == EPI_STORE ? 1 : epilogue == EPI_STORE_DUALK ? 2 : 0;  // 0: never split
  auto with_chunk = [&](TileShape t) {
    GemmChoice c = {t, passes ? split_chunk(L, dt, t, passes) : 0};
    if (c.kchunk && dt == MODSE_BF16 && t.bm > 32 && gemm_cost(L, epilogue, t, c.kchunk / 64) > gemm_cost(L, epilogue, t, 0))
      c.kchunk = 0;
    return c;
  };
  const double r = (double)L.T * L.k / L.N;
  const bool swiglu = epilogue == EPI_SWIGLU;  // `bn` columns of each of the two matrices
  if (dt == MODSE_F32) {
    // 128 x 128 tiles (a wave then needs four LDS reads per sixteen matrix instructions) where their rounds, two tiles per
    // CU, fit the work; 64 x 64 ones are up to 10 % slower but leave less of a last round empty (d = 1024, 4096 tokens:
    // down-projection of 544 large tiles 509 us, 462 with small ones; up-projection of 2992 large tiles 788, 821)
    const TileShape t = swiglu ? TileShape{128, 64} : TileShape{128, 128}, t64 = {64, 64};
    const double slots = 2 * GEMM_CUS, rounds = gemm_work(L, epilogue, t).tiles / slots;
    const double small = gemm_work(L, epilogue, t64).tiles / (swiglu ? 2 : 4) / slots;  // in units of a large tile's work
    const GemmChoice c = with_chunk(rounds >= 1 && rounds + 0.3 <= 1.07 * small + 0.15 ? t : t64);
    // Fewer than one and a half 64 x 64 tiles per CU leave matrix pipes idle and each K loop's chain of latencies exposed: 32 x
    // 32 tiles, four to a CU, whose four waves share out the K slices, unless the 64 x 64 ones fill the CUs once (or twice) and
    // the others mean a further part of a round.  Estimates in K steps of a 64 x 64 tile alone on its CU (two of them take
    // 1.7), fitted to four products each of 100 layers, d = 32 ... 2528.  Sum of the four products in us, 64 -> 32: eight
    // experts, d = d_ff = 256, 512 tokens (80 tiles) 48 -> 36, 1500 tokens (204) 49 -> 57, 2048 tokens (272) 73 -> 70; d = d_ff =
    // 1024, 100 tokens (128) 129 -> 92, 384 tokens (256) 132 -> 157, 500 tokens (320) 226 -> 196.  One K step is enough
    // to share out: d = d_ff = 32, 256 tokens 16.1 -> 14.8, d = d_ff = 64 20.2 -> 18.2.
    const Work w = gemm_work(L, epilogue, t64), w32 = gemm_work(L, epilogue, TileShape{32, 32});
    const double large = std::max(w.longest, w.tiles > GEMM_CUS ? 1.7 * w.steps / w.tiles : 0.0);
    const bool few = epilogue != EPI_STORE_F32 && c.kchunk == 0 && 2 * w.tiles < 3 * GEMM_CUS &&
                     0.35 * w.longest + 0.25 * w32.steps / GEMM_CUS < large;
    return few ? GemmChoice{TileShape{32, 32}, 0} : c;
  }
  // The products with d columns: 32-row tiles for decode-sized batches (20 KiB a K step, four of them in flight), 64-row
  // tiles as long as they hold an expert's rows.  d = 2048, eight experts: 32 rows (T = 130) 32 against 64 rows 54 / 56
  // us with 64 / 128-row tiles, 97 rows 74 / 71.
  if (passes) {
    if (passes == 1 && r <= split_rows_max(32)) return with_chunk(TileShape{32, 128});
    if (r <= split_rows_max(64)) return with_chunk(TileShape{64, 128});
  }
  GemmChoice best = {swiglu ? TileShape{256, 128} : TileShape{256, 256}, 0};
  // (loads less even than assumed cost the large tiles more, hence the 5 %)
  double cost = 1.05 * gemm_cost(L, epilogue, best.tile, 0);
  for (int bm = 128; bm >= 64; bm -= 64) {
    if (bm == 64 && (passes || epilogue == EPI_STORE_F32)) break;
    // (weight gradients of many tiles are bound by their stores, which the larger tiles do better)
    if (epilogue == EPI_STORE_F32 && gemm_work(L, epilogue, best.tile).tiles > 16 * GEMM_CUS) break;
    const GemmChoice c = with_chunk(swiglu ? TileShape{bm, 64} : TileShape{bm, 128});
    const double mine = gemm_cost(L, epilogue, c.tile, c.kchunk / 64);
    if (mine < cost) {
      cost = mine;
      best = c;
    }
  }
  return best;
}

// Calls visit(T', kchunk) with token counts T' <= L.T among which is the one whose split product has the largest partial
// sums.  For a given tile the chunk length goes by the number of row blocks of an expert's mean rows, so the largest T' of
// each number of them does (whether such a batch really takes that tile does not matter for an upper bound).  At most a few
// hundred visits, for layers of a few narrow experts; usually one to twenty.
template <typename Visit>
inline void for_each_split(LayerDims L, modse_dtype dt, int epilogue, Visit visit) {
  const int64_t T = L.T;
  const int passes = epilogue == EPI_STORE ? 1 : 2;
  for (int bm = dt == MODSE_BF16 && passes == 1 ? 32 : 64; bm <= 128; bm *= 2) {
    const TileShape t = {bm, dt == MODSE_F32 ? bm : 128};
    // (bf16: the tiles of 32 and 64 rows are for that many mean rows per expert only)
    const int64_t most = std::min(T, dt == MODSE_BF16 && bm < 128 ? (int64_t)split_rows_max(bm) * L.N / L.k : T);
    for (int64_t blocks = 1;; ++blocks) {
      const int64_t tokens = std::min(most, blocks * bm * L.N / L.k);
      L.T = (int32_t)tokens;
      const int kchunk = split_chunk(L, dt, t, passes);
      if (kchunk == 0) break;  // nor for more rows
      visit(tokens, kchunk);
      if (tokens == most) break;
    }
  }
}

}  // namespace modse_gemm
