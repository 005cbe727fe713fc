// C ABI of libmodse: argument checks, workspace carving and the launch sequence of the MoDSE layer
// (forward: route -> permute -> grouped up-GEMM + SwiGLU -> grouped down-GEMM -> combine; backward: the
// chain rule through the same steps).  Nothing here allocates device memory or synchronises, except the
// opt-in per-stage timing.
#include <algorithm>
#include <cstring>

#include "bwd_dwg.h"
#include "common.h"
#include "gemm_choice.h"

namespace {
using modse_gemm::GemmChoice;
using modse_gemm::gemm_choice;

struct Carver {
  size_t off = 0;
  size_t take(size_t bytes) {
    const size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  }
};

size_t esize_of(modse_dtype dt) { return dt == MODSE_F32 ? 4 : 2; }

modse_status check_desc(const modse_desc* desc, int64_t T) {
  if (!desc || !desc->d_ff) return MODSE_ERR_INVALID_ARG;
  if (T < 0) return MODSE_ERR_INVALID_ARG;
  // (the field is read as an integer: a caller may have put any value there, and loading a value that is none of
  // the enumerators through the enumeration type is undefined)
  static_assert(sizeof(modse_dtype) == sizeof(int32_t), "enumeration stored as a 32-bit integer");
  int32_t dtype_bits;
  std::memcpy(&dtype_bits, &desc->dtype, sizeof dtype_bits);
  if (dtype_bits != (int32_t)MODSE_F32 && dtype_bits != (int32_t)MODSE_BF16) return MODSE_ERR_UNSUPPORTED;
  if (desc->n_experts < 1 || desc->d_model < 1) return MODSE_ERR_INVALID_ARG;
  if (desc->top_k < 1 || desc->top_k > desc->n_experts) return MODSE_ERR_INVALID_ARG;
  if (desc->n_experts > MODSE_MAX_EXPERTS) return MODSE_ERR_UNSUPPORTED;
  if (desc->top_k > 2) return MODSE_ERR_UNSUPPORTED;
  if (desc->d_model % 32 != 0) return MODSE_ERR_INVALID_ARG;
  int64_t fmax = 0;
  for (int e = 0; e < desc->n_experts; ++e) {
    const int32_t f = desc->d_ff[e];
    if (f <= 0 || f % 32 != 0) return MODSE_ERR_INVALID_ARG;
    fmax = std::max<int64_t>(fmax, f);
  }
  // kernels index rows and per-expert matrices with 32-bit element offsets
  const int64_t lim = (int64_t)1 << 31;
  if (T * desc->top_k + 64 * desc->n_experts + 64 >= lim / 64) return MODSE_ERR_UNSUPPORTED;
  if ((T + 64) * std::max<int64_t>(fmax, desc->d_model) >= lim) return MODSE_ERR_UNSUPPORTED;
  if (fmax * desc->d_model >= lim) return MODSE_ERR_UNSUPPORTED;
  return MODSE_OK;
}

LayerDims make_dims(const modse_desc* desc, int64_t T) {
  LayerDims L;
  std::memset(&L, 0, sizeof(L));
  L.d = desc->d_model;
  L.N = desc->n_experts;
  L.k = desc->top_k;
  L.T = (int32_t)T;
  for (int e = 0; e < L.N; ++e) {
    L.f[e] = desc->d_ff[e];
    L.foff[e + 1] = L.foff[e] + L.f[e];
    L.order[e] = e;
  }
  std::stable_sort(L.order, L.order + L.N, [&](int a, int b) { return L.f[a] > L.f[b]; });
  return L;
}

// Upper bound of sum_e n_e * d_ff[e]: every token picks top_k distinct experts, so at worst all tokens
// pick the top_k widest ones.
size_t hidden_elems_max(const LayerDims& L) {
  size_t s = 0;
  for (int j = 0; j < L.k; ++j) s += (size_t)L.f[L.order[j]];
  return s * (size_t)L.T;
}

// scratch of the routing kernels (see RouteBufs)
struct RouteScratch {
  size_t blockhist, near_flag, wpad, total;
};
void carve_route(Carver& c, const LayerDims& L, modse_dtype dt, RouteScratch& r) {
  const size_t nb = ((size_t)L.T + MODSE_ROUTE_TOKENS_PER_BLOCK - 1) / MODSE_ROUTE_TOKENS_PER_BLOCK;
  r.blockhist = c.take(nb * (L.N + 1) * 4);
  r.near_flag = c.take((size_t)L.T * 4);
  r.wpad = c.take(route_wpad_bytes(L, esize_of(dt)));
  r.total = c.off;
}
RouteBufs route_bufs(char* base, const RouteScratch& r, void* wt) {
  return RouteBufs{reinterpret_cast<int32_t*>(base + r.blockhist), reinterpret_cast<int32_t*>(base + r.near_flag),
                   base + r.wpad, wt};
}
// W_gate's columns, for the routers that want them: behind the scratch, if there is room
void* wt_behind(char* base, const RouteScratch& r, size_t bytes, const LayerDims& L, modse_dtype dt) {
  return bytes - r.total >= route_wt_bytes(L, esize_of(dt)) ? base + r.total : nullptr;
}

struct FwdLayout {
  RouteScratch route;
  size_t topk_idx, topk_w, counts, offsets, row_of, src_of, near_tie, plan_up, plan_down, Xp, H, O, total;
};

// Float32 partial sums of a product with d columns whose K = f_e is cut into chunks of kchunk (once per operand pair);
// they lie behind the rest of a workspace.
size_t partial_sum_bytes(const LayerDims& L, int kchunk, int passes) {
  if (kchunk == 0) return 0;
  const int fmax = L.f[L.order[0]];
  return align_up((size_t)passes * ((fmax + kchunk - 1) / kchunk) * L.T * L.k * L.d * 4, 256);
}

// with_saved: the call is given the buffer that carries activations to the backward pass; the permuted rows,
// the hidden activations and the expert outputs then live there and take no workspace
FwdLayout fwd_layout(const LayerDims& L, modse_dtype dt, bool with_saved) {
  FwdLayout w;
  Carver c;
  const size_t es = esize_of(dt), Tk = (size_t)L.T * L.k;
  carve_route(c, L, dt, w.route);
  w.topk_idx = c.take(Tk * 4);
  w.topk_w = c.take(Tk * 4);
  w.counts = c.take(L.N * 4);
  w.offsets = c.take((L.N + 1) * 4);
  w.row_of = c.take(Tk * 4);
  w.src_of = c.take(Tk * 4);
  w.near_tie = c.take(4);
  w.plan_up = c.take(sizeof(GemmPlan));
  w.plan_down = c.take(sizeof(GemmPlan));
  w.Xp = c.take(with_saved ? 0 : Tk * L.d * es);
  w.H = c.take(with_saved ? 0 : hidden_elems_max(L) * es);
  w.O = c.take(with_saved ? 0 : Tk * L.d * es);
  w.total = c.off;
  return w;
}

struct SavedLayout {
  size_t dHdA, dHdB, H, O, Xp, total;
};

SavedLayout saved_layout(const LayerDims& L, modse_dtype dt) {
  SavedLayout s;
  Carver c;
  const size_t es = esize_of(dt), h = hidden_elems_max(L) * es;
  s.dHdA = c.take(h);
  s.dHdB = c.take(h);
  s.H = c.take(h);
  s.O = c.take((size_t)L.T * L.k * L.d * es);
  s.Xp = c.take((size_t)L.T * L.k * L.d * es);  // permuted token rows: the weight-gradient GEMMs read them again
  s.total = c.off;
  return s;
}

struct BwdLayout {
  size_t plan[3], dO, dA, dB, dXp, dg, dl, du, dgamma_part, dWg_partial, Wt, total;
};

BwdLayout bwd_layout(const LayerDims& L, modse_dtype dt) {
  BwdLayout w;
  Carver c;
  const size_t es = esize_of(dt), Tk = (size_t)L.T * L.k;
  const size_t h = hidden_elems_max(L) * es;
  const size_t nb = ((size_t)L.T + MODSE_ROUTE_TOKENS_PER_BLOCK - 1) / MODSE_ROUTE_TOKENS_PER_BLOCK;
  for (int i = 0; i < 3; ++i) w.plan[i] = c.take(sizeof(GemmPlan));
  w.dO = c.take(Tk * L.d * es);
  w.dA = c.take(h);
  w.dB = c.take(h);
  w.dXp = c.take(Tk * L.d * es);
  w.dg = c.take(Tk * 4);
  w.dl = c.take((size_t)L.T * L.N * 4);
  w.du = c.take((size_t)L.T * L.N * 4);
  w.dgamma_part = c.take((((size_t)L.T + 63) / 64) * 4);
  w.dWg_partial = c.take((nb + 1) * L.d * L.N * 4);  // (W_gate and W_noise: twice one per 64 tokens)
  w.Wt = c.take((size_t)L.d * L.N * es);
  w.total = c.off;
  return w;
}

// A workspace that serves every batch of at most L.T tokens.  The parts of a layout grow with the batch, but the partial
// sums of a split product do not: batches of a middling size have the most of them, and large ones none.  Sized for one
// batch alone, the workspace of a program's largest one would leave the smaller ones without room for theirs.
template <typename Layout>
size_t workspace_bytes(const LayerDims& L, modse_dtype dt, int epilogue, Layout layout_bytes) {
  size_t bytes = layout_bytes(L);
  modse_gemm::for_each_split(L, dt, epilogue, [&](int64_t tokens, int kchunk) {
    LayerDims M = L;
    M.T = (int32_t)tokens;
    bytes = std::max(bytes, layout_bytes(M) + partial_sum_bytes(M, kchunk, epilogue == EPI_STORE ? 1 : 2));
  });
  return bytes;
}

// Upper bound of the number of tiles of a GEMM whose rows are the experts' token rows (top_k * T in all, at most T of
// one expert) and whose columns are the hidden width (n_is_f) or d.  The row blocks number at most
// floor(rows / bm) + 1 per expert together, and the bound gives as many of them as can be to the widest experts.
int64_t tiles_bound(const LayerDims& L, const TileShape& t, bool n_is_f) {
  int64_t s = 0, full = (int64_t)L.T * L.k / t.bm;
  for (int i = 0; i < L.N; ++i) {
    const int64_t nt = ((n_is_f ? L.f[L.order[i]] : L.d) + t.bn - 1) / t.bn;
    const int64_t mine = std::min<int64_t>(full, (L.T + t.bm - 1) / t.bm - 1);
    full -= mine;
    s += (mine + 1) * nt;
  }
  return s;
}
// the same for a product with d columns whose K = f_e is cut into chunks
int64_t split_tiles_bound(const LayerDims& L, const TileShape& t, int kchunk, int passes) {
  const int64_t nt = (L.d + t.bn - 1) / t.bn;
  int64_t s = 0, full = (int64_t)L.T * L.k / t.bm;
  for (int i = 0; i < L.N; ++i) {
    const int64_t mine = std::min<int64_t>(full, (L.T + t.bm - 1) / t.bm - 1);
    full -= mine;
    s += (mine + 1) * nt * passes * ((L.f[L.order[i]] + kchunk - 1) / kchunk);
  }
  return s;
}
// the launch option that goes with such tiles
int spread(const LayerDims& L, modse_dtype dt, const TileShape& t) { return modse_gemm::spread_k(L, dt, t) ? GEMM_SPREAD_K : 0; }
// problems of a split product: the chunks of all experts
int split_problems(const LayerDims& L, int kchunk, int passes) {
  int n = 0;
  for (int e = 0; e < L.N; ++e) n += passes * ((L.f[e] + kchunk - 1) / kchunk);
  return n;
}
// tiles of the weight-gradient launch (their number does not depend on the routing)
int64_t wgrad_tiles(const LayerDims& L, const TileShape& t) {
  int64_t s = 0;
  for (int e = 0; e < L.N; ++e)
    s += 2 * (int64_t)((L.f[e] + t.bm - 1) / t.bm) * ((L.d + t.bn - 1) / t.bn) +
         (int64_t)((L.d + t.bm - 1) / t.bm) * ((L.f[e] + t.bn - 1) / t.bn);
  return s;
}

// ---------------------------------------------------------------- stage timing
struct StageTimer {
  bool on = false;
  static constexpr int MAXEV = 24;
  hipEvent_t ev[2][MAXEV];
  int stage[2][MAXEV];
  int n[2] = {0, 0};
  bool created = false;
};
StageTimer g_timer;

struct Stamp {
  int which;
  hipStream_t s;
  bool on;
  Stamp(int w, hipStream_t st) : which(w), s(st), on(g_timer.on) {
    if (on) {
      g_timer.n[which] = 0;
      mark(-1);
    }
  }
  void mark(int stage) {
    if (!on) return;
    int& n = g_timer.n[which];
    if (n >= StageTimer::MAXEV) return;
    g_timer.stage[which][n] = stage;
    (void)hipEventRecord(g_timer.ev[which][n], s);
    ++n;
  }
};

#define HIP_TRY(expr)                            \
  do {                                           \
    if ((expr) != hipSuccess) return MODSE_ERR_HIP; \
  } while (0)

RoutingPtrs routing_from(const modse_routing* r, char* ws, const FwdLayout& w) {
  RoutingPtrs R;
  if (r) {
    R = {r->topk_idx, r->topk_w, r->counts, r->offsets, r->row_of, r->src_of, r->near_tie_count};
  } else {
    R = {reinterpret_cast<int32_t*>(ws + w.topk_idx), reinterpret_cast<float*>(ws + w.topk_w),
         reinterpret_cast<int32_t*>(ws + w.counts),   reinterpret_cast<int32_t*>(ws + w.offsets),
         reinterpret_cast<int32_t*>(ws + w.row_of),   reinterpret_cast<int32_t*>(ws + w.src_of),
         reinterpret_cast<int32_t*>(ws + w.near_tie)};
  }
  return R;
}

bool routing_complete(const modse_routing* r) {
  return r && r->topk_idx && r->topk_w && r->counts && r->offsets && r->row_of && r->src_of && r->near_tie_count;
}

// A gate extension is usable when every pointer its switched-on parts need is there.
bool ext_complete(const modse_gate_ext* e) {
  if (!e) return true;
  if (e->W_noise && (!e->gamma || !e->noise_pre || !(e->eps >= 0.f))) return false;
  if (e->probs && (!e->aux_f || !e->aux_P || !e->aux_loss)) return false;
  return true;
}

GateExtPtrs ext_ptrs(const modse_gate_ext* e) {
  return GateExtPtrs{e->W_noise, e->gamma, e->eps, e->noise_pre, e->aux_alpha, e->probs, e->aux_f, e->aux_P, e->aux_loss};
}

}  // namespace

extern "C" {

const char* modse_status_string(modse_status s) {
  int32_t code;  // (read as an integer: a C caller may pass any value)
  static_assert(sizeof(modse_status) == sizeof(int32_t), "enumeration stored as a 32-bit integer");
  std::memcpy(&code, &s, sizeof code);
  switch (code) {
    case MODSE_OK: return "ok";
    case MODSE_ERR_INVALID_ARG: return "invalid argument";
    case MODSE_ERR_UNSUPPORTED: return "unsupported configuration";
    case MODSE_ERR_WORKSPACE: return "workspace too small";
    case MODSE_ERR_HIP: return "HIP launch failed";
  }
  return "unknown status";
}

modse_status modse_workspace_size(const modse_desc* desc, int64_t T, int need_bwd, size_t* bytes) {
  if (!bytes) return MODSE_ERR_INVALID_ARG;
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  const LayerDims L = make_dims(desc, T);
  if (need_bwd != MODSE_WS_FWD && need_bwd != MODSE_WS_BWD && need_bwd != MODSE_WS_FWD_SAVED) return MODSE_ERR_INVALID_ARG;
  const modse_dtype dt = desc->dtype;
  if (need_bwd == MODSE_WS_BWD)
    *bytes = workspace_bytes(L, dt, EPI_STORE_DUALK, [&](const LayerDims& M) { return bwd_layout(M, dt).total; });
  else
    *bytes = workspace_bytes(L, dt, EPI_STORE,
                             [&](const LayerDims& M) { return fwd_layout(M, dt, need_bwd == MODSE_WS_FWD_SAVED).total; });
  return MODSE_OK;
}

modse_status modse_saved_size(const modse_desc* desc, int64_t T, size_t* bytes) {
  if (!bytes) return MODSE_ERR_INVALID_ARG;
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  *bytes = saved_layout(make_dims(desc, T), desc->dtype).total;
  return MODSE_OK;
}

modse_status modse_route(const modse_desc* desc, int64_t T, const void* x, const void* W_gate,
                         const float* logit_bias, const modse_routing* out, void* ws, size_t ws_bytes,
                         void* hip_stream) {
  return modse_route_ext(desc, T, x, W_gate, logit_bias, nullptr, out, ws, ws_bytes, hip_stream);
}

modse_status modse_route_ext(const modse_desc* desc, int64_t T, const void* x, const void* W_gate,
                             const float* logit_bias, const modse_gate_ext* ext, const modse_routing* out, void* ws,
                             size_t ws_bytes, void* hip_stream) {
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  if (T == 0) return MODSE_OK;
  if (!x || !W_gate || !ws || !routing_complete(out) || !ext_complete(ext)) return MODSE_ERR_INVALID_ARG;
  GateExtPtrs G;
  if (ext) G = ext_ptrs(ext);
  const LayerDims L = make_dims(desc, T);
  RouteScratch w;  // the routing scratch is the head of the forward workspace; this call needs no more of it
  Carver c;
  carve_route(c, L, desc->dtype, w);
  if (ws_bytes < w.total) return MODSE_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const RoutingPtrs R = {out->topk_idx, out->topk_w, out->counts, out->offsets, out->row_of, out->src_of, out->near_tie_count};
  HIP_TRY(launch_route(L, desc->dtype, x, W_gate, logit_bias, R,
                       route_bufs(static_cast<char*>(ws), w, wt_behind(static_cast<char*>(ws), w, ws_bytes, L, desc->dtype)), nullptr,
                       ext ? &G : nullptr, s));
  return MODSE_OK;
}

// ---------------------------------------------------------------- modse_route without a workspace
// For callers that cannot hand over a workspace they allocated (HIP graph capture, serving loops that must
// not allocate): the router's scratch -- per-block histograms and near-tie flags -- lives in a device array
// of this library.  Every GPU holds its own copy at its own address; the name below is only the host-side
// handle of the symbol, the address comes from hipGetSymbolAddress, once per device.
// Behind the scratch: W_gate's columns.
static __device__ __align__(256) unsigned char g_route_scratch[MODSE_ROUTE_STATIC_SCRATCH_BYTES + ROUTE_WT_MAX];

namespace {
constexpr int kMaxDevices = 64;
void* g_route_scratch_ptr[kMaxDevices] = {};

}  // namespace

modse_status modse_route_static(const modse_desc* desc, int64_t T, const void* x, const void* W_gate,
                                const float* logit_bias, const modse_routing* out, void* hip_stream) {
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  if (T == 0) return MODSE_OK;
  if (!x || !W_gate || !routing_complete(out)) return MODSE_ERR_INVALID_ARG;
  const LayerDims L = make_dims(desc, T);
  RouteScratch w;
  Carver c;
  carve_route(c, L, desc->dtype, w);
  if (w.total > MODSE_ROUTE_STATIC_SCRATCH_BYTES) return MODSE_ERR_WORKSPACE;  // more tokens than the array serves
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MODSE_ERR_HIP;
  if (!g_route_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_route_scratch)) != hipSuccess || !p) return MODSE_ERR_HIP;
    g_route_scratch_ptr[dev] = p;
  }
  char* scratch = static_cast<char*>(g_route_scratch_ptr[dev]);
  const RoutingPtrs R = {out->topk_idx, out->topk_w, out->counts, out->offsets, out->row_of, out->src_of, out->near_tie_count};
  // every word of the scratch that a kernel reads has been written by an earlier kernel of this call
  HIP_TRY(launch_route(L, desc->dtype, x, W_gate, logit_bias, R,
                       route_bufs(scratch, w, scratch + MODSE_ROUTE_STATIC_SCRATCH_BYTES), nullptr, nullptr,
                       static_cast<hipStream_t>(hip_stream)));
  return MODSE_OK;
}

modse_status modse_routing_stats(const modse_desc* desc, int64_t T, const modse_routing* routing,
                                 int32_t* slot_counts, float* summary, void* hip_stream) {
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  if (!routing || !routing->topk_idx || !slot_counts || !summary) return MODSE_ERR_INVALID_ARG;
  const LayerDims L = make_dims(desc, T);
  HIP_TRY(launch_routing_stats(L, routing->topk_idx, slot_counts, summary, static_cast<hipStream_t>(hip_stream)));
  return MODSE_OK;
}

modse_status modse_layer_fwd(const modse_desc* desc, int64_t T, const void* x, const void* W_gate,
                             const float* logit_bias, const void* W1, const void* W3, const void* W2, void* y,
                             const modse_routing* routing_out, void* saved, void* ws, size_t ws_bytes,
                             void* hip_stream) {
  return modse_layer_fwd_ext(desc, T, x, W_gate, logit_bias, nullptr, W1, W3, W2, y, routing_out, saved, ws, ws_bytes,
                             hip_stream);
}

modse_status modse_layer_fwd_ext(const modse_desc* desc, int64_t T, const void* x, const void* W_gate,
                                 const float* logit_bias, const modse_gate_ext* ext, const void* W1, const void* W3,
                                 const void* W2, void* y, const modse_routing* routing_out, void* saved, void* ws,
                                 size_t ws_bytes, void* hip_stream) {
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  if (T == 0) return MODSE_OK;
  if (!x || !W_gate || !W1 || !W3 || !W2 || !y || !ws || !ext_complete(ext)) return MODSE_ERR_INVALID_ARG;
  GateExtPtrs G;
  if (ext) G = ext_ptrs(ext);
  if (routing_out && !routing_complete(routing_out)) return MODSE_ERR_INVALID_ARG;
  const modse_dtype dt = desc->dtype;
  const LayerDims L = make_dims(desc, T);
  const FwdLayout w = fwd_layout(L, dt, saved != nullptr);
  if (ws_bytes < w.total) return MODSE_ERR_WORKSPACE;
  GemmChoice down = gemm_choice(L, dt, EPI_STORE);
  if (ws_bytes - w.total < partial_sum_bytes(L, down.kchunk, 1)) down.kchunk = 0;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  char* wsb = static_cast<char*>(ws);
  const RoutingPtrs R = routing_from(routing_out, wsb, w);
  // (W_gate's N columns lie where the experts' outputs will: those are T k rows of d, more than N where a router wants
  // the columns, and written long after the routing)
  void* const wt = saved ? static_cast<char*>(saved) + saved_layout(L, dt).O : wsb + w.O;
  const RouteBufs RB = route_bufs(wsb, w.route, wt);
  Stamp stamp(0, s);

  // with a backward pass to follow, the permuted rows go straight into the saved buffer
  void* Xp = saved ? static_cast<char*>(saved) + saved_layout(L, dt).Xp : wsb + w.Xp;
  HIP_TRY(launch_router(L, dt, x, W_gate, logit_bias, R, RB, ext ? &G : nullptr, s));
  stamp.mark(MODSE_STAGE_ROUTE);

  FwdPlanArgs pa;
  std::memset(&pa, 0, sizeof(pa));
  pa.Xp = Xp; pa.W1 = W1; pa.W3 = W3; pa.W2 = W2;
  if (saved) {
    const SavedLayout sl = saved_layout(L, dt);
    char* sb = static_cast<char*>(saved);
    pa.dHdA = sb + sl.dHdA; pa.dHdB = sb + sl.dHdB; pa.H = sb + sl.H; pa.O = sb + sl.O;
  } else {
    pa.H = wsb + w.H; pa.O = wsb + w.O;
  }
  pa.up = reinterpret_cast<GemmPlan*>(wsb + w.plan_up);
  pa.down = reinterpret_cast<GemmPlan*>(wsb + w.plan_down);
  pa.up_tile = gemm_choice(L, dt, EPI_SWIGLU).tile;
  pa.down_tile = down.tile;
  const int kchunk = down.kchunk;
  pa.kchunk = kchunk;
  pa.Opart = reinterpret_cast<float*>(wsb + w.total);
  // histogram, scan (which also writes the tile plans), stable scatter: one launch for all of it up to 4096 tokens
  HIP_TRY(launch_permute(L, dt, x, R, RB, Xp, ext ? &G : nullptr, &pa, s));
  stamp.mark(MODSE_STAGE_PERMUTE);

  HIP_TRY(launch_grouped_gemm(dt, EPI_SWIGLU, pa.up_tile, pa.up, L.N, 0, (saved ? GEMM_SAVE_TERMS : 0) | spread(L, dt, pa.up_tile),
                              tiles_bound(L, pa.up_tile, true), s));
  stamp.mark(MODSE_STAGE_UP);
  if (kchunk) {
    const int64_t bound = split_tiles_bound(L, pa.down_tile, kchunk, 1);
    HIP_TRY(launch_grouped_gemm(dt, EPI_STORE_F32, pa.down_tile, pa.down, split_problems(L, kchunk, 1), 0,
                                spread(L, dt, pa.down_tile), bound, s, LAYOUT_TN));
    stamp.mark(MODSE_STAGE_DOWN);
    HIP_TRY(launch_combine_split(L, dt, pa.Opart, kchunk, R, saved ? pa.O : nullptr, y, s));
    stamp.mark(MODSE_STAGE_COMBINE);
    return MODSE_OK;
  }
  HIP_TRY(launch_grouped_gemm(dt, EPI_STORE, pa.down_tile, pa.down, L.N, 0, spread(L, dt, pa.down_tile),
                              tiles_bound(L, pa.down_tile, false), s));
  stamp.mark(MODSE_STAGE_DOWN);
  HIP_TRY(launch_combine(L, dt, pa.O, R, y, s));
  stamp.mark(MODSE_STAGE_COMBINE);
  return MODSE_OK;
}

modse_status modse_layer_bwd(const modse_desc* desc, int64_t T, const void* x, const void* W_gate, const void* W1,
                             const void* W3, const void* W2, const modse_routing* routing, const void* saved,
                             const void* dY, void* dX, float* dW_gate, float* dW1, float* dW3, float* dW2,
                             int accumulate, void* ws, size_t ws_bytes, void* hip_stream) {
  return modse_layer_bwd_ext(desc, T, x, W_gate, nullptr, 0.f, W1, W3, W2, routing, saved, dY, dX, dW_gate, nullptr,
                             nullptr, dW1, dW3, dW2, accumulate, ws, ws_bytes, hip_stream);
}

modse_status modse_layer_bwd_ext(const modse_desc* desc, int64_t T, const void* x, const void* W_gate,
                                 const modse_gate_ext* ext, float aux_grad, const void* W1, const void* W3,
                                 const void* W2, const modse_routing* routing, const void* saved, const void* dY,
                                 void* dX, float* dW_gate, float* dW_noise, float* dgamma, float* dW1, float* dW3,
                                 float* dW2, int accumulate, void* ws, size_t ws_bytes, void* hip_stream) {
  const modse_status st = check_desc(desc, T);
  if (st != MODSE_OK) return st;
  if (T == 0) return MODSE_OK;
  if (!x || !W_gate || !W1 || !W3 || !W2 || !saved || !dY || !dX || !dW_gate || !dW1 || !dW3 || !dW2 || !ws)
    return MODSE_ERR_INVALID_ARG;
  if (!ext_complete(ext) || (ext && ext->W_noise && (!dW_noise || !dgamma))) return MODSE_ERR_INVALID_ARG;
  GateExtPtrs G;
  if (ext) G = ext_ptrs(ext);
  if (!routing_complete(routing)) return MODSE_ERR_INVALID_ARG;
  const modse_dtype dt = desc->dtype;
  const LayerDims L = make_dims(desc, T);
  const BwdLayout w = bwd_layout(L, dt);
  if (ws_bytes < w.total) return MODSE_ERR_WORKSPACE;
  GemmChoice dx = gemm_choice(L, dt, EPI_STORE_DUALK);
  if (ws_bytes - w.total < partial_sum_bytes(L, dx.kchunk, 2)) dx.kchunk = 0;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  char* wsb = static_cast<char*>(ws);
  const SavedLayout sl = saved_layout(L, dt);
  const char* sb = static_cast<const char*>(saved);
  const RoutingPtrs R = {routing->topk_idx, routing->topk_w, routing->counts, routing->offsets,
                         routing->row_of,   routing->src_of, routing->near_tie_count};
  Stamp stamp(1, s);

  const void* Xp = sb + sl.Xp;
  void* dO = wsb + w.dO;
  float* dg = reinterpret_cast<float*>(wsb + w.dg);
  BwdPlanArgs pa;
  std::memset(&pa, 0, sizeof(pa));
  pa.Xp = Xp; pa.dO = dO; pa.H = sb + sl.H; pa.dHdA = sb + sl.dHdA; pa.dHdB = sb + sl.dHdB;
  pa.W1 = W1; pa.W3 = W3; pa.W2 = W2;
  pa.dA = wsb + w.dA; pa.dB = wsb + w.dB; pa.dXp = wsb + w.dXp;
  pa.dW1 = dW1; pa.dW3 = dW3; pa.dW2 = dW2;
  pa.dXpart = reinterpret_cast<float*>(wsb + w.total);
  pa.dx_kchunk = dx.kchunk;
  pa.dh = reinterpret_cast<GemmPlan*>(wsb + w.plan[0]);
  pa.dx = reinterpret_cast<GemmPlan*>(wsb + w.plan[1]);
  pa.wg = reinterpret_cast<GemmPlan*>(wsb + w.plan[2]);
  pa.dh_tile = gemm_choice(L, dt, EPI_SWIGLU_BWD).tile;
  pa.dx_tile = dx.tile;
  pa.wg_tile = gemm_choice(L, dt, EPI_STORE_F32).tile;
  const BwdRouterBufs rb = {reinterpret_cast<float*>(wsb + w.dl), reinterpret_cast<float*>(wsb + w.du),
                            reinterpret_cast<float*>(wsb + w.dgamma_part),
                            reinterpret_cast<float*>(wsb + w.dWg_partial), wsb + w.Wt};
  HIP_TRY(launch_bwd_prep(L, dt, dY, sb + sl.O, R, dO, dg, pa, ext ? &G : nullptr, aux_grad, W_gate, rb, s));
  stamp.mark(MODSE_STAGE_BWD_PREP);

  HIP_TRY(launch_grouped_gemm(dt, EPI_SWIGLU_BWD, pa.dh_tile, pa.dh, L.N, 0, spread(L, dt, pa.dh_tile),
                              tiles_bound(L, pa.dh_tile, true), s));
  // Gradients of more than half the memory-side cache (256 MB) would be gone from it before anybody reads them, and with
  // them what the launches around this one leave for each other (partial sums of dX, activations, weights): they are stored
  // with the non-temporal hint, and old ones that are added to are read with it.  1.1 GB of gradients: this launch takes as
  // long, but the router's backward pass behind it 26 us in place of 40, a training pass of 1021 tokens 856 in place of 888, and
  // reading with the hint takes a step of two such passes from 1882 to 1849.  Smaller gradients are still in the cache when the
  // next micro-batch adds to them; the hint changes nothing there (two passes with 48 MB 595 us with it, 597 without).
  const bool stream = 3 * (size_t)L.foff[L.N] * L.d * sizeof(float) > ((size_t)128 << 20);
  const int n_dx = pa.dx_kchunk ? split_problems(L, pa.dx_kchunk, 2) : L.N, wg_option = stream ? GEMM_STREAM_C : 0;
  const int64_t dx_tiles =
      pa.dx_kchunk ? split_tiles_bound(L, pa.dx_tile, pa.dx_kchunk, 2) : tiles_bound(L, pa.dx_tile, false);
  const int64_t wg_tiles = wgrad_tiles(L, pa.wg_tile);
  const int dx_option = spread(L, dt, pa.dx_tile);
  const bool wg_beside = wgrad_beside_dx(dt, pa.dx_tile, pa.wg_tile);
  // (of a plain gate: the gradient of the logits is there)
  const bool dwg_done = dwg_beside_dx(dt, pa.dx_tile, pa.wg_tile) && bwd_gate_is_plain(L, ext ? &G : nullptr, aux_grad);
  if (dwg_beside_dx(dt, pa.dx_tile, pa.wg_tile)) {
    const DwgArgs dwg = dwg_args(L, x, rb, 1);
    HIP_TRY(launch_dx(dt, pa.dx_tile, pa.dx_kchunk != 0, pa.dx, n_dx, dx_tiles, dx_option, wg_beside ? pa.wg : nullptr, 3 * L.N, wg_tiles,
                      accumulate, wg_option, dwg_done ? &dwg : nullptr, s));
  } else if (pa.dx_kchunk) {
    HIP_TRY(launch_grouped_gemm(dt, EPI_STORE_F32, pa.dx_tile, pa.dx, n_dx, 0, dx_option, dx_tiles, s, LAYOUT_B_KN));
  } else {
    HIP_TRY(launch_grouped_gemm(dt, EPI_STORE_DUALK, pa.dx_tile, pa.dx, n_dx, 0, dx_option, dx_tiles, s));
  }
  stamp.mark(MODSE_STAGE_BWD_DGRAD);  // (and the weight gradients, where they are in that launch)
  if (!wg_beside) {
    HIP_TRY(launch_grouped_gemm(dt, EPI_STORE_F32, pa.wg_tile, pa.wg, 3 * L.N, accumulate, wg_option, wg_tiles, s));
    stamp.mark(MODSE_STAGE_BWD_WGRAD);
  }

  const DxRows rows = {pa.dXp, pa.dXpart, pa.dx_kchunk};
  HIP_TRY(launch_bwd_router(L, dt, x, W_gate, rows, dg, R, ext ? &G : nullptr, aux_grad, rb, dX, dW_gate, dW_noise,
                            dgamma, accumulate, dwg_done, s));
  stamp.mark(MODSE_STAGE_BWD_ROUTER);
  return MODSE_OK;
}

modse_status modse_stage_timing_enable(int on) {
  if (on && !g_timer.created) {
    for (int w = 0; w < 2; ++w)
      for (int i = 0; i < StageTimer::MAXEV; ++i)
        if (hipEventCreate(&g_timer.ev[w][i]) != hipSuccess) return MODSE_ERR_HIP;
    g_timer.created = true;
  }
  g_timer.on = on != 0;
  g_timer.n[0] = g_timer.n[1] = 0;
  return MODSE_OK;
}

modse_status modse_stage_times(float* ms) {
  if (!ms) return MODSE_ERR_INVALID_ARG;
  for (int i = 0; i < MODSE_N_STAGES; ++i) ms[i] = 0.f;
  if (!g_timer.created) return MODSE_OK;
  for (int w = 0; w < 2; ++w) {
    const int n = g_timer.n[w];
    if (n < 2) continue;
    if (hipEventSynchronize(g_timer.ev[w][n - 1]) != hipSuccess) return MODSE_ERR_HIP;
    for (int i = 1; i < n; ++i) {
      float t = 0.f;
      if (hipEventElapsedTime(&t, g_timer.ev[w][i - 1], g_timer.ev[w][i]) != hipSuccess) return MODSE_ERR_HIP;
      const int st = g_timer.stage[w][i];
      if (st >= 0 && st < MODSE_N_STAGES) ms[st] += t;
    }
  }
  return MODSE_OK;
}

}  // extern "C"
