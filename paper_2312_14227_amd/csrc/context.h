// Shared state of the step executor: the context behind the C ABI, the workspace planner, the
// timed regions of the profiler (Section 5) and the GEMM launch helpers used by the per-model
// forward / backward chains.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "et.h"
#include "kernels.h"

using et::bf16;

namespace et_exec {

constexpr uint32_t SEG_ELEMS = 16384;  // elements per chunk of the importance / update tables

enum Phase { PH_FWD = 0, PH_DW = 1, PH_DY = 2, PH_UPD = 3 };

struct Share {  // part of a timed region's time that belongs to a piece (phase, tensor) of the time model
  int phase, tensor;
  double weight;
};

struct TensorInfo {
  std::string name;
  size_t numel;
  int32_t dtype;
};

struct Scope {  // one timed region of the profile; its time is divided among the shares in proportion to their weights
  std::vector<Share> shares;
  hipEvent_t e0, e1;
};

struct KernelRecord {  // one timed kernel launch (measurement support)
  int cls;
  double work;
  hipEvent_t e0, e1;
};

struct VitBlockBufs {
  float *h_in, *h_mid, *mean1, *rstd1, *mean2, *rstd2, *lse;
  bf16 *a1, *qkv, *p, *o, *a2, *u, *ga;
  bf16* o_rest = nullptr;   // what rounding o to bf16 left out (long sequences only)
};

// activations kept by one convolution + affine (+ReLU) unit of the ResNet
struct ConvUnit {
  int t;                      // tensor index of the convolution weight (gain t+1, shift t+2)
  int H, W, Cin, Ho, Wo, Cout, k, stride, Kc;   // Kc: padded column count of the im2col matrix
  const bf16* in;             // input activation [B,H,W,Cin]
  bf16* cols;                 // im2col matrix [B*Ho*Wo][Kc] (null: the input itself is the matrix)
  bf16* z;                    // convolution output [B*Ho*Wo][Cout]
  bf16* y;                    // after affine (+ReLU); for the last unit of a block: the block output
  bf16* wflip;                // mirrored weight [Cin][3][3][Cout] of a unit whose dy() is an implicit convolution
};
struct ResBlockBufs {
  int t;
  bool proj;
  ConvUnit c1, c2, c3, sc;
  const bf16* x;              // block input
  bf16* y;                    // block output (after the closing ReLU)
};

// activations kept by one inverted-residual block (MobileNetV2 family)
struct MbBlockBufs {
  int t, t_dw;                 // tensor index of the block's first weight and of its depthwise weight
  int Cin, hid, Cout, stride, H, W, Ho, Wo;
  bool expand, shortcut;
  const bf16* x;               // block input [B,H,W,Cin]
  bf16 *z_exp, *y_exp;         // expansion: convolution output, after affine + ReLU6   [B,H,W,hid]
  bf16 *z_dw, *y_dw;           // depthwise: the same                                   [B,Ho,Wo,hid]
  bf16 *z_proj, *y;            // projection output and the block output                [B,Ho,Wo,Cout]
};

}  // namespace et_exec
using namespace et_exec;

struct et_ctx {
  et_model_desc desc;
  hipStream_t stream = nullptr;
  std::vector<TensorInfo> tensors;
  int32_t state_slots = 0;
  bool bf16_model = false;

  // workspace plan (offsets in bytes)
  size_t ws_bytes = 0;
  // At its end lie two parts that work with less room than they can use (see place_tail): the scratch of split reductions, of which the largest single
  // product has to find its part, and the gradients that are kept
  size_t ws_min = 0, tail_at = 0, group_most = 0, keep_most = 0;
  std::vector<std::pair<void**, size_t>> plan;  // (where to store the pointer, offset)

  // bound buffers
  bool bound = false;
  std::vector<void*> w;
  std::vector<float*> grad;
  std::vector<float*> state;
  unsigned char* ws = nullptr;

  // MLP buffers
  std::vector<float*> act;  // act[i]: input of layer i (act[0] is x itself, not in the workspace)
  float *logits = nullptr, *dlogits = nullptr, *loss = nullptr, *dbuf[2] = {nullptr, nullptr};

  // ViT buffers
  std::vector<VitBlockBufs> blk;
  float *e = nullptr, *h_out = nullptr, *s_f32 = nullptr, *meanf = nullptr, *rstdf = nullptr, *dh = nullptr;
  bf16 *zc = nullptr, *dl16 = nullptr, *dz = nullptr, *dh16 = nullptr, *da = nullptr, *du = nullptr, *dattn = nullptr,
       *dqkv = nullptr, *ds = nullptr, *de = nullptr;
  float* gemm_partials = nullptr;
  size_t gemm_partial_elems = 0;   // what one product may take (fixed by the shapes, so that a split is)

  // column sums of the backward pass that wait for their second step: partial rows in sum_arena (bump allocated), finished
  // together by one launch at the end of the pass, or earlier when the arena is full
  float* sum_arena = nullptr;
  size_t sum_arena_elems = 0, sum_used = 0;
  std::vector<et::SumJob> sum_jobs;
  std::vector<int> sum_tensors;
  // weight gradients that run together at the end of a backward pass, and the arena (bump allocated) for the gradients they read: what
  // each layer's gradient is stored in if its weight is selected, instead of the scratch buffer that the next layer overwrites
  bf16* keep_arena = nullptr;
  size_t keep_elems = 0, keep_used = 0, group_elems = 0;   // group_elems: what the products of a group may take of gemm_partials
  std::vector<et::DwJob> dw_jobs;
  std::vector<int> dw_tensors;
  std::vector<et::DwGroupPlan> dw_plans;   // one per group (a group ends where the scratch of split reductions does)
  // transformer: share of a launch's time that the column sums riding on it take, measured by et_profile ([the last block's few rows][kernel])
  double sum_cost[2][3] = {};

  // ResNet buffers
  ConvUnit stem;
  std::vector<ResBlockBufs> rblk;
  bf16 *stem_w8 = nullptr, *pool_y = nullptr, *pooled = nullptr, *rd[3] = {nullptr, nullptr, nullptr}, *rdsum = nullptr,
       *rdsc = nullptr, *rdcols = nullptr;
  uint8_t* pool_arg = nullptr;
  float *stem_dw8 = nullptr, *stem_z32 = nullptr;
  bf16* stem_xpad = nullptr;   // ResNet stem as a gathered GEMM: the image padded to 4 channels and by the window
  int stem_hp = 0, stem_wp = 0;

  // plain convolution stack (VGG family): one unit per convolution (y: after bias + ReLU),
  // per stage the pooled output and the chosen taps, the inputs of the linear layers
  std::vector<ConvUnit> vconv;
  std::vector<int> vstage;
  std::vector<bf16*> vpool;
  std::vector<uint8_t*> varg;
  std::vector<bf16*> vact;
  std::vector<int> vdims;           // vdims[j] -> vdims[j+1]: linear layer j
  float* fc_z32 = nullptr;          // reduced sum of a linear layer's split forward product

  // inverted-residual network: blocks; the stem and the last convolution are ConvUnits (`stem`, `mlast`)
  std::vector<MbBlockBufs> mblk;
  ConvUnit mlast;

  // tables for importance / update
  std::vector<uint32_t> seg_begin;  // [N+1]
  uint32_t n_segs = 0;
  et::TensorSeg* imp_segs_dev = nullptr;
  et::UpdateSeg* upd_segs_dev = nullptr;
  uint32_t* seg_begin_dev = nullptr;
  uint32_t* upd_selected_dev = nullptr;   // indices of the chunks of the tensors selected by upd_mask
  std::vector<uint32_t> upd_selected;
  std::vector<uint8_t> upd_mask;          // the mask upd_selected_dev was built for
  double *imp_partial_dev = nullptr, *imp_out_dev = nullptr;
  std::vector<et::UpdateSeg> upd_segs_host;
  std::vector<et::TensorSeg> imp_segs_host;

  // launch accounting and profiling
  int32_t launches[4] = {0, 0, 0, 0};
  int cur_phase = PH_FWD;
  bool profiling = false;
  std::vector<Scope> scopes;
  std::vector<hipEvent_t> event_pool;
  size_t events_used = 0;
  hipError_t hip_err = hipSuccess;

  // per-kernel-class timing
  bool ktiming = false;
  std::vector<KernelRecord> kcal;   // event pairs with nothing between them, recorded when timing is enabled
  std::vector<KernelRecord> krecs;
  std::vector<hipEvent_t> kevent_pool;
  size_t kevents_used = 0;
};

namespace et_exec {

#define ET_HIP(expr)                       \
  do {                                     \
    hipError_t e__ = (expr);               \
    if (e__ != hipSuccess) {               \
      c->hip_err = e__;                    \
      return ET_EHIP;                      \
    }                                      \
  } while (0)

// kernel launch through a wrapper that returns hipError_t; counts the launches
#define ET_K(n, expr)                      \
  do {                                     \
    hipError_t e__ = (expr);               \
    if (e__ != hipSuccess) {               \
      c->hip_err = e__;                    \
      return ET_EHIP;                      \
    }                                      \
    c->launches[c->cur_phase] += (n);      \
  } while (0)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int round8(int v) { return (v + 7) & ~7; }

template <typename T>
inline void reserve(et_ctx* c, T** where, size_t bytes) {
  c->plan.emplace_back(reinterpret_cast<void**>(where), c->ws_bytes);
  c->ws_bytes += align_up(bytes, 256);
}

inline hipError_t get_event(et_ctx* c, hipEvent_t* ev) {
  if (c->events_used == c->event_pool.size()) {
    hipEvent_t e;
    hipError_t r = hipEventCreate(&e);
    if (r != hipSuccess) return r;
    c->event_pool.push_back(e);
  }
  *ev = c->event_pool[c->events_used++];
  return hipSuccess;
}

// timed region: events are recorded only while profiling
struct Region {
  et_ctx* c;
  bool on;
  size_t idx = 0;
  Region(et_ctx* ctx, int phase, int tensor) : c(ctx), on(ctx->profiling) {
    const Share one = {phase, tensor, 1.0};
    begin(phase, &one, 1);
  }
  // `phase`: what the launches are counted as
  Region(et_ctx* ctx, int phase, const Share* shares, size_t n) : c(ctx), on(ctx->profiling) { begin(phase, shares, n); }
  void begin(int phase, const Share* shares, size_t n) {
    c->cur_phase = phase;
    if (!on) return;
    Scope s;
    s.shares.assign(shares, shares + n);
    if (get_event(c, &s.e0) != hipSuccess || get_event(c, &s.e1) != hipSuccess) {
      on = false;
      c->hip_err = hipErrorOutOfMemory;
      return;
    }
    (void)hipEventRecord(s.e0, c->stream);
    idx = c->scopes.size();
    c->scopes.push_back(s);
  }
  ~Region() {
    if (on) (void)hipEventRecord(c->scopes[idx].e1, c->stream);
  }
};

// ---- column sums (see et_ctx::sum_arena)
// workspace for the partial sums of a backward pass: `total` floats hold every sum at once, `largest` the largest group that is
// allocated together; beyond 64 MB the pass finishes what it has and starts over
inline void reserve_sums(et_ctx* c, size_t total, size_t largest) {
  c->sum_arena_elems = std::max(std::max(largest, (size_t)64), std::min(total, (size_t)16 << 20));
  reserve(c, &c->sum_arena, sizeof(float) * c->sum_arena_elems);
}
inline size_t sum_elems(size_t rows, size_t cols) { return (rows * cols + 63) / 64 * 64; }

inline int sums_finish(et_ctx* c) {
  if (c->sum_jobs.empty()) return ET_OK;
  std::vector<Share> shares;
  if (c->profiling)
    for (size_t i = 0; i < c->sum_jobs.size(); i++) shares.push_back({PH_DW, c->sum_tensors[i], (double)c->sum_jobs[i].rows * c->sum_jobs[i].cols});
  Region r(c, PH_DW, shares.data(), shares.size());
  int n = 0;
  const hipError_t e = et::sum_finish(c->sum_jobs.data(), (int)c->sum_jobs.size(), c->stream, &n);
  c->launches[PH_DW] += n;
  c->sum_jobs.clear();
  c->sum_tensors.clear();
  c->sum_used = 0;
  if (e != hipSuccess) { c->hip_err = e; return ET_EHIP; }
  return ET_OK;
}
// makes room for a group of sums that one kernel produces
inline int sums_room(et_ctx* c, size_t elems) { return c->sum_used + elems > c->sum_arena_elems ? sums_finish(c) : ET_OK; }
// partial rows of one sum, to be finished into the gradient of `tensor`
inline float* sum_job(et_ctx* c, int tensor, int rows, int cols) {
  float* p = c->sum_arena + c->sum_used;
  c->sum_used += sum_elems(rows, cols);
  c->sum_jobs.push_back({p, c->grad[tensor], rows, cols, 0});
  c->sum_tensors.push_back(tensor);
  return p;
}
// gradient of `tensor` = column sum of a [rows][cols] matrix (times the normalised h)
inline int colsum_dw(et_ctx* c, int tensor, const bf16* d, const float* d32, long long d_stride, int rows, int cols, const float* h = nullptr,
                     long long h_stride = 0, const float* mean = nullptr, const float* rstd = nullptr, long long stat_stride = 1) {
  const int parts = et::colsum_parts(rows, cols);
  const int rc = sums_room(c, sum_elems(parts, cols));
  if (rc != ET_OK) return rc;
  Region r(c, PH_DW, tensor);
  float* part = sum_job(c, tensor, parts, cols);
  ET_K(1, et::colsum_part(d, d32, d_stride, h, h_stride, mean, rstd, stat_stride, part, rows, cols, c->stream));
  return ET_OK;
}

// split of the reduction dimension for a weight gradient [Mo][No] reduced over K rows
inline int split_for(int Mo, int No, int K) {
  int tile, split;
  et::gemm_bf16_plan_split(Mo, No, K, &tile, &split);
  return split;
}

// Y[M][N] = X[M][K] W[N][K]^T (+ bias) ...
inline et::GemmDesc linear_fwd(const bf16* X, const bf16* W, const bf16* bias, int M, int N, int K) {
  et::GemmDesc g;
  g.A = X; g.lda = K; g.B = W; g.ldb = K; g.M = M; g.N = N; g.K = K; g.bias = bias; g.ldc = N;
  return g;
}
// dX[M][K] = dY[M][N] W[N][K]
inline et::GemmDesc linear_dx(const bf16* dY, const bf16* W, int M, int N, int K) {
  et::GemmDesc g;
  g.A = dY; g.lda = N; g.B = W; g.b_t = true; g.ldb = K; g.M = M; g.N = K; g.K = N; g.ldc = K;
  return g;
}
// dW[N][K] = dY[M][N]^T X[M][K], fp32, split over the rows
inline et::GemmDesc linear_dw(et_ctx* c, const bf16* dY, int ldy, const bf16* X, int ldx, float* dW, int M, int N, int K) {
  et::GemmDesc g;
  g.A = dY; g.a_t = true; g.lda = ldy; g.B = X; g.b_t = true; g.ldb = ldx; g.M = N; g.N = K; g.K = M;
  g.C = dW; g.ldc = K; g.c_f32 = true;
  et::gemm_bf16_plan_split(N, K, M, &g.tile, &g.split_k);
  g.partials = c->gemm_partials;
  if (et::gemm_bf16_partial_elems(N, K, g.split_k) > c->gemm_partial_elems) { g.split_k = 1; g.tile = 0; }
  return g;
}

// ---- weight gradients at the end of the pass (see et_ctx::keep_arena)
// `total`: elements of all the gradients that weight gradients are taken from; beyond 24 GB, or the room that is given, weight gradients run at once
inline void reserve_keep(et_ctx* c, size_t total) { c->keep_most = std::min(total, (size_t)12 << 30); }
inline size_t keep_size(size_t elems) { return (elems + 127) / 128 * 128; }
// where the gradient in front of a weight is to be stored: kept for the end of the pass if the weight is selected
inline bf16* keep(et_ctx* c, bool selected, size_t elems, bf16* scratch) {
  if (!selected || c->keep_used + keep_size(elems) > c->keep_elems) return scratch;
  bf16* p = c->keep_arena + c->keep_used;
  c->keep_used += keep_size(elems);
  return p;
}
inline bool kept(const et_ctx* c, const bf16* d) { return d == c->dl16 || (d >= c->keep_arena && d < c->keep_arena + c->keep_elems); }
inline void dw_defer(et_ctx* c, int tensor, const et::DwJob& j) {
  c->dw_jobs.push_back(j);
  c->dw_tensors.push_back(tensor);
}
// partial sums of split products: room for the largest single one (`elems`), and for all weight gradients of a pass (`all`) up to 1.5 GB
inline void reserve_partials(et_ctx* c, size_t elems, size_t all) {
  c->gemm_partial_elems = elems;
  c->group_most = std::max(std::max<size_t>(elems, 64), std::min((size_t)384 << 20, all));
}
// behind everything else: the sizes of a workspace
inline void reserve_tail(et_ctx* c) {
  c->tail_at = c->ws_min = c->ws_bytes;
  if (c->group_most == 0) return;   // (a model that keeps no gradients)
  c->ws_min += align_up(sizeof(float) * std::max<size_t>(c->gemm_partial_elems, 64), 256);
  c->ws_bytes += align_up(sizeof(float) * c->group_most, 256) + align_up(sizeof(bf16) * c->keep_most, 256);
}
// divides what is there beyond the least between both parts as they could use it
inline void place_tail(et_ctx* c, size_t bytes) {
  if (c->group_most == 0) return;
  bytes = std::min(bytes, c->ws_bytes) / 256 * 256;
  const size_t least = c->ws_min - c->tail_at, most = align_up(sizeof(float) * c->group_most, 256);
  const size_t extra = bytes - c->ws_min, extra_most = c->ws_bytes - c->ws_min;
  const size_t scratch = extra == extra_most ? most : least + (size_t)((double)(most - least) * ((double)extra / (double)extra_most)) / 256 * 256;
  c->gemm_partials = (float*)(c->ws + c->tail_at);
  c->group_elems = scratch / sizeof(float);
  c->keep_arena = (bf16*)(c->ws + c->tail_at + scratch);
  c->keep_elems = (bytes - c->tail_at - scratch) / sizeof(bf16);
}

// bracket a launch with events while per-kernel timing is on
struct KernelTimer {
  et_ctx* c;
  bool on = false;
  size_t idx = 0;
  KernelTimer(et_ctx* ctx, int cls, double work) : c(ctx) {
    if (!c->ktiming) return;
    KernelRecord r;
    r.cls = cls;
    r.work = work;
    for (hipEvent_t* ev : {&r.e0, &r.e1}) {
      if (c->kevents_used == c->kevent_pool.size()) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) { c->hip_err = hipErrorOutOfMemory; return; }
        c->kevent_pool.push_back(e);
      }
      *ev = c->kevent_pool[c->kevents_used++];
    }
    (void)hipEventRecord(r.e0, c->stream);
    idx = c->krecs.size();
    c->krecs.push_back(r);
    on = true;
  }
  ~KernelTimer() {
    if (on) (void)hipEventRecord(c->krecs[idx].e1, c->stream);
  }
};

inline int launch_gemm(et_ctx* c, const et::GemmDesc& g) {
  int n = 0;
  const int cls = g.a_t ? 2 : (g.b_t ? 1 : 0);
  KernelTimer kt(c, cls, 2.0 * g.M * g.N * (double)g.K * g.z_outer * g.z_inner);
  hipError_t e = et::gemm_bf16(g, c->stream, &n);
  if (e != hipSuccess) { c->hip_err = e; return ET_EHIP; }
  c->launches[c->cur_phase] += n;
  return ET_OK;
}
#define ET_G(g)                            \
  do {                                     \
    int r__ = launch_gemm(c, (g));         \
    if (r__ != ET_OK) return r__;          \
  } while (0)

// weight gradient of `tensor`, dW[N][K] = dY[M][N]^T X[M][K]: with the others at the end of the pass if dY stays, else at once (and while
// kernels are timed, each with a record of its own)
inline int weight_grad(et_ctx* c, int tensor, const bf16* dY, int ldy, const bf16* X, int ldx, int M, int N, int K) {
  et::DwJob j;
  j.A = dY; j.lda = ldy; j.B = X; j.ldb = ldx; j.C = c->grad[tensor]; j.M = N; j.N = K; j.K = M;
  const et::GemmDesc g = linear_dw(c, dY, ldy, X, ldx, c->grad[tensor], M, N, K);
  j.split = g.split_k;
  if (!c->ktiming && kept(c, dY) && et::dw_group_takes(j)) {
    dw_defer(c, tensor, j);
    return ET_OK;
  }
  Region r(c, PH_DW, tensor);
  ET_G(g);
  return ET_OK;
}

// runs what has been deferred, in groups whose split reductions find room in the scratch
inline int dw_finish(et_ctx* c) {
  hipError_t e = hipSuccess;
  const int n = (int)c->dw_jobs.size();
  for (int at = 0, group = 0; at < n && e == hipSuccess; group++) {
    int end = at;
    for (size_t used = 0; end < n && end - at < et::DW_GROUP_MAX; end++) {
      used += et::dw_group_elems(c->dw_jobs[end]);
      if (used > c->group_elems && end > at) break;
    }
    // the plan depends on the shapes alone and is kept while they stay the same
    et::DwGroupPlan& plan = c->dw_plans[group];
    e = et::dw_group_plan(c->dw_jobs.data() + at, end - at, plan);
    if (e == hipSuccess) {
      std::vector<Share> shares;
      if (c->profiling)
        for (int i = at; i < end; i++) shares.push_back({PH_DW, c->dw_tensors[i], plan.cost[i - at]});
      Region r(c, PH_DW, shares.data(), shares.size());
      int launches = 0;
      e = et::dw_group(c->dw_jobs.data() + at, end - at, plan, c->gemm_partials, c->stream, &launches);
      c->launches[PH_DW] += launches;
    }
    at = end;
  }
  c->dw_jobs.clear();
  c->dw_tensors.clear();
  if (e != hipSuccess) { c->hip_err = e; return ET_EHIP; }
  return ET_OK;
}

}  // namespace et_exec

// per-model chains (each in its own file)
int build_resnet(et_ctx* c);
// mask (nullable = keep everything): the forward pass stores a backward-only tensor only if the
// masked backward pass will read it
int resnet_forward(et_ctx* c, const void* x, const int32_t* y, const uint8_t* mask);
int resnet_backward(et_ctx* c, const void* x, const uint8_t* mask);
int build_mobilenet(et_ctx* c);
int mobilenet_forward(et_ctx* c, const void* x, const int32_t* y, const uint8_t* mask);
int mobilenet_backward(et_ctx* c, const void* x, const uint8_t* mask);
int build_vgg(et_ctx* c);
int vgg_forward(et_ctx* c, const void* x, const int32_t* y);
int vgg_backward(et_ctx* c, const void* x, const uint8_t* mask);
