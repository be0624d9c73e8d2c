// Convolution units shared by the convolutional chains: a convolution is a GEMM over the rows of
// an im2col matrix (a 1x1 stride-1 convolution reads the activation itself): forward cols * W^T,
// dw() d^T * cols (split over the rows), dy() d * W followed by the gather-form adjoint of im2col.
// A 3x3 convolution of stride 1 or 2 (and a strided 1x1 one) with channel counts in multiples of 64 never
// writes that matrix: the forward product and dw() gather its rows from the activation inside the GEMM; dy()
// of a stride-1 3x3 convolution is the same kind of convolution of the output gradient with the mirrored
// weight, dy() of the strided ones goes through a float32 column gradient and the adjoint of im2col.
#pragma once
#include "context.h"

namespace et_exec {

// launch of an HBM-bound kernel of this workload: counted, and timed as kernel class 7 with its
// algorithmic bytes (operands read once, results written once)
#define ET_KB(n, bytes, expr)              \
  do {                                     \
    KernelTimer kt__(c, 7, (double)(bytes)); \
    ET_K(n, expr);                         \
  } while (0)

// Gradient that reaches an affine, before the activation's mask and the shortcut's share have been applied: ((d + add) where
// 0 < y < hi); `tensor` is the one whose dy() handed it over.  Whoever else reads the finished gradient finds it in `dmid`.
// from_z: the activation is the affine's own, its openness follows from z where z is stored.
struct Incoming {
  const bf16 *d = nullptr, *add = nullptr, *y = nullptr;
  bf16* dmid = nullptr;
  float hi = __builtin_inff();
  int tensor = -1;
  bool from_z = false;
};

// The per-channel pieces of a folded-BN affine y = z * gain + shift (tensors tg = gain, tg + 1 = shift) on the
// gradient d [M][C] of y: dw(shift) = column sum of d, dw(gain) = column sum of d * z (z bf16, or float32 z32),
// dy(gain): dout = d * gain.  One kernel reads d once for whichever of the three are wanted (the order of a sum does not
// depend on the others), and finishes d first; the profile divides its time by the bytes each of them adds.  dy_used = false
// skips dy(gain) although the chain passes the tensor: a projection shortcut's scaled gradient has no reader when its weight
// is not selected and nothing in front of the block is (the time model then charges a few microseconds that are not spent).
// *done (if given) tells whether the kernel ran, i.e. whether in.dmid is written.
inline int affine_back(et_ctx* c, const uint8_t* mask, int jstar, int tg, const Incoming& in, const bf16* z, const float* z32,
                       bf16* dout, long long M, int C, bool dy_used = true, bool* done = nullptr) {
  if (done) *done = false;
  const double zb = z32 ? 4.0 : 2.0;
  const bool scaled = tg > jstar && dy_used;
  if (!mask[tg] && !mask[tg + 1] && !scaled) return ET_OK;
  const int parts = et::affine_back_parts((int)M, C);
  const int rc = sums_room(c, 2 * sum_elems(parts, C));
  if (rc != ET_OK) return rc;
  et::AffineBack a;
  a.d = in.d; a.add = in.add; a.dmid = in.dmid; a.hi = in.hi; a.rows = (int)M; a.cols = C;
  a.mask_from_z = in.y && in.from_z && mask[tg];
  a.y = a.mask_from_z ? nullptr : in.y;
  a.z = mask[tg] ? z : nullptr; a.z32 = mask[tg] ? z32 : nullptr;
  a.gain = (const bf16*)c->w[tg]; a.shift = (const bf16*)c->w[tg + 1];
  Share shares[4];
  size_t n = 0;
  double bytes = 2.0;
  if (scaled) { shares[n++] = {PH_DY, tg, 4.0}; bytes += 2.0; }
  if (mask[tg + 1]) shares[n++] = {PH_DW, tg + 1, 0.5};
  if (mask[tg]) { shares[n++] = {PH_DW, tg, zb}; bytes += zb; }
  const double extra = (a.add ? 2.0 : 0.0) + (a.y ? 2.0 : 0.0) + (a.dmid ? 2.0 : 0.0);
  const bool alone = scaled && n == 1;
  if (extra > 0.0) shares[n++] = {PH_DY, in.tensor, extra};
  a.dout = scaled ? dout : nullptr;
  a.part_sum = mask[tg + 1] ? sum_job(c, tg + 1, parts, C) : nullptr;
  a.part_mul = mask[tg] ? sum_job(c, tg, parts, C) : nullptr;
  Region r(c, alone ? PH_DY : PH_DW, shares, n);
  ET_KB(1, (bytes + extra) * M * C, et::affine_back_part(a, c->stream));
  if (done) *done = true;
  return ET_OK;
}

inline et::ConvGeom geom(const et_ctx* c, const ConvUnit& u) {
  et::ConvGeom g;
  g.B = c->desc.batch; g.H = u.H; g.W = u.W; g.C = u.Cin; g.k = u.k; g.stride = u.stride; g.pad = (u.k - 1) / 2;
  g.Ho = u.Ho; g.Wo = u.Wo; g.Kc = u.Kc;
  return g;
}

inline void init_unit(ConvUnit& u, int t, int H, int W, int Cin, int Cout, int k, int stride) {
  u.t = t; u.H = H; u.W = W; u.Cin = Cin; u.Cout = Cout; u.k = k; u.stride = stride;
  const int pad = (k - 1) / 2;
  u.Ho = (H + 2 * pad - k) / stride + 1;
  u.Wo = (W + 2 * pad - k) / stride + 1;
  u.Kc = round8(k * k * Cin);
  u.in = nullptr; u.cols = nullptr; u.z = nullptr; u.y = nullptr; u.wflip = nullptr;
}

inline size_t rows_of(const et_ctx* c, const ConvUnit& u) { return (size_t)c->desc.batch * u.Ho * u.Wo; }
inline bool needs_cols(const ConvUnit& u) { return u.k > 1 || u.stride > 1; }
// which of the three products of a unit run as implicit GEMMs
// (3x3 of stride 1 or 2 and strided 1x1 convolutions gather their rows inside the GEMM)
inline bool gathered_kind(const ConvUnit& u) { return (u.k == 3 && (u.stride == 1 || u.stride == 2)) || (u.k == 1 && u.stride == 2); }
inline bool implicit_fwd(const ConvUnit& u) { return gathered_kind(u) && (u.Cin % 64) == 0; }
inline bool implicit_dy(const ConvUnit& u) { return u.k == 3 && u.stride == 1 && (u.Cout % 64) == 0 && (u.Cin % 8) == 0; }
inline bool implicit_dw(const et_ctx*, const ConvUnit& u) {
  return gathered_kind(u) && (u.Cin % 8) == 0 && u.H < 4096 && u.W < 4096;
}
// tile and split of a unit's implicit forward (or, with the channel roles exchanged, gradient-passing) product
// (a plain stack's forward pass has `fixed_sums`: in front of a max pooling, near-ties of bf16 values are decided by the last bit,
// and with another order of the sums another tap wins here and there, which moves gradients by some per cent; so the order
// stays that of one plan while the tile is free)
inline void plan_implicit(et_ctx* c, et::GemmDesc& g, bool fixed_sums = false) {
  if (const int tile = fixed_sums ? 0 : et::conv_raster_tile(g)) {   // (sums over chunks of channels, then taps)
    g.tile = tile;
    g.split_k = 1;
    return;
  }
  et::gemm_bf16_plan_conv(g.M, g.N, g.K, &g.tile, &g.split_k, fixed_sums);
  g.partials = c->gemm_partials;
  if (et::gemm_bf16_partial_elems(g.M, g.N, g.split_k) > c->gemm_partial_elems) g.split_k = 1;
  if (et::conv_halo_pays(g)) g.tile = et::CONV_TILE_HALO;   // (not a split one; the sums are in the same order)
}
inline size_t conv_split_partials(const et_ctx* c, const ConvUnit& u, bool fixed_sums = false) {
  size_t n = 0;
  int tile, split;
  const int M = (int)rows_of(c, u);
  if (implicit_fwd(u)) {
    et::gemm_bf16_plan_conv(M, u.Cout, u.k * u.k * u.Cin, &tile, &split, fixed_sums);
    n = std::max(n, et::gemm_bf16_partial_elems(M, u.Cout, split));
  }
  if (implicit_dy(u)) {
    et::gemm_bf16_plan_conv(M, u.Cin, 9 * u.Cout, &tile, &split);
    n = std::max(n, et::gemm_bf16_partial_elems(M, u.Cin, split));
  }
  return n;
}
// fp32 partial elements of a unit's weight gradient with the split its plan chooses
inline size_t conv_dw_partials(const et_ctx* c, const ConvUnit& u) {
  const int M = (int)rows_of(c, u);
  int tile, split;
  if (implicit_dw(c, u)) {
    et::gemm_bf16_plan_conv_dw(u.Cout, u.k * u.k * u.Cin, M, &tile, &split);
    return et::gemm_bf16_partial_elems(u.Cout, u.k * u.k * u.Cin, split);
  }
  return et::gemm_bf16_partial_elems(u.Cout, u.Kc, split_for(u.Cout, u.Kc, M));
}

// z = cols(in) * Wm^T; with gain/shift the GEMM epilogue also writes y = max(z * gain + shift, 0)
inline int conv_forward(et_ctx* c, const ConvUnit& u, const bf16* in, const bf16* Wm, void* z, bool z_f32,
                 const bf16* gain = nullptr, const bf16* shift = nullptr, bf16* y = nullptr, const bf16* branch = nullptr,
                 const bf16* gain2 = nullptr, const bf16* shift2 = nullptr) {
  const bf16* A = in;
  if (needs_cols(u) && !implicit_fwd(u)) {
    ET_KB(1, 2.0 * ((double)c->desc.batch * u.H * u.W * u.Cin + (double)rows_of(c, u) * u.Kc),
          et::im2col(in, u.cols, geom(c, u), c->stream));
    A = u.cols;
  }
  et::GemmDesc g = linear_fwd(A, Wm, nullptr, (int)rows_of(c, u), u.Cout, u.Kc);
  if (implicit_fwd(u)) { g.conv_h = u.H; g.conv_w = u.W; g.conv_c = u.Cin; g.conv_taps = u.k; g.conv_stride = u.stride; }
  g.C = z; g.c_f32 = z_f32;
  if (gain) {
    g.mode = et::EPI_AFFINE_RELU; g.gain = gain; g.bias = shift; g.C2 = y;
    if (branch) {   // the other branch of a block end, inside the same ReLU
      g.mode = et::EPI_AFFINE_ADD_RELU; g.U = branch; g.gain2 = gain2; g.bias2 = shift2;
    }
  }
  if (implicit_fwd(u) && !z_f32 && !branch) plan_implicit(c, g);
  ET_G(g);
  return ET_OK;
}

// weight gradient of a unit, from the gradient d of its convolution's output: with the others at the end of the pass if d stays, else at once
inline int conv_dw(et_ctx* c, const ConvUnit& u, const bf16* in, const bf16* d) {
  const int t = u.t;
  if (implicit_dw(c, u)) {   // B operand: the activation standing for its im2col matrix
    et::GemmDesc g;
    const int kk = u.k * u.k * u.Cin;
    g.A = d; g.a_t = true; g.lda = u.Cout; g.B = in; g.b_t = true; g.ldb = kk;
    g.M = u.Cout; g.N = kk; g.K = (int)rows_of(c, u);
    g.C = c->grad[t]; g.ldc = kk; g.c_f32 = true;
    g.conv_h = u.H; g.conv_w = u.W; g.conv_c = u.Cin; g.conv_taps = u.k; g.conv_stride = u.stride;
    et::gemm_bf16_plan_conv_dw(g.M, g.N, g.K, &g.tile, &g.split_k);
    g.partials = c->gemm_partials;
    if (et::gemm_bf16_partial_elems(g.M, g.N, g.split_k) > c->gemm_partial_elems) g.split_k = 1;
    et::DwJob j;
    j.A = d; j.lda = u.Cout; j.B = in; j.ldb = kk; j.C = c->grad[t]; j.M = g.M; j.N = g.N; j.K = g.K;
    j.conv_h = u.H; j.conv_w = u.W; j.conv_c = u.Cin; j.conv_taps = u.k; j.conv_stride = u.stride; j.split = g.split_k;
    if (!c->ktiming && kept(c, d) && et::dw_group_takes(j)) {
      dw_defer(c, t, j);
      return ET_OK;
    }
    Region r(c, PH_DW, t);
    ET_G(g);
    return ET_OK;
  }
  return weight_grad(c, t, d, u.Cout, needs_cols(u) ? u.cols : in, u.Kc, (int)rows_of(c, u), u.Cout, u.Kc);
}

// Gradient of the column matrix: dcols[M][Kc] = d[M][Cout] * Wm[Cout][Kc].  For a 1x1 convolution this is the
// input gradient itself, stored as bf16 like every tensor handed from one operation to the next.  For a larger
// kernel it is an intermediate whose shifted copies the adjoint of im2col has yet to add: it stays float32, so
// that the input gradient is rounded once, after the sum, as in the implicit-GEMM form of the same operation.
inline bool dcols_f32(const ConvUnit& u) { return u.k > 1; }
inline size_t dcols_bytes(const et_ctx* c, const ConvUnit& u) { return rows_of(c, u) * u.Kc * (dcols_f32(u) ? 4 : 2); }
inline int conv_dcols(et_ctx* c, const ConvUnit& u, const bf16* d, const bf16* Wm, void* dcols) {
  et::GemmDesc g = linear_dx(d, Wm, (int)rows_of(c, u), u.Cout, u.Kc);
  g.C = dcols;
  g.c_f32 = dcols_f32(u);
  ET_G(g);
  return ET_OK;
}


// room for the mirrored weight of a unit
inline void reserve_flip(et_ctx* c, ConvUnit& u) {
  if (implicit_dy(u)) reserve(c, &u.wflip, sizeof(bf16) * (size_t)u.Cout * 9 * u.Cin);
}
// the mirrored weights of all units that this backward pass takes dy() of (the weights stand until its update)
inline int mirror_weights(et_ctx* c, const std::vector<const ConvUnit*>& units, int jstar) {
  std::vector<et::FlipJob> jobs;
  std::vector<Share> shares;
  for (const ConvUnit* u : units)
    if (implicit_dy(*u) && u->t > jstar) {
      jobs.push_back({(const bf16*)c->w[u->t], u->wflip, u->Cout, u->Cin, 0});
      shares.push_back({PH_DY, u->t, (double)u->Cout * u->Cin});
    }
  if (jobs.empty()) return ET_OK;
  Region r(c, PH_DY, shares.data(), shares.size());
  int n = 0;
  const hipError_t e = et::flip3x3(jobs.data(), (int)jobs.size(), c->stream, &n);
  c->launches[PH_DY] += n;
  if (e != hipSuccess) { c->hip_err = e; return ET_EHIP; }
  return ET_OK;
}

// dy() of a 3x3 / stride 1 unit as an implicit GEMM: out = (convolution of d with the mirrored weight), times
// the ReLU mask (relu_y > 0) if given
inline int conv_dy_implicit(et_ctx* c, const ConvUnit& u, const bf16* d, const bf16* relu_y, bf16* out) {
  et::GemmDesc g = linear_fwd(d, u.wflip, nullptr, (int)rows_of(c, u), u.Cin, 9 * u.Cout);
  g.conv_h = u.H; g.conv_w = u.W; g.conv_c = u.Cout;
  g.C = out;
  if (relu_y) { g.mode = et::EPI_RELU_MASK; g.U = relu_y; }
  plan_implicit(c, g);
  ET_G(g);
  return ET_OK;
}

}  // namespace et_exec
