// Internal launch interface of the HIP kernels (gfx950).  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace et {

typedef __bf16 bf16;

// ------------------------------------------------------------------------------------------
// bf16 MFMA GEMM:  D[i][j] = alpha * sum_k A(i,k) * B(j,k)   (fp32 accumulation)
//   A(i,k) = a_t ? A[k*lda + i] : A[i*lda + k]      (a_t: the reduction index is the slow one)
//   B(j,k) = b_t ? B[k*ldb + j] : B[j*ldb + k]
// so forward (X W^T) is (a_t,b_t) = (0,0), input gradient (dY W) is (0,1) and weight gradient
// (dY^T X) is (1,1).  Requirements (checked on the host): 16-byte aligned bases, lda/ldb multiples
// of 8, ldc and the C batch strides multiples of 4; an operand that is not transposed must have
// finite data up to K rounded up to 8 in every row (the tail is multiplied by zeros or must itself
// be zero).  Only the (layout, epilogue) pairs the training step uses are built: a residual needs
// fp32 output and (0,0); GELU forward needs (0,0), GELU backward (0,1), split-K (1,1).
// ------------------------------------------------------------------------------------------
enum EpiMode : int {
  EPI_PLAIN = 0,     // C = v
  EPI_GELU_FWD = 1,  // C = gelu'(v) (bf16, kept for the backward pass), C2 = gelu(v) (bf16)
  EPI_GELU_BWD = 2,  // C = v * U, U = the stored gelu'(u)
  EPI_AFFINE_RELU = 3,  // C = z = v (bf16), C2 = max(z * gain[j] + bias[j], 0) (bf16), z as rounded to bf16
  EPI_BIAS_RELU = 6,    // C = max(v + bias, 0) (bf16)
  EPI_RELU_MASK = 7,    // C = U > 0 ? v : 0 (bf16): gradient through a ReLU whose output U was stored
  EPI_GELU_ONLY = 5,    // C = gelu(v) (bf16): the forward of a layer whose backward will not run
  EPI_AFFINE_ADD_RELU = 4,  // C = z, C2 = max(z * gain + bias + U * gain2 + bias2, 0); gain2 null: + U
};

// compute units of the current device (a multiple of 8): what a resident kernel's grid is
int compute_units();

struct GemmDesc {
  const bf16* A = nullptr;
  const bf16* B = nullptr;
  int M = 0, N = 0, K = 0;
  // a row-major operand is read up to K rounded up to 8: finite values there, and zeros in one of two row-major operands
  int lda = 0, ldb = 0;
  bool a_t = false, b_t = false;
  // batching: blockIdx.z = outer * z_inner + inner; offsets in elements
  int z_outer = 1, z_inner = 1;
  long long sAo = 0, sAi = 0, sBo = 0, sBi = 0, sCo = 0, sCi = 0;
  // split-K (weight gradients): > 1 writes fp32 partials to `partials` and reduces them in a
  // fixed order with a second kernel; batching must then be off
  int split_k = 1;
  float* partials = nullptr;
  // epilogue: v = alpha * acc + bias[j] + residual[i][j]
  float alpha = 1.f;
  const bf16* bias = nullptr;      // per output column
  const bf16* gain = nullptr;      // EPI_AFFINE_RELU / EPI_AFFINE_ADD_RELU, per output column
  const bf16* gain2 = nullptr;     // EPI_AFFINE_ADD_RELU (nullable, then bias2 is ignored too)
  const bf16* bias2 = nullptr;
  const float* residual = nullptr; // fp32 [M][ldr]
  int ldr = 0;
  int mode = EPI_PLAIN;
  // the AFFINE modes' activation is a clamp to [act_lo, act_hi] (defaults: ReLU; 0, 6: ReLU6; -inf, +inf: none);
  // EPI_RELU_MASK passes where 0 < U < mask_hi
  float act_lo = 0.f, act_hi = __builtin_inff(), mask_hi = __builtin_inff();
  void* C = nullptr;               // bf16 or fp32 [M][ldc]; may be null for the AFFINE modes (z not kept)
  int ldc = 0;
  bool c_f32 = false;
  bf16* C2 = nullptr;              // EPI_GELU_FWD
  float* colsum = nullptr;         // EPI_GELU_BWD (nullable): (M + 31) / 32 rows of N partial column sums of C as rounded, over 32 rows each
  const bf16* U = nullptr;         // EPI_GELU_BWD, EPI_AFFINE_ADD_RELU, EPI_RELU_MASK: same leading dimension as C
  // implicit convolution (conv_c > 0), 3x3 with zero padding 1 (conv_taps = 3) or 1x1 (conv_taps = 1), stride
  // conv_stride (1 or 2): A is the NHWC activation [batch, conv_h, conv_w, conv_c] itself, standing for its im2col
  // matrix [M = batch Ho Wo][K = taps^2 conv_c] (column (tap, c); Ho = (conv_h - 1) / stride + 1); conv_c must be a
  // multiple of 64; row-major operands, no batching; split_k > 1 (with `partials`, ldc == N, bf16 outputs, not with
  // the ADD / GELU modes) reduces in a second kernel that also applies the epilogue.
  // With a_t and b_t (weight gradient): B is the activation standing for [K = batch Ho Wo output pixels]
  // [N = taps^2 conv_c]; conv_c % 8 == 0, K a multiple of 64 (any K on the ring tile), fp32 output, split allowed
  int conv_h = 0, conv_w = 0, conv_c = 0, conv_taps = 3, conv_stride = 1;
  int tile = 0;                    // 0 = choose by shape; else a TileId (tuning/tests)
};

// 3x3 / stride 1 convolution of 64 channels from tiles of the input with their border (conv_halo.hip); tile id of that kernel in GemmDesc::tile
constexpr int CONV_TILE_HALO = 31;
bool conv_halo_takes(const GemmDesc& d);
bool conv_halo_pays(const GemmDesc& d);
hipError_t conv_halo(const GemmDesc& d, hipStream_t s);
// the same with many channels on small images (conv_raster.hip)
constexpr int CONV_TILE_RASTER = 33, CONV_TILE_RASTER_256 = 35;   // 128 or 256 positions per workgroup
bool conv_raster_takes(const GemmDesc& d);
int conv_raster_tile(GemmDesc d);   // the tile id where this kernel is to be used, without a split; else 0
hipError_t conv_raster(const GemmDesc& d, hipStream_t s);

// returns hipSuccess, or hipErrorInvalidValue when a requirement above is violated
// *launches (nullable) receives the number of kernels launched (1, or 2 with split-K)
hipError_t gemm_bf16(const GemmDesc& d, hipStream_t s, int* launches = nullptr);
// tile id that a plain product without a split runs with
int gemm_bf16_tile(const GemmDesc& d);
// fp32 partial elements needed for a split-K call
size_t gemm_bf16_partial_elems(int M, int N, int split_k);
// tile and split for a weight gradient [M][N] reduced over K rows (a cost model over tile shapes
// and split counts); pass both on in GemmDesc::tile and GemmDesc::split_k
void gemm_bf16_plan_split(int M, int N, int K, int* tile, int* split_k);
// the same for the implicit forward / gradient-passing 3x3 convolution [M pixels][N channels], K = 9 input channels:
// layers with few pixels split the reduction, and a second kernel sums the parts and applies the epilogue
// fixed_sums: the split, and with it the order of every sum, is that of the plan for the wide tiles whichever tile is chosen
void gemm_bf16_plan_conv(int M, int N, int K, int* tile, int* split_k, bool fixed_sums = false);
// the same for the implicit weight gradient of a 3x3 convolution (M output channels, N = 9 input channels, K pixels); taps = 7: of a
// 7x7 stem (N = 256)
void gemm_bf16_plan_conv_dw(int M, int N, int K, int* tile, int* split_k, int taps = 3);

// The weight gradients of a backward pass together: C[M][N] (fp32, rows without padding) = sum over K rows of A[k][m] B[k][n], plain or, with
// conv_c > 0, with B gathered from the NHWC activation [.., conv_h, conv_w, conv_c] (M output channels, N = taps^2 conv_c, K output pixels).
struct DwJob {
  const bf16* A = nullptr;
  const bf16* B = nullptr;
  float* C = nullptr;
  int M = 0, N = 0, K = 0, lda = 0, ldb = 0;
  int conv_h = 0, conv_w = 0, conv_c = 0, conv_taps = 3, conv_stride = 1;
  int split = 1;   // chunks of the reduction: the plan of the product on its own (a gradient has the same bits whatever runs beside it)
};
// One launch of a group: tile, and the jobs in the order of their units
struct DwGroupLaunch {
  struct Part { int job, split, per; long long tiles; };   // chunks of the reduction, of `per` slices of 64 rows; tiles of each
  bool direct = false, gathered = false;
  int bm = 64, bn = 64;
  double cost = 0.0;     // estimate, us
  std::vector<Part> parts;
};
// Which kernels run a group, in which order; a function of the jobs' shapes alone
struct DwGroupPlan {
  std::vector<long long> shapes;
  std::vector<DwGroupLaunch> launches;
  std::vector<double> cost;   // per job: estimated share of the time, in arbitrary units
};
// whether a gradient can take part (an implicit one of 14 GFLOP and more is better off on its own)
bool dw_group_takes(const DwJob& j);
// floats of scratch that its chunks take
inline size_t dw_group_elems(const DwJob& j) { return j.split > 1 ? (size_t)j.split * j.M * j.N : 0; }
constexpr int DW_GROUP_MAX = 120;   // jobs of a group
// makes `plan` that of the jobs, unless it is
hipError_t dw_group_plan(const DwJob* jobs, int n, DwGroupPlan& plan);
// Runs them, in few launches; the gradients are bit-reproducible.  partials: scratch for dw_group_elems of all jobs, 16-byte aligned
hipError_t dw_group(const DwJob* jobs, int n, const DwGroupPlan& plan, float* partials, hipStream_t s, int* launches);

// ------------------------------------------------------------------------------------------
// fp32 GEMM (true fp32 FMA), same operand convention, for the fp32 MLP workload
//   relu_out: C = max(v, 0);  mask: C = v * (mask[i][j] > 0)  (ReLU backward, ldmask = ldc)
// ------------------------------------------------------------------------------------------
struct GemmF32Desc {
  const float* A = nullptr;
  const float* B = nullptr;
  float* C = nullptr;
  int M = 0, N = 0, K = 0, lda = 0, ldb = 0, ldc = 0;
  bool a_t = false, b_t = false;
  bool relu_out = false;
  const float* mask = nullptr;
};
hipError_t gemm_f32(const GemmF32Desc& d, hipStream_t s);

// ------------------------------------------------------------------------------------------
// row-wise and reduction kernels (HBM bound)
// ------------------------------------------------------------------------------------------
// LayerNorm forward over rows of an fp32 matrix; in_stride = elements between consecutive rows
hipError_t layernorm_fwd(const float* h, long long in_stride, const bf16* gain, const bf16* shift, float eps,
                         bf16* out, float* mean, float* rstd, int rows, int D, hipStream_t s);
// LayerNorm backward over `rows` rows of D elements: dh = skip + LN'(d), in fp32 and bf16; and, where a part_* pointer is given
// (D <= LAYERNORM_SUMS_MAX_D), layernorm_bwd_parts(rows) rows of D partial column sums of
//   d * xhat (gain gradient), d (shift gradient), dh (gradient of the bias added in front of the LayerNorm's input).
// Strides in elements between consecutive rows: d, h, the statistics, and dh / dh16 / skip; skip may be null, and is
// added only to every skip_period-th row if that is above 1.
struct LayerNormBwd {
  const bf16* d = nullptr;
  const float *h = nullptr, *mean = nullptr, *rstd = nullptr;
  const bf16* gain = nullptr;
  const float* skip = nullptr;
  float* dh = nullptr;
  bf16* dh16 = nullptr;
  float *part_gain = nullptr, *part_shift = nullptr, *part_bias = nullptr;
  long long d_stride = 0, h_stride = 0, stat_stride = 1, out_stride = 0;
  int rows = 0, D = 0, skip_period = 1;
};
constexpr int LAYERNORM_SUMS_MAX_D = 2048;
int layernorm_bwd_parts(int rows);
hipError_t layernorm_bwd(const LayerNormBwd& a, hipStream_t s);

// Column sums over rows come in two steps.  A first kernel leaves partial sums, colsum_parts(rows, cols) rows of `cols`
// floats; sum_finish adds the partial rows of any number of such jobs in one launch, in a fixed order.
//   colsum_part: sum_r d[r][c] * (h ? (h[r][c]-mean[r])*rstd[r] : 1);  d is bf16 (d_f32 == nullptr) or fp32
struct SumJob {
  const float* part;   // [rows][cols], 16-byte aligned
  float* out;          // [cols]
  int rows, cols;      // cols a multiple of 4
  int block0;          // filled in by sum_finish
};
hipError_t colsum_part(const bf16* d, const float* d_f32, long long d_stride, const float* h, long long h_stride, const float* mean,
                       const float* rstd, long long stat_stride, float* part, int rows, int cols, hipStream_t s);
hipError_t sum_finish(SumJob* jobs, int n, hipStream_t s, int* launches);
int colsum_parts(int rows, int cols);
// Backward of a per-channel affine, rows x cols, cols a multiple of 8.  With m = (d + add) where the activation is open, else 0 (as
// rounded to bf16): dmid = m; dout = m * gain; part_sum, part_mul: affine_back_parts(rows, cols) rows of partial sums of m and of
// m * z.  Every output is nullable, dmid may alias d or add.  Open: everywhere; or where 0 < y < hi; or (mask_from_z) where
// 0 < clamp(z * gain + shift, 0, hi) < hi, rounded as the forward pass stores it.  z is bf16, or z32 fp32 (then no add, no y).
struct AffineBack {
  const bf16 *d = nullptr, *add = nullptr, *y = nullptr, *z = nullptr, *gain = nullptr, *shift = nullptr;
  const float* z32 = nullptr;
  bf16 *dmid = nullptr, *dout = nullptr;
  float *part_sum = nullptr, *part_mul = nullptr;
  float hi = __builtin_inff();
  bool mask_from_z = false;
  int rows = 0, cols = 0;
};
int affine_back_parts(int rows, int cols);
hipError_t affine_back_part(const AffineBack& a, hipStream_t s);
// sum over the batch: out[t][c] = sum_b d[b][t][c]   (t < T_out; fp32 in/out)
hipError_t batchsum(const float* d, float* out, int B, long long batch_stride, int n, hipStream_t s);

// softmax over the first `cols` entries of each fp32 row (ld elements apart); bf16 result, tail zeroed
hipError_t softmax_rows(const float* s, bf16* p, int rows, int cols, int ld, hipStream_t stream);
// dS = scale * P * (dP - sum(dP*P)); bf16 result, tail zeroed
hipError_t softmax_bwd_rows(const float* dp, const bf16* p, bf16* ds, float scale, int rows, int cols, int ld,
                            hipStream_t stream);

// fused attention core (head size 64): up to 224 tokens one workgroup per (batch, head), beyond that one per 128 queries
// (or keys) of a (batch, head):
//   forward: out[b][t][h*64+d] = softmax(Q K^T * scale) V, lse[b][h][t] = log-sum-exp of the scaled scores
//   backward: dqkv (same layout as qkv) from dout, recomputing the probabilities from lse; `out` is the stored
//   forward output (rowsum(P * dP) = dout . out)
bool attention_fused_supported(int T, int head_dim);
//   rest (more than 224 tokens, attention_wants_rest(T); nullable): what rounding left out of `out`, as bf16; the forward pass leaves it and the
//   backward pass takes rowsum(P * dP) from out + rest (null: from `out` alone)
hipError_t attention_fwd(const bf16* qkv, bf16* out, bf16* rest, float* lse, int B, int T, int H, int head_dim, float scale,
                         hipStream_t s);
bool attention_wants_rest(int T);
// part (nullable): attention_bwd_parts(B, T) rows of partial sums over the rows of dqkv, 3 * 64 H columns each
hipError_t attention_bwd(const bf16* qkv, const bf16* out, const bf16* rest, const bf16* dout, const float* lse, bf16* dqkv, int B, int T, int H,
                         int head_dim, float scale, hipStream_t s, float* part = nullptr);
int attention_bwd_parts(int B, int T);
// backward when only the first token's row of dout is read (the others are zeros that need not be stored): dqkv complete; part
// (nullable): B rows of partial sums
hipError_t attention_bwd_cls(const bf16* qkv, const bf16* out, const bf16* rest, const bf16* dout, const float* lse, bf16* dqkv, int B, int T, int H,
                             int head_dim, float scale, hipStream_t s, float* part = nullptr);
// the same for sequences of any length, streamed (attention_fwd / _bwd choose)
hipError_t attention_long_fwd(const bf16* qkv, bf16* out, bf16* rest, float* lse, int B, int T, int H, float scale, hipStream_t s);
hipError_t attention_long_bwd(const bf16* qkv, const bf16* out, const bf16* rest, const bf16* dout, const float* lse, bf16* dqkv, int B, int T,
                              int H, float scale, hipStream_t s, float* part = nullptr);
int attention_long_bwd_parts(int B, int T);

// mean softmax cross-entropy: dlogits fp32 and (if not null) a bf16 copy [B][ld16], zero padded; `loss` points to
// 64 + B floats: the loss in element 0, the per-row terms from element 64 on (two launches)
hipError_t xent(const float* logits, const int32_t* y, int B, int C, float* loss, float* dlogits, bf16* dlogits_bf16,
                int ld16, hipStream_t s);

// ViT embedding: h0[b][0] = cls + pos[0]; h0[b][t] = e[b][t-1] + pos[t]  (e fp32 [B*(T-1)][D])
hipError_t embed_assemble(const float* e, const bf16* cls, const bf16* pos, float* h0, int B, int T, int D, hipStream_t s);
// drop the CLS rows: out[b*(T-1)+t-1] = bf16(d[b][t]) for t >= 1
hipError_t gather_patch_rows(const float* d, bf16* out, int B, int T, int D, hipStream_t s);
// fill with zeros (a kernel, so that it may be captured in a graph)
hipError_t fill_zero(void* p, size_t bytes, hipStream_t s);

// ------------------------------------------------------------------------------------------
// convolutional workload: NHWC bf16 activations, a convolution is a GEMM over an im2col matrix
// ------------------------------------------------------------------------------------------
struct ConvGeom {
  int B, H, W, C;      // input [B][H][W][C]
  int k, stride, pad;  // square kernel
  int Ho, Wo;          // output size, (H + 2 pad - k) / stride + 1
  int Kc;              // row length of the column matrix: k*k*C rounded up to a multiple of 8
};
// cols[B*Ho*Wo][Kc], column order (ky, kx, c); out-of-image taps and the row tail are zero
hipError_t im2col(const bf16* x, bf16* cols, const ConvGeom& g, hipStream_t s);
// first convolution of a chain (3x3, at most three input channels), no column matrix.  w [N][3][3][C].  With gain: z (nullable) =
// the convolution as rounded, y = clamp(z * gain + shift, lo, hi); without: y = max(convolution + shift, 0)
bool conv_first_supported(int k, int C);
hipError_t conv_first(const bf16* x, const bf16* w, const ConvGeom& g, int N, const bf16* gain, const bf16* shift, bf16* z, bf16* y, float lo,
                      float hi, hipStream_t s);
// out[B][H][W][C] = (adjoint of im2col applied to dcols  + add) * (mask > 0); add, mask nullable; C % 8 == 0;
// dcols is float32 [B*Ho*Wo][Kc] (dcols_f32) or bf16; the taps are added in float32, the result is rounded once
hipError_t col2im(const void* dcols, bool dcols_f32, const bf16* add, const bf16* mask, bf16* out, const ConvGeom& g,
                  hipStream_t s);
// folded BatchNorm: out = act(z1*g1 + b1 + t), t = z2*g2 + b2 (g2 given), z2 (g2 null) or 0 (z2 null);
// z1 is bf16, or fp32 when z1_f32 is given; rows x C, C % 8 == 0
hipError_t affine_act(const bf16* z1, const float* z1_f32, const bf16* g1, const bf16* b1, const bf16* z2,
                      const bf16* g2, const bf16* b2, bool relu, bf16* out, long long rows, int C, hipStream_t s);
// out = (a + b) * (mask > 0), n elements (n % 8 == 0); b nullable; out may alias a or b
hipError_t add_mask(const bf16* a, const bf16* b, const bf16* mask, bf16* out, long long n, hipStream_t s,
                    float mask_hi = __builtin_inff());
// stem pooling: y = relu(z*gain + shift) in fp32, then 3x3 / stride 2 / pad 1 maximum, first maximum in
// (ky, kx) order; arg holds the chosen tap (one byte per output element)
hipError_t maxpool3x3s2_fwd(const float* z, const bf16* gain, const bf16* shift, bf16* out, uint8_t* arg, int B, int H,
                            int W, int C, hipStream_t s);
// out[B][H][W][C] = (d routed back to the chosen taps) * (y > 0)
hipError_t maxpool3x3s2_bwd(const bf16* d, const uint8_t* arg, const bf16* y, bf16* out, int B, int H, int W, int C,
                            hipStream_t s);
// p[b][c] = mean over the HW positions; backward: out[b][t][c] = dp[b][c] / HW * (y[b][t][c] > 0)
hipError_t avgpool_fwd(const bf16* x, bf16* p, int B, int HW, int C, hipStream_t s);
hipError_t avgpool_bwd_relu(const bf16* dp, const bf16* y, bf16* out, int B, int HW, int C, hipStream_t s,
                            float mask_hi = __builtin_inff());
// 2x2 / stride 2 max pooling of y [B][H][W][C] (H, W even), first maximum in (dy, dx) order; arg: one byte per output
hipError_t maxpool2x2_fwd(const bf16* y, bf16* out, uint8_t* arg, int B, int H, int W, int C, hipStream_t s);
// out[B][H][W][C] = (d routed back to the chosen tap of its window) * (y > 0)
hipError_t maxpool2x2_bwd(const bf16* d, const uint8_t* arg, const bf16* y, bf16* out, int B, int H, int W, int C,
                          hipStream_t s);
// rows of K elements <-> rows of Kc >= K elements (zero tail)
// 3x3 depthwise convolution, zero padding 1, stride 1 or 2, NHWC, C % 8 == 0, weights [C][9] (bf16):
//   fwd: z (nullable: not kept) = the convolution, rounded; y = clamp(z * gain + shift, 0, 6)
//   dx:  out[B][H][W][C] = (adjoint applied to d [B][Ho][Wo][C] + add) * (0 < relu6_y < 6); add, relu6_y nullable
//   dw:  part[R][C * 9] fp32 partial sums of R = depthwise3x3_dw_rows(..) workgroups; their column sum (sum_finish) is the
//        gradient [C][9]
hipError_t depthwise3x3_fwd(const bf16* x, const bf16* w, const bf16* gain, const bf16* shift, bf16* z, bf16* y, int B, int H,
                            int W, int C, int stride, hipStream_t s);
hipError_t depthwise3x3_dx(const bf16* d, const bf16* w, const bf16* add, const bf16* relu6_y, bf16* out, int B, int H, int W,
                           int C, int stride, hipStream_t s);
int depthwise3x3_dw_rows(int B, int H, int W, int C, int stride);
hipError_t depthwise3x3_dw(const bf16* d, const bf16* x, float* part, int B, int H, int W, int C, int stride, hipStream_t s);
// out[rows][N] (bf16) = max(z[rows][N] + bias[N], 0), z fp32; N % 4 == 0
hipError_t bias_relu_rows(const float* z, const bf16* bias, bf16* out, int rows, int N, hipStream_t s);
// out[C][3][3][O] = w[O][3][3][C] with mirrored taps: the weight of the 3x3 convolution that maps an output
// gradient to the input gradient; any number of weights in one launch.  O, C multiples of 8, 16-byte aligned.
struct FlipJob {
  const bf16* w;
  bf16* out;
  int O, C;
  int block0;          // filled in by flip3x3
};
hipError_t flip3x3(FlipJob* jobs, int n, hipStream_t s, int* launches);
hipError_t pad_rows(const bf16* in, bf16* out, int rows, int K, int Kc, hipStream_t s);
hipError_t strip_rows(const float* in, float* out, int rows, int K, int Kc, hipStream_t s);
// operands of the stem convolution (7x7 / stride 2 / zero padding 3, C <= 4 input channels) for its gathered GEMM:
// the image padded to [B][Hp][Wp][4] (pixel (h, w) at (h + 3, w + 3)), the weight widened to [O][8][8][4], and the
// float32 weight gradient [O][8][8][4] brought back to [O][7][7][C]
hipError_t stem_pad_image(const bf16* x, bf16* out, int B, int H, int W, int C, int Hp, int Wp, hipStream_t s);
hipError_t stem_pack_weight(const bf16* w, bf16* out, int O, int C, hipStream_t s);
hipError_t stem_unpack_dw(const float* in, float* out, int O, int C, hipStream_t s);

// ------------------------------------------------------------------------------------------
// importance (Eq. 2) and masked optimizer update over a table of tensors
// ------------------------------------------------------------------------------------------
struct TensorSeg {       // one chunk of one tensor
  const float* g;        // gradient
  const void* w;         // current weights (bf16 or fp32)
  const void* w_snap;    // snapshot
  uint32_t n;            // elements in this chunk
  uint32_t tensor;       // tensor index
};
// stage 1: one block per segment -> partial[seg]; stage 2: per tensor, fixed-order sum -> double
// metric 0: sum g (w_snap - w) (Eq. 2); 1: sum |w|; 2: sum |g| (w_snap is not read for 1 and 2)
hipError_t importance_reduce(const TensorSeg* segs_dev, int n_segs, const uint32_t* seg_begin_dev, int n_tensors,
                             bool bf16_weights, double* partial_dev, double* out_dev, hipStream_t s, int metric = 0);

struct UpdateSeg {
  const float* g;
  void* w;        // model weights (bf16 or fp32)
  float* master;  // fp32 master weights (bf16 models), else null
  float* m;
  float* v;       // Adam only
  uint32_t n;
  uint32_t tensor;
};
struct OptParams {
  int kind;       // 0 Adam, 1 SGDW
  float lr, beta1, beta2, eps, momentum, wd;
  float bc1, bc2; // 1 - beta1^t, 1 - beta2^t
  int dry;        // 1: compute, then store the values that were loaded (timing without side effects)
};
// segs_dev lists the chunks of ALL tensors, selected_dev the indices of the n_selected chunks that belong to
// selected tensors: one workgroup per listed chunk, nothing else is touched
hipError_t masked_update(const UpdateSeg* segs_dev, const uint32_t* selected_dev, int n_selected, bool bf16_weights,
                         OptParams p, hipStream_t s);

}  // namespace et
