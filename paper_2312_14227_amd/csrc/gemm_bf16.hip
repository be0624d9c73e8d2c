// Host side of the bf16 MFMA GEMM: argument checks, tile choice, split-K reduction.
#include <algorithm>
#include <cmath>

#include "gemm_bf16_kernels.h"
#include "gemm_bf16_ring.h"

namespace et {
namespace {

// out[i] = sum_z part[z][i], z ascending: the same order on every run
__global__ void splitk_reduce_kernel(const float4* __restrict__ part, float4* __restrict__ out, size_t n4, int splits) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n4) return;
  float4 s = part[i];
  for (int z = 1; z < splits; z++) {
    const float4 p = part[(size_t)z * n4 + i];
    s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
  }
  out[i] = s;
}

// many chunks, few outputs: 16 lanes share one output vector, lane g adds the chunks g, g + 16, ... in
// order, then the 16 sums are added in lane order (through LDS): again the same order on every run
__global__ __launch_bounds__(256) void splitk_reduce_wide_kernel(const float4* __restrict__ part, float4* __restrict__ out,
                                                                 size_t n4, int splits) {
  __shared__ float4 sh[16][16];
  const int o = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const size_t i = blockIdx.x * (size_t)16 + o;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n4)
    for (int z = grp; z < splits; z += 16) {
      const float4 p = part[(size_t)z * n4 + i];
      s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
    }
  sh[grp][o] = s;
  __syncthreads();
  if (grp == 0 && i < n4) {
    float4 t = sh[0][o];
    for (int k = 1; k < 16; k++) {
      const float4 p = sh[k][o];
      t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
    }
    out[i] = t;
  }
}

// Split implicit convolution: out = epilogue(sum_z part[z]), z ascending.  mode: 0 bf16 copy, 1 max(v + bias, 0),
// 2 0 < U < mask_hi ? v : 0, 3 z = bf16(v) (kept if zout), y = clamp(z * gain + bias, lo, hi)
struct ReduceEpi {
  const float4* part;
  size_t n4;
  int splits, N, mode;
  const bf16* bias;
  const bf16* gain;
  const bf16* U;
  bf16* out;
  bf16* zout;
  float lo, hi, mask_hi;
};

__global__ __launch_bounds__(256) void splitk_reduce_epilogue_kernel(ReduceEpi e) {
  typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= e.n4) return;
  float4 s = e.part[i];
  for (int z = 1; z < e.splits; z++) {
    const float4 p = e.part[(size_t)z * e.n4 + i];
    s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
  }
  float v[4] = {s.x, s.y, s.z, s.w};
  const int col = (int)((i * 4) % (size_t)e.N);
  bf16x4 o;
  if (e.mode == 1) {
    const bf16x4 b = *(const bf16x4*)(e.bias + col);
#pragma unroll
    for (int j = 0; j < 4; j++) o[j] = (bf16)fmaxf(v[j] + (float)b[j], 0.f);
  } else if (e.mode == 2) {
    const bf16x4 u = ((const bf16x4*)e.U)[i];
#pragma unroll
    for (int j = 0; j < 4; j++) o[j] = ((float)u[j] > 0.f && (float)u[j] < e.mask_hi) ? (bf16)v[j] : (bf16)0.f;
  } else if (e.mode == 3) {
    const bf16x4 g = *(const bf16x4*)(e.gain + col), b = *(const bf16x4*)(e.bias + col);
    bf16x4 z;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      z[j] = (bf16)v[j];
      o[j] = (bf16)fminf(fmaxf((float)z[j] * (float)g[j] + (float)b[j], e.lo), e.hi);
    }
    if (e.zout) ((bf16x4*)e.zout)[i] = z;
  } else {
#pragma unroll
    for (int j = 0; j < 4; j++) o[j] = (bf16)v[j];
  }
  ((bf16x4*)e.out)[i] = o;
}

// tiles of the plain products; the implicit convolutions have a kernel of their own for 11, 13 (256x192), 15 (256x128) and 17 .. 21
enum TileId : int { T_AUTO = 0, T_128x128 = 1, T_128x64 = 3, T_DMA_256x256 = 5, T_DMA_256x128 = 7, T_DIRECT_256x256 = 11, T_DIRECT_192x256 = 13,
              T_DIRECT_128x256 = 15, T_PP_256x256 = 11, T_PP_256x192 = 13, T_PP_256x128 = 15, T_PP_512x64 = 17, T_PP_128x256 = 19, T_PP_64x512 = 21,
              T_RING_64x64 = 23, T_RING_64x128 = 25, T_RING_128x64 = 27, T_RING_128x128 = 29 };

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Cost model behind the tile and split choice of the gathered convolutions and the chunks of large weight gradients (seconds, one launch):
//   rounds of workgroups over the 256 CUs x time of one workgroup at the rate a CU sustains with
//   that tile (about 3.3 TFLOP/s per CU with 256x256 through registers, 3.0 with 256x192), plus, for a split
//   reduction, writing and re-reading the fp32 partials.
struct Plan { int tile, split; double cost; };

struct TileRate { int tile, bm, bn; double rate; };

Plan plan_tiles(int M, int N, int K, bool may_split, const TileRate* cand, int n_cand) {
  Plan best = {T_AUTO, 1, 1e30};
  const int slices = (K + gemm::PBK - 1) / gemm::PBK;
  const int max_split = may_split ? std::max(1, std::min(256, slices / 4)) : 1;
  for (int ci = 0; ci < n_cand; ci++) {
    const TileRate& c = cand[ci];
    const long long tiles = (long long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    for (int s = 1; s <= max_split; s++) {
      const int per = (slices + s - 1) / s;
      const int chunks = (slices + per - 1) / per;
      if (chunks != s) continue;   // this split leaves empty chunks: the same work as a smaller one
      const long long rounds = (tiles * s + 255) / 256;
      double t = rounds * (2.0 * c.bm * c.bn * per * gemm::PBK / c.rate);
      if (s > 1) t += (2.0 * s + 1.0) * M * N * 4.0 / 3.5e12 + 4e-6;   // partial traffic and one more launch
      if (t < best.cost) best = {c.tile, s, t};
    }
  }
  return best;
}

// weight gradient of a convolution, [M = output channels][N = 9 input channels] reduced over the pixels:
// few output channels take the tiles that are narrow in M (rates measured on the VGG16 shapes)
Plan plan_conv_dw(int M, int N, int K) {
  static const TileRate cand[4] = {{T_PP_256x256, 256, 256, 3.3e12}, {T_PP_256x192, 256, 192, 3.0e12},
                                   {T_PP_128x256, 128, 256, 2.4e12}, {T_PP_64x512, 64, 512, 2.0e12}};
  return plan_tiles(M, N, K, true, cand, 4);
}

// implicit convolution (forward, gradient passing): the same cost model over the four tiles, with the rates a
// CU sustains on the VGG16 layer shapes (the shifted rows of the nine taps hit in the L2, so the wide tiles
// run faster here than on a stored matrix)
int choose_conv_tile(const GemmDesc& d) {
  if (d.tile == T_PP_256x256 || d.tile == T_PP_256x192 || d.tile == T_PP_256x128 || d.tile == T_PP_512x64 || d.tile == T_RING_64x64 ||
      d.tile == T_RING_64x128 || d.tile == T_RING_128x64 || d.tile == T_RING_128x128)
    return d.tile;
  static const TileRate cand[4] = {{T_PP_256x256, 256, 256, 4.5e12}, {T_PP_256x192, 256, 192, 4.0e12},
                                   {T_PP_256x128, 256, 128, 3.3e12}, {T_PP_512x64, 512, 64, 2.6e12}};
  return plan_tiles(d.M, d.N, d.K, false, cand, 4).tile;
}

// Small and medium products: the tile with the least estimated time (seconds) for `count` batch entries or chunks.  Fixed
// cost apart, a CU works through its share of the tiles one slice after the other, whether one or three workgroups
// share it (us per slice of 64 and per tile, measured on [788 .. 6304 rows] x [64 .. 4096] x [16 .. 4096]):
//   ring 64x64     0.175 (0.205 with one tile per CU) + 0.5: any K; 1.6 - 3.6 x faster than the register-staged tiles on
//                  long K ([788 x 768 x 3072] 36.2 -> 13.9 us, [1568 x 512 x 2048] 25.3 -> 10.0, [1024 x 1024] over 6304
//                  rows 69.8 -> 26.6, all unsplit), equal at 3 - 5 slices;
//   ring 64x128    0.30 (0.33) + 1.0: [4616 x 384 x 1536] 12.5 us against 13.3, [6272 x 256 x 1024] 8.9 against 9.3;
//   ring 128x128   0.55 + 2.3, one workgroup per CU: [25088 x 128 x 512] 11.1 us against 12.9, [1568 x 2048 x 512] 9.1 against 10.6;
//   staged 128x64  0.33 + 0.75, but a memory round trip of 0.75 per slice when a CU has one tile only;
//   staged 128x128 0.66 + 1.2, the same: ahead where tiles are many and short, by halving or quartering the operand
//                  re-reads and the per-tile cost ([100352 x 256 x 64] 17.6 us against 23.3, [25088 x 512 x 128] 12.5
//                  against 15.1).
Plan plan_small(int M, int N, int K, int count) {
  struct Cand { int tile, bm, bn; double slice, solo, fixed; };
  static const Cand cand[5] = {{T_RING_64x64, 64, 64, 0.175e-6, 0.205e-6, 0.5e-6},
                               {T_RING_64x128, 64, 128, 0.30e-6, 0.33e-6, 1.0e-6},
                               {T_RING_128x128, 128, 128, 0.55e-6, 0.55e-6, 2.3e-6},
                               {T_128x64, 128, 64, 0.33e-6, 0.75e-6, 0.75e-6},
                               {T_128x128, 128, 128, 0.66e-6, 0.85e-6, 1.2e-6}};
  Plan best = {T_128x64, 1, 1e30};
  const int slices = (K + gemm::SBK - 1) / gemm::SBK;
  for (const Cand& c : cand) {
    const long long tiles = (long long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * count;
    const long long per_cu = (tiles + 255) / 256;
    const double t = std::max(per_cu * (slices * c.slice + c.fixed), slices * c.solo + c.fixed);
    if (t < best.cost) best = {c.tile, 1, t};
  }
  return best;
}

// A ring tile with its reduction split so that the estimated time is least: a CU's share of the units, one after the
// other (`solo` / `loaded` seconds per slice of 64 with one / several workgroups per CU, `fixed` per unit), at least the time the
// operands take to stream in with as many CUs as there are units (an activation read by nine taps counts once); a split adds the partials' traffic and a second launch (3 us).
struct RingTile { int tile, bm, bn; double solo, loaded, fixed; };

template <int N_TILES>
Plan plan_ring(int M, int N, int K, bool may_split, double operand_elems, const RingTile (&tiles)[N_TILES], int only_split = 0) {
  const int slices = (K + gemm::PBK - 1) / gemm::PBK;
  const double stream = 2.0 * operand_elems / 4e12;
  const int max_split = may_split && (N & 3) == 0 ? std::max(1, std::min(256, slices / 4)) : 1;
  Plan best = {T_RING_64x64, 1, 1e30};
  for (const RingTile& r : tiles)
    for (int s = 1; s <= max_split; s++) {
      if (only_split && s != only_split) continue;
      const int per = (slices + s - 1) / s;
      if ((slices + per - 1) / per != s) continue;   // this split leaves empty chunks
      const long long units = (long long)((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn) * s;
      const double load = stream * 256.0 / (double)std::min<long long>(units, 256);
      const double ring = units <= 256 ? per * r.solo + r.fixed : (double)((units + 255) / 256) * (per * r.loaded + r.fixed);
      double t = std::max(load, ring);
      if (s > 1) t += (2.0 * s + 1.0) * M * N * 4.0 / 3.5e12 + 3e-6;
      if (t < best.cost * 0.999) best = {r.tile, s, t};
    }
  return best;
}

// Rates measured per tile.  Weight gradients [rows of A^T][B^T], any layout of a split reduction (plan_small has the 64x64 rates):
// [1152 x 384] over 4616 rows in 4 chunks 9.8 us on 64x128, 10.5 on 64x64.
const RingTile kRingDw[2] = {{T_RING_64x64, 64, 64, 0.25e-6, 0.175e-6, 0.5e-6}, {T_RING_64x128, 64, 128, 0.36e-6, 0.33e-6, 1.0e-6}};
// Implicit convolutions, 32 images, best 64x64 plan / chosen: 28x28x128 18.7 / 14.9 us (128x128), 14x14x256 17.7 / 15.8 (64x128),
// 224x224x64 257 / 220 (128x64).
const RingTile kRingConv[4] = {{T_RING_64x64, 64, 64, 0.28e-6, 0.19e-6, 0.5e-6}, {T_RING_64x128, 64, 128, 0.38e-6, 0.33e-6, 1.0e-6},
                               {T_RING_128x64, 128, 64, 0.45e-6, 0.33e-6, 1.0e-6}, {T_RING_128x128, 128, 128, 0.56e-6, 0.56e-6, 2.5e-6}};
// Their weight gradients: 28x28x128 20.2 / 17.8 us, 14x14x256 20.6 / 18.2 (128x64), 224x224x64 219 / 185 (64x128).
const RingTile kRingConvDw[3] = {{T_RING_64x64, 64, 64, 0.365e-6, 0.24e-6, 0.5e-6}, {T_RING_64x128, 64, 128, 0.46e-6, 0.36e-6, 1.0e-6},
                                 {T_RING_128x64, 128, 64, 0.36e-6, 0.34e-6, 1.0e-6}};

// Large products with K in slices of 64: rounds of workgroups over the 256 CUs x (slices x time per slice + fixed part), us.  A slice takes longer the more
// CUs are at work (`load` more with all of them: the clock follows the load); an epilogue with more arithmetic or with an fp32 residual adds per
// round, a residual its memory traffic.  Fitted (relative error 3 - 5 %) to 161 products of [1576 .. 17000 rows] x [384 .. 4096] x [512 .. 4096]; the
// epilogues' terms of the direct tiles corrected by 140 others with six epilogues each, [724 .. 12600 rows] x [256 .. 4096] x [256 .. 4096], 8 GFLOP
// and more: 26.4 ms with this choice, 26.4 the best tile of each, 28.7 with the tiles through registers (256x256, 256x192, 256x128) that the
// direct ones replace, no product more than 3 % behind what it took with those: [12608 x 3072 x 768] 78 -> 68 us, with GELU 106 -> 94,
// [12608 x 768 x 3072] 73 -> 62, with residual 92 -> 73.  Between 6 and 8 GFLOP it would be 0.99x in the sum and 0.8x for tall reductions
// ([1377 x 640 x 4032] 18.1 -> 22.5): those stay with plan_small.
int choose_large_tile(const GemmDesc& d, int K) {
  struct Cand { int tile, bm, bn; double slice, load, rounds2, fixed, once, gelu, gelu_back, res, res_elem, elem; };
  static const Cand cand[5] = {{T_DIRECT_256x256, 256, 256, 0.870, 0.525, 0.0, 2.79, 3.68, 9.81, 3.56, 3.99, 0.632e-6, 0.238e-6},
                               {T_DIRECT_192x256, 192, 256, 0.686, 0.536, 0.0, 3.48, 2.62, 8.18, 3.15, 2.80, 0.679e-6, 0.110e-6},
                               {T_DIRECT_128x256, 128, 256, 0.644, 0.345, 0.0, 2.92, 2.41, 6.16, 2.74, 1.99, 0.785e-6, 0.041e-6},
                               {T_RING_64x128, 64, 128, 0.227, 0.092, 0.00065, 1.00, 3.90, 1.38, 0.02, 0.0, 0.640e-6, 0.0},
                               {T_RING_128x128, 128, 128, 0.431, 0.147, 0.0, 2.11, 2.14, 3.31, 0.0, 0.0, 0.715e-6, 0.317e-6}};
  const bool gelu = d.mode == EPI_GELU_FWD || d.mode == EPI_GELU_ONLY, gelu_back = d.mode == EPI_GELU_BWD;
  const double slices = (K + gemm::PBK - 1) / gemm::PBK, batch = (double)d.z_outer * d.z_inner * std::max(1, d.split_k), elems = (double)d.M * d.N * batch;
  int best = T_DIRECT_128x256;
  double least = 1e30;
  for (const Cand& c : cand) {
    // (the epilogues of a folded BatchNorm need more registers than the tallest tiles leave)
    if (d.mode == EPI_AFFINE_RELU && c.tile == T_DIRECT_256x256) continue;
    if (d.mode == EPI_AFFINE_ADD_RELU && (c.tile == T_DIRECT_256x256 || c.tile == T_DIRECT_192x256)) continue;
    const double tiles = (double)((d.M + c.bm - 1) / c.bm) * ((d.N + c.bn - 1) / c.bn) * batch, rounds = std::ceil(tiles / 256.0);
    double t = rounds * (slices * (c.slice + c.load * tiles / rounds / 256.0 + c.rounds2 * rounds) + c.fixed) + c.once + c.elem * elems;
    if (d.residual) t += rounds * c.res + c.res_elem * elems;
    if (gelu || gelu_back) t += rounds * (gelu ? c.gelu : c.gelu_back);
    if (t < least) { least = t; best = c.tile; }
  }
  return best;
}

// Chunks of a weight gradient's reduction [M][N] over K rows, from the shape alone: they fix the order of the sums, and so a gradient's bits, whichever
// kernel runs it, alone or in a group.  The error of an fp32 sum grows with the length of its chunk: against 64 bits (2-norms), [2304 x 768] over
// 12608 rows 2.6e-7 with these 7 chunks and 4.0e-7 with 3, [2304 x 768] over 6304 1.7e-7 with 8 and 3.4e-7 with 2, twice to three times as much
// where the activations have a mean.  3 chunks would write less: a full step of 12 such blocks takes 10.24 ms with 3, 10.53 ms with these.
// 16 GFLOP and more: over a multiple of 64 rows the least of rounds of 256 x 256 or 256 x 192 tiles and the partials' traffic; over a multiple of
// 32, about 256 tiles in all and at most 8 chunks.  Else the plan of the ring tiles.
int split_of_dw(int M, int N, int K) {
  if (M >= 256 && N >= 256 && 2.0 * M * N * (double)K >= 1.6e10) {
    static const TileRate cand[2] = {{T_AUTO, 256, 256, 3.3e12}, {T_AUTO, 256, 192, 3.0e12}};
    if ((K % gemm::PBK) == 0) return plan_tiles(M, N, K, (N & 3) == 0, cand, 2).split;
    if ((K % gemm::DBK) == 0 && K >= 128 * gemm::DBK) {
      const int slices = (K + gemm::PBK - 1) / gemm::PBK, tiles = ((M + 255) / 256) * ((N + 255) / 256);
      const int wanted = (N & 3) == 0 ? std::max(1, std::min(8, 256 / tiles)) : 1, per = (slices + wanted - 1) / wanted;
      return (slices + per - 1) / per;   // (no empty chunks)
    }
  }
  return plan_ring(M, N, K, true, ((double)M + N) * K, kRingDw).split;
}

// Tile of a weight gradient of 4 GFLOP and more that runs by itself, in those chunks: the least estimated time (us).  As above, with the
// partials' traffic and the second launch; the time per slice of a ring tile grows with the length of its chunk (its operand re-reads).  Fitted to
// 85 shapes of [384 .. 4096] x [384 .. 1024] over 1576 .. 17000 rows with up to a dozen plans each (relative error 5 - 8 %).
int tile_of_dw(int M, int N, int K, int split) {
  struct Cand { int tile, bm, bn; double slice, slice2, load, solo, fixed, once, part, elem, split, rounds2; };
  static const Cand cand[5] = {{T_DIRECT_256x256, 256, 256, 0.833, 0.0, 0.696, 0.0, 5.38, 5.92, 0.880e-6, 0.0, 0.0, 0.0},
                               {T_DIRECT_192x256, 192, 256, 0.841, 0.0, 0.419, 0.0, 3.84, 4.65, 0.890e-6, 0.0, 1.80, 0.0},
                               {T_DIRECT_128x256, 128, 256, 0.765, 0.0, 0.304, 0.0, 2.35, 5.45, 0.744e-6, 0.0, 2.41, 0.0},
                               {T_RING_64x128, 64, 128, 0.179, 0.00069, 0.0, 0.0, 0.0, 5.61, 1.377e-6, 0.750e-6, 2.53, 0.0228},
                               {T_RING_64x64, 64, 64, 0.116, 0.00047, 0.0, 0.0179, 0.0, 5.95, 1.581e-6, 0.189e-6, 1.00, 0.0122}};
  const int slices = (K + gemm::PBK - 1) / gemm::PBK, per = (slices + split - 1) / split;
  int best = T_RING_64x128;
  double least = 1e30;
  for (const Cand& c : cand) {
    const double units = (double)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * split, elems = (double)M * N, rounds = std::ceil(units / 256.0);
    double t = rounds * (per * (c.slice + c.slice2 * per + c.load * units / rounds / 256.0 + c.rounds2 * rounds) + c.fixed) + c.once + c.elem * elems;
    if (rounds == 1.0) t += c.solo * per;
    if (split > 1) t += c.part * split * elems + c.split;
    if (t < least) { least = t; best = c.tile; }
  }
  return best;
}

int choose_tile(const GemmDesc& d, int k_per_block) {
  const bool dma_ok = (d.K % gemm::DBK) == 0 && (k_per_block % gemm::DBK) == 0;
  const bool slices_ok = (d.K % gemm::PBK) == 0 && (k_per_block % gemm::PBK) == 0;
  // the direct tiles take any number of rows of a weight gradient, and split no other product; their lanes' offsets within a slice are 32 bits wide
  const bool direct_ok = ((d.a_t && d.b_t) || (slices_ok && d.split_k <= 1)) && d.lda < (1 << 22) && d.ldb < (1 << 22);
  if (d.tile == T_DIRECT_256x256 || d.tile == T_DIRECT_192x256 || d.tile == T_DIRECT_128x256) {
    if (!direct_ok) return dma_ok ? T_DMA_256x256 : T_128x128;
    if (d.mode == EPI_AFFINE_ADD_RELU) return T_DIRECT_128x256;
    return d.mode == EPI_AFFINE_RELU && d.tile == T_DIRECT_256x256 ? T_DIRECT_192x256 : d.tile;
  }
  if (d.tile == T_PP_512x64 || d.tile == T_PP_128x256 || d.tile == T_PP_64x512) return slices_ok ? d.tile : T_128x128;   // (by id only: tests, tuning)
  if (d.tile == T_DMA_256x256 || d.tile == T_DMA_256x128) return dma_ok ? d.tile : T_128x128;
  if (d.tile != T_AUTO) return d.tile;
  // large problems (8 GFLOP and more; a ViT-L layer at batch 32 has 13): the tile with the least estimated time where K comes in
  // slices of 64, else the direct-to-LDS tile with slices of 32.
  const int batch = d.z_outer * d.z_inner;
  if (d.M >= 512 && d.N >= 256 && 2.0 * d.M * d.N * (double)k_per_block * batch >= 8e9) {
    const long long big_tiles = (long long)((d.M + 255) / 256) * ((d.N + 255) / 256) * batch;
    if (direct_ok && k_per_block >= 4 * gemm::PBK) return choose_large_tile(d, k_per_block);
    if (dma_ok && k_per_block >= 4 * gemm::DBK && big_tiles >= 128) return d.N >= 2560 ? T_DMA_256x128 : T_DMA_256x256;
  }
  return plan_small(d.M, d.N, k_per_block, batch * std::max(1, d.split_k)).tile;
}

}  // namespace

int gemm_bf16_tile(const GemmDesc& d) { return choose_tile(d, d.K); }

// number of compute units of the current device (256 on an MI355X), looked up once per device; a multiple of 8
// (one share per XCD) as the resident kernels' unit order assumes whenever a workgroup takes a second unit
int compute_units() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
    cus[dev] = n & ~7;
  }
  return cus[dev];
}

size_t gemm_bf16_partial_elems(int M, int N, int split_k) { return split_k > 1 ? (size_t)M * N * split_k : 0; }

// Implicit convolutions: the ring tiles up to 32 GFLOP (weight gradients: 14) and for at most 64 output channels, the two-group
// tiles beyond.  Measured at batch 32, forward (two-group plan / ring): 7x7x512 27.9 / 20, 14x14x256 27.6 / 15.8, 56x56x64
// 24.5 / 20, 224x224x64 285 / 220 us, 14x14x512 45.8 / 42, but 112x112x128 155 / 170; weight gradients: 14x14x256 32.0 / 20,
// 56x56x64 43.5 / 23, 224x224x64 390 / 195, but 14x14x512 52 / 54, 56x56 128 -> 256 81 / 110.
static bool conv_on_ring(int rows, int channels, int K, double most) { return channels <= 64 || 2.0 * rows * channels * (double)K < most; }

void gemm_bf16_plan_conv(int M, int N, int K, int* tile, int* split_k, bool fixed_sums) {
  static const TileRate cand[4] = {{T_PP_256x256, 256, 256, 4.5e12}, {T_PP_256x192, 256, 192, 4.0e12},
                                   {T_PP_256x128, 256, 128, 3.3e12}, {T_PP_512x64, 512, 64, 2.6e12}};
  const bool ring = conv_on_ring(M, N, K, 3.2e10);
  const Plan wide = !ring || fixed_sums ? plan_tiles(M, N, K, (N & 3) == 0, cand, 4) : Plan{T_AUTO, 0, 0.0};
  const Plan pl = ring ? plan_ring(M, N, K, true, K / 9.0 * M + (double)N * K, kRingConv, wide.split) : wide;
  *tile = pl.tile;
  *split_k = pl.split;
}

void gemm_bf16_plan_conv_dw(int M, int N, int K, int* tile, int* split_k, int taps) {
  // a pixel count that is not a multiple of 64 runs on the ring tile whatever its size; a 7x7 stem always on the two-group tiles, the only
  // ones built for its window (64 x 256 over 401 408 pixels: 46 us in 251 chunks of 128 x 256; with the 128 that the ring plan asks for 77)
  const bool ring = taps != 7 && ((K % gemm::PBK) || conv_on_ring(K, M, N, 1.4e10));
  const Plan pl = ring ? plan_ring(M, N, K, true, (M + N / 9.0) * K, kRingConvDw) : plan_conv_dw(M, N, K);
  *tile = pl.tile;
  *split_k = pl.split;
}

void gemm_bf16_plan_split(int M, int N, int K, int* tile, int* split_k) {
  *tile = T_AUTO;
  *split_k = 1;
  *split_k = split_of_dw(M, N, K);
  if (2.0 * M * N * (double)K >= 4e9 && M >= 256 && N >= 256 && K >= 4 * gemm::PBK) *tile = tile_of_dw(M, N, K, *split_k);
  else if (*split_k > 1) *tile = plan_ring(M, N, K, true, ((double)M + N) * K, kRingDw).tile;   // (unsplit: whichever tile choose_tile prefers)
}

hipError_t gemm_bf16(const GemmDesc& d, hipStream_t s, int* launches) {
  if (launches) *launches = 0;
  const bool c_optional = d.mode == EPI_AFFINE_RELU || d.mode == EPI_AFFINE_ADD_RELU;
  if (!d.A || !d.B || (!d.C && !c_optional) || d.M <= 0 || d.N <= 0 || d.K <= 0) return hipErrorInvalidValue;
  if (!aligned(d.A, 16) || !aligned(d.B, 16) || !aligned(d.C, 16) || (d.lda & 7) || (d.ldb & 7)) return hipErrorInvalidValue;
  if ((d.sAo | d.sAi | d.sBo | d.sBi) & 7) return hipErrorInvalidValue;
  if ((d.sCo | d.sCi) & 3) return hipErrorInvalidValue;
  if (d.z_outer < 1 || d.z_inner < 1) return hipErrorInvalidValue;
  // rows must be long enough for the 16-byte loads of the contiguous index
  if (!d.a_t && d.conv_c <= 0 && d.lda < ((d.K + 7) & ~7)) return hipErrorInvalidValue;
  if (!d.b_t && d.ldb < ((d.K + 7) & ~7)) return hipErrorInvalidValue;
  if (d.a_t && d.lda < ((d.M + 7) & ~7)) return hipErrorInvalidValue;
  if (d.b_t && !(d.conv_c > 0 && d.a_t) && d.ldb < ((d.N + 7) & ~7)) return hipErrorInvalidValue;
  if (d.bias && !aligned(d.bias, 8)) return hipErrorInvalidValue;
  const bool conv = d.conv_c > 0;
  const bool conv_dw = conv && d.a_t && d.b_t;
  const int taps2 = d.conv_taps * d.conv_taps;
  int conv_ho = 0, conv_wo = 0;
  const bool stem = conv && d.conv_taps == 7;
  if (stem) {   // padded image [.., conv_h, conv_w, 4]; the window is widened to 8 x 8
    if (d.conv_c != 4 || d.conv_stride != 2 || d.conv_h < 8 || d.conv_w < 8 || (d.conv_w & 1) || d.conv_h > 4095 || d.conv_w > 4095 ||
        d.z_outer != 1 || d.z_inner != 1)
      return hipErrorInvalidValue;
    conv_ho = (d.conv_h - 8) / 2 + 1;
    conv_wo = (d.conv_w - 8) / 2 + 1;
    if (conv_dw ? (d.N != 256 || (d.K % (conv_ho * conv_wo)) || (d.K % gemm::PBK) || !d.c_f32)
                : (d.K != 256 || (d.M % (conv_ho * conv_wo)) || d.a_t || d.b_t || d.split_k > 1 || d.mode != EPI_PLAIN || !d.c_f32 ||
                   d.residual))
      return hipErrorInvalidValue;
  } else if (conv) {
    if ((d.conv_taps != 1 && d.conv_taps != 3) || (d.conv_stride != 1 && d.conv_stride != 2) || d.conv_h < 1 || d.conv_w < 1 ||
        d.conv_h > 4095 || d.conv_w > 4095)
      return hipErrorInvalidValue;
    conv_ho = (d.conv_h - 1) / d.conv_stride + 1;
    conv_wo = (d.conv_w - 1) / d.conv_stride + 1;
  }
  if (stem) {
  } else if (conv_dw) {   // B is the activation; the reduction runs over the output pixels
    if ((d.conv_c & 7) || d.N != taps2 * d.conv_c || (d.K % (conv_ho * conv_wo)) || d.z_outer != 1 || d.z_inner != 1 || !d.c_f32)
      return hipErrorInvalidValue;
  } else if (conv) {
    if ((d.conv_c % gemm::PBK) || d.K != taps2 * d.conv_c || (d.M % (conv_ho * conv_wo)) || d.a_t || d.b_t || d.z_outer != 1 ||
        d.z_inner != 1)
      return hipErrorInvalidValue;
    // a split reduction finishes in a second kernel that applies the epilogue: outputs without padding
    if (d.split_k > 1 && (!d.partials || !aligned(d.partials, 16) || d.ldc != d.N || (d.N & 3) || d.c_f32 || d.residual ||
                          d.alpha != 1.f || d.mode == EPI_AFFINE_ADD_RELU || d.mode == EPI_GELU_FWD || d.mode == EPI_GELU_BWD ||
                          d.mode == EPI_GELU_ONLY || (d.mode == EPI_PLAIN && d.bias)))
      return hipErrorInvalidValue;
    if (d.split_k > 1 && ((d.mode == EPI_AFFINE_RELU && (!d.C2 || !d.gain || !d.bias || !aligned(d.C2, 8) || !aligned(d.gain, 8))) ||
                          (d.mode == EPI_RELU_MASK && (!d.U || !aligned(d.U, 8))) || (d.mode == EPI_BIAS_RELU && !d.bias)))
      return hipErrorInvalidValue;
  }
  if (conv && !conv_dw && !stem && (d.tile == CONV_TILE_HALO || d.tile == CONV_TILE_RASTER || d.tile == CONV_TILE_RASTER_256)) {
    const hipError_t e = d.tile == CONV_TILE_HALO ? conv_halo(d, s) : conv_raster(d, s);   // (each checks its own requirements)
    if (e == hipSuccess && launches) *launches = 1;
    return e;
  }
  const bool conv_split = conv && !conv_dw && d.split_k > 1;
  if (d.residual && (d.ldr < d.N || (d.ldr & 3) || !aligned(d.residual, 16))) return hipErrorInvalidValue;

  gemm::Params p;
  p.A = d.A; p.B = d.B; p.M = d.M; p.N = d.N; p.K = d.K; p.lda = d.lda; p.ldb = d.ldb;
  p.z_inner = d.z_inner;
  p.sAo = d.sAo; p.sAi = d.sAi; p.sBo = d.sBo; p.sBi = d.sBi; p.sCo = d.sCo; p.sCi = d.sCi;
  p.split_k = 1; p.k_chunk = 0;
  p.alpha = d.alpha; p.bias = d.bias; p.gain = d.gain; p.gain2 = d.gain2; p.bias2 = d.bias2; p.residual = d.residual; p.ldr = d.ldr;
  p.C = d.C; p.ldc = d.ldc; p.C2 = d.C2; p.U = d.U;
  p.cH = d.conv_h; p.cW = d.conv_w; p.cC = d.conv_c;
  p.cT = stem ? 8 : d.conv_taps; p.cS = d.conv_stride; p.cHo = conv_ho; p.cWo = conv_wo;
  p.act_lo = d.act_lo; p.act_hi = d.act_hi; p.mask_hi = d.mask_hi;
  p.colsum = d.colsum;
  int zdim = d.z_outer * d.z_inner;
  int epi;
  int k_per_block = d.K;
  if (d.split_k > 1) {
    if (!conv_split && (zdim != 1 || !d.partials || !d.c_f32 || d.bias || d.residual || d.mode != EPI_PLAIN || d.alpha != 1.f ||
                        d.ldc != d.N || (d.N & 3) || !aligned(d.partials, 16)))
      return hipErrorInvalidValue;
    const int slices = (d.K + gemm::SBK - 1) / gemm::SBK;
    const int per = (slices + d.split_k - 1) / d.split_k;
    p.k_chunk = per * gemm::SBK;
    p.split_k = (slices + per - 1) / per;  // no empty chunks
    k_per_block = p.k_chunk;
  }
  if (p.split_k > 1) {
    p.C = d.partials;
    zdim = p.split_k;
    epi = gemm::E_PARTIAL;
  } else {
    p.split_k = 1;
    if (d.ldc < d.N || (d.ldc & 3)) return hipErrorInvalidValue;
    if (d.mode == EPI_GELU_FWD) {
      if (!d.C2 || d.c_f32 || d.residual || !aligned(d.C2, 8)) return hipErrorInvalidValue;
      epi = gemm::E_GELU_FWD;
    } else if (d.mode == EPI_BIAS_RELU) {
      if (d.c_f32 || d.residual || d.a_t || d.b_t) return hipErrorInvalidValue;
      epi = gemm::E_BIAS_RELU;
    } else if (d.mode == EPI_GELU_ONLY) {
      if (d.c_f32 || d.residual || d.a_t || d.b_t) return hipErrorInvalidValue;
      epi = gemm::E_GELU_ONLY;
    } else if (d.mode == EPI_AFFINE_RELU) {
      if (!d.C2 || !d.gain || !d.bias || d.c_f32 || d.residual || d.a_t || d.b_t || !aligned(d.C2, 8)) return hipErrorInvalidValue;
      epi = gemm::E_AFFINE;
    } else if (d.mode == EPI_AFFINE_ADD_RELU) {
      if (!d.C2 || !d.gain || !d.bias || !d.U || (d.gain2 && !d.bias2) || d.c_f32 || d.residual || d.a_t || d.b_t ||
          !aligned(d.C2, 8) || !aligned(d.U, 8))
        return hipErrorInvalidValue;
      epi = gemm::E_AFFINE_ADD;
    } else if (d.mode == EPI_RELU_MASK) {
      if (!d.U || d.c_f32 || d.residual || d.bias || !aligned(d.U, 8)) return hipErrorInvalidValue;
      epi = gemm::E_RELU_MASK;
    } else if (d.mode == EPI_GELU_BWD) {
      if (!d.U || d.c_f32 || d.residual || d.bias || !aligned(d.U, 8) || (d.colsum && zdim != 1)) return hipErrorInvalidValue;
      epi = gemm::E_GELU_BWD;
    } else if (d.c_f32) {
      epi = d.residual ? gemm::E_F32_RES : gemm::E_F32;
    } else {
      if (d.residual) return hipErrorInvalidValue;
      epi = gemm::E_BF16;
    }
  }
  int BM, BN;
  gemm::LaunchFn fn;
  const bool conv_general = conv && !(d.conv_taps == 3 && d.conv_stride == 1);   // geometry as launch arguments
  bool resident = true;   // the two-group kernels keep one workgroup per CU that walks over the tiles
  if (conv_dw && !stem && (d.tile == T_RING_64x64 || d.tile == T_RING_64x128 || d.tile == T_RING_128x64)) {
    BM = d.tile == T_RING_128x64 ? 128 : 64; BN = d.tile == T_RING_64x128 ? 128 : 64; resident = false;
    fn = d.tile == T_RING_64x64 ? gemm::ring_convdw_64x64(epi) : d.tile == T_RING_64x128 ? gemm::ring_convdw_64x128(epi) : gemm::ring_convdw_128x64(epi);
  } else if (conv_dw) {
    if (d.K % gemm::PBK) return hipErrorInvalidValue;
    int tile = d.tile;
    if (tile != T_PP_256x256 && tile != T_PP_256x192 && tile != T_PP_128x256 && tile != T_PP_64x512) {
      if (tile != T_AUTO && d.split_k > 1) return hipErrorInvalidValue;   // (a split belongs to the tile that it was planned with)
      tile = plan_conv_dw(d.M, d.N, k_per_block).tile;
    }
    switch (tile) {
      case T_PP_64x512: BM = 64; BN = 512; fn = gemm::pp_convdw_64x512(epi, conv_general); break;
      case T_PP_128x256: BM = 128; BN = 256; fn = gemm::pp_convdw_128x256(epi, conv_general); break;
      case T_PP_256x192: BM = 256; BN = 192; fn = gemm::pp_convdw_256x192(epi, conv_general); break;
      default: BM = 256; BN = 256; fn = gemm::pp_convdw_256x256(epi, conv_general); break;
    }
  } else if (stem) {   // few output channels, fp32 result
    BM = 512; BN = 64; fn = gemm::pp_conv_512x64(epi, conv_general);
  } else if (conv) {
    switch (choose_conv_tile(d)) {
      case T_RING_64x64: BM = 64; BN = 64; fn = gemm::ring_conv_64x64(epi); resident = false; break;
      case T_RING_64x128: BM = 64; BN = 128; fn = gemm::ring_conv_64x128(epi); resident = false; break;
      case T_RING_128x64: BM = 128; BN = 64; fn = gemm::ring_conv_128x64(epi); resident = false; break;
      case T_RING_128x128: BM = 128; BN = 128; fn = gemm::ring_conv_128x128(epi); resident = false; break;
      case T_PP_512x64: BM = 512; BN = 64; fn = gemm::pp_conv_512x64(epi, conv_general); break;
      case T_PP_256x128: BM = 256; BN = 128; fn = gemm::pp_conv_256x128(epi, conv_general); break;
      case T_PP_256x192: BM = 256; BN = 192; fn = gemm::pp_conv_256x192(epi, conv_general); break;
      default: BM = 256; BN = 256; fn = gemm::pp_conv_256x256(epi, conv_general); break;
    }
  } else
  switch (choose_tile(d, k_per_block)) {
    case T_PP_64x512: BM = 64; BN = 512; fn = gemm::pp_64x512(d.a_t, d.b_t, epi); break;
    case T_PP_128x256: BM = 128; BN = 256; fn = gemm::pp_128x256(d.a_t, d.b_t, epi); break;
    case T_PP_512x64: BM = 512; BN = 64; fn = gemm::pp_512x64(d.a_t, d.b_t, epi); break;
    case T_128x64: BM = 128; BN = 64; fn = gemm::staged_128x64(d.a_t, d.b_t, epi); resident = false; break;
    case T_RING_64x64: BM = 64; BN = 64; fn = gemm::ring_64x64(d.a_t, d.b_t, epi); resident = false; break;
    case T_RING_64x128: BM = 64; BN = 128; fn = gemm::ring_64x128(d.a_t, d.b_t, epi); resident = false; break;
    case T_RING_128x128: BM = 128; BN = 128; fn = gemm::ring_128x128(d.a_t, d.b_t, epi); resident = false; break;
    case T_DMA_256x256: BM = 256; BN = 256; fn = gemm::dma_256x256(d.a_t, d.b_t, epi); resident = false; break;
    case T_DMA_256x128: BM = 256; BN = 128; fn = gemm::dma_256x128(d.a_t, d.b_t, epi); resident = false; break;
    case T_DIRECT_256x256: BM = 256; BN = 256; fn = gemm::direct_256x256(d.a_t, d.b_t, epi); break;
    case T_DIRECT_192x256: BM = 192; BN = 256; fn = gemm::direct_192x256(d.a_t, d.b_t, epi); break;
    case T_DIRECT_128x256: BM = 128; BN = 256; fn = gemm::direct_128x256(d.a_t, d.b_t, epi); break;
    default: BM = 128; BN = 128; fn = gemm::staged_128x128(d.a_t, d.b_t, epi); resident = false; break;
  }
  // a lone 64x64 tile per CU with a long reduction waits for memory: five slices in flight instead of three.  [788 x 768 x 3072] with weights
  // from memory 14.3 -> 13.3 us, with both operands from memory 14.4 -> 13.3; the same times a transposed weight 13.6 -> 13.4 and 13.9 -> 13.3,
  // x 2304 10.9 -> 11.0 and 11.3 -> 11.1, in a training pass 11.9 -> 11.1.  At 32 slices 10.2 -> 10.2 and 10.6 -> 10.3, transposed 10.1 -> 10.3
  // and 10.4 -> 10.4, hence the later start there.  With both operands in the L2, which no pass over a model leaves, it costs 4 - 6 %; so does
  // the LDS that it takes with two or more tiles per CU ([788 x 3072 x 768] 12.4 -> 13.7)
  if (fn && !conv && BM == 64 && BN == 64 && !resident && k_per_block >= (d.b_t ? 36 : 32) * gemm::PBK &&
      (long long)((d.M + 63) / 64) * ((d.N + 63) / 64) * zdim <= 256) {
    const gemm::LaunchFn deep = gemm::ring_64x64_deep(d.a_t, d.b_t, epi);
    if (deep) fn = deep;
  }
  if (!fn) return hipErrorInvalidValue;  // this (layout, epilogue) pair is not part of the training step
  const int tiles = ((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN);
  if ((long long)tiles * zdim >= (1ll << 23)) return hipErrorInvalidValue;   // (the resident kernels' unit arithmetic)
  p.units = tiles * zdim;
  // resident kernels: every workgroup takes the same number of units (600 tiles run as 200 workgroups of 3 rather than
  // 256 of 2 or 3: the launch takes 3 tile times either way, and the CUs left idle lower the load the others run under)
  int resident_grid = p.units;
  const int cus = compute_units();
  if (resident_grid > cus) {
    const int rounds = (p.units + cus - 1) / cus;
    resident_grid = std::min(cus, ((p.units + rounds - 1) / rounds + 7) & ~7);
  }
  hipError_t e = resident ? fn(p, dim3(resident_grid, 1, 1), s) : fn(p, dim3(tiles, 1, zdim), s);
  if (e != hipSuccess) return e;
  if (launches) *launches = 1;
  if (p.split_k > 1 && conv_split) {
    ReduceEpi r;
    r.part = (const float4*)d.partials; r.n4 = (size_t)d.M * d.N / 4; r.splits = p.split_k; r.N = d.N;
    r.mode = d.mode == EPI_BIAS_RELU ? 1 : d.mode == EPI_RELU_MASK ? 2 : d.mode == EPI_AFFINE_RELU ? 3 : 0;
    r.bias = d.bias; r.gain = d.gain; r.U = d.U;
    r.out = d.mode == EPI_AFFINE_RELU ? d.C2 : (bf16*)d.C;
    r.zout = d.mode == EPI_AFFINE_RELU ? (bf16*)d.C : nullptr;
    r.lo = d.act_lo; r.hi = d.act_hi; r.mask_hi = d.mask_hi;
    hipLaunchKernelGGL(splitk_reduce_epilogue_kernel, dim3((unsigned)((r.n4 + 255) / 256)), dim3(256), 0, s, r);
    e = hipGetLastError();
    if (launches) *launches = 2;
  } else if (p.split_k > 1) {
    const size_t n4 = (size_t)d.M * d.N / 4;
    if (p.split_k > 32)
      hipLaunchKernelGGL(splitk_reduce_wide_kernel, dim3((unsigned)((n4 + 15) / 16)), dim3(256), 0, s,
                         (const float4*)d.partials, (float4*)d.C, n4, p.split_k);
    else
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                         (const float4*)d.partials, (float4*)d.C, n4, p.split_k);
    e = hipGetLastError();
    if (launches) *launches = 2;
  }
  return e;
}

}  // namespace et
