// LDS layout, MFMA fragments and row stores shared by the attention kernels (head size 64): attention.hip holds a whole
// head on chip, attention_long.hip streams one through LDS in chunks of 64 rows.
#pragma once
#include "kernels.h"

namespace et {
namespace attn {

typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int DH = 64;
// LDS rows are the 128 bytes of 64 bf16 without padding; the 16-byte chunk c of row r sits at chunk position
// c ^ swz(r).  Every tile is read two ways and both must spread over the 64 banks:
//   - row-major fragments (ds_read_b128, 16 consecutive rows x one chunk per 16 lanes): rows alternate between the
//     two 128-byte halves of the 256-byte bank span, so the 8 even rows of a group need 8 different positions;
//   - transposing fragments (ds_read_b64_tr_b16, 4 consecutive rows x 64 contiguous bytes per 32 lanes): rows
//     r and r + 2 share a half, so their 64-byte pieces must land in different quarters.
// swz(r) = bit 1 of r as the high bit, bits 2..3 of r as the low bits, does both (a plain (r >> 1) & 7 leaves the
// transposing reads two-way conflicted, as did padded rows of 160 bytes: 41-45 % conflict cycles measured).
constexpr int PITCH = 128;
__device__ __forceinline__ int swz(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

__device__ __forceinline__ bf16x4 lds_read_tr(const unsigned char* p) {
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
  return __builtin_bit_cast(bf16x4, v);
}

// A- or B-operand fragment of rows [row0, row0+32) for reduction slice ks (16 of the 64 columns):
// lane l gets row row0 + l%32, columns ks*16 + (l/32)*8 .. +7
__device__ __forceinline__ bf16x8 frag_direct(const unsigned char* m, int row0, int ks, int lane) {
  const int row = row0 + (lane & 31);
  return *(const bf16x8*)(m + row * PITCH + (((ks * 2 + (lane >> 5)) ^ swz(row)) << 4));
}

// B-operand fragment for a reduction over ROWS of a matrix stored [row][64]: lane l gets column
// col0 + l%32 and the 8 rows  row0 + (e/4)*8 + (l/32)*4 + e%4  (e = 0..7)
__device__ __forceinline__ bf16x8 frag_rows_tr(const unsigned char* m, int row0, int col0, int lane) {
  const int g = lane >> 4, r16 = lane & 15;
  // (rows r and r + 8 differ in bit 3, which is bit 1 of swz: the second address is computed on its own)
  const int row = row0 + (g >> 1) * 4 + (r16 >> 2);
  const int byte = (col0 + (g & 1) * 16 + 4 * (r16 & 3)) * 2;      // 8-byte piece inside the logical row
  const int chunk = byte >> 4, half = byte & 8;
  const unsigned char* p = m + row * PITCH + ((chunk ^ swz(row)) << 4) + half;
  const unsigned char* p8 = m + (row + 8) * PITCH + ((chunk ^ swz(row + 8)) << 4) + half;
  const bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p8);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// element r of an MFMA result tile: row offset inside the 32x32 tile
__device__ __forceinline__ int tile_row(int r, int lane) { return (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3); }

// Store a 32 x 64 result tile (lane = row l%32, registers t[dt][a*4 + e] = column dt*32 + a*8 + (l/32)*4 + e), times
// `mul`, as bf16 rows of `ld` elements starting at `base` (row 0 of the tile), rows >= `rows` left out.  Straight
// from the registers a store instruction would put 16 bytes into each of 32 rows (8-byte pieces of two lanes);
// written that way the 19 MB of a ViT-B forward output cost 6 us.  The tile goes through a wave-private 4 KiB LDS
// area instead (16-byte chunks XORed with (row >> 1) & 7: even and odd rows lie in different halves of the 256-byte
// bank span, so 16 consecutive rows of one column are spread over all 64 banks) and
// leaves as whole 128-byte rows, 8 lanes x 16 bytes each.  LDS instructions of one wave execute in order, so no
// barrier is needed between the writes and the reads, nor between two tiles through the same area.
constexpr int STORE_AREA = 32 * 128;
// `sums` (nullable, wave-private, in LDS): receives the column sums of the stored rows, 64 floats, as rounded.  Each lane adds the
// pieces it stores, then the eight lanes of a column share out the adding (7 shuffles).  With the addition over the waves the sums
// lengthen a backward launch of 64 x 12 heads from 64.6 to 68.6 us (as 32 two-byte LDS reads per column to 71); another
// pass over dQ, dK and dV took 8.5 to 11 and a launch.
__device__ __forceinline__ void store_tile(unsigned char* area, const f32x16 (&t)[2], float mul, bf16* base, long long ld,
                                           int rows, int lane, float* sums = nullptr) {
  asm volatile("" : "+v"(lane));   // (addresses below are computed here, not kept live through the caller's main loop)
  const int l32 = lane & 31, khalf = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; e++) v[e] = (bf16)(t[dt][a * 4 + e] * mul);
      *(bf16x4*)(area + l32 * 128 + (((dt * 4 + a) ^ ((l32 >> 1) & 7)) << 4) + khalf * 8) = v;
    }
  float s8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int row = i * 8 + (lane >> 3), chunk = lane & 7;
    const bf16x8 v = *(const bf16x8*)(area + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
    if (row < rows) *(bf16x8*)(base + row * ld + chunk * 8) = v;
    if (sums && row < rows)
#pragma unroll
      for (int e = 0; e < 8; e++) s8[e] += (float)v[e];
  }
  if (!sums) return;
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
  float s4[4], s2[2];
#pragma unroll
  for (int e = 0; e < 4; e++) s4[e] = (b5 ? s8[e + 4] : s8[e]) + __shfl_xor(b5 ? s8[e] : s8[e + 4], 32, 64);
#pragma unroll
  for (int e = 0; e < 2; e++) s2[e] = (b4 ? s4[e + 2] : s4[e]) + __shfl_xor(b4 ? s4[e] : s4[e + 2], 16, 64);
  const float s1 = (b3 ? s2[1] : s2[0]) + __shfl_xor(b3 ? s2[0] : s2[1], 8, 64);
  sums[(lane & 7) * 8 + (b5 ? 4 : 0) + (b4 ? 2 : 0) + (b3 ? 1 : 0)] = s1;
}

// 16 bytes per lane from global memory straight into LDS at (base in M0) + 16 * lane
__device__ __forceinline__ void dma16(const void* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(gptr) : "memory");
}

}  // namespace attn
}  // namespace et
