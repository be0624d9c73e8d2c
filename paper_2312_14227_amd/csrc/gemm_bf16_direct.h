// Two-group kernel with operands loaded straight to LDS: the large plain products (K a multiple of 64; weight gradients over any number of rows).
//
// The schedule is that of gemm_pp_kernel (gemm_bf16_kernels.h): eight waves in two groups of one wave per SIMD, which alternate
// every barrier interval between the matrix instructions of half a slice of 64 k values and fetching the fragments of the
// next half.  The slices travel by global_load_lds_dwordx4: no registers hold operands in flight, nothing is stored to LDS, and a wave requests
// its pieces in its fetching phases, where a full address queue stalls no matrix instruction.  A CU takes 10 ns for a wave-wide load of
// 1 KB, so the 64 loads of a slice are spread evenly over its four intervals.  Measured on one CU, clocks per interval of 512 matrix clocks:
// 580 (registers and LDS stores: 643; requests between the matrix instructions 674, all of them in two of the four intervals 761).  Tile
// 256 x 256, K = 768: 1.0 - 1.1 us per slice with all CUs at work against 1.3 - 1.4.
//
// One tile is 64 MI x 256 (MI = 4, 3, 2), the waves 2 x 4, each 32 MI x 64; three stages of the A operand, two of B.  In intervals, with the
// fetching phase M(t, h) and the multiplication C(t, h) of half h of slice t:
//   group 0:  M(t,0) 4t | C(t,0) 4t+1 | M(t,1) 4t+2 | C(t,1) 4t+3           group 1: one interval later
// A stage of slice t is read for the last time in interval 4t + 3.  M(t,0) requests B(t + 1) into the stage of B(t - 1), M(t,1) requests A(t + 2) into
// that of A(t - 1); slice t + 1 is waited for at the end of interval 4t + 3 with the A requests of M(t,1) left in flight.  Slices are
// counted through all the units of work of a resident workgroup, so the first slices of the next tile arrive under the last
// multiplications and the epilogue of the current one, whose staging area is the A stage of the last slice t (requested again in M(t+1,1), a
// barrier after the last wave has left the epilogue).  The groups meet for the epilogue, so that its instructions and waits overlap.
#pragma once
#include "gemm_bf16_kernels.h"

namespace et {
namespace gemm {

__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const unsigned long long v = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (const char*)(((unsigned long long)hi << 32) | lo);
}

// 16 bytes per lane to LDS (lds_base + 16 * lane) from base + off, both bases the same for all lanes
__device__ __forceinline__ void dma16_off(unsigned off, const void* base, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(off),
               "s"(uniform_ptr(base))
               : "memory");
}

// Epilogue of one wave with 4 KB of staging: 32 rows of 128 bytes, i.e. 64 columns of bf16 or 32 of fp32, the eight 16-byte chunks of
// row r XORed with (r >> 1) & 7 (no bank conflicts either way).  The accumulators' layout is that of wave_epilogue_impl; every global access is a
// whole 128-byte line of 8 rows per instruction.  A second operand in bf16 (GELU backward, a block's other branch) goes through the same area first.
constexpr int kEpiStage = 4096;

template <int EPI, int MI, bool FULL>
__device__ __forceinline__ void direct_epilogue(const Params& g, f32x16 (&acc)[MI][2], unsigned char* stage, int row0, int col0, long long c_off,
                                                int lane) {
  const int l32 = lane & 31, khalf = lane >> 5, r8 = lane >> 3, c8 = lane & 7;
  const int ld = EPI == E_PARTIAL ? g.N : g.ldc;
  const auto at = [&](int row, int chunk) { return stage + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); };
  if constexpr (EPI != E_F32 && EPI != E_F32_RES && EPI != E_PARTIAL) {
    constexpr bool TWO = EPI == E_GELU_FWD || EPI == E_AFFINE || EPI == E_AFFINE_ADD, HAS_U = EPI == E_GELU_BWD || EPI == E_AFFINE_ADD;
    constexpr bool AFFINE = EPI == E_AFFINE || EPI == E_AFFINE_ADD;
    bf16x4 bias_q[2][4], gain_q[AFFINE ? 2 : 1][4], bias2_q[EPI == E_AFFINE_ADD ? 2 : 1][4], gain2_q[EPI == E_AFFINE_ADD ? 2 : 1][4];
    const bool has_bias = EPI != E_GELU_BWD && g.bias != nullptr;
    const bool keep_c = !AFFINE || g.C != nullptr;   // z is kept only if the gain's gradient will be computed
#pragma unroll
    for (int ni = 0; ni < 2; ni++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int col = col0 + ni * 32 + q * 8 + khalf * 4;
        auto four = [&](const bf16* p, float otherwise) {
          bf16x4 b;
#pragma unroll
          for (int j = 0; j < 4; j++) b[j] = (bf16)otherwise;
          if (p) {
            if (FULL || col + 3 < g.N) {
              b = *(const bf16x4*)(p + col);
            } else {
              for (int j = 0; j < 4 && col + j < g.N; j++) b[j] = p[col + j];
            }
          }
          return b;
        };
        bias_q[ni][q] = four(has_bias ? g.bias : nullptr, 0.f);
        if constexpr (AFFINE) gain_q[ni][q] = four(g.gain, 1.f);
        if constexpr (EPI == E_AFFINE_ADD) {
          gain2_q[ni][q] = four(g.gain2, 1.f);
          bias2_q[ni][q] = four(g.gain2 ? g.bias2 : nullptr, 0.f);
        }
      }
    const int col = col0 + c8 * 8;
    const bool wide = FULL || (col + 7 < g.N && (ld & 7) == 0 && (c_off & 7) == 0 && ((uintptr_t)g.C & 15) == 0 && ((uintptr_t)g.C2 & 15) == 0 &&
                               ((uintptr_t)g.U & 15) == 0);
    // the 32 rows in the staging area to out, 8 columns per lane
    auto rows_out = [&](bf16* out, int row, bf16x8 (&v)[4]) {
      constexpr int TURN = TWO ? 2 : 4;   // (rows of both outputs at once would spill)
#pragma unroll
      for (int t = 0; t < 4; t += TURN) {
#pragma unroll
        for (int it = t; it < t + TURN; it++) v[it] = *(const bf16x8*)at(it * 8 + r8, c8);
#pragma unroll
        for (int it = t; it < t + TURN; it++) {
          const int r = row + it * 8 + r8;
          if (!FULL && r >= g.M) continue;
          bf16* p = out + c_off + (long long)r * ld + col;
          if (wide) {
            *(bf16x8*)p = v[it];
          } else {
#pragma unroll
            for (int j = 0; j < 8; j++)
              if (col + j < g.N) p[j] = v[it][j];
          }
        }
        if (TURN < 4) __builtin_amdgcn_sched_barrier(0);
      }
    };
    bf16x8 u[4];
    auto load_u = [&](int row) {
#pragma unroll
      for (int it = 0; it < 4; it++) {
        const int r = row + it * 8 + r8;
        bf16x8 v = {};
        if (FULL || r < g.M) {
          const bf16* p = g.U + c_off + (long long)r * ld + col;
          if (wide) {
            v = *(const bf16x8*)p;
          } else {
#pragma unroll
            for (int j = 0; j < 8; j++)
              if (col + j < g.N) v[j] = p[j];
          }
        }
        u[it] = v;
      }
    };
    if (HAS_U) load_u(row0);
#pragma unroll
    for (int mi = 0; mi < MI; mi++) {
      bf16x4 second[TWO ? 8 : 1];
      bf16x4 uq[HAS_U ? 8 : 1];
      if constexpr (HAS_U) {
#pragma unroll
        for (int it = 0; it < 4; it++) *(bf16x8*)at(it * 8 + r8, c8) = u[it];
        if (mi + 1 < MI) load_u(row0 + (mi + 1) * 32);
#pragma unroll
        for (int k = 0; k < 8; k++) uq[k] = *(const bf16x4*)(at(l32, k) + khalf * 8);
      }
      if constexpr (EPI == E_AFFINE_ADD) {   // (kept packed: as floats the four sets would take 128 registers)
#pragma unroll
        for (int k = 0; k < 8; k++) {
          asm volatile("" : "+v"(bias_q[k >> 2][k & 3]), "+v"(gain_q[k >> 2][k & 3]));
          asm volatile("" : "+v"(bias2_q[k >> 2][k & 3]), "+v"(gain2_q[k >> 2][k & 3]));
        }
      }
#pragma unroll
      for (int ni = 0; ni < 2; ni++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          bf16x4 o;
#pragma unroll
          for (int j = 0; j < 4; j++) {
            const float a = acc[mi][ni][q * 4 + j];
            if constexpr (EPI == E_GELU_BWD) {
              o[j] = (bf16)(a * g.alpha * (float)uq[ni * 4 + q][j]);
            } else if constexpr (AFFINE) {
              o[j] = (bf16)(a * g.alpha);
              float y = (float)o[j] * (float)gain_q[ni][q][j] + (float)bias_q[ni][q][j];
              if constexpr (EPI == E_AFFINE_ADD) y += (float)uq[ni * 4 + q][j] * (float)gain2_q[ni][q][j] + (float)bias2_q[ni][q][j];
              second[ni * 4 + q][j] = (bf16)fminf(fmaxf(y, g.act_lo), g.act_hi);
            } else {
              const float v = a * g.alpha + (float)bias_q[ni][q][j];
              if (EPI == E_GELU_FWD) {
                float gv, dgv;
                gelu_both(v, gv, dgv);
                o[j] = (bf16)dgv;
                second[TWO ? ni * 4 + q : 0][j] = (bf16)gv;
              } else if (EPI == E_GELU_ONLY) {
                o[j] = (bf16)gelu_only(v);
              } else if (EPI == E_BIAS_RELU) {
                o[j] = (bf16)fmaxf(v, 0.f);
              } else {
                o[j] = (bf16)v;
              }
            }
          }
          *(bf16x4*)(at(l32, ni * 4 + q) + khalf * 8) = o;   // (LDS operations of one wave complete in order)
          if ((EPI == E_GELU_FWD && q & 1) || EPI == E_AFFINE_ADD) __builtin_amdgcn_sched_barrier(0);   // (few elements at a time: more would spill)
        }
      bf16x8 v[4];
      if (keep_c) rows_out((bf16*)g.C, row0 + mi * 32, v);
      if constexpr (TWO) {
#pragma unroll
        for (int k = 0; k < 8; k++) *(bf16x4*)(at(l32, k) + khalf * 8) = second[k];
        rows_out(g.C2, row0 + mi * 32, v);
      }
      if constexpr (EPI == E_GELU_BWD) {
        // column sums of these 32 rows as rounded: per lane over its 4 rows, then over the 8 lanes of a column, in pairs (one after the other the
        // error is 1.1 - 1.2 times as large)
        if (g.colsum && row0 + mi * 32 < g.M) {
          float s[8];
#pragma unroll
          for (int j = 0; j < 8; j++) {
            float r[4];
#pragma unroll
            for (int it = 0; it < 4; it++) r[it] = FULL || row0 + mi * 32 + it * 8 + r8 < g.M ? (float)v[it][j] : 0.f;
            s[j] = (r[0] + r[1]) + (r[2] + r[3]);
          }
          float* f = (float*)stage;    // [8 lanes of a column][64 columns], 2 KB
          *(float4*)(f + r8 * 64 + c8 * 8) = make_float4(s[0], s[1], s[2], s[3]);
          *(float4*)(f + r8 * 64 + c8 * 8 + 4) = make_float4(s[4], s[5], s[6], s[7]);
          float t[8];
#pragma unroll
          for (int k = 0; k < 8; k++) t[k] = f[k * 64 + lane];
          const float sum = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
          if (FULL || col0 + lane < g.N) g.colsum[(long long)((row0 + mi * 32) >> 5) * g.N + col0 + lane] = sum;
        }
      }
    }
  } else {
    static_assert(EPI == E_F32 || EPI == E_F32_RES || EPI == E_PARTIAL, "epilogue");
    constexpr bool RES = EPI == E_F32_RES;
    constexpr int BLOCKS = MI * 2, AHEAD = RES ? 3 : 1;
    // residual pieces of block b = (mi, ni), requested AHEAD blocks before they are used
    float4 res[AHEAD][4];
    auto load_res = [&](int b) {
      const int col = col0 + (b & 1) * 32 + c8 * 4;
#pragma unroll
      for (int it = 0; it < 4; it++) {
        const int r = row0 + (b >> 1) * 32 + it * 8 + r8;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (FULL || r < g.M) {
          const float* p = g.residual + (long long)r * g.ldr + col;
          if (FULL || col + 3 < g.N) {
            v = *(const float4*)p;
          } else {
            if (col < g.N) v.x = p[0];
            if (col + 1 < g.N) v.y = p[1];
            if (col + 2 < g.N) v.z = p[2];
          }
        }
        res[b % AHEAD][it] = v;
      }
    };
    if (RES) {
#pragma unroll
      for (int b = 0; b < AHEAD; b++) load_res(b);
    }
    float bias[2][4] = {};
    if (EPI != E_PARTIAL && g.bias) {
#pragma unroll
      for (int ni = 0; ni < 2; ni++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const int col = col0 + ni * 32 + c8 * 4 + j;
          if (FULL || col < g.N) bias[ni][j] = (float)g.bias[col];
        }
    }
#pragma unroll
    for (int b = 0; b < BLOCKS; b++) {
      const int mi = b >> 1, ni = b & 1;
#pragma unroll
      for (int q = 0; q < 4; q++)
        *(float4*)at(l32, q * 2 + khalf) = make_float4(acc[mi][ni][q * 4], acc[mi][ni][q * 4 + 1], acc[mi][ni][q * 4 + 2], acc[mi][ni][q * 4 + 3]);
      float4 v[4];
#pragma unroll
      for (int it = 0; it < 4; it++) v[it] = *(const float4*)at(it * 8 + r8, c8);
      const int col = col0 + ni * 32 + c8 * 4;
#pragma unroll
      for (int it = 0; it < 4; it++) {
        const int r = row0 + mi * 32 + it * 8 + r8;
        if (!FULL && r >= g.M) continue;
        float4 x = v[it];
        if (EPI != E_PARTIAL)
          x = make_float4(x.x * g.alpha + bias[ni][0], x.y * g.alpha + bias[ni][1], x.z * g.alpha + bias[ni][2], x.w * g.alpha + bias[ni][3]);
        if (RES) {
          const float4 t = res[b % AHEAD][it];
          x.x += t.x; x.y += t.y; x.z += t.z; x.w += t.w;
        }
        float* p = (float*)g.C + c_off + (long long)r * ld + col;
        if (FULL || col + 3 < g.N) {
          *(float4*)p = x;
        } else {
          if (col < g.N) p[0] = x.x;
          if (col + 1 < g.N) p[1] = x.y;
          if (col + 2 < g.N) p[2] = x.z;
        }
      }
      if (RES && b + AHEAD < BLOCKS) load_res(b + AHEAD);
    }
  }
}

// GROUP: the units are those of a group of weight gradients (AT, BT, E_PARTIAL)
template <int MI, bool AT, bool BT, int EPI, bool GROUP = false>
__global__ __launch_bounds__(512) void gemm_direct_kernel(std::conditional_t<GROUP, GroupParams<false>, Params> g) {
  static_assert(!GROUP || (AT && BT && EPI == E_PARTIAL), "groups of weight gradients");
  constexpr int BM = 64 * MI, BN = 256, NW = 8, NI = 2, TM = 32 * MI, TN = 64;
  constexpr int A_BYTES = BM * PBK * 2, B_BYTES = BN * PBK * 2;
  constexpr int A_LOADS = MI, B_LOADS = 4, LOADS = A_LOADS + B_LOADS;   // wave-wide 1 KiB pieces per wave and slice
  // LDS: three stages of A, two of B, and what the A stages lack for a staging area of 4 KB per wave
  constexpr int B_AT = 3 * A_BYTES, REST_AT = B_AT + 2 * B_BYTES, IN_STAGE = A_BYTES / kEpiStage;
  constexpr int SMEM = REST_AT + (IN_STAGE < NW ? (NW - IN_STAGE) * kEpiStage : 0);
  static_assert(SMEM <= 160 * 1024, "LDS");
  // transposed operands: [64 k-rows][tile width], chunk j of k-row k at j ^ ((k & 3) << shift) (see gemm_pp_kernel)
  constexpr int TSH_A = (BM % 128 == 0) ? 2 : 1, TSH_B = 2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave >> 2, wave_n = wave & 3, group = wave_m;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  // where unit w lies: tile corner, operands, offset of the result, number of slices and k values of the last one, all uniform
  struct Unit { int m0, n0, k_begin, nk, rem, M, N, lda, ldb; const bf16 *A, *B; long long c_off; void* C; };
  auto unit = [&](int w) {
    Unit u;
    int z, k_end;
    if constexpr (GROUP) {
      const int at = __builtin_amdgcn_readfirstlane(group_unit(w, (int)gridDim.x, g.units));
      const GroupJob& j = g.job[__builtin_amdgcn_readfirstlane(group_job<false>(g, at))];
      u.M = j.M; u.N = j.N; u.lda = j.lda; u.ldb = j.ldb; u.A = j.A; u.B = j.B; u.C = j.C;
      group_tile<BM, BN>(u.M, u.N, at - j.unit0, u.m0, u.n0, z);
      z = __builtin_amdgcn_readfirstlane(z);
      u.k_begin = z * j.k_chunk;
      k_end = min(j.K, u.k_begin + j.k_chunk);
      u.c_off = (long long)z * u.M * u.N;
    } else {
      u.M = g.M; u.N = g.N; u.lda = g.lda; u.ldb = g.ldb; u.C = g.C;
      unit_coords<BM, BN>(g, w, u.m0, u.n0, z);
      z = __builtin_amdgcn_readfirstlane(z);
      batch_offsets(g, z, u.A, u.B, u.c_off, u.k_begin, k_end);
    }
    u.m0 = __builtin_amdgcn_readfirstlane(u.m0);
    u.n0 = __builtin_amdgcn_readfirstlane(u.n0);
    u.nk = (k_end - u.k_begin + PBK - 1) / PBK;
    u.rem = k_end - u.k_begin - (u.nk - 1) * PBK;
    return u;
  };
  // The next slice of either operand to request: its unit (>= g.units: nothing left), position and how many follow it in that unit
  // (uniform), and per lane the byte offsets of this wave's pieces.  (Lane-dependent values come from an opaque copy of the thread index: they
  // are recomputed per unit instead of kept in registers.)
  int a_w = blockIdx.x, b_w = blockIdx.x, a_left, b_left, a_rem, b_rem;
  const char *pa, *pb;
  long long a_step, b_step;
  unsigned oa[A_LOADS], ob[B_LOADS];
  auto setup_a = [&]() {
    const Unit u = unit(a_w);
    a_left = u.nk;
    a_rem = u.rem;
    pa = uniform_ptr(AT ? u.A + (long long)u.k_begin * u.lda : u.A + (long long)u.m0 * u.lda + u.k_begin);
    a_step = (AT ? (long long)PBK * u.lda : PBK) * 2;
    int s_tid = tid;
    asm volatile("" : "+v"(s_tid));
    const int lane = s_tid & 63;
#pragma unroll
    for (int i = 0; i < A_LOADS; i++) {
      const int q = wave * A_LOADS + i;
      if (!AT) {   // 8 rows x 128 B; 16-byte chunk c of row r lands at chunk position c ^ ((r >> 1) & 7)
        const int row = q * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
        oa[i] = (unsigned)(min(row, u.M - 1 - u.m0) * u.lda + chunk * 8) * 2u;
      } else {
        const int pos = q * 64 + lane, k = pos / (BM / 8), j = (pos % (BM / 8)) ^ ((k & 3) << TSH_A);
        int gi = u.m0 + j * 8;
        if (gi + 8 > ((u.M + 7) & ~7)) gi = 0;
        oa[i] = (unsigned)(k * u.lda + gi) * 2u;
      }
    }
  };
  auto setup_b = [&]() {
    const Unit u = unit(b_w);
    b_left = u.nk;
    b_rem = u.rem;
    pb = uniform_ptr(BT ? u.B + (long long)u.k_begin * u.ldb : u.B + (long long)u.n0 * u.ldb + u.k_begin);
    b_step = (BT ? (long long)PBK * u.ldb : PBK) * 2;
    int s_tid = tid;
    asm volatile("" : "+v"(s_tid));
    const int lane = s_tid & 63;
#pragma unroll
    for (int i = 0; i < B_LOADS; i++) {
      const int q = wave * B_LOADS + i;
      if (!BT) {
        const int row = q * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
        ob[i] = (unsigned)(min(row, u.N - 1 - u.n0) * u.ldb + chunk * 8) * 2u;
      } else {
        const int pos = q * 64 + lane, k = pos / (BN / 8), j = (pos % (BN / 8)) ^ ((k & 3) << TSH_B);
        int gj = u.n0 + j * 8;
        if (gj + 8 > ((u.N + 7) & ~7)) gj = 0;
        ob[i] = (unsigned)(k * u.ldb + gj) * 2u;
      }
    }
  };
  // one 1 KiB piece of the next slice into a stage (0..2 of A, 0..1 of B); then on to the slice after it, of this unit or the next
  auto piece_a = [&](int j, int stage) { dma16_off(oa[j], pa, lds0 + stage * A_BYTES + (wave * A_LOADS + j) * 1024); };
  auto piece_b = [&](int j, int stage) { dma16_off(ob[j], pb, lds0 + B_AT + stage * B_BYTES + (wave * B_LOADS + j) * 1024); };
  // the same in a last slice of fewer than 64 k values (weight gradients, over any number of rows): zeros beyond them
  constexpr bool RAGGED = AT && BT;
  auto tail_a = [&](int j, int stage) {
    const int k = ((wave * A_LOADS + j) * 64 + lane) / (BM / 8);
    dma16(k < a_rem ? pa + oa[j] : (const char*)kZeroBlock, __builtin_amdgcn_readfirstlane(lds0 + stage * A_BYTES + (wave * A_LOADS + j) * 1024));
  };
  auto tail_b = [&](int j, int stage) {
    const int k = ((wave * B_LOADS + j) * 64 + lane) / (BN / 8);
    dma16(k < b_rem ? pb + ob[j] : (const char*)kZeroBlock, __builtin_amdgcn_readfirstlane(lds0 + B_AT + stage * B_BYTES + (wave * B_LOADS + j) * 1024));
  };
  auto advance_a = [&]() {
    pa += a_step;
    if (--a_left == 0) {
      a_w += (int)gridDim.x;
      if (a_w < g.units) setup_a();
    }
  };
  auto advance_b = [&]() {
    pb += b_step;
    if (--b_left == 0) {
      b_w += (int)gridDim.x;
      if (b_w < g.units) setup_b();
    }
  };
  // this wave's share of the next slice of an operand; there is one
  auto request_a = [&](int stage) {
    if (RAGGED && a_left == 1 && a_rem < PBK) {
#pragma unroll
      for (int j = 0; j < A_LOADS; j++) tail_a(j, stage);
    } else {
#pragma unroll
      for (int j = 0; j < A_LOADS; j++) piece_a(j, stage);
    }
    advance_a();
  };
  auto request_b = [&](int stage) {
    if (RAGGED && b_left == 1 && b_rem < PBK) {
#pragma unroll
      for (int j = 0; j < B_LOADS; j++) tail_b(j, stage);
    } else {
#pragma unroll
      for (int j = 0; j < B_LOADS; j++) piece_b(j, stage);
    }
    advance_b();
  };

  f32x16 acc[MI][NI];
  const int l32 = lane & 31, khalf = lane >> 5;
  const int grp16 = lane >> 4, r16 = lane & 15;
  const int tr_col = (grp16 & 1) * 16 + 4 * (r16 & 3);
  const int tr_krow = (grp16 >> 1) * 8 + (r16 >> 2);
  const int tr_row = r16 >> 2;

  auto load_a = [&](const unsigned char* st, int ks, int mi) -> bf16x8 {
    const int rbase = wave_m * TM + mi * 32;
    if (!AT) {
      const int row = rbase + l32, chunk = ks * 2 + khalf;
      return *(const bf16x8*)(st + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
    } else {
      const int col = rbase + tr_col;
      const unsigned char* p = st + (ks * 16 + tr_krow) * (BM * 2) + (((col >> 3) ^ (tr_row << TSH_A)) << 4) + ((col >> 2) & 1) * 8;
      bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * (BM * 2));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  auto load_b = [&](const unsigned char* st, int ks, int ni) -> bf16x8 {
    const int rbase = wave_n * TN + ni * 32;
    if (!BT) {
      const int row = rbase + l32, chunk = ks * 2 + khalf;
      return *(const bf16x8*)(st + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
    } else {
      const int col = rbase + tr_col;
      const unsigned char* p = st + (ks * 16 + tr_krow) * (BN * 2) + (((col >> 3) ^ (tr_row << TSH_B)) << 4) + ((col >> 2) & 1) * 8;
      bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * (BN * 2));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  int sa = 0, sb = 0;            // stages of the slice being multiplied
  bf16x8 fa[2][MI], fb[2][NI];   // fragments of the two k-steps of a half slice
  auto fetch = [&](int half) {
    const unsigned char *at = smem + sa * A_BYTES, *bt = smem + B_AT + sb * B_BYTES;
#pragma unroll
    for (int k = 0; k < 2; k++) {
#pragma unroll
      for (int mi = 0; mi < MI; mi++) fa[k][mi] = load_a(at, half * 2 + k, mi);
#pragma unroll
      for (int ni = 0; ni < NI; ni++) fb[k][ni] = load_b(bt, half * 2 + k, ni);
    }
  };
  auto multiply = [&](auto first_tag) {   // the matrix instructions of half a slice
    constexpr bool FIRST = decltype(first_tag)::value;
    const f32x16 zero = {};
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int k = 0; k < 2; k++)
#pragma unroll
      for (int mi = 0; mi < MI; mi++)
#pragma unroll
        for (int ni = 0; ni < NI; ni++)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[k][ni], fa[k][mi], FIRST && k == 0 ? zero : acc[mi][ni], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  auto fetched = [&]() {   // fragments have arrived; meet the others
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0) (the builtin: the compiler then knows that no further wait is needed)
    block_barrier();
  };
  // everything requested has landed but for the A slice requested last, if it was
  auto landed = [&](bool a_requested) {
    if (a_requested) wait_vmcnt<A_LOADS>();
    else wait_vmcnt<0>();
  };

  // slices 0 and 1 (of the workgroup's units one after the other)
  int w = blockIdx.x;
  setup_a();
  setup_b();
  bool two = false;
#pragma unroll
  for (int s = 0; s < 2; s++)
    if (a_w < g.units) {
      request_a(s);
      request_b(s);
      two = s == 1;
    }
  if (two) wait_vmcnt<LOADS>();
  else wait_vmcnt<0>();
  block_barrier();
  bool started = false;   // B(1) is requested above
  constexpr std::true_type yes;
  constexpr std::false_type no;
  auto slice = [&](auto first_tag) {
    fetch(0);
    __builtin_amdgcn_sched_barrier(0);
    if (started && b_w < g.units) request_b(sb ^ 1);
    fetched();
    multiply(first_tag);
    block_barrier();
    fetch(1);
    __builtin_amdgcn_sched_barrier(0);
    const bool fresh = a_w < g.units;   // the youngest request is A(t + 2)
    if (fresh) request_a(sa == 0 ? 2 : sa - 1);
    if (group == 1) landed(fresh);
    fetched();
    multiply(no);
    if (group == 0) landed(fresh);
    block_barrier();
    started = true;
    sa = sa == 2 ? 0 : sa + 1;
    sb ^= 1;
  };
  for (;;) {
    const Unit u = unit(w);
    if (group == 1) block_barrier();
    slice(yes);
    for (int kt = 1; kt < u.nk; kt++) slice(no);
    if (group == 0) block_barrier();
    int e_tid = tid;
    asm volatile("" : "+v"(e_tid));
    const int e_lane = e_tid & 63;
    const int last = sa == 0 ? 2 : sa - 1;
    unsigned char* area = smem + (wave < IN_STAGE ? last * A_BYTES + wave * kEpiStage : REST_AT + (wave - IN_STAGE) * kEpiStage);
    const int row0 = u.m0 + wave_m * TM, col0 = u.n0 + wave_n * TN;
    bool full = row0 + TM <= u.M && col0 + TN <= u.N;
    if constexpr (GROUP) {
      Params e;
      e.M = u.M; e.N = u.N; e.C = u.C;
      if (full) direct_epilogue<EPI, MI, true>(e, acc, area, row0, col0, u.c_off, e_lane);
      else direct_epilogue<EPI, MI, false>(e, acc, area, row0, col0, u.c_off, e_lane);
    } else {
      if (EPI != E_F32 && EPI != E_F32_RES && EPI != E_PARTIAL)
        full = full && (g.ldc & 7) == 0 && (u.c_off & 7) == 0 && (((uintptr_t)g.C | (uintptr_t)g.C2 | (uintptr_t)g.U) & 15) == 0;
      if (full) direct_epilogue<EPI, MI, true>(g, acc, area, row0, col0, u.c_off, e_lane);
      else direct_epilogue<EPI, MI, false>(g, acc, area, row0, col0, u.c_off, e_lane);
    }
    w += (int)gridDim.x;
    if (w >= g.units) break;
  }
}

}  // namespace gemm
}  // namespace et
