// Attention core for sequences longer than the on-chip kernels hold (head size 64, any number of tokens).  A workgroup of
// four waves owns 128 rows of one (batch, head), 32 per wave, with their fragments in registers, and streams the other
// side through LDS in chunks of 64 rows (two buffers of 16 KB, direct-to-LDS loads of the next chunk under the current
// one's work):
//   forward   own queries, stream K and V: running maximum and sum per query (a lane holds one query), the result is
//             rescaled when the maximum of a chunk exceeds what was seen before;
//   backward  one launch, two kinds of workgroups: own queries, stream K and V -> dQ; own keys, stream Q and dO -> dK, dV.
//             Both recompute the probabilities from the stored log-sum-exp; rowsum(P * dP) of a query is dO . O, with O as the
//             stored bf16 value plus a second one, `rest`, that the forward pass leaves.  From the stored output alone,
//             dP - rowsum(P * dP) keeps the rounding error of O wherever values share a mean across tokens (relative error of dQ at 577
//             tokens, values of mean 3: 1.0e-2, against 3.0e-3 from materialised bf16 probabilities and 2.4e-3 with the rest).
//             out + rest is the result divided by the sum of the probabilities as rounded, so that what all keys share is exact.
//             It costs 2.0 us of the forward pass and 1.0 of the backward (times below).
// The register layout (transposed scores, no LDS round trip between the two products) is that of attention.hip.
// No score ever goes to memory: at 577 tokens, 8 x 6 heads, the former path (scores, softmax, batched products: eight launches
// for a layer's forward and backward, 64 MB of fp32 scores written and read several times) took about 170 us per layer, these
// two take 19.8 and 40.7 us; the full step of 12 such layers went from 5357 to 3929 us.  Up to 224 tokens the kernels that
// hold a head on chip stay ahead (64 x 12 heads of 197 tokens: 24.5 / 63.8 us against 28.7 / 88.5 here).
// Workgroups of one (batch, head) are dealt to the same XCD, whose L2 then holds the streamed rows.
#include "attention_tiles.h"

namespace et {
namespace {

using namespace attn;

constexpr int LW = 4, LTHREADS = LW * 64, OWN = LW * 32;   // waves, threads and own rows of a workgroup
constexpr int CH = 64, MAT = CH * PITCH;                   // rows of a chunk; bytes of one streamed matrix

// workgroup -> (batch, head) item and block of own rows; blocks of an item share an XCD (ids are dealt round-robin over 8)
__device__ __forceinline__ bool locate(int blocks, int items, int& item, int& blk) {
  const int x = blockIdx.x;
  item = x / (8 * blocks) * 8 + x % 8;
  blk = x / 8 % blocks;
  return item < items;
}

// one chunk of two [T][64] matrices (row strides ld0, ld1) into an LDS buffer: 16 one-KiB pieces of 8 rows, 4 per wave; rows
// beyond the sequence repeat the last one
__device__ __forceinline__ void issue_chunk(const bf16* m0, long long ld0, const bf16* m1, long long ld1, int row0, int T, unsigned lds_base, int tid) {
  asm volatile("" : "+v"(tid));   // (addresses are recomputed per chunk, not kept in registers)
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int p = wave * 4 + i, rp = p & 7;
    const int row = rp * 8 + (lane >> 3), pos = lane & 7;
    const long long r = min(row0 + row, T - 1);
    const bf16* src = (p >> 3 ? m1 + r * ld1 : m0 + r * ld0) + ((pos ^ swz(row)) << 3);
    dma16(src, __builtin_amdgcn_readfirstlane(lds_base + (p >> 3) * MAT + rp * 1024));
  }
}
__device__ __forceinline__ void chunk_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // this wave's pieces have landed, its reads of the other buffer too
  asm volatile("s_barrier" ::: "memory");
}
// own rows as an operand: row l%32 of the wave's 32, 8 consecutive columns per half-wave and slice of 16
__device__ __forceinline__ void load_own(const bf16* m, long long ld, int row, bf16x8 (&f)[4], int khalf) {
#pragma unroll
  for (int ks = 0; ks < 4; ks++) f[ks] = *(const bf16x8*)(m + (long long)row * ld + ks * 16 + khalf * 8);
}

__global__ __launch_bounds__(LTHREADS) void attention_long_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ out, bf16* __restrict__ rest,
                                                                      float* __restrict__ lse, int T, int H, float scale, int items, int blocks) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * 2 * MAT + LW * STORE_AREA];
  int item, blk;
  if (!locate(blocks, items, item, blk)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, khalf = lane >> 5;
  const int b = item / H, h = item % H, D = H * DH;
  const long long ld = 3LL * D;
  const bf16* q = qkv + (long long)b * T * ld + h * DH;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  const float c = scale * 1.44269504088896341f;
  const int own0 = blk * OWN + wave * 32;

  bf16x8 qf[4];
  load_own(q, ld, min(own0 + l32, T - 1), qf, khalf);
  issue_chunk(q + D, ld, q + 2 * D, ld, 0, T, lds0, tid);
  float m = -INFINITY, sum = 0.f;
  f32x16 o[2], sum16;   // sum16: of the rounded probabilities, a product with ones (the same sum in every register)
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; e++) ones[e] = (bf16)1.f;
#pragma unroll
  for (int r = 0; r < 16; r++) sum16[r] = 0.f;
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[dt][r] = 0.f;
  const int chunks = (T + CH - 1) / CH;
  for (int ch = 0; ch < chunks; ch++) {
    chunk_barrier();
    if (ch + 1 < chunks) issue_chunk(q + D, ld, q + 2 * D, ld, (ch + 1) * CH, T, lds0 + ((ch + 1) & 1) * 2 * MAT, tid);
    const unsigned char* sk = smem + (ch & 1) * 2 * MAT;
    const unsigned char* sv = sk + MAT;
    f32x16 st[2];
#pragma unroll
    for (int kt = 0; kt < 2; kt++) {
#pragma unroll
      for (int r = 0; r < 16; r++) st[kt][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ks++)
        st[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_direct(sk, kt * 32, ks, lane), qf[ks], st[kt], 0, 0, 0);
    }
    if (ch + 1 == chunks) {   // keys beyond the sequence
#pragma unroll
      for (int kt = 0; kt < 2; kt++)
#pragma unroll
        for (int r = 0; r < 16; r++) st[kt][r] = ch * CH + kt * 32 + tile_row(r, lane) < T ? st[kt][r] : -INFINITY;
    }
    float mx = m;
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
#pragma unroll
      for (int r = 0; r < 16; r++) mx = fmaxf(mx, st[kt][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));   // finite: the first key of a chunk exists
    if (__any(mx > m)) {
      const float f = __builtin_amdgcn_exp2f((m - mx) * c);   // (0 for the first chunk)
      sum *= f;
#pragma unroll
      for (int r = 0; r < 16; r++) sum16[r] *= f;
#pragma unroll
      for (int dt = 0; dt < 2; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[dt][r] *= f;
      m = mx;
    }
    const float mc = -m * c;
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
#pragma unroll
      for (int j = 0; j < 2; j++) {
        bf16x8 pf;
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float p = __builtin_amdgcn_exp2f(fmaf(st[kt][j * 8 + e], c, mc));
          sum += p;
          pf[e] = (bf16)p;
        }
        sum16 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pf, sum16, 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < 2; dt++)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_tr(sv, kt * 32 + j * 16, dt * 32, lane), pf, o[dt], 0, 0, 0);
      }
  }
  const float S = sum + __shfl_xor(sum, 32, 64), inv = 1.f / S, inv16 = 1.f / sum16[0];
  const int row = own0 + l32;
  if (khalf == 0 && row < T) lse[((long long)b * H + h) * T + row] = m * scale + logf(S);
  unsigned char* area = smem + 2 * 2 * MAT + wave * STORE_AREA;
  const long long at = ((long long)b * T + own0) * D + h * DH;
  store_tile(area, o, inv, out + at, D, T - own0, lane);
  if (!rest) return;
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[dt][r] = o[dt][r] * inv16 - (float)(bf16)(o[dt][r] * inv);
  store_tile(area, o, 1.f, rest + at, D, T - own0, lane);
}

// sum += x . (y + r), 8 elements; r nullable
__device__ __forceinline__ void add_dot(float& sum, const bf16* x, const bf16* y, const bf16* r) {
  const bf16x8 a = *(const bf16x8*)x, b = *(const bf16x8*)y;
  bf16x8 c = {};
  if (r) c = *(const bf16x8*)r;
#pragma unroll
  for (int e = 0; e < 8; e++) sum += (float)a[e] * ((float)b[e] + (float)c[e]);
}

__global__ __launch_bounds__(LTHREADS) void attention_long_bwd_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ out, const bf16* __restrict__ rest,
                                                                      const bf16* __restrict__ dout, const float* __restrict__ lse,
                                                                      bf16* __restrict__ dqkv, float* __restrict__ part, int T, int H, float scale, int items, int blocks) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * 2 * MAT + LW * STORE_AREA];
  __shared__ __attribute__((aligned(16))) float s_lse[2][CH], s_dot[2][CH];
  __shared__ float s_sum[2][LW][DH];   // column sums of dQ, or of dK and dV, per wave
  int item, blk;
  if (!locate(2 * blocks, items, item, blk)) return;
  const bool keys = blk >= blocks;       // own keys (dK, dV); the first `blocks` workgroups own queries (dQ)
  if (keys) blk -= blocks;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, khalf = lane >> 5;
  const int b = item / H, h = item % H, D = H * DH;
  const long long ld = 3LL * D;
  const bf16* q = qkv + (long long)b * T * ld + h * DH;
  const bf16* dO = dout + (long long)b * T * D + h * DH;
  const bf16* oo = out + (long long)b * T * D + h * DH;
  const bf16* orest = rest ? rest + (long long)b * T * D + h * DH : nullptr;
  const float* ls = lse + ((long long)b * H + h) * T;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  const float log2e = 1.44269504088896341f, c = scale * log2e;   // exp(scale * s - lse) = 2^(c s - lse log2(e))
  const int own0 = blk * OWN + wave * 32;
  const int own = min(own0 + l32, T - 1);
  const int chunks = (T + CH - 1) / CH;
  unsigned char* area = smem + 2 * 2 * MAT + wave * STORE_AREA;

  if (!keys) {
    issue_chunk(q + D, ld, q + 2 * D, ld, 0, T, lds0, tid);
    bf16x8 qf[4], dof[4];
    load_own(q, ld, own, qf, khalf);
    load_own(dO, D, own, dof, khalf);
    float dot = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      const long long at = (long long)own * D + ks * 16 + khalf * 8;
      add_dot(dot, dO + at, oo + at, orest ? orest + at : nullptr);
    }
    dot += __shfl_xor(dot, 32, 64);
    const float my_lse = ls[own] * log2e;
    f32x16 dq[2];
#pragma unroll
    for (int dt = 0; dt < 2; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) dq[dt][r] = 0.f;
    for (int ch = 0; ch < chunks; ch++) {
      chunk_barrier();
      if (ch + 1 < chunks) issue_chunk(q + D, ld, q + 2 * D, ld, (ch + 1) * CH, T, lds0 + ((ch + 1) & 1) * 2 * MAT, tid);
      const unsigned char* sk = smem + (ch & 1) * 2 * MAT;
      const unsigned char* sv = sk + MAT;
      const int left = T - ch * CH;   // keys of this chunk inside the sequence (rows beyond repeat the last key)
#pragma unroll
      for (int kt = 0; kt < 2; kt++) {
        f32x16 st, dp;
#pragma unroll
        for (int r = 0; r < 16; r++) { st[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
          st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_direct(sk, kt * 32, ks, lane), qf[ks], st, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_direct(sv, kt * 32, ks, lane), dof[ks], dp, 0, 0, 0);
        }
        if (left < CH) {
#pragma unroll
          for (int r = 0; r < 16; r++) st[r] = kt * 32 + tile_row(r, lane) < left ? st[r] : -INFINITY;
        }
#pragma unroll
        for (int j = 0; j < 2; j++) {
          bf16x8 dsf;
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const int r = j * 8 + e;
            dsf[e] = (bf16)(__builtin_amdgcn_exp2f(fmaf(st[r], c, -my_lse)) * (dp[r] - dot));
          }
#pragma unroll
          for (int dt = 0; dt < 2; dt++)
            dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_tr(sk, kt * 32 + j * 16, dt * 32, lane), dsf, dq[dt], 0, 0, 0);
        }
      }
    }
    store_tile(area, dq, scale, dqkv + ((long long)b * T + own0) * ld + h * DH, ld, T - own0, lane,
               part ? s_sum[0][wave] : nullptr);
    if (!part) return;
    __syncthreads();
    if (tid < DH) {   // row (b, blk) of the partial sums [B * blocks][3 D]
      float s = s_sum[0][0][tid];
#pragma unroll
      for (int k = 1; k < LW; k++) s += s_sum[0][k][tid];
      part[(b * blocks + blk) * ld + h * DH + tid] = s;
    }
    return;
  }

  // ---- own keys
  // log-sum-exp and dO . O of a chunk's 64 queries: four threads per query, 16 columns each
  auto chunk_scalars = [&](int ch) {
    const int r = tid >> 2, part = tid & 3, row = ch * CH + r;
    const long long at = (long long)min(row, T - 1) * D + part * 16;
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < 2; i++) add_dot(dot, dO + at + i * 8, oo + at + i * 8, orest ? orest + at + i * 8 : nullptr);
    dot += __shfl_xor(dot, 1, 64);
    dot += __shfl_xor(dot, 2, 64);
    if (part == 0) {
      s_dot[ch & 1][r] = dot;
      s_lse[ch & 1][r] = row < T ? ls[row] * log2e : INFINITY;   // queries beyond the sequence: probability zero
    }
  };
  issue_chunk(q, ld, dO, D, 0, T, lds0, tid);
  chunk_scalars(0);
  bf16x8 kf[4], vf[4];
  load_own(q + D, ld, own, kf, khalf);
  load_own(q + 2 * D, ld, own, vf, khalf);
  f32x16 dk[2], dv[2];
#pragma unroll
  for (int dt = 0; dt < 2; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) { dk[dt][r] = 0.f; dv[dt][r] = 0.f; }
  for (int ch = 0; ch < chunks; ch++) {
    chunk_barrier();
    if (ch + 1 < chunks) {
      issue_chunk(q, ld, dO, D, (ch + 1) * CH, T, lds0 + ((ch + 1) & 1) * 2 * MAT, tid);
      chunk_scalars(ch + 1);
    }
    const unsigned char* sq = smem + (ch & 1) * 2 * MAT;
    const unsigned char* sdo = sq + MAT;
#pragma unroll 1
    for (int qt = 0; qt < 2; qt++) {
      f32x16 st, dp;
#pragma unroll
      for (int r = 0; r < 16; r++) { st[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < 4; ks++) {
        st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_direct(sq, qt * 32, ks, lane), kf[ks], st, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_direct(sdo, qt * 32, ks, lane), vf[ks], dp, 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < 2; j++) {
        bf16x8 pf, dsf;
#pragma unroll
        for (int a = 0; a < 2; a++) {
          const int at = qt * 32 + (j * 2 + a) * 8 + khalf * 4;
          const float4 l4 = *(const float4*)(s_lse[ch & 1] + at), d4 = *(const float4*)(s_dot[ch & 1] + at);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const int r = j * 8 + a * 4 + e;
            const float p = __builtin_amdgcn_exp2f(fmaf(st[r], c, -lv[e]));
            pf[a * 4 + e] = (bf16)p;
            dsf[a * 4 + e] = (bf16)(p * (dp[r] - dv4[e]));
          }
        }
#pragma unroll
        for (int dt = 0; dt < 2; dt++) {
          dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_tr(sdo, qt * 32 + j * 16, dt * 32, lane), pf, dv[dt], 0, 0, 0);
          dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows_tr(sq, qt * 32 + j * 16, dt * 32, lane), dsf, dk[dt], 0, 0, 0);
        }
      }
    }
  }
  bf16* drow0 = dqkv + ((long long)b * T + own0) * ld + h * DH;
  store_tile(area, dk, scale, drow0 + D, ld, T - own0, lane, part ? s_sum[0][wave] : nullptr);
  store_tile(area, dv, 1.f, drow0 + 2 * D, ld, T - own0, lane, part ? s_sum[1][wave] : nullptr);
  if (!part) return;
  __syncthreads();
  if (tid < 2 * DH) {
    const int which = tid / DH, col = tid % DH;
    float s = s_sum[which][0][col];
#pragma unroll
    for (int k = 1; k < LW; k++) s += s_sum[which][k][col];
    part[(b * blocks + blk) * ld + (1 + which) * D + h * DH + col] = s;
  }
}

// grid: items rounded up to a multiple of 8 (one share per XCD) times the blocks of an item
bool grid_of(int B, int T, int H, int per_item, unsigned* grid) {
  const long long items8 = ((long long)B * H + 7) / 8 * 8;
  const long long n = items8 * per_item;
  if (n > 0x7fffffffll || (long long)B * H > 0x7ffffff0ll) return false;
  *grid = (unsigned)n;
  return true;
}

}  // namespace

hipError_t attention_long_fwd(const bf16* qkv, bf16* out, bf16* rest, float* lse, int B, int T, int H, float scale, hipStream_t s) {
  const int blocks = (T + OWN - 1) / OWN;
  unsigned grid;
  if (B < 1 || H < 1 || T < 1 || !grid_of(B, T, H, blocks, &grid)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attention_long_fwd_kernel, dim3(grid), dim3(LTHREADS), 0, s, qkv, out, rest, lse, T, H, scale, B * H, blocks);
  return hipGetLastError();
}

hipError_t attention_long_bwd(const bf16* qkv, const bf16* out, const bf16* rest, const bf16* dout, const float* lse, bf16* dqkv, int B, int T,
                              int H, float scale, hipStream_t s, float* part) {
  const int blocks = (T + OWN - 1) / OWN;
  unsigned grid;
  if (B < 1 || H < 1 || T < 1 || !out || !grid_of(B, T, H, 2 * blocks, &grid)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attention_long_bwd_kernel, dim3(grid), dim3(LTHREADS), 0, s, qkv, out, rest, dout, lse, dqkv, part, T, H, scale, B * H, blocks);
  return hipGetLastError();
}

int attention_long_bwd_parts(int B, int T) { return B * ((T + OWN - 1) / OWN); }

}  // namespace et
